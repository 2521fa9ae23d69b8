// Host driver of tests/test_grown_box.py: the interface box grown by g cells
// (GrownBox) against its definition, over every box on one axis of a small
// lattice with a box of one cell in the middle of the two others.
#include <cstdio>
#include <cstdlib>
#include <set>
#include <vector>

#include "fslbm_adjoint.hpp"

using namespace fslbm;

static int bad = 0;

static void check(int axis, int n, int o, int e, int g)
{
    int ext[3] = {13, 13, 13}, lo[3] = {6, 6, 6}, len[3] = {1, 1, 1};
    ext[axis] = n;
    lo[axis] = o;
    len[axis] = e;
    const GrownBox box(CellRange{lo[0], lo[1], lo[2], len[0], len[1], len[2]}, ext[0], ext[1], ext[2], g);
    // the definition: a coordinate within g cells of the box, on the circle
    std::vector<char> in[3];
    for (int a = 0; a < 3; ++a) {
        in[a].assign(ext[a], 0);
        for (int v = lo[a] - g; v < lo[a] + len[a] + g; ++v) in[a][((v % ext[a]) + ext[a]) % ext[a]] = 1;
    }
    std::set<int> want, got;
    bool same = true;
    for (int z = 0; z < ext[2]; ++z)
        for (int y = 0; y < ext[1]; ++y)
            for (int x = 0; x < ext[0]; ++x) {
                const bool w = in[0][x] && in[1][y] && in[2][z];
                if (w) want.insert(x + ext[0] * (y + ext[1] * z));
                same &= box.contains(x, y, z) == w;
            }
    for (int k = 0; k < box.r.size(); ++k) got.insert(box.at(k).at(0, 0, 0));
    same &= got == want && (int)got.size() == box.r.size();
    if (!same) {
        ++bad;
        std::printf("axis %d extent %d box start %d length %d grown by %d\n", axis, n, o, e, g);
    }
}

int main()
{
    int cases = 0;
    for (int axis = 0; axis < 3; ++axis)
        for (int g : {2, FD_GROW})
            for (int n = g == 2 ? 3 : 10; n <= 20; ++n)  // the extents that the LSQR and FD models take
                for (int o = 0; o < n; ++o)
                    for (int e = 1; o + e <= n; ++e, ++cases) check(axis, n, o, e, g);
    std::printf("%d boxes, %d wrong\n", cases, bad);
    return bad != 0;
}
