// Cell-type conversion, interface-list compaction, obstacle fill reflection.
//
// The paper keeps the liquid / interface / gas classification of Sec. II
// (an interface cell has liquid and gas D3Q19 neighbours, only interface
// cells hold 0 < phi < 1) and defers the conversion rules to Koerner et al.
// This library uses the following rules, per step:
//   1  interface cells fill when m > (1 + eps) rho and empty when
//      m < -eps rho (classified in the stream-collide kernel);
//   2  filling wins: an emptying cell with a filling D3Q19 neighbour stays;
//   3  gas neighbours of filling cells and liquid neighbours of emptying
//      cells become interface cells; those from gas get
//      f' = feq(mean rho, mean u) of their liquid/interface neighbours and
//      m = 0, those from liquid keep f' and get m = rho;
//   4  closure of the interface layer (Sec. II.D: an interface cell has gas
//      and liquid D3Q19 neighbours): on the types after rules 1-3, a layer
//      cell without a gas neighbour becomes liquid; then, on the updated
//      types, one without a liquid neighbour becomes gas;
//   5  every cell that leaves the layer hands on m - rho (to liquid) or m
//      (to gas), split equally over its D3Q19 neighbours that are interface
//      cells after the step; with no such neighbour the amount goes to a
//      reservoir;
//   6  the cells take their new types.
// Rule 4 starts from a closed layer (creation closes it), so only cells of
// the step's layer (old interface cells and new cells) can break it.
// Three launches per step, all of which return at once when no cell converts
// (the last one then only sets phi = m / rho):
//   k_conv_mark    one wavefront per filling or emptying cell (rules 2-3),
//   k_conv_close   one thread per cell of the layer (rule 4) and one half
//                  wavefront per new cell (the f' of rule 3),
//   k_conv_gather  one thread per cell of the layer (rules 5-6), the new
//                  interface list and its box.
// The work is latency: a few hundred cells per step, each with two rings of
// scattered neighbours. So the cells are spread over lanes (one lane per
// neighbour), and a cell's neighbour types are loaded together rather than
// one after the other. Each output value has one writer, or several writers
// storing the identical value. New cells are tagged in `mark` with the step
// number, so no clearing pass is needed. Measured per step, FP32: 34 us
// (7 + 10 + 17) on a bubble carried through 97 x 61 x 83 at u = 0.05, 22 us
// on the 256 x 256 x 128 sessile drop; with one thread per converting cell
// (each computing the f' of up to 18 new cells from 342 neighbour loads in
// turn), neighbours tested one by one and the list copied by a launch of its
// own, the chain took five launches and 228 and 79 us there.
#pragma once

#include "fslbm_device.hpp"
#include "fslbm_stream.hpp"

namespace fslbm {

constexpr int LIST_GRID = 256;  // blocks per lattice of the grid-stride list kernels (of 256 threads)
// Threads of a block of the list kernels whose threads work alone (gradients
// and stencils over list cells: some 50 scattered loads a thread). A list
// holds tens to a thousand wavefronts: blocks of one wavefront spread them
// over the CUs, where four to a block share one CU's cache and leave most of
// the others idle. Per launch, 256 -> 64 threads: reverse pass over phi = m / rho
// 7.6 -> 5.0 us and transposed gradient 8.9 -> 5.8 (128^3 sessile drop; both
// with their loads moved ahead), normals 7.1 -> 6.2 there and 9.4 -> 8.3 on
// the 256 x 256 x 128 drop; the LSQR fit, bound by its FP64 chain, is equal.
constexpr int LIST_NT = 64;

__device__ inline int list_count(const DevScalars *sc) { return *(volatile const int *)&sc->icount; }

// The interface list: the step that rebuilds it writes the other of the two
// buffers, and its last block makes that one current.
template <class P>
__device__ inline const int32_t *interface_list(const Fields<P> &F)
{
    return F.sc->lsel ? F.ilist_tmp : F.ilist;
}

// A new cell of this step (tagged 1 from gas or 2 from liquid; 3 marks an
// old-list cell that leaves the layer).
__device__ inline bool is_new(uint32_t mk, uint32_t tag) { return (mk & ~3u) == tag && (mk & 3u) != 3u; }

__device__ inline int wrap_one(int v, int n) { return v < 0 ? v + n : (v >= n ? v - n : v); }

// Rules 2 and 3, one wavefront per cell that the stream-collide listed as
// filling or emptying (clist, nconv entries). Lane q < 19 looks at the
// neighbour in direction q: rule 2 drops an emptying cell next to a filling
// one (it reads only its neighbours' filling, which dropping never changes),
// rule 3 tags the new interface cells and lists them once. The wavefront
// then stamps the 7x7x7 box around the cell in `near` with the low byte of
// the step number: the closure of rule 4 can only change a cell within two
// cells of a converting one (the layer was closed before the step), and the
// excess of rule 5 moves one cell further. A stale stamp that happens to
// match only makes a cell be checked. The fluid box grows by every new cell
// (a new cell from gas is fluid whether it stays in the layer or closes to
// liquid).
template <class P>
__device__ inline void conv_mark(const Fields<P> &F, int nc, int wave, int waves)
{
    const uint32_t tag = F.sc->step << 2;
    const uint8_t s8 = uint8_t(tag >> 2);
    const int lane = threadIdx.x & 63;
    const int q = lane < NQ ? lane : 0;  // lanes without a direction read the cell itself
    for (int c = wave; c < nc; c += waves) {
        const int i = F.clist[c];
        const Nbr nb(i, F.nx, F.ny, F.nz);
        const int j = nb.at(dir_x(q), dir_y(q), dir_z(q));
        const uint8_t st = F.conv[i], cj = F.conv[j], fj = F.flags[j];
        if (st == CV_EMPTY && __any(q != 0 && (fj & FL_IF) && cj == CV_FILL)) {
            if (lane == 0) F.conv[i] = CV_NONE;
            continue;
        }
        const uint8_t tj = fj & FL_TYPE;
        const bool hit = q != 0 && tj == (st == CV_FILL ? FL_GAS : FL_LIQ);
        bool fresh = false;
        if (hit) {
            const uint32_t mk = tag | (st == CV_FILL ? 1u : 2u);
            // the first wavefront to tag j lists it as a new interface cell
            fresh = (atomicExch(&F.mark[j], mk) & ~3u) != tag;
            F.conv[j] = CV_NONE;
        }
        const unsigned long long fm = __ballot(fresh);
        if (fm) {
            int base = 0;
            if (lane == 0) base = atomicAdd(&F.sc->nnew, __popcll(fm));
            base = __shfl(base, 0, 64);
            if (fresh) {
                F.newlist[base + __popcll(fm & ((1ull << lane) - 1ull))] = j;
                const int yz = j / F.nx, z = yz / F.ny;
                const int v[3] = {j - yz * F.nx, yz - z * F.ny, z};
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    if (v[k] < F.sc->fbox[k]) atomicMin(&F.sc->fbox[k], v[k]);
                    if (v[k] > F.sc->fbox[3 + k]) atomicMax(&F.sc->fbox[3 + k], v[k]);
                }
            }
        }
        for (int t = lane; t < 343; t += 64) {  // one wrap covers an offset of 3 for extents >= 3
            const int dx = t % 7 - 3, dy = (t / 7) % 7 - 3, dz = t / 49 - 3;
            F.near[wrap_one(nb.x + dx, F.nx) + F.nx * (wrap_one(nb.y + dy, F.ny) + F.ny * wrap_one(nb.z + dz, F.nz))] = s8;
        }
    }
}
template <class P>
__global__ __launch_bounds__(256) void k_conv_mark(const Batch<P> B)
{
    const Fields<P> &F = B.f[blockIdx.y];
    const int nc = *(volatile const int *)&F.sc->nconv;
    const int waves = blockDim.x >> 6;
    if (nc != 0) conv_mark(F, nc, blockIdx.x * waves + (threadIdx.x >> 6), gridDim.x * waves);
}

// Cell type after rules 1-3 (CLOSE_* codes read as interface) from a cell's
// flags, mark and status: the classification rule 4 starts from. A cell that
// is tagged as leaving in the same launch reads the same before and after.
__device__ inline uint8_t type_after(uint8_t f, uint32_t mk, uint8_t st, uint32_t tag)
{
    if (is_new(mk, tag)) return FL_IF;
    if (!(f & FL_IF)) return f & FL_TYPE;
    return st == CV_FILL ? FL_LIQ : (st == CV_EMPTY ? FL_GAS : FL_IF);
}

// The types of cell c's neighbours in the directions 1..18, loaded together.
template <class P>
__device__ inline void neighbour_types(const Fields<P> &F, const Nbr &nb, uint32_t tag, uint8_t (&t)[NQ])
{
    uint8_t f[NQ], st[NQ];
    uint32_t mk[NQ];
#pragma unroll
    for (int q = 1; q < NQ; ++q) {
        const int j = nb.at(dir_x(q), dir_y(q), dir_z(q));
        f[q] = F.flags[j];
        mk[q] = F.mark[j];
        st[q] = F.conv[j];
    }
#pragma unroll
    for (int q = 1; q < NQ; ++q) t[q] = type_after(f[q], mk[q], st[q], tag);
}

// Cell k of the step's layer: the old list, then the new cells.
template <class P>
__device__ inline int layer_cell(const Fields<P> &F, const int32_t *list, int k, int n)
{
    return k < n ? list[k] : F.newlist[k - n];
}

// f' of a new cell (rule 3), by the 32 lanes of a half wavefront. From gas:
// feq(mean rho, mean u) of its liquid / interface neighbours (types before
// the step), lane p holding the moments of neighbour p, added in direction
// order; m = 0. From liquid: f' stays, rho is its sum in direction order and
// m = rho.
template <class P>
__device__ inline void init_new_cell(const Fields<P> &F, int j, int lane)
{
    using T = typename P::T;
    using R = typename P::R;
    const typename P::S *f = F.fdst;
    const int p = lane < NQ ? lane : 0;
    if ((F.mark[j] & 3u) == 1u) {
        const Nbr nj(j, F.nx, F.ny, F.nz);
        const int w = nj.at(dir_x(p), dir_y(p), dir_z(p));
        const int fluid = p != 0 && (F.flags[w] & FL_FLUID) ? 1 : 0;
        T r = 0, ux = 0, uy = 0, uz = 0;
        if (fluid) {
            T fw[NQ];
#pragma unroll
            for (int s = 0; s < NQ; ++s) {
                switch (s) {
#define FSLBM_LD(QQ) case QQ: fw[s] = load_f<P, QQ>(plane<P, QQ>(f, F.NS), w); break;
                    FSLBM_LD(0) FSLBM_LD(1) FSLBM_LD(2) FSLBM_LD(3) FSLBM_LD(4) FSLBM_LD(5)
                    FSLBM_LD(6) FSLBM_LD(7) FSLBM_LD(8) FSLBM_LD(9) FSLBM_LD(10) FSLBM_LD(11)
                    FSLBM_LD(12) FSLBM_LD(13) FSLBM_LD(14) FSLBM_LD(15) FSLBM_LD(16)
                    FSLBM_LD(17) FSLBM_LD(18)
#undef FSLBM_LD
                }
            }
            moments(fw, r, ux, uy, uz);
        }
        T rs = 0, usx = 0, usy = 0, usz = 0;
        int cnt = 0;
        for (int s = 1; s < NQ; ++s) {
            const T a = __shfl(r, s, 32), bx = __shfl(ux, s, 32), by = __shfl(uy, s, 32), bz = __shfl(uz, s, 32);
            if (!__shfl(fluid, s, 32)) continue;
            rs += a; usx += bx; usy += by; usz += bz;
            ++cnt;
        }
        const T rm = rs / T(cnt), vx = usx / T(cnt), vy = usy / T(cnt), vz = usz / T(cnt);
        const T v = feq<T>(p, rm, vx, vy, vz, vx * vx + vy * vy + vz * vz);
        typename P::S *dst = F.fdst + (size_t)p * (size_t)F.NS + j;
        if (lane < NQ) {
            if constexpr (P::SHIFT) store_rn(dst, (v - weight<T>(p)) * T(P::SCALE));
            else __builtin_nontemporal_store(v, dst);
        }
        if (lane == 0) {
            F.rho[j] = R(rm);
            F.m[j] = R(0);
        }
    } else {
        T v = 0;
        if constexpr (P::SHIFT) v = weight<T>(p) + to_float(f[(size_t)p * (size_t)F.NS + j]) * T(1.0 / P::SCALE);
        else v = f[(size_t)p * (size_t)F.NS + j];
        T r = 0;
        for (int s = 0; s < NQ; ++s) r += __shfl(v, s, 32);
        if (lane == 0) {
            F.rho[j] = R(r);
            F.m[j] = R(r);
        }
    }
}

// Rule 4, both passes in one launch: without a gas neighbour a cell becomes
// liquid; otherwise, without a neighbour that is liquid after the first pass
// (liquid, or a layer cell without a gas neighbour), it becomes gas. Each
// cell writes only its own status, and a neighbour's first-pass result is
// evaluated, not read, so no thread depends on another's write. The second
// pass looks two cells out only for a cell without a liquid neighbour after
// rules 1-3, which is rare. Every old-list cell that leaves the layer is
// tagged tag | 3, which k_conv_gather tells it by. The new cells' f' (an
// independent job) rides on the same launch, in its last blocks first, which
// have no cell of the layer on a small lattice. Block b of nb blocks.
template <class P>
__device__ inline void conv_close(const Fields<P> &F, int b, int nb)
{
    if (b == 0 && threadIdx.x == 0) {  // counters of the list rebuild in k_conv_gather
        F.sc->nkeep = 0;
        F.sc->done = 0;
        F.sc->bbox[0] = F.nx; F.sc->bbox[1] = F.ny; F.sc->bbox[2] = F.nz;
        F.sc->bbox[3] = -1; F.sc->bbox[4] = -1; F.sc->bbox[5] = -1;
    }
    const uint32_t tag = F.sc->step << 2;
    const uint8_t s8 = uint8_t(tag >> 2);
    const int n = list_count(F.sc), nn = *(volatile const int *)&F.sc->nnew, nt = blockDim.x;
    const int32_t *list = interface_list(F);
    for (int m = (nb - 1 - b) * (nt >> 5) + (int)(threadIdx.x >> 5); m < nn; m += nb * (nt >> 5))
        init_new_cell(F, F.newlist[m], threadIdx.x & 31);
    const int lane = threadIdx.x & 63;
    for (int k0 = b * nt; k0 < n + nn; k0 += nb * nt) {
        const int k = k0 + (int)threadIdx.x;
        const int i = k < n + nn ? layer_cell(F, list, k, n) : 0;
        const bool on = k < n + nn && F.near[i] == s8;
        const bool leaves = on && F.conv[i] != CV_NONE;
        if (leaves && k < n) F.mark[i] = tag | 3u;
        bool gas = true, liquid = true;
        if (on && !leaves) {
            uint8_t t[NQ];
            neighbour_types(F, Nbr(i, F.nx, F.ny, F.nz), tag, t);
            gas = liquid = false;
#pragma unroll
            for (int q = 1; q < NQ; ++q) {
                gas |= t[q] == FL_GAS;
                liquid |= t[q] == FL_LIQ;
            }
        }
        // the second pass, by the whole wavefront for one cell after the
        // other: lane q asks whether neighbour q lacks a gas neighbour
        unsigned long long need = __ballot(gas && !liquid);
        while (need) {
            const int l = __ffsll(need) - 1;
            need &= need - 1;
            const Nbr nc(__shfl(i, l, 64), F.nx, F.ny, F.nz);
            const int q = lane < NQ ? lane : 0;
            const int j = nc.at(dir_x(q), dir_y(q), dir_z(q));
            bool ok = false;
            if (q != 0 && type_after(F.flags[j], F.mark[j], F.conv[j], tag) == FL_IF) {
                uint8_t u[NQ];
                neighbour_types(F, Nbr(j, F.nx, F.ny, F.nz), tag, u);
                ok = true;
#pragma unroll
                for (int p = 1; p < NQ; ++p) ok &= u[p] != FL_GAS;
            }
            const bool found = __any(ok);
            if (lane == l) liquid = found;
        }
        if (gas && liquid) continue;
        F.conv[i] = gas ? CV_CLOSE_GAS : CV_CLOSE_LIQ;
        if (k < n) F.mark[i] = tag | 3u;
    }
}
template <class P>
__global__ __launch_bounds__(256) void k_conv_close(const Batch<P> B)
{
    const Fields<P> &F = B.f[blockIdx.y];
    if (F.sc->nconv != 0) conv_close(F, blockIdx.x, gridDim.x);
}

// Rule 5 for a cell w that leaves the layer: its excess, and the number of
// its neighbours that receive (cells of the layer that stay; every converter
// has a status, so the types that k_conv_gather rewrites do not enter).
template <class P>
__device__ inline int receivers(const Fields<P> &F, const Nbr &nw, uint32_t tag)
{
    uint8_t f[NQ], st[NQ];
    uint32_t mk[NQ];
#pragma unroll
    for (int q = 1; q < NQ; ++q) {
        const int j = nw.at(dir_x(q), dir_y(q), dir_z(q));
        f[q] = F.flags[j];
        mk[q] = F.mark[j];
        st[q] = F.conv[j];
    }
    int cnt = 0;
#pragma unroll
    for (int q = 1; q < NQ; ++q) cnt += ((f[q] & FL_IF) || (mk[q] & ~3u) == tag) && st[q] == CV_NONE;
    return cnt;
}
template <class P>
__device__ inline typename P::R excess_mass(const Fields<P> &F, int w)
{
    return cv_to_liquid(F.conv[w]) ? F.m[w] - F.rho[w] : F.m[w];
}

// The shares that reach cell j, in direction order: the neighbours that
// leave are collected first, then evaluated one after the other (one or two
// per receiving cell, so the lanes of a wavefront share the few rounds).
template <class P>
__device__ inline typename P::R gathered_excess(const Fields<P> &F, int j, uint32_t tag)
{
    using R = typename P::R;
    const Nbr nb(j, F.nx, F.ny, F.nz);
    uint32_t mk[NQ], from = 0;
    uint8_t st[NQ];
#pragma unroll
    for (int q = 1; q < NQ; ++q) {
        const int w = nb.at(dir_x(q), dir_y(q), dir_z(q));
        mk[q] = F.mark[w];
        st[q] = F.conv[w];
    }
#pragma unroll
    for (int q = 1; q < NQ; ++q) from |= (mk[q] & ~3u) == tag && st[q] != CV_NONE ? 1u << q : 0u;
    R acc = 0;
    while (from) {
        const int q = __ffs(from) - 1;
        from &= from - 1;
        const int w = nb.at(dir_x(q), dir_y(q), dir_z(q));
        const Nbr nw(w, F.nx, F.ny, F.nz);
        acc += excess_mass(F, w) / R(receivers(F, nw, tag));
    }
    return acc;
}

__device__ inline int block_exclusive_scan(int v, int *lds_wave, int &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) lds_wave[wave] = x;
    __syncthreads();
    int off = 0, tot = 0;
    const int nw = blockDim.x >> 6;
    for (int w = 0; w < nw; ++w) {
        if (w < wave) off += lds_wave[w];
        tot += lds_wave[w];
    }
    total = tot;
    __syncthreads();
    return off + x - v;
}

// Block-wide min / max of a box contribution; thread 0 issues the atomics.
template <int NT>
__device__ inline void block_box_update(int (&lo)[3], int (&hi)[3], int *box)
{
    __shared__ int red[6][NT / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            lo[c] = min(lo[c], __shfl_xor(lo[c], d, 64));
            hi[c] = max(hi[c], __shfl_xor(hi[c], d, 64));
        }
    if (lane == 0)
        for (int c = 0; c < 3; ++c) {
            red[c][wave] = lo[c];
            red[3 + c][wave] = hi[c];
        }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < NT / 64; ++w)
            for (int c = 0; c < 3; ++c) {
                red[c][0] = min(red[c][0], red[c][w]);
                red[3 + c][0] = max(red[3 + c][0], red[3 + c][w]);
            }
        if (red[3][0] >= 0)
            for (int c = 0; c < 3; ++c) {
                atomicMin(&box[c], red[c][0]);
                atomicMax(&box[3 + c], red[3 + c][0]);
            }
    }
    __syncthreads();
}

template <class P>
__device__ inline void box_add(const Fields<P> &F, int i, int (&lo)[3], int (&hi)[3])
{
    const int yz = i / F.nx, z = yz / F.ny, y = yz - z * F.ny, x = i - yz * F.nx;
    lo[0] = min(lo[0], x); lo[1] = min(lo[1], y); lo[2] = min(lo[2], z);
    hi[0] = max(hi[0], x); hi[1] = max(hi[1], y); hi[2] = max(hi[2], z);
}

// Rules 5 and 6, one thread per cell of the layer (the old list, then the
// new cells): receivers add their neighbours' shares, cells that leave take
// their type (their excess goes to the reservoir when nobody receives it),
// and the cells that stay are appended to the other list buffer, in order
// within each 256-cell chunk; the last block to finish makes that buffer
// current. The order of the list does not enter any result (every per-cell
// computation is independent). Also sets phi = m / rho of every interface
// cell for the new time level, so it runs in every step; without conversions
// that is all it does. Block b of nb blocks of NT threads.
template <class P, int NT>
__device__ inline void conv_gather(const Fields<P> &F, bool frozen, int b, int nb)
{
    using R = typename P::R;
    const int n = list_count(F.sc);
    const int32_t *list = interface_list(F);
    if (F.sc->nconv == 0) {
        for (int k = b * NT + threadIdx.x; k < n; k += nb * NT) {
            const int i = list[k];
            const R ph = F.m[i] / F.rho[i];
            F.phi[i] = ph;
            // a frozen window stays on one smooth piece of the step only while
            // every interface fill lies strictly inside (0, 1); one pair of
            // atomics per wavefront, for most windows have such cells
            const unsigned long long out = __ballot(frozen && !(ph > R(0) && ph < R(1)));
            if (out && (threadIdx.x & 63) == (unsigned)(__ffsll(out) - 1)) {
                atomicAdd(&F.sc->fill_out, __popcll(out));
                atomicMin(&F.sc->fill_out_step, F.sc->step);
            }
        }
        return;
    }
    __shared__ int lw[NT / 64];
    __shared__ int base_s;
    const uint32_t tag = F.sc->step << 2;
    const uint8_t s8 = uint8_t(tag >> 2);
    const int nl = n + *(volatile const int *)&F.sc->nnew;
    int32_t *out = F.sc->lsel ? F.ilist : F.ilist_tmp;
    int lo[3] = {1 << 30, 1 << 30, 1 << 30}, hi[3] = {-1, -1, -1};
    for (int k0 = b * NT; k0 < nl; k0 += nb * NT) {
        const int k = k0 + (int)threadIdx.x;
        bool keep = false;
        int i = 0;
        if (k < nl) {
            i = layer_cell(F, list, k, n);
            const uint8_t st = F.conv[i];
            keep = st == CV_NONE;
            if (keep) {
                // only a cell near a filling or emptying cell can receive
                const R mn = F.m[i] + (F.near[i] == s8 ? gathered_excess(F, i, tag) : R(0));
                F.m[i] = mn;
                F.phi[i] = mn / F.rho[i];
                if (k >= n) F.flags[i] = (F.flags[i] & FL_NEAR_OBST) | FL_IF;
            } else {
                const Nbr nb(i, F.nx, F.ny, F.nz);
                if (receivers(F, nb, tag) == 0) reservoir_add(F.sc, (double)excess_mass(F, i));
                F.phi[i] = cv_to_liquid(st) ? R(1) : R(0);
                F.flags[i] = (F.flags[i] & FL_NEAR_OBST) | (cv_to_liquid(st) ? FL_LIQ : FL_GAS);
            }
        }
        int tot;
        const int ex = block_exclusive_scan(keep ? 1 : 0, lw, tot);
        if (threadIdx.x == 0) base_s = tot > 0 ? atomicAdd(&F.sc->nkeep, tot) : 0;
        __syncthreads();
        if (keep) {
            out[base_s + ex] = i;
            box_add(F, i, lo, hi);
        }
    }
    block_box_update<NT>(lo, hi, F.sc->bbox);
    // no fence (it would write the whole L2 back): the last block reads
    // nothing of the others but nkeep, whose additions have returned before
    // their blocks count themselves here
    if (threadIdx.x == 0) {
        if (atomicAdd(&F.sc->done, 1) == nb - 1) {
            F.sc->icount = atomicAdd(&F.sc->nkeep, 0);
            F.sc->lsel ^= 1;
        }
    }
}
template <class P>
__global__ __launch_bounds__(256) void k_conv_gather(const Batch<P> B)
{
    conv_gather<P, 256>(B.f[blockIdx.y], B.p[blockIdx.y].frozen != 0, blockIdx.x, gridDim.x);
}

// The whole chain of a small layer in one block per lattice: the phases of
// the three launches above with barriers between them. A step without
// conversions is then one launch instead of three (each costs about 3 us on
// the device whatever it does). Between two phases every wavefront
// waits until its stores are in the L2, where the atomics act, and then drops
// what the CU's cache holds of words that the atomics changed. The host
// takes it for lattices of at most CONV_BLOCK_CELLS interface cells (one
// thread each) when they were last sized: there a few converting cells fit the
// block's 16 wavefronts. A layer that has grown since is walked in rounds.
// Per pass, FP64: droplet 24^3 (5 steps) 204 -> 180 us; 48^3 bubble between
// walls (20 steps, with the launch that the walls share with the volume sum)
// 1157 -> 925 us.
constexpr int CONV_BLOCK = 1024;
constexpr int CONV_BLOCK_CELLS = 1024;

template <class P>
__global__ __launch_bounds__(CONV_BLOCK) void k_conv_block(const Batch<P> B)
{
    const Fields<P> &F = B.f[blockIdx.y];
    const int nc = *(volatile const int *)&F.sc->nconv;
    if (nc != 0) {
        conv_mark(F, nc, threadIdx.x >> 6, CONV_BLOCK / 64);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        conv_close(F, 0, 1);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    conv_gather<P, CONV_BLOCK>(F, B.p[blockIdx.y].frozen != 0, 0, 1);
}

// The current list back into ilist (state copies hold that buffer alone):
// the entries, then the selector.
template <class P>
__global__ __launch_bounds__(256) void k_list_home(Fields<P> F)
{
    if (!F.sc->lsel) return;
    const int n = list_count(F.sc);
    for (int k = blockIdx.x * 256 + threadIdx.x; k < n; k += gridDim.x * 256) F.ilist[k] = F.ilist_tmp[k];
}
__global__ void k_list_reset(DevScalars *sc)
{
    sc->lsel = 0;
    sc->done = 0;
}

// ----------------------------------------------------------- compaction
// Ascending list of the cells whose flags match `want`: each block covers
// 1024 consecutive cells (4 per thread); per-block counts, one scan block,
// then the write pass with a wavefront-ballot / shuffle prefix sum.
constexpr int CMP_CELLS = 1024;


// Cells k = base .. base+3 of a range (x fastest): hit[s] and their indices.
__device__ inline int cells_matching(const uint8_t *flags, const CellRange &r, int nx, int ny, int base,
                                     uint8_t want, bool (&hit)[4], int (&idx)[4])
{
    const int n = r.size();
    int c = 0;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int k = base + s;
        idx[s] = k < n ? r.cell(k, nx, ny) : 0;
        hit[s] = k < n && (flags[idx[s]] & want);
        c += hit[s];
    }
    return c;
}

// which = 0: interface cells (flags & FL_IF) into ilist / icount (at
// creation); which = 1: the static list of obstacle cells next to
// non-obstacle cells (conv bit 0) into olist / ocount; which = 2: the static
// list of non-obstacle cells next to obstacle cells (conv bit 1) into
// wlist / wcount.
template <class P>
__device__ inline void compact_source(const Fields<P> &F, int which, const uint8_t *&src, uint8_t &want,
                                      int32_t *&list, int *&count, CellRange &range)
{
    range = which == 0 ? CellRange::from(F.sc->fbox) : CellRange::whole(F.nx, F.ny, F.nz);
    src = which == 0 ? F.flags : F.conv;
    want = which == 0 ? FL_IF : (which == 1 ? 1 : 2);
    list = which == 0 ? F.ilist : (which == 1 ? F.olist : F.wlist);
    count = which == 0 ? &F.sc->icount : (which == 1 ? &F.sc->ocount : &F.sc->wcount);
}

// A fixed grid of CMP_GRID blocks per lattice; block b owns a contiguous run
// of 1024-cell tiles, so the list stays in ascending order.
constexpr int CMP_GRID = 256;

__device__ inline void tile_range(int N, int &t0, int &t1)
{
    const int ntiles = (N + CMP_CELLS - 1) / CMP_CELLS;  // N: cells of the range
    const int per = (ntiles + gridDim.x - 1) / gridDim.x;
    t0 = min(ntiles, (int)blockIdx.x * per);
    t1 = min(ntiles, t0 + per);
}

template <class P>
__global__ __launch_bounds__(256) void k_compact_count(const Batch<P> B, int which)
{
    const Fields<P> &F = B.f[blockIdx.y];
    const uint8_t *src; uint8_t want; int32_t *list; int *count; CellRange range;
    compact_source(F, which, src, want, list, count, range);
    __shared__ int lw[4];
    int t0, t1;
    tile_range(range.size(), t0, t1);
    int sum = 0;
    for (int t = t0; t < t1; ++t) {
        bool hit[4];
        int idx[4];
        const int c = cells_matching(src, range, F.nx, F.ny, t * CMP_CELLS + threadIdx.x * 4, want, hit, idx);
        int total;
        block_exclusive_scan(c, lw, total);
        sum += total;
    }
    if (threadIdx.x == 0) F.counts[blockIdx.x] = sum;
}

// One block per lattice: exclusive scan of the block counts, list length;
// the interface bounding box is reset for the write pass.
template <class P>
__global__ __launch_bounds__(1024) void k_compact_scan(const Batch<P> B, int which, int nblocks)
{
    const Fields<P> &F = B.f[blockIdx.y];
    const uint8_t *src; uint8_t want; int32_t *list; int *count; CellRange range;
    compact_source(F, which, src, want, list, count, range);
    __shared__ int lw[16];
    int carry = 0;
    for (int b0 = 0; b0 < nblocks; b0 += 1024) {
        const int b = b0 + threadIdx.x;
        const int v = b < nblocks ? F.counts[b] : 0;
        int total;
        const int ex = block_exclusive_scan(v, lw, total);
        if (b < nblocks) F.counts[b] = carry + ex;
        carry += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *count = carry;
        if (which == 0) {
            F.sc->bbox[0] = F.nx; F.sc->bbox[1] = F.ny; F.sc->bbox[2] = F.nz;
            F.sc->bbox[3] = -1; F.sc->bbox[4] = -1; F.sc->bbox[5] = -1;
        }
    }
}

template <class P>
__global__ __launch_bounds__(256) void k_compact_write(const Batch<P> B, int which)
{
    const Fields<P> &F = B.f[blockIdx.y];
    const uint8_t *src; uint8_t want; int32_t *list; int *count; CellRange range;
    compact_source(F, which, src, want, list, count, range);
    __shared__ int lw[4];
    int t0, t1;
    tile_range(range.size(), t0, t1);
    int base = F.counts[blockIdx.x];
    int lo[3] = {F.nx, F.ny, F.nz}, hi[3] = {-1, -1, -1};
    for (int t = t0; t < t1; ++t) {
        bool hit[4];
        int idx[4];
        const int c = cells_matching(src, range, F.nx, F.ny, t * CMP_CELLS + threadIdx.x * 4, want, hit, idx);
        int total;
        int pos = base + block_exclusive_scan(c, lw, total);
#pragma unroll
        for (int s = 0; s < 4; ++s)
            if (hit[s]) {
                const int i = idx[s];
                list[pos++] = i;
                const int yz = i / F.nx, x = i - yz * F.nx, z = yz / F.ny, y = yz - z * F.ny;
                lo[0] = min(lo[0], x); lo[1] = min(lo[1], y); lo[2] = min(lo[2], z);
                hi[0] = max(hi[0], x); hi[1] = max(hi[1], y); hi[2] = max(hi[2], z);
            }
        base += total;
    }
    if (which == 0 && hi[0] >= 0) {
        for (int k = 0; k < 3; ++k) {
            atomicMin(&F.sc->bbox[k], lo[k]);
            atomicMax(&F.sc->bbox[3 + k], hi[k]);
        }
    }
}

// Static wall lists: bit 0 marks obstacle cells with a non-obstacle D3Q19
// neighbour, bit 1 non-obstacle cells with an obstacle D3Q19 neighbour.
__global__ __launch_bounds__(256) void k_mark_wall_cells(const uint8_t *flags, uint8_t *out, int nx, int ny,
                                                         int nz, int N)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= N) return;
    const bool obst = flags[i] & FL_OBST;
    const Nbr nb(i, nx, ny, nz);
    bool other = false;
#pragma unroll
    for (int q = 1; q < NQ; ++q) other |= ((flags[nb.at(dir_x(q), dir_y(q), dir_z(q))] & FL_OBST) != 0) != obst;
    out[i] = other ? (obst ? 1 : 2) : 0;
}

// ------------------------------------------------ obstacle fill (Sec. II.A)
// phi(x_o) = sum |nw.c^_q| phi(x_o + c_q) / sum |nw.c^_q| over fluid
// neighbours with aperture |nw.c^_q| > sqrt(2)/2 (strict; the 45-degree
// links are excluded), nw the normalised sum of the directions from x_o to
// its non-obstacle neighbours.
// The 18 types of a cell come in together, then the 18 fill levels of a cell
// with a fluid neighbour (away from the liquid most have none). FROM_M: the
// interface cells' fill levels are computed from m and rho, with
// k_conv_gather's division, so that the fill does not wait for that kernel;
// only for steps in which no cell converts. Thread t of nt.
template <class P, bool FROM_M>
__device__ inline void obstacle_fill(const Fields<P> &F, int t, int nt)
{
    using R = typename P::R;
    const int n = F.sc->ocount;
    const double alpha = 0.70710678118654752440 + 1e-12;
    for (int k = t; k < n; k += nt) {
        const int i = F.olist[k];
        const Nbr nb(i, F.nx, F.ny, F.nz);
        uint8_t fl[NQ];
#pragma unroll
        for (int q = 1; q < NQ; ++q) fl[q] = F.flags[nb.at(dir_x(q), dir_y(q), dir_z(q))];
        int sx = 0, sy = 0, sz = 0;
        bool fluid = false;
#pragma unroll
        for (int q = 1; q < NQ; ++q) {
            fluid |= (fl[q] & FL_FLUID) != 0;
            if (!(fl[q] & FL_OBST)) {
                sx += dir_x(q); sy += dir_y(q); sz += dir_z(q);
            }
        }
        double num = 0, den = 0;
        if (fluid && (sx | sy | sz) != 0) {
            R ph[NQ], m[NQ], rho[NQ];
#pragma unroll
            for (int q = 1; q < NQ; ++q) {
                const int j = nb.at(dir_x(q), dir_y(q), dir_z(q));
                ph[q] = F.phi[j];
                if constexpr (FROM_M) {
                    m[q] = F.m[j];
                    rho[q] = F.rho[j];
                }
            }
            const double len = sqrt(double(sx * sx + sy * sy + sz * sz));
            const double wx = sx / len, wy = sy / len, wz = sz / len;
#pragma unroll
            for (int q = 1; q < NQ; ++q) {
                if (!(fl[q] & FL_FLUID)) continue;
                const double cl = sqrt(double(dir_len2(q)));
                const double w = fabs((wx * dir_x(q) + wy * dir_y(q) + wz * dir_z(q)) / cl);
                if (w > alpha) {
                    if constexpr (FROM_M)
                        if (fl[q] & FL_IF) ph[q] = m[q] / rho[q];
                    num += w * double(ph[q]);
                    den += w;
                }
            }
        }
        F.phi[i] = R(den > 0 ? num / den : 0.0);
        if (F.snap) F.snap[(size_t)SNAP * F.sc->icount + k] = R(den > 0 ? num / den : 0.0);
    }
}
template <class P>
__global__ __launch_bounds__(256) void k_obstacle_fill(const Batch<P> B)
{
    obstacle_fill<P, false>(B.f[blockIdx.y], blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

// phi = m / rho (blocks before ng) and the obstacle fill (the others, none
// without walls) of a step with frozen cell types in one launch: 5.0 us on
// the 128^3 sessile drop, 4.7 + 5.3 in two.
template <class P>
__global__ __launch_bounds__(LIST_NT) void k_gather_walls(const Batch<P> B, int ng)
{
    const int b = blockIdx.x;
    if (b < ng) conv_gather<P, LIST_NT>(B.f[blockIdx.y], true, b, ng);
    else obstacle_fill<P, true>(B.f[blockIdx.y], (b - ng) * LIST_NT + threadIdx.x, ((int)gridDim.x - ng) * LIST_NT);
}

// ------------------------------------------------ bubble model (Sec. III.A.1)
// The whole gas of a lattice is one bubble with isothermal pressure,
// p_g(t) V(t) = p_g(0) V(0), so rho_gas(t) = rho_gas V0 / V(t) with the gas
// volume V = (non-obstacle cells) - (liquid cells + sum of phi over
// interface cells). The liquid volume is summed over the fluid box in a
// fixed partition (VOL_CHUNKS chunks, fixed order within each), after the
// step's conversions.
// Four chunks to a block, and the block that finishes last adds the chunk
// sums and sets rho_gas(t): no launch of its own. The obstacle fill (blocks
// before `nw`) reads other cells than it writes and none of the sum's, so the
// two share a launch. Per launch 10.0 us on the 96^3 bubble between walls
// (FP64), where fill, chunk sums and final sum took 4.9 + 5.7 + 4.1 in three
// (48^3: 8.0; 9.4 with a barrier at each level of the two trees).
constexpr int VOL_CHUNKS = 1024;
constexpr int VOL_NT = 1024;                       // threads per block, 256 to a chunk
constexpr int VOL_GRID = VOL_CHUNKS / (VOL_NT / 256);

template <class P>
__global__ __launch_bounds__(VOL_NT) void k_bubble_walls(const Batch<P> B, int nw)
{
    const Fields<P> &F = B.f[blockIdx.y];
    if ((int)blockIdx.x < nw) {  // 256 cells to a block: the loads of a wavefront per SIMD
        if (threadIdx.x < 256) obstacle_fill<P, false>(F, blockIdx.x * 256 + threadIdx.x, nw * 256);
        return;
    }
    const Params &prm = B.p[blockIdx.y];
    if (!prm.bubble) return;
    __shared__ double s[VOL_NT];
    __shared__ int last;
    // one barrier, then the first wavefront of the values adds them in the
    // order of a halving tree (w = n / 2, ..., 1: s[t] += s[t + w])
    auto wave_tree = [](double v) {
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) v += __shfl_down(v, w, 64);
        return v;
    };
    const int t = threadIdx.x & 255, c = ((int)blockIdx.x - nw) * (VOL_NT / 256) + (int)(threadIdx.x >> 8);
    const CellRange box = CellRange::from(F.sc->fbox);
    const int n = box.size();
    const int chunk = (n + VOL_CHUNKS - 1) / VOL_CHUNKS;
    const int b0 = min(n, c * chunk), b1 = min(n, b0 + chunk);
    double acc = 0.0;
    for (int k = b0 + t; k < b1; k += 256) {
        const int i = box.cell(k, F.nx, F.ny);
        const uint8_t fl = F.flags[i];
        if (fl & FL_LIQ) acc += 1.0;
        else if (fl & FL_IF) acc += double(F.phi[i]);
    }
    s[threadIdx.x] = acc;
    __syncthreads();
    if (t < 64) {
        const double *v = s + threadIdx.x;
        acc = wave_tree((v[0] + v[128]) + (v[64] + v[192]));
    }
    // the chunk sums go by atomic exchanges, which have taken effect for the
    // whole device when they return: no fence, which would write the L2 back
    // in each of the 256 blocks (12 us)
    auto *part = reinterpret_cast<unsigned long long *>(F.part);
    if (t == 0) {
        const unsigned long long was = atomicExch(&part[c], (unsigned long long)__double_as_longlong(acc));
        asm volatile("" ::"v"(was));  // waits for the return
    }
    __syncthreads();
    if (threadIdx.x == 0) last = atomicInc(&F.sc->vdone, unsigned(VOL_GRID - 1)) == unsigned(VOL_GRID - 1);
    __syncthreads();
    if (!last) return;
    s[threadIdx.x] = __longlong_as_double((long long)atomicOr(&part[threadIdx.x], 0ull));
    __syncthreads();
    if (threadIdx.x >= 64) return;
    double e[VOL_NT / 64];
#pragma unroll
    for (int k = 0; k < VOL_NT / 64; ++k) e[k] = s[threadIdx.x + 64 * k];
#pragma unroll
    for (int h = VOL_NT / 128; h > 0; h >>= 1)
#pragma unroll
        for (int k = 0; k < h; ++k) e[k] += e[k + h];
    const double sum = wave_tree(e[0]);
    if (threadIdx.x == 0) {
        const double v = prm.n_free - sum;
        if (F.sc->bubble_init) {
            F.sc->gas_v0 = v;
            F.sc->bubble_init = 0;
        }
        F.sc->rho_gas_t = v > 0.0 ? prm.rho_gas * F.sc->gas_v0 / v : prm.rho_gas;
    }
}

}  // namespace fslbm
