"""The two forms of the tiled FD curvature (few tiles: 512 threads and columns
of cells; many tiles: 256 threads) give the same bits: lattices stepped alone
are under the line between them, the same lattices in one batch over it.
Against the oracle both are covered by the parity tests.
"""
import math

import numpy as np
import pytest

from paper_1509_07691_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fs():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1509_07691_amd import fslbm

    return fslbm


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_few_and_many_tiles(fs, precision):
    lats = []
    for k in range(3):  # a drop on a wall, a droplet over a periodic boundary, a droplet at the centre
        if k == 0:
            fill, obst = I.sessile_droplet(75, 71, 40, 33.0, noise=1e-6, seed=3)
        else:
            fill, obst = I.droplet(77, 28.0, noise=1e-6, seed=k), None
            fill = np.roll(fill[0], 31 * (2 - k), axis=(0, 1, 2))
        kw = dict(precision=precision, curv_model="fd", sigma=1e-3, tau=0.8, theta=math.radians(70.0))
        lats.append([fs.Lattice(fill, obst, **kw) for _ in range(2)])
    counts = [a.interface_list().size for a, _ in lats]
    assert max(counts) < 512 * 64 < sum(counts)
    batch = fs.Batch([b for _, b in lats])
    for n in (1, 9):
        batch.step(n)
        for a, b in lats:
            a.step(n)
            for name in ("flags", "fill", "curvature", "normal", "velocity"):
                assert np.array_equal(getattr(a, name)(), getattr(b, name)()), name
    batch.close()
    for a, b in lats:
        a.close()
        b.close()
