"""The one-block conversion chain of small interface layers and the launches
that share the obstacle fill, HIP path against the FP64 oracle: layers within
one round of the block, just below its bound and above it (the launches of
larger layers), two lattices a launch, walls with and without the bubble
model.

Bars as in test_gpu_edge_cases.py: cell types and interface lists exact,
fields within 1e-10 relative (FP64).
"""
import numpy as np
import pytest

import oracle as O
from paper_1509_07691_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fslbm():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1509_07691_amd import fslbm as mod

    return mod


def body(radius, gas, walls):
    n = int(2 * radius) + 9
    shape = (n + 2, n + 1, n)
    c = (n / 2 + 0.3, n / 2 + 0.4, n / 2 + 0.2)
    fill = np.clip(I.sphere_fraction(shape, c, radius), 0.0, 1.0)
    fill = I.perturb_interface(1.0 - fill if gas else fill, 1e-6, 4)
    u = np.zeros((3,) + shape)
    u[0], u[1] = 0.09, -0.06
    obst = None
    if walls:
        obst = np.zeros(shape, np.uint8)
        obst[0] = obst[-1] = 1
        fill[obst != 0] = 0.0
        u[:, obst != 0] = 0.0
    return fill, obst, u


# radius 4: about 300 layer cells; 7.4 and 8.4: just below and above 1024; two
# of radius 27: more than 16384, the bound of the blocks of one wavefront
@pytest.mark.parametrize("radius,below,gas,walls,bubble", [
    (r, r < 8, *k) for r in (4.0, 7.4, 8.4)
    for k in ((False, False, False), (True, True, True), (True, True, False), (True, False, True))
] + [(27.0, False, False, False, False)])
def test_small_layers_against_oracle(fslbm, radius, below, gas, walls, bubble):
    fill, obst, u = body(radius, gas, walls)
    model = dict(sigma=1e-3, tau=0.8)
    pair = [fslbm.Lattice(fill, obst, precision="f64", curv_model=c, bubble=bubble, **model) for c in ("lsqr", "fd")]
    ref = [O.Oracle(fill, obst, curv_model=c, bubble=bubble, **model) for c in (O.CURV_LSQR, O.CURV_FD)]
    for g, o in zip(pair, ref):
        g.set_equilibrium(1.0, u)
        o.set_equilibrium(np.ones(fill.shape), u)
        assert (g.interface_list().size <= 1024) == below
    batch = fslbm.Batch(pair)
    changed = 0
    for _ in range(5):
        before = ref[0].flags()
        batch.step(3)
        for g, o in zip(pair, ref):
            o.step(3)
            now = o.flags()
            assert np.array_equal(g.flags(), now)
            assert np.array_equal(g.interface_list(), o.interface_list())
            fluid = (now == O.LIQUID) | (now == O.INTERFACE)
            for a, b in ((g.fill(), o.fill()), (g.pressure(), o.pressure()), (g.velocity(), o.velocity())):
                assert np.linalg.norm((a - b)[..., fluid]) < 1e-10 * np.linalg.norm(b[..., fluid])
        changed += int((ref[0].flags() != before).sum())
    assert changed > 20
    if radius > 20:
        assert sum(g.interface_list().size for g in pair) > 16384
    for g in pair:
        g.close()
