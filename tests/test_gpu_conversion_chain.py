"""Cell conversions in bulk, HIP path against the FP64 oracle (through the C
ABI): more converting cells per step than a wavefront, a block or the
smallest grid of the conversion kernels holds, on extents where the 7x7x7
neighbourhood of a converting cell wraps onto itself, and with the interface
list in either of its two buffers when the state is saved.

Bars as in test_gpu_edge_cases.py: cell types and interface lists exact,
fields within 1e-10 relative (FP64).
"""
import numpy as np
import pytest

import oracle as O
from paper_1509_07691_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Lattice():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1509_07691_amd.fslbm import Lattice as L

    return L


def body(name):
    """(fill, velocity) of a moving body."""
    if name == "thin":  # a cylinder, 3 cells along its axis
        shape = (3, 41, 45)
        fill = I.cylinder_fraction(shape, (22.0, 20.0), 12.0)
        u = (0.09, -0.05, 0.0)
    elif name == "narrow":  # 6 cells: the 7-cell box covers the axis and one cell twice
        shape = (6, 37, 33)
        fill = I.cylinder_fraction(shape, (16.0, 18.0), 11.0)
        u = (-0.06, 0.08, 0.0)
    else:  # hundreds of conversions a step
        shape = (70, 74, 67)
        fill = I.sphere_fraction(shape, (33.0, 37.0, 35.0), 25.0)
        u = (0.08, 0.06, -0.07)
    fill = I.perturb_interface(np.clip(fill, 0.0, 1.0), 1e-6, 4)
    vel = np.zeros((3,) + shape)
    vel[0], vel[1], vel[2] = u
    return fill, vel


@pytest.mark.parametrize("name,steps,least", [("thin", 24, 40), ("narrow", 24, 40), ("ball", 8, 1500)])
def test_conversions_against_oracle(Lattice, name, steps, least):
    fill, u = body(name)
    kw = dict(sigma=1e-3, tau=0.8)
    g = Lattice(fill, None, precision="f64", curv_model="lsqr", **kw)
    o = O.Oracle(fill, None, curv_model=O.CURV_LSQR, **kw)
    g.set_equilibrium(1.0, u)
    o.set_equilibrium(np.ones(fill.shape), u)
    changed, before = 0, o.flags()
    for _ in range(steps // 4):
        g.step(4)
        o.step(4)
        now = o.flags()
        changed += int((now != before).sum())
        before = now
        assert np.array_equal(g.flags(), now)
        assert np.array_equal(g.interface_list(), o.interface_list())
        fluid = (now == O.LIQUID) | (now == O.INTERFACE)
        for a, b in ((g.fill(), o.fill()), (g.pressure(), o.pressure()), (g.velocity(), o.velocity())):
            assert np.linalg.norm((a - b)[..., fluid]) < 1e-10 * np.linalg.norm(b[..., fluid])
    assert changed > least
    g.close()


@pytest.mark.parametrize("precision", ["f64", "bf16"])
def test_saved_state_of_every_step(Lattice, precision):
    """A run that is saved and loaded into another lattice after every step
    (the interface list changes buffer in each step that converts a cell)
    is the uninterrupted run, bit for bit."""
    fill, u = body("narrow")
    kw = dict(precision=precision, curv_model="lsqr", sigma=1e-3, tau=0.8)
    a, b, c = (Lattice(fill, None, **kw) for _ in range(3))
    for lat in (a, b, c):
        lat.set_equilibrium(1.0, u)
    for _ in range(10):
        a.step(1)
        b.step(1)
        c.load_state(b.save_state())
        b, c = c, b
        assert np.array_equal(a.flags(), b.flags())
        assert np.array_equal(a.interface_list(), b.interface_list())
        assert np.array_equal(a.fill(), b.fill()) and np.array_equal(a.velocity(), b.velocity())
    for lat in (a, b, c):
        lat.close()
