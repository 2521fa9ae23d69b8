"""Gradients of a frozen window where the wall lies across a periodic
boundary: one sessile drop on two obstacle layers, rolled along the wall's
axis so that the interface box starts at the first plane (the wall is then
at the last two), at the second plane, in the middle, or spans the boundary;
the wall normal to z or to x. The window knows nothing of the position, so
the gradients are those of the first position, and each agrees with the
oracle's tangent-linear build.

Bar 1e-9 relative, as the other comparisons with the tangent-linear build:
both sides are derivatives of the same FP64 map, 24 steps long, and differ
in the order of their sums.
"""
import math

import numpy as np
import pytest

import oracle as O
from paper_1509_07691_amd import inputs as I

pytestmark = pytest.mark.gpu

T_STEPS, K_CK = 24, 5
MODELS = {"fd": O.CURV_FD, "lsqr": O.CURV_LSQR}
PRM = dict(sigma=5e-3, tau=0.8, theta=math.radians(70.0))
# shift of the drop along the wall's axis (16 planes, wall at the first two)
SHIFTS = {"middle": 3, "starts at plane 0": -2, "starts at plane 1": -1, "spans the boundary": 11}


@pytest.fixture(scope="module")
def Lattice():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1509_07691_amd.fslbm import Lattice as L

    return L


def problem(axis, shift):
    """(fill, obstacle, target, seed field) of the drop rolled by shift."""
    shape = (16, 21, 22)
    fill = I.sphere_fraction(shape, (11.0, 10.5, 2.0), 6.0)
    obst = np.zeros(shape, dtype=np.uint8)
    obst[:2] = 1
    fill[:2] = 0.0
    fill = I.perturb_interface(fill, 1e-6, 5)
    rng = np.random.default_rng(11)
    target = rng.uniform(0.0, 1.0, shape)
    v = rng.uniform(-1.0, 1.0, shape) * ((fill > 1e-3) & (fill < 1 - 1e-3))
    turn = (lambda a: a) if axis == "z" else (lambda a: np.moveaxis(a, 0, 2))
    return [np.ascontiguousarray(turn(np.roll(a, shift, axis=0))) for a in (fill, obst, target, v)]


def gradients(Lattice, model, axis, shift):
    fill, obst, target, v = problem(axis, shift)
    g = Lattice(fill, obst, precision="f64", curv_model=model, **PRM)
    g.adjoint_forward(T_STEPS, K_CK)
    seed = 2.0 * (g.fill() - target) * (obst == 0)
    d0, ds, dt = g.adjoint_backward(seed)
    ifc = np.argwhere(g.flags() == 2)
    g.close()
    a = 0 if axis == "z" else 2
    return d0.cpu().numpy(), ds, dt, (ifc[:, a].min(), ifc[:, a].max())


@pytest.mark.parametrize("where", list(SHIFTS))
@pytest.mark.parametrize("axis", ["z", "x"])
@pytest.mark.parametrize("model", ["lsqr", "fd"])
def test_gradients_do_not_depend_on_the_boundary(Lattice, model, axis, where):
    shift = SHIFTS[where]
    fill, obst, target, v = problem(axis, shift)
    d0, ds, dt, span = gradients(Lattice, model, axis, shift)
    assert span == {"middle": (5, 10), "starts at plane 0": (0, 5), "starts at plane 1": (1, 6),
                    "spans the boundary": (0, 15)}[where]

    def dL(**seed):
        t = O.TangentLinear(fill, obst, curv_model=MODELS[model], **PRM, **seed)
        t.step(T_STEPS)
        val, der = t.fill_and_derivative()
        return float((2.0 * (val - target) * (obst == 0) * der).sum())

    pairs = {"sigma": (ds, dL(dsigma=1.0)), "theta": (dt, dL(dtheta=1.0)),
             "fill": (float((d0 * v).sum()), dL(fill_dot=v))}
    print(model, axis, where, {k: f"{a:.12e} tl {b:.12e}" for k, (a, b) in pairs.items()})
    for k, (a, b) in pairs.items():
        assert abs(a - b) <= 1e-9 * abs(b), f"{k}: adjoint {a} vs tangent-linear {b}"
    # cell by cell against the drop away from the boundary
    ref = gradients(Lattice, model, axis, SHIFTS["middle"])[0]
    ref = np.roll(ref, shift - SHIFTS["middle"], axis=0 if axis == "z" else 2)
    assert np.abs(d0 - ref).max() <= 1e-9 * np.abs(ref).max()
