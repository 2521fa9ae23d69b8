"""The launches over the interface list follow the layer as it grows: by a
loaded state, and by stepping with read-outs. The form changes, the results
do not."""
import numpy as np
import pytest

from paper_1509_07691_amd import inputs as I

pytestmark = pytest.mark.gpu

BLOCK_CELLS = 1024  # bound of the one-block form


@pytest.fixture(scope="module")
def fs():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1509_07691_amd import fslbm

    return fslbm


def fields(lat):
    return {"flags": lat.flags(), "fill": lat.fill(), "pressure": lat.pressure(), "velocity": lat.velocity(),
            "curvature": lat.curvature(), "ilist": lat.interface_list()}


def conversion_ms(fs, lats, steps):
    """Device time per step of the conversion phase of each lattice; the
    least of five runs, the lattices in turn."""
    best = [float("inf")] * len(lats)
    for _ in range(5):
        for k, lat in enumerate(lats):
            fs.fslbm_set_option(lat.handle, fs.FSLBM_OPT_TIMING, 1)
            fs.fslbm_reset_timing(lat.handle)
            lat.step(steps)
            ms, n = fs.fslbm_read_timing(lat.handle)
            fs.fslbm_set_option(lat.handle, fs.FSLBM_OPT_TIMING, 0)
            assert n == steps
            best[k] = min(best[k], ms[2] / steps)
    return best


def test_loaded_layer_sizes_the_launches(fs):
    """A lattice created with a small drop that loads a state of some 24,000
    interface cells converts as fast as the lattice that saved it: the same
    launches, so the times differ by noise (a fifth, with launches of some
    10 us). Bar: a factor of 2; one block for all these cells takes 18 times
    as long."""
    kw = dict(precision="f32", curv_model="lsqr", sigma=1e-3, tau=0.8)
    big = fs.Lattice(I.droplet(96, 36.0, noise=1e-6, seed=1)[0], None, **kw)
    small = fs.Lattice(I.droplet(96, 6.0, noise=1e-6, seed=2)[0], None, **kw)
    assert small.interface_list().size <= BLOCK_CELLS and big.interface_list().size > 20 * BLOCK_CELLS
    u = np.zeros((3, 96, 96, 96))
    u[0] = 0.03
    big.set_equilibrium(1.0, u)
    big.step(10)
    start = big.save_state()
    small.load_state(start)
    want, got = conversion_ms(fs, [big, small], 20)
    print(f"conversion {want * 1e3:.1f} us a step where it was created, {got * 1e3:.1f} us where it was loaded")
    a, b = fields(big), fields(small)
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    assert got <= 2.0 * want
    big.close()
    small.close()


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("precision,model", [("f64", "fd"), ("f32", "lsqr")])
def test_growing_layer_changes_the_form(fs, precision, model, graph):
    """A drop in a straining flow flattens across the bound of the one-block
    form. One lattice is read every 20 steps, so its launches follow the
    count; the other is read at the end alone and keeps its form: same bits."""
    import torch

    shape = (28, 44, 44)
    fill = I.perturb_interface(I.sphere_fraction(shape, (22.0, 22.0, 14.0), 7.6), 1e-6, 3)
    z, y, x = np.meshgrid(*[np.arange(n) + 0.5 - n / 2 for n in shape], indexing="ij")
    u = np.clip(0.006 * np.stack([x, y, -2 * z]), -0.1, 0.1) * (fill > 0)
    stream = torch.cuda.Stream() if graph else None
    pair = [fs.Lattice(fill, None, precision=precision, curv_model=model, sigma=1e-4, tau=0.6, stream=stream)
            for _ in range(2)]
    for lat in pair:
        fs.fslbm_set_option(lat.handle, fs.FSLBM_OPT_GRAPH, int(graph))
        lat.set_equilibrium(1.0, u)
    counts = [pair[0].interface_list().size]
    for _ in range(8):
        pair[0].step(20)
        counts.append(pair[0].interface_list().size)
    pair[1].step(160)
    assert counts[0] <= BLOCK_CELLS < 1.25 * counts[0] < counts[-1], counts
    a, b = [fields(lat) for lat in pair]
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    for lat in pair:
        lat.close()
