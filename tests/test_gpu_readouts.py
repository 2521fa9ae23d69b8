"""Read-outs on extents around the sizes their kernels work in (64 cells per
bit word, 16 flags per load, 1024 cells per block), and on device buffers of
any alignment. The references are plain numpy on the library's own fields.

n_inner and the interface list are whole numbers and must be equal. dp is
(mean density - rho_gas) / 3 with densities near 1 summed over at most 1e5
cells: two orders of summation differ by less than 1e5 ulp of 1, 2.3e-11,
and dp by a third of it; the bar is 1e-11.
"""
import numpy as np
import pytest

from paper_1509_07691_amd import inputs as I

pytestmark = pytest.mark.gpu

SHAPES = [(14, 12, 3), (12, 9, 5), (9, 11, 63), (10, 9, 64), (9, 10, 65), (11, 9, 66), (8, 12, 130), (31, 33, 35)]


@pytest.fixture(scope="module")
def fs():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1509_07691_amd import fslbm

    return fslbm


def layered(shape):
    """A liquid slab with a tilted, periodic surface, rolled so that it
    crosses the x and z boundaries."""
    nz, ny, nx = shape
    z = np.arange(nz)[:, None, None]
    h = 0.7 * nz + 0.3 + 0.1 * np.sin(2 * np.pi * np.arange(nx) / nx)[None, None, :] \
        + 0.1 * np.cos(2 * np.pi * np.arange(ny) / ny)[None, :, None]
    fill = np.clip(h - z, 0.0, 1.0)
    fill[0] = 0.5
    return np.roll(fill, (nz // 3, 2, -1), axis=(0, 1, 2))


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("precision", ["f64", "f16"])
def test_readouts_against_numpy(fs, shape, precision):
    import torch

    lat = fs.Lattice(layered(shape), None, precision=precision, curv_model="lsqr", sigma=1e-3, tau=0.8)
    lat.step(3)
    flags = lat.flags()
    # the list, and the flags on an unaligned device buffer
    assert np.array_equal(lat.interface_list(), np.flatnonzero(flags == fs.FSLBM_INTERFACE))
    assert np.array_equal(fs.fslbm_read_interface_list_noalloc(lat.handle), np.flatnonzero(flags == fs.FSLBM_INTERFACE))
    buf = torch.full((lat.n + 32,), 9, dtype=torch.uint8, device="cuda:0")
    for at in (0, 1, 16):
        buf.fill_(9)
        fs.fslbm_read_flags(lat.handle, buf[at:at + lat.n], device=True)
        got = buf.cpu().numpy()
        assert np.array_equal(got[at:at + lat.n], flags.reshape(-1))
        assert (got[:at] == 9).all() and (got[at + lat.n:] == 9).all()
    # inner liquid cells: no gas or interface cell within a distance of sqrt(6)
    surf = (flags == fs.FSLBM_GAS) | (flags == fs.FSLBM_INTERFACE)
    near = np.zeros(shape, bool)
    r = range(-2, 3)
    for d in [(a, b, c) for a in r for b in r for c in r if a * a + b * b + c * c <= 6]:
        near |= np.roll(surf, d, axis=(0, 1, 2))
    inner = (flags == fs.FSLBM_LIQUID) & ~near
    d = lat.diagnostics()
    assert d["n_inner"] == inner.sum()
    if inner.any():
        assert abs(d["dp"] - (lat.pressure()[inner].mean() - 1.0 / 3.0)) < 1e-11
    # fields on the host and on the device, scalar and vector
    for name, comps in (("fill", 1), ("pressure", 1), ("curvature", 1), ("plic", 1), ("mass_field", 1),
                        ("velocity", 3), ("normal", 3)):
        host = getattr(lat, name)()
        dev = torch.full((comps * lat.n + 2,), np.nan, dtype=torch.float64, device="cuda:0")
        getattr(fs, "fslbm_read_" + name)(lat.handle, dev[1:-1], device=True)
        got = dev.cpu().numpy()
        assert np.array_equal(got[1:-1], host.reshape(-1)), name
        assert np.isnan(got[0]) and np.isnan(got[-1])
        if name in ("curvature", "normal", "plic", "mass_field"):
            assert not host[..., flags != fs.FSLBM_INTERFACE].any()
    assert np.abs(lat.normal()[:, flags == fs.FSLBM_INTERFACE]).sum() > 0
    lat.close()
