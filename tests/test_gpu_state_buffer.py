"""The bytes of a saved state follow from the lattice alone: they do not depend
on what the buffer held before, on its alignment or on whether the lattice
got the state by stepping or by a load, and a load takes a buffer of any
alignment. A drop whose fluid box covers part of the lattice; extents whose
regions are not multiples of 256 bytes.
"""
import math

import numpy as np
import pytest

from paper_1509_07691_amd import inputs as I

pytestmark = pytest.mark.gpu

FORMS = [("f64", "lsqr"), ("f32", "fd"), ("f16", "lsqr"), ("bf16", "fd")]


@pytest.fixture(scope="module")
def fs():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_1509_07691_amd import fslbm

    return fslbm


def make(fs, precision, model, radius=6.0, seed=1):
    fill, obst = I.sessile_droplet(27, 25, 15, radius, noise=1e-6, seed=seed)
    return fs.Lattice(fill, obst, precision=precision, curv_model=model, sigma=2e-3, tau=0.8,
                      theta=math.radians(60.0))


def save(fs, lat, byte, offset=0):
    """The saved state as a device tensor that starts `offset` bytes into a
    buffer prefilled with `byte`; the bytes beside it must stay."""
    import torch

    n = fs.fslbm_state_bytes(lat.handle)
    buf = torch.full((n + 64,), byte, dtype=torch.uint8, device=lat.device)
    assert buf.data_ptr() % 256 == 0
    fs.fslbm_save_state(lat.handle, buf.data_ptr() + offset, n)
    assert bool((buf[:offset] == byte).all()) and bool((buf[offset + n:] == byte).all())
    return buf[offset:offset + n]


def fields(lat):
    return {"flags": lat.flags(), "fill": lat.fill(), "pressure": lat.pressure(), "velocity": lat.velocity(),
            "curvature": lat.curvature(), "ilist": lat.interface_list()}


@pytest.mark.parametrize("precision,model", FORMS)
def test_saved_bytes_follow_from_the_state(fs, precision, model):
    lat = make(fs, precision, model)
    lat.step(10)
    a, b = save(fs, lat, 0xA5), save(fs, lat, 0x5A)
    assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())
    # one more step and back: a save after a load is the loaded buffer
    lat.step(1)
    lat.load_state(a)
    assert np.array_equal(save(fs, lat, 0x33).cpu().numpy(), a.cpu().numpy())
    # also in a lattice that held another drop
    other = make(fs, precision, model, radius=4.0, seed=3)
    other.step(4)
    other.load_state(a)
    assert np.array_equal(save(fs, other, 0x77).cpu().numpy(), a.cpu().numpy())
    lat.close()
    other.close()


@pytest.mark.parametrize("offset", [1, 2, 8, 16])
@pytest.mark.parametrize("precision,model", FORMS)
def test_buffer_alignment(fs, precision, model, offset):
    lat = make(fs, precision, model)
    lat.step(10)
    plain = save(fs, lat, 0xA5)
    odd = save(fs, lat, 0x5A, offset)
    assert np.array_equal(plain.cpu().numpy(), odd.cpu().numpy())
    again = save(fs, lat, 0xA5)
    assert np.array_equal(plain.cpu().numpy(), again.cpu().numpy())
    lat.step(15)
    want = fields(lat)
    for buf in (plain, odd):
        lat.load_state(buf)
        lat.step(15)
        got = fields(lat)
        for k in want:
            assert np.array_equal(got[k], want[k]), k
    lat.close()


@pytest.mark.parametrize("precision,model", FORMS)
def test_buffer_in_pinned_host_memory(fs, precision, model):
    """A buffer outside the lattice's device memory (pinned host memory here,
    another device's elsewhere) goes by copies of the runtime: the same
    bytes, and a load from it continues the run."""
    import torch

    lat = make(fs, precision, model)
    lat.step(10)
    ref = save(fs, lat, 0xA5).cpu().numpy()
    buf = torch.empty(ref.size, dtype=torch.uint8, pin_memory=True)
    buf.fill_(0x5A)
    fs.fslbm_save_state(lat.handle, buf.data_ptr(), ref.size)
    assert np.array_equal(buf.numpy(), ref)
    lat.step(15)
    want = fields(lat)
    fs.fslbm_load_state(lat.handle, buf.data_ptr(), ref.size)
    lat.step(15)
    got = fields(lat)
    for k in want:
        assert np.array_equal(got[k], want[k]), k
    lat.close()
