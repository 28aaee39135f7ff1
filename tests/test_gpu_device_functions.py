"""Device functions of the library in test kernels of their own
(tests/kernels)."""
import ctypes
import importlib.util
import os

import numpy as np
import pytest
import torch

from gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu
HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "kernels")


@pytest.fixture(scope="module")
def kernels():
    need_gpu()
    path = os.path.join(HERE, "libtest_kernels.so")
    if not os.path.exists(path):
        spec = importlib.util.spec_from_file_location("test_kernels_build", os.path.join(HERE, "build.py"))
        b = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(b)
        b.build()
    return ctypes.CDLL(path)


def stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def hash3(b):
    p = b.astype(np.uint32) * np.array([73856093, 19349669, 83492791], np.uint32)
    return p[:, 0] ^ p[:, 1] ^ p[:, 2]


@pytest.mark.parametrize("slots,nrefs,n", [(256, 64, 1), (256, 64, 15), (256, 128, 31), (512, 512, 64)])
def test_tile_cache_of_512_threads_keeps_its_pairs(kernels, slots, nrefs, n):
    """More threads than the finer levels' LDS hash has slots: the walk that
    writes the pairs back stays inside the hash, so the tile's pairs are those
    put in, no more, and again after a round through memory (n below a quarter
    of the room: unused pairs stay too)."""
    rng = np.random.default_rng(n)
    blocks, seen = [], set()
    while len(blocks) < n:                       # homes apart, so that every pair finds a place
        b = rng.integers(-6, 6, 3).astype(np.int32)
        h = int(hash3(b[None])[0] & np.uint32(slots - 1))
        if h not in seen:
            seen.add(h)
            blocks.append(b)
    blocks = np.array(blocks, np.int32)
    tab = torch.zeros((nrefs, 2), dtype=torch.int64, device="cuda")
    count = torch.zeros(1, dtype=torch.int32, device="cuda")
    dev = torch.from_numpy(blocks).cuda()
    for again in (0, 1):
        rc = kernels.tile_cache_round_trip(ctypes.c_void_p(tab.data_ptr()), ctypes.c_void_p(count.data_ptr()), nrefs,
                                           slots, ctypes.c_void_p(dev.data_ptr()), n, again, stream())
        assert rc == 0
        assert int(count.item()) == n
        t = tab.cpu().numpy()
        key = t[1:n + 1, 0]
        got = np.stack([((key >> s) & 0x1FFFFF) - (1 << 20) for s in (0, 21, 42)], 1)
        slot = (t[1:n + 1, 1] & 0xFFFFFFFF).astype(np.int64)
        assert sorted(map(tuple, np.c_[got, slot])) == sorted(map(tuple, np.c_[blocks, np.arange(n)]))
        assert (t[n + 1:] == 0).all()            # nothing past them


def test_reciprocal_of_every_float(kernels):
    """rcp_rn, on which the integration's bit-exactness rests: the IEEE 1 / x for
    all 2^32 bit patterns (any NaN for a NaN)."""
    bad = torch.zeros(1, dtype=torch.int64, device="cuda")
    assert kernels.check_rcp_f32(ctypes.c_void_p(bad.data_ptr()), stream()) == 0
    assert int(bad.item()) == 0


@pytest.mark.parametrize("e0,ne", [(-100, 200), (-1000, 2000)])
def test_reciprocal_of_doubles(kernels, e0, ne):
    """rcp_f64, the solve's reciprocal pivots: the division for 2^32 random
    values, over the magnitudes of pivots and over nearly all normal ones."""
    bad = torch.zeros(1, dtype=torch.int64, device="cuda")
    assert kernels.check_rcp_f64(e0, ne, ctypes.c_void_p(bad.data_ptr()), stream()) == 0
    assert int(bad.item()) == 0


def test_reciprocal_of_special_doubles(kernels):
    x = np.array([0.0, -0.0, np.inf, -np.inf, np.nan, 1.0, -3.0, 2.0 ** -1000, 2.0 ** 1000])
    with np.errstate(divide="ignore"):
        want = 1.0 / x
    dx = torch.from_numpy(x).cuda()
    dy = torch.zeros_like(dx)
    rc = kernels.rcp_f64_values(ctypes.c_void_p(dx.data_ptr()), ctypes.c_void_p(dy.data_ptr()), len(x), stream())
    assert rc == 0
    y = dy.cpu().numpy()
    np.testing.assert_array_equal(y, want)
    assert (np.signbit(y) == np.signbit(want))[~np.isnan(x)].all()
