"""The frame's block list and the free blocks' export over hash sizes: a chunk
a workgroup, part of a wavefront's loads, several rounds of loads; sparse and
nearly full tables; room for fewer free blocks than there are."""
import ctypes

import numpy as np
import pytest
import torch

import oracle as O
from gpu_helpers import dev_pose, gpu_keyset, need_gpu, sort_keys

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rf():
    return need_gpu()


@pytest.mark.parametrize("free_blocks", [0, 1])
@pytest.mark.parametrize("bits", [9, 10, 14, 18, 22])
def test_lists_over_hash_sizes(rf, bits, free_blocks):
    W, H, s, tau = 48, 36, 0.02, 0.06
    intr = (40.0, 40.0, (W - 1) / 2, (H - 1) / 2)
    rng = np.random.default_rng(bits)
    params = rf.MapParams(s, tau, 5.0, 1 << bits, 1 << 12, 255, 1, "fp32", W * H)
    params.free_blocks = bool(free_blocks)
    m = rf.Map(params)
    o = O.OracleMap(s, tau, 5.0, 255, 1, real_bits=32, free_blocks=free_blocks)
    for k in range(3):
        # a tilted wall near enough for the smallest table (2^9 buckets)
        depth = (0.55 + 0.1 * k + 0.1 * np.linspace(0, 1, W)[None] + 0.005 * rng.uniform(size=(H, W))).astype(np.float32)
        rgb = rng.integers(0, 256, (H, W, 3)).astype(np.uint8)
        T = np.eye(4)
        g, f = rf.Frame.from_numpy(depth, rgb, *intr), O.Frame(depth, rgb, *intr)
        m.allocate(g, dev_pose(T))
        want = np.asarray(o.allocate(f, T)).reshape(-1, 3)
        assert np.array_equal(gpu_keyset(m.frame_blocks()), want[sort_keys(want)])
        m.integrate(g, dev_pose(T))
        o.integrate(f, T)
    assert m.status()[0] == 0
    if not free_blocks:
        return
    fk, fw = [t.cpu().numpy() for t in m.export_free()]
    ok, ow = o.export_free()
    i = sort_keys(fk)
    assert len(ok) > 20 and np.array_equal(fk[i], ok) and np.array_equal(fw[i], ow.astype(np.float32))
    cap = len(ok) // 2
    keys = torch.full((len(ok), 3), 1 << 30, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    st = m.L.hashmap_export_free(m.h, ctypes.c_void_p(keys.data_ptr()), None, cap, ctypes.c_void_p(cnt.data_ptr()), None)
    assert st == 0 and int(cnt.item()) == len(ok)
    part = keys.cpu().numpy()
    assert (part[cap:] == 1 << 30).all()
    assert {tuple(x) for x in part[:cap]} <= {tuple(x) for x in ok} and len({tuple(x) for x in part[:cap]}) == cap
