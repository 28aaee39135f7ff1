"""Stage outputs of the dynamic mask that share buffers: a shared buffer keeps
the last stage written to it (raw, eroded, filled, mask), and the mask itself
does not depend on who shares."""
import ctypes

import numpy as np
import pytest
import torch

import synth
from gpu_helpers import dev_pose, gpu_frame, map_params, need_gpu

pytestmark = pytest.mark.gpu
STAGES = ("raw", "eroded", "filled", "final")


@pytest.fixture(scope="module")
def scene():
    rf = need_gpu()
    seq = synth.dynamic_room(n_frames=13, width=160, height=120, n_clusters=2, movers="in_view")
    m = rf.Map(map_params(rf, seq))
    for k in range(0, 12, 3):
        mask = torch.from_numpy((seq.labels[k] > 0).astype(np.uint8)).cuda()
        m.allocate(gpu_frame(rf, seq, k), dev_pose(seq.poses[k]), mask)
        m.integrate(gpu_frame(rf, seq, k), dev_pose(seq.poses[k]), mask)
    g, P, mp = gpu_frame(rf, seq, 12), dev_pose(seq.poses[12]), rf.MaskParams()
    apart = {k: v.cpu().numpy() for k, v in m.dynamic_mask(g, P, mp, stages=True).items()}
    assert all(apart[k].any() for k in STAGES)
    assert all((apart[a] != apart[b]).any() for a in STAGES for b in STAGES if a < b)
    return rf, m, g, P, mp, apart


# a letter per stage: equal letters share a buffer, "-" is not asked for
@pytest.mark.parametrize("share", ["aabc", "abca", "-aba", "aaba", "aabb", "aaab", "aaaa", "abaa", "abbc", "abbb",
                                   "abab", "abac", "-aab", "-abb"])
def test_stages_that_share_buffers(scene, share):
    rf, m, g, P, mp, apart = scene
    shape = apart["raw"].shape
    bufs = {c: torch.full(shape, 9, dtype=torch.uint8, device="cuda") for c in share if c != "-"}
    ptr = [None if c == "-" else ctypes.c_void_p(bufs[c].data_ptr()) for c in share]
    c = mp.c()
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        rc = rf.lib().compute_dynamic_mask_stages(m.h, ctypes.byref(g.s), ctypes.c_void_p(P.data_ptr()),
                                                  ctypes.byref(c), *ptr, None, stream)
        assert rc == 0
        for letter, buf in bufs.items():
            last = STAGES[max(i for i, x in enumerate(share) if x == letter)]
            np.testing.assert_array_equal(buf.cpu().numpy(), apart[last])
