"""A reset map holds nothing of its former contents: rebuilt from other frames
it exports what a fresh map does, voxels that no frame observed included."""
import numpy as np
import pytest
import torch

import synth
from gpu_helpers import dev_pose, gpu_export_sorted, gpu_frame, map_params, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rf():
    return need_gpu()


def build(rf, m, seq, frames):
    for k in frames:
        m.allocate(gpu_frame(rf, seq, k), dev_pose(seq.poses[k]))
        m.integrate(gpu_frame(rf, seq, k), dev_pose(seq.poses[k]))


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("free_blocks", [False, True])
@pytest.mark.parametrize("before", ["frames", "full pool", "import", "reset"])
def test_reset_map_equals_a_fresh_one(rf, storage, free_blocks, before):
    seq = synth.static_room(n_frames=40, width=160, height=120)
    params = map_params(rf, seq, storage=storage, max_blocks=1 << 16)
    params.free_blocks = free_blocks
    params.carve_stride = 2 if free_blocks else params.carve_stride
    if before == "full pool":
        params.max_blocks = 200
    m = rf.Map(params)
    if before == "import":
        rng = np.random.default_rng(3)
        n = 300
        keys = rng.permutation(20 ** 3)[:n]
        keys = np.stack([keys % 20, keys // 20 % 20, keys // 400], 1).astype(np.int32)
        m.import_(*[torch.from_numpy(x).cuda() for x in (
            keys, rng.uniform(-0.01, 0.01, (n, 512)).astype(np.float32), np.ones((n, 512), np.float32),
            rng.integers(0, 256, (n, 512, 3)).astype(np.uint8))])
    else:
        build(rf, m, seq, (0, 39))
    full = m.status()[0] & rf.RF_FLAG_POOL_FULL
    assert bool(full) == (before == "full pool")
    for _ in range(2 if before == "reset" else 1):
        m.L.hashmap_reset(m.h, None)
    assert m.status()[:2] == (0, 0)
    build(rf, m, seq, (20,))
    params.max_blocks = 1 << 16
    fresh = rf.Map(params)
    build(rf, fresh, seq, (20,))
    a, b = gpu_export_sorted(m), gpu_export_sorted(fresh)
    if before == "full pool":  # which blocks got a slot is not fixed: each voxel is the fresh map's or unobserved
        at = {tuple(k): i for i, k in enumerate(b[0])}
        sel = [at[tuple(k)] for k in a[0]]
        b = [x[sel] for x in b]
    assert len(a[0]) > 100
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
