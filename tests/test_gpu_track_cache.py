"""The tracking block cache (per level and tile, in the map's arena) never
changes a result: tracking with warm caches, after a reset, and after new
blocks were allocated (absent-block entries of an older allocation epoch)
gives bit for bit what a fresh map gives."""
import numpy as np
import pytest
import torch

import synth
from gpu_helpers import gpu_frame, map_params, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rf():
    return need_gpu()


def build(rf, m, seq, frames):
    for k in frames:
        P = torch.as_tensor(seq.poses[k]).cuda().contiguous()
        f = gpu_frame(rf, seq, k)
        m.allocate(f, P)
        m.integrate(f, P)


def track(rf, m, seq, k, start):
    P = torch.as_tensor(seq.poses[start]).cuda().contiguous()
    stats = torch.zeros(16, dtype=torch.float64, device="cuda")
    m.track(gpu_frame(rf, seq, k), P, rf.TrackParams(3, 6), stats=stats)
    torch.cuda.synchronize()
    return P.cpu().numpy(), stats.cpu().numpy()


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
def test_block_cache_never_changes_results(rf, storage):
    seq = synth.static_room(n_frames=9, width=320, height=240)
    mp = map_params(rf, seq, storage=storage, max_blocks=1 << 16)
    warm = rf.Map(mp)
    build(rf, warm, seq, range(6))
    cold_pose, cold_stats = track(rf, warm, seq, 6, 5)      # first call: caches fill level by level
    for _ in range(2):                                      # warm caches
        p, st = track(rf, warm, seq, 6, 5)
        assert np.array_equal(p, cold_pose) and np.array_equal(st, cold_stats)
    fresh = rf.Map(mp)
    build(rf, fresh, seq, range(6))
    p, st = track(rf, fresh, seq, 6, 5)
    assert np.array_equal(p, cold_pose) and np.array_equal(st, cold_stats)
    # new blocks: the absent-block entries the caches hold are of an older epoch
    build(rf, warm, seq, [6])
    build(rf, fresh, seq, [6])
    other = rf.Map(mp)
    build(rf, other, seq, range(7))
    a = track(rf, warm, seq, 7, 6)
    b = track(rf, fresh, seq, 7, 6)
    c = track(rf, other, seq, 7, 6)
    for x, y, z in zip(a, b, c):
        assert np.array_equal(x, z) and np.array_equal(y, z)
    # a reset clears the caches (slots of the rebuilt map differ)
    warm.L.hashmap_reset(warm.h, None)
    build(rf, warm, seq, range(3, 7))
    ref = rf.Map(mp)
    build(rf, ref, seq, range(3, 7))
    for x, y in zip(track(rf, warm, seq, 7, 6), track(rf, ref, seq, 7, 6)):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("voxel,tau,adaptive", [(0.004, 0.02, False), (0.01, 0.03, True), (0.02, 0.06, False)])
def test_block_cache_over_jumping_frames(rf, voxel, tau, adaptive):
    """Tiles with more blocks than a cache entry holds and blocks outside its
    window (depth steps at small voxels), pairs kept over several launches,
    and frames from poses far apart in turn: a warm map's registrations equal
    those of a map that has tracked nothing before."""
    seq = synth.static_room(n_frames=61, width=320, height=240)
    mp = map_params(rf, seq, max_blocks=1 << 18)
    mp.voxel_size, mp.truncation = voxel, tau
    warm = rf.Map(mp)
    build(rf, warm, seq, (0, 30, 60))
    tp = rf.TrackParams(4, 5, adaptive=adaptive)

    def run(m, k, start):
        P = torch.as_tensor(seq.poses[start]).cuda().contiguous()
        m.track(gpu_frame(rf, seq, k), P, tp)
        out = m.normal_equations(gpu_frame(rf, seq, k), P, level=0)
        return P.cpu().numpy(), out.cpu().numpy()

    for k, start in ((30, 31), (60, 59), (0, 1), (60, 58), (30, 29)):
        a = run(warm, k, start)
        fresh = rf.Map(mp)
        build(rf, fresh, seq, (0, 30, 60))
        b = run(fresh, k, start)
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
        assert a[1][28] > 1000


@pytest.mark.parametrize("free_blocks", [False, True])
@pytest.mark.parametrize("width,height", [(320, 240), (77, 53)])
def test_residual_with_and_without_cached_pairs(rf, width, height, free_blocks):
    """The mask's residual on a map that has not tracked (tiles look up the
    hash table) and on one that has (through the tile cache) is the same."""
    seq = synth.static_room(n_frames=5, width=width, height=height)
    mp = map_params(rf, seq, max_blocks=1 << 16)
    mp.free_blocks = free_blocks
    res = []
    for tracked in (False, True):
        m = rf.Map(mp)
        build(rf, m, seq, range(3))
        if tracked:
            track(rf, m, seq, 4, 2)
        out = torch.empty((height, width), dtype=torch.float32, device="cuda")
        P = torch.as_tensor(seq.poses[4]).cuda().contiguous()
        m.dynamic_mask(gpu_frame(rf, seq, 4), P, rf.MaskParams(), residual=out)
        res.append(out.cpu().numpy())
    assert (res[0] >= 0).sum() > res[0].size // 4
    assert np.array_equal(res[0], res[1])
