"""Virtual depth (raycast_depth, Sec. III-E) through the C ABI against the
oracle: bit-exact against the FP32 mirror on analytic maps and on a fused
map, close to the FP64 reference; the fill mode keeps valid depths; the
VirtualDepth helper refines the holes of real frames from an n-frame model."""
import numpy as np
import pytest
import torch

import oracle as O
import synth
from gpu_helpers import dev_pose, gpu_frame, map_params, need_gpu, orc_frame, oracle_maps
from synth import analytic as A

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rf():
    return need_gpu()


def import_both(rf, keys, sdf, w, rgb, s, tau):
    mp = rf.MapParams(s, tau, 5.0, 1 << 16, 1 << 15, 255, 4, "fp32", 64 * 64)
    m = rf.Map(mp)
    sdf32 = sdf.astype(np.float32)
    m.import_(torch.from_numpy(keys).cuda(), torch.from_numpy(sdf32).cuda(),
              torch.from_numpy(w.astype(np.float32)).cuda(), torch.from_numpy(rgb).cuda())
    oms = []
    for bits in (32, 64):
        o = O.OracleMap(s, tau, 5.0, 255, 4, real_bits=bits)
        o.import_(keys, sdf32.astype(np.float64), w, rgb)
        oms.append(o)
    return m, oms[0], oms[1]


def frames_for(rf, W, H, f, depth):
    g = rf.Frame(torch.from_numpy(depth).cuda(), torch.zeros((H, W, 3), dtype=torch.uint8, device="cuda"),
                 f, f, (W - 1) / 2.0, (H - 1) / 2.0, 1.0)
    o = O.Frame(depth, np.zeros((H, W, 3), np.uint8), f, f, (W - 1) / 2.0, (H - 1) / 2.0)
    return g, o


@pytest.mark.parametrize("shape", ["sphere", "plane"])
def test_raycast_of_analytic_map_matches_oracle(rf, shape):
    s, tau = 0.01, 0.05
    if shape == "sphere":
        c, r = np.array([0.05, -0.03, 1.2]), 0.3
        ang, pol = np.linspace(0, 2 * np.pi, 90), np.linspace(0, np.pi, 45)
        pts = c + r * np.array([[np.cos(a) * np.sin(b), np.sin(a) * np.sin(b), np.cos(b)] for a in ang for b in pol])
        keys = A.blocks_near(pts, s, 1)
        fn = lambda x: np.clip(np.linalg.norm(x - c, axis=-1) - r, -tau, tau)
    else:
        n = np.array([0.0, np.sin(0.3), np.cos(0.3)])
        B = 8 * s
        keys = np.array([[x, y, z] for x in range(-11, 11) for y in range(-9, 9) for z in range(10, 28)], np.int32)
        fn = lambda x: np.clip(1.4 - x @ n, -tau, tau)
    k, sdf, w, rgb = A.fill_map(keys, s, fn)
    m, o32, o64 = import_both(rf, k, sdf, w, rgb, s, tau)
    W, H = 64, 48
    g, o = frames_for(rf, W, H, 50.0, np.zeros((H, W), np.float32))
    T = np.eye(4)
    T[:3, 3] = [0.01, -0.02, 0.03]
    zg = m.raycast(g, dev_pose(T), only_invalid=False).cpu().numpy()
    z32 = o32.raycast(o, T, only_invalid=False)
    z64 = o64.raycast(o, T, only_invalid=False)
    assert (zg > 0).sum() > 500
    assert np.array_equal(zg, z32)                                # bit-exact vs the FP32 mirror
    both = (zg > 0) & (z64 > 0)
    assert both.sum() >= 0.99 * (zg > 0).sum()
    assert np.abs(zg[both] - z64[both]).max() < 1e-4              # FP64 reference


@pytest.mark.parametrize("storage,orc_storage", [("fp32", 0), ("fp16", 1)])
def test_raycast_of_fused_map_fills_holes_like_the_oracle(rf, storage, orc_storage):
    seq = synth.parity_room(n_frames=5)
    m = rf.Map(map_params(rf, seq, storage))
    o64, o32 = oracle_maps(seq, orc_storage)
    for k in range(4):
        g = gpu_frame(rf, seq, k)
        P = dev_pose(seq.poses[k])
        m.allocate(g, P)
        m.integrate(g, P)
        for o in (o64, o32):
            o.allocate(orc_frame(seq, k), seq.poses[k])
            o.integrate(orc_frame(seq, k), seq.poses[k])
    rng = np.random.default_rng(5)
    depth = seq.depth[4].copy()
    holes = rng.uniform(size=depth.shape) < 0.2
    depth[holes] = 0
    g = rf.Frame.from_numpy(depth, seq.rgb[4], *seq.intrinsics, depth_scale=seq.depth_scale)
    o = O.Frame(depth, seq.rgb[4], *seq.intrinsics, depth_scale=seq.depth_scale)
    zg = m.raycast(g, dev_pose(seq.poses[4]), far_value=4.0).cpu().numpy()
    z32 = o32.raycast(o, seq.poses[4], far_value=4.0)
    assert np.array_equal(zg, z32)
    truth = seq.depth[4].astype(np.float32) * np.float32(seq.depth_scale if seq.depth.dtype == np.uint16 else 1.0)
    keep = ~holes & (seq.depth[4] > 0)
    assert np.array_equal(zg[keep], truth[keep])                  # valid depths untouched
    filled = holes & (seq.depth[4] > 0) & (zg != 4.0)
    assert filled.sum() > 0.5 * holes.sum()
    assert np.median(np.abs(zg[filled] - truth[filled])) < 0.01   # the model explains the holes


def test_virtual_depth_helper_refines_holes(rf):
    seq = synth.dynamic_room(n_frames=6, width=160, height=120, n_clusters=1, movers="in_view")
    vd = rf.VirtualDepth(map_params(rf, seq), n=6, far_value=5.0)
    rng = np.random.default_rng(1)
    outs, holes = [], []
    for k in range(6):
        d = seq.depth[k].copy()
        h = rng.uniform(size=d.shape) < 0.15
        d[h] = 0
        holes.append(h & (seq.depth[k] > 0))
        outs = vd.push(rf.Frame.from_numpy(d, seq.rgb[k], *seq.intrinsics, depth_scale=seq.depth_scale),
                       dev_pose(seq.poses[k]))
        assert (len(outs) == 0) == (k < 5)
    assert len(outs) == 6
    errs = []
    for k, (f, P) in enumerate(outs):
        z = f.depth.cpu().numpy()
        truth = seq.depth[k].astype(np.float32) * np.float32(seq.depth_scale)
        sel = holes[k] & (z < 5.0)
        errs.append(np.abs(z[sel] - truth[sel]))
        assert (z[seq.depth[k] == 0] > 0).all()                    # no zero is left
    assert np.median(np.concatenate(errs)) < 0.01


@pytest.mark.parametrize("storage,orc_storage", [("fp32", 0), ("fp16", 1)])
@pytest.mark.parametrize("W,H,holes,s,tau", [
    (1, 1, 1.0, 0.01, 0.05), (17, 15, 1.0, 0.01, 0.05), (47, 33, 0.05, 0.01, 0.05), (47, 33, 0.16, 0.01, 0.05),
    (64, 48, 0.5, 0.01, 0.05), (64, 48, 1.0, 0.02, 0.01), (33, 31, 1.0, 0.02, 0.4), (40, 40, 1.0, 0.006, 0.02),
])
def test_raycast_paths_match_the_mirror(rf, W, H, holes, s, tau, storage, orc_storage):
    """Few and many rays a tile, ragged tiles, samples shorter than a voxel
    and longer than a block, more blocks than the tile's table holds, rays
    through blocks that are absent, partly observed, free and mixed, and a
    pose far off the origin: bit-exact against the FP32 mirror."""
    rng = np.random.default_rng(7)
    far = 0.0 if holes < 1.0 else 40.0
    c, r = np.array([0.05 + far, -0.03, 1.0]), 0.25
    B = 8 * s
    lo = np.floor((c - [0.9, 0.7, 0.9]) / B).astype(int)
    hi = np.ceil((c + [0.9, 0.7, 0.6]) / B).astype(int)
    keys = np.array([[x, y, z] for x in range(lo[0], hi[0]) for y in range(lo[1], hi[1]) for z in range(lo[2], hi[2])],
                    np.int32)
    keys = keys[rng.uniform(size=len(keys)) > 0.03]               # some blocks are absent
    keys = keys[rng.permutation(len(keys))[:30000]]
    k, sdf, w, rgb = A.fill_map(keys, s, lambda x: np.clip(np.minimum(np.linalg.norm(x - c, axis=-1) - r,
                                                                     1.45 - x[..., 2]), -tau, tau))
    w = np.where(rng.uniform(size=w.shape) < 2e-5, 0.0, w)         # and a few voxels unobserved
    mp = rf.MapParams(s, tau, 5.0, 1 << 17, 1 << 15, 255, 4, storage, 64 * 64)
    m = rf.Map(mp)
    sdf32 = sdf.astype(np.float32)
    m.import_(torch.from_numpy(k).cuda(), torch.from_numpy(sdf32).cuda(),
              torch.from_numpy(w.astype(np.float32)).cuda(), torch.from_numpy(rgb).cuda())
    o32 = O.OracleMap(s, tau, 5.0, 255, 4, real_bits=32, storage=orc_storage)
    # the mirror imports values as they are, so it gets what the map holds (16-bit storage rounds)
    ke, se, we, ce = [t.cpu().numpy() for t in m.export()]
    o32.import_(ke, se.astype(np.float64), we.astype(np.float64), ce)
    depth = np.where(rng.uniform(size=(H, W)) < holes, 0.0, 1.5).astype(np.float32)
    g, o = frames_for(rf, W, H, 0.8 * max(W, 16), depth)
    T = np.eye(4)
    T[:3, :3] = [[0.96, 0.0, 0.28], [0.0, 1.0, 0.0], [-0.28, 0.0, 0.96]]
    T[:3, 3] = [far - 0.25, 0.02, 0.03]
    for only in ([True, False] if holes < 1.0 else [False]):
        zg = m.raycast(g, dev_pose(T), z_near=0.1, z_far=2.0, far_value=4.0, only_invalid=only).cpu().numpy()
        z32 = o32.raycast(o, T, z_near=0.1, z_far=2.0, far_value=4.0, only_invalid=only)
        assert W == 1 or tau < 0.02 or (zg > 0).mean() > 0.2
        assert np.array_equal(zg, z32)


def test_raycast_through_free_blocks_matches_the_mirror(rf):
    """Compact free space: rays step over free blocks and blocks with voxels."""
    seq = synth.parity_room(n_frames=4)
    mp = map_params(rf, seq)
    mp.free_blocks = True
    m = rf.Map(mp)
    o32 = O.OracleMap(seq.voxel_size, seq.truncation, seq.depth_max, 255, seq.carve_stride, real_bits=32,
                      free_blocks=True)
    for k in range(3):
        g, P = gpu_frame(rf, seq, k), dev_pose(seq.poses[k])
        m.allocate(g, P)
        m.integrate(g, P)
        o32.allocate(orc_frame(seq, k), seq.poses[k])
        o32.integrate(orc_frame(seq, k), seq.poses[k])
    zg = m.raycast(gpu_frame(rf, seq, 3), dev_pose(seq.poses[3]), only_invalid=False).cpu().numpy()
    z32 = o32.raycast(orc_frame(seq, 3), seq.poses[3], z_far=seq.depth_max, only_invalid=False)
    assert (zg > 0).mean() > 0.5
    assert np.array_equal(zg, z32)
