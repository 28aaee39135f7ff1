"""Mesh extraction (marching tetrahedra) through the C ABI against the oracle:
bit-exact against the FP32 mirror (triangles compared as sorted lists), close
to the FP64 reference, on an analytic sphere map and on maps fused from
frames (FP32 and FP16 storage); capacity overflow and the empty map."""
import ctypes

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


def sorted_tris(T):
    T = np.asarray(T, np.float64).reshape(len(T), 9)
    return T[np.lexsort(T.T[::-1])]


def sphere_inputs(c, r, s=0.01, tau=0.05):
    ang = np.linspace(0, 2 * np.pi, 90)
    pol = np.linspace(0, np.pi, 45)
    pts = c + r * np.array([[np.cos(a) * np.sin(b), np.sin(a) * np.sin(b), np.cos(b)] for a in ang for b in pol])
    keys = A.blocks_near(pts, s, 1)
    return A.fill_map(keys, s, lambda x: np.clip(np.linalg.norm(x - c, axis=-1) - r, -tau, tau))


def test_mesh_of_analytic_sphere_matches_oracle(rf):
    s, tau = 0.01, 0.05
    c, r = np.array([0.013, -0.007, 0.021]), 0.17
    keys, sdf, w, rgb = sphere_inputs(c, r, s, tau)
    mp = rf.MapParams(s, tau, 5.0, 1 << 16, 1 << 14, 255, 4, "fp32", 64 * 64)
    m = rf.Map(mp)
    m.import_(torch.from_numpy(keys).cuda(), torch.from_numpy(sdf.astype(np.float32)).cuda(),
              torch.from_numpy(w.astype(np.float32)).cuda(), torch.from_numpy(rgb).cuda())
    g = m.mesh().cpu().numpy()
    o32 = O.OracleMap(s, tau, 5.0, 255, 4, real_bits=32)
    o32.import_(keys, sdf.astype(np.float32).astype(np.float64), w, rgb)
    o64 = O.OracleMap(s, tau, 5.0, 255, 4, real_bits=64)
    o64.import_(keys, sdf.astype(np.float32).astype(np.float64), w, rgb)
    t32, t64 = o32.mesh(), o64.mesh()
    assert len(g) == len(t32) == len(t64) > 10000
    a, b = sorted_tris(g), sorted_tris(t32)
    assert np.array_equal(a, b)                                   # bit-exact vs the FP32 mirror
    assert np.abs(t64 - t32).max() < 1e-6                         # FP64 reference, same emission order
    V = g.reshape(-1, 3).astype(np.float64)
    assert np.abs(np.linalg.norm(V - c, axis=1) - r).max() < 3 * s * s / (8 * r) * 1.01 + 1e-6


@pytest.mark.parametrize("storage,orc_storage", [("fp32", 0), ("fp16", 1)])
def test_mesh_of_fused_map_matches_mirror(rf, storage, orc_storage):
    seq = synth.parity_room(n_frames=4)
    m = rf.Map(map_params(rf, seq, storage))
    o64, o32 = oracle_maps(seq, orc_storage)
    for k in range(4):
        g = gpu_frame(rf, seq, k)
        P = dev_pose(seq.poses[k])
        m.allocate(g, P)
        m.integrate(g, P)
        fr = orc_frame(seq, k)
        for o in (o64, o32):
            o.allocate(fr, seq.poses[k])
            o.integrate(fr, seq.poses[k])
    torch.cuda.synchronize()
    gm = m.mesh().cpu().numpy()
    t32 = o32.mesh()
    assert len(gm) == len(t32) > 1000
    assert np.array_equal(sorted_tris(gm), sorted_tris(t32))
    t64 = o64.mesh()
    # the FP64 map differs from the FP32 one by rounding, so compare the
    # surfaces: every GPU vertex lies within a voxel of the FP64 mesh's vertices
    from scipy.spatial import cKDTree
    d, _ = cKDTree(t64.reshape(-1, 3)).query(gm.reshape(-1, 3).astype(np.float64))
    assert np.percentile(d, 99) < 1e-3 and d.max() < seq.voxel_size


def test_mesh_capacity_overflow_and_empty_map(rf):
    s, tau = 0.01, 0.05
    keys, sdf, w, rgb = sphere_inputs(np.zeros(3), 0.08, s, tau)
    mp = rf.MapParams(s, tau, 5.0, 1 << 14, 1 << 12, 255, 4, "fp32", 64 * 64)
    empty = rf.Map(mp)
    assert empty.mesh().shape[0] == 0
    m = rf.Map(mp)
    m.import_(torch.from_numpy(keys).cuda(), torch.from_numpy(sdf.astype(np.float32)).cuda(),
              torch.from_numpy(w.astype(np.float32)).cuda(), torch.from_numpy(rgb).cuda())
    full = m.mesh().cpu().numpy()
    cap = len(full) // 3
    tris = torch.full((cap, 3, 3), -7.0, dtype=torch.float32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    L = m.L
    assert L.extract_mesh(m.h, ctypes.c_void_p(tris.data_ptr()), cap, ctypes.c_void_p(cnt.data_ptr()), None) == 0
    torch.cuda.synchronize()
    assert int(cnt.item()) == len(full)                          # the total, beyond the capacity
    part = tris.cpu().numpy()
    assert np.array_equal(part, full[:cap])                      # the first cap triangles, in order
    assert L.extract_mesh(m.h, None, 10, ctypes.c_void_p(cnt.data_ptr()), None) != 0   # NULL triangles, cap > 0


@pytest.mark.parametrize("storage,orc_storage", [("fp32", 0), ("fp16", 1)])
@pytest.mark.parametrize("density,holes,absent", [(0.5, 0.0, 0.0), (0.5, 0.02, 0.3), (0.02, 0.01, 0.6), (1.0, 0.3, 0.0)])
def test_mesh_of_random_blocks_matches_mirror(rf, density, holes, absent, storage, orc_storage):
    """Every corner pattern, at every face, edge and corner of a block, with
    and without the neighbours, unobserved voxels and voxels at the band's
    limit: the triangles bit-exact against the FP32 mirror, the same again, and
    the marks of the blocks gone afterwards (the next frame list is right)."""
    rng = np.random.default_rng(11)
    s, tau = 0.02, 0.06
    keys = np.array([[x, y, z] for x in range(-2, 3) for y in range(-2, 2) for z in range(3, 7)], np.int32)
    keys = keys[rng.uniform(size=len(keys)) >= absent]
    shape = (len(keys), 512)
    sdf = rng.uniform(-tau, tau, shape)
    sdf = np.where(rng.uniform(size=shape) < density, sdf, tau)    # the rest: free space
    sdf[rng.uniform(size=shape) < 0.01] = 0.0
    sdf[rng.uniform(size=shape) < 0.01] = -tau
    w = (rng.uniform(size=shape) >= holes).astype(np.float32)
    rgb = np.zeros(shape + (3,), np.uint8)
    m = rf.Map(rf.MapParams(s, tau, 5.0, 1 << 12, 1 << 10, 255, 4, storage, 64 * 48))
    m.import_(torch.from_numpy(keys).cuda(), torch.from_numpy(sdf.astype(np.float32)).cuda(),
              torch.from_numpy(w).cuda(), torch.from_numpy(rgb).cuda())
    ke, se, we, ce = [t.cpu().numpy() for t in m.export()]          # as stored
    o32 = O.OracleMap(s, tau, 5.0, 255, 4, real_bits=32, storage=orc_storage)
    o32.import_(ke, se.astype(np.float64), we.astype(np.float64), ce)
    g, t32 = m.mesh().cpu().numpy(), o32.mesh()
    assert len(g) == len(t32) and (len(g) > 0) == (density >= 0.5)  # 2%: no cube has all corners in the band
    assert np.array_equal(sorted_tris(g), sorted_tris(t32))
    assert np.array_equal(m.mesh().cpu().numpy(), g)
    f = rf.Frame(torch.full((48, 64), 0.9, dtype=torch.float32, device="cuda"),
                 torch.zeros((48, 64, 3), dtype=torch.uint8, device="cuda"), 60.0, 60.0, 31.5, 23.5, 1.0)
    fresh = rf.Map(m.params)
    lists = []
    for q in (m, fresh):
        q.allocate(f, dev_pose(np.eye(4)))
        k = q.frame_blocks().cpu().numpy()
        lists.append(k[np.lexsort(k.T)])
    assert np.array_equal(lists[0], lists[1])


def test_mesh_of_many_blocks(rf):
    """More blocks than a workgroup of the write pass lists at once: the
    surface's blocks among 530 000 of free space give the same triangles."""
    s, tau = 0.01, 0.05
    c = np.array([0.3, 0.2, 0.1])
    keys, sdf, w, rgb = sphere_inputs(c, 0.15, s, tau)
    arr = [torch.from_numpy(x).cuda() for x in (keys, sdf.astype(np.float32), w.astype(np.float32), rgb)]
    small = rf.Map(rf.MapParams(s, tau, 5.0, 1 << 12, 1 << 11, 255, 4, "fp16", 64 * 64))
    small.import_(*arr)
    n = 530000
    m = rf.Map(rf.MapParams(s, tau, 5.0, 1 << 21, n + (1 << 12), 255, 4, "fp16", 64 * 64))
    grid = torch.arange(n, device="cuda", dtype=torch.int32)
    far = torch.stack([100 + grid % 100, 100 + (grid // 100) % 100, 100 + grid // 10000], 1).contiguous()
    half = n // 2
    tau_block = torch.full((half, 512), tau, dtype=torch.float32, device="cuda")
    one = torch.ones((half, 512), dtype=torch.float32, device="cuda")
    black = torch.zeros((half, 512, 3), dtype=torch.uint8, device="cuda")
    m.import_(far[:half], tau_block, one, black)
    m.import_(*arr)
    m.import_(far[half:2 * half], tau_block, one, black)
    a, b = small.mesh().cpu().numpy(), m.mesh().cpu().numpy()
    assert len(a) == len(b) > 5000
    assert np.array_equal(sorted_tris(a), sorted_tris(b))
