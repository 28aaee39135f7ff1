"""The solve of a registration step: against a pivoted solve on the host, and
the same wherever it runs (the last launch of a pass, the start of an
evaluation, a launch of its own)."""
import numpy as np
import pytest
import torch

import oracle as O
import synth
from gpu_helpers import dev_pose, gpu_frame, map_params, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rf():
    return need_gpu()


@pytest.fixture(scope="module")
def scene(rf):
    seq = synth.static_room(n_frames=3, width=160, height=120)
    m = rf.Map(map_params(rf, seq))
    m.allocate(gpu_frame(rf, seq, 0), dev_pose(seq.poses[0]))
    m.integrate(gpu_frame(rf, seq, 0), dev_pose(seq.poses[0]))
    return seq, m


def twist(rng, r):
    return np.r_[rng.normal(size=3) * 0.01, rng.normal(size=3) * r]


@pytest.mark.parametrize("lam", [0.0, 0.5])
@pytest.mark.parametrize("r", [0.001, 0.02, 0.2])
def test_one_step_against_a_host_solve(rf, scene, lam, r):
    """Small and large rotations (the series and the closed form of the
    exponential).  Both sides solve the same totals in FP64: a backward-stable
    solve errs by about cond(H) 2^-53 times its dimension, taken 16 times."""
    seq, m = scene
    rng = np.random.default_rng(int(1000 * r))
    T = O.pose_left_update(twist(rng, r), seq.poses[0])
    g = gpu_frame(rf, seq, 1)
    ne = m.normal_equations(g, dev_pose(T), 0, 0.025).cpu().numpy()
    P = dev_pose(T)
    m.track(g, P, rf.TrackParams(1, 1, 0.025, min_valid=6, lm_lambda=lam))
    H = np.zeros((6, 6))
    H[np.triu_indices(6)] = ne[:21]
    H = np.triu(H) + np.triu(H, 1).T
    H[np.diag_indices(6)] *= 1.0 + lam
    d = np.linalg.solve(H, -ne[21:27])
    want = O.pose_left_update(d, T)
    tol = 16 * 6 * np.linalg.cond(H) * 2.0 ** -53 * max(1.0, np.abs(d).max()) * max(1.0, np.abs(want).max())
    assert np.abs(P.cpu().numpy() - want).max() <= tol


def test_solve_at_every_place(rf, scene):
    """Three steps at once (the first two solved at the start of the next
    evaluation) equal three passes of one step, each solved by the last launch."""
    seq, m = scene
    g = gpu_frame(rf, seq, 2)
    P, Q = dev_pose(seq.poses[0]), dev_pose(seq.poses[0])
    m.track(g, P, rf.TrackParams(1, 3))
    for _ in range(3):
        m.track(g, Q, rf.TrackParams(1, 1))
    torch.cuda.synchronize()
    assert np.array_equal(P.cpu().numpy(), Q.cpu().numpy())


@pytest.mark.parametrize("adaptive", [False, True])
def test_solve_in_a_launch_of_its_own(rf, adaptive):
    """A level of 3600 workgroups (1280x720), above the 3072 from which on the
    solve is a launch of its own: three Gauss-Newton steps at once equal three
    passes of one step, whose only solve is the last launch's, and a pass of
    four Levenberg-Marquardt evaluations equals itself after another pass has
    left other contents in the state buffers."""
    seq = synth.static_room(n_frames=2, width=1280, height=720)
    m = rf.Map(map_params(rf, seq))
    m.allocate(gpu_frame(rf, seq, 0), dev_pose(seq.poses[0]))
    m.integrate(gpu_frame(rf, seq, 0), dev_pose(seq.poses[0]))
    assert m.status()[0] == 0
    g = gpu_frame(rf, seq, 1)
    P, Q = dev_pose(seq.poses[0]), dev_pose(seq.poses[0])
    if adaptive:
        tp = rf.TrackParams(1, 4, lm_lambda=1e-3, adaptive=True)
        m.track(g, P, tp)
        m.track(g, dev_pose(seq.poses[0]), rf.TrackParams(2, 3, lm_lambda=10.0, adaptive=True))
        m.track(g, Q, tp)
    else:
        m.track(g, P, rf.TrackParams(1, 3))
        for _ in range(3):
            m.track(g, Q, rf.TrackParams(1, 1))
    torch.cuda.synchronize()
    assert m.status()[0] == 0 and np.array_equal(P.cpu().numpy(), Q.cpu().numpy())
    assert np.abs(P.cpu().numpy() - seq.poses[0]).max() > 1e-4         # it moved


@pytest.mark.parametrize("adaptive", [False, True])
@pytest.mark.parametrize("lam", [1e200, 1e300, 1e308, np.inf])
def test_damping_without_bound_keeps_the_pose(rf, scene, lam, adaptive):
    """Damping up to infinity is accepted: the reciprocal pivots go to zero, so
    every step is applied and changes nothing.  Steps are at most |g| / (lambda
    min diag H) < 1e20 / 1e200 per component; an infinite damping gives exactly
    zero.  Under Levenberg-Marquardt the first step starts from lambda itself."""
    seq, m = scene
    P = dev_pose(seq.poses[0])
    stats = torch.zeros(16, dtype=torch.float64, device="cuda")
    n = 2 if adaptive else 3
    m.track(gpu_frame(rf, seq, 1), P, rf.TrackParams(1, n, lm_lambda=lam, adaptive=adaptive), None, stats)
    words = stats.cpu().numpy().view(np.uint32)
    assert int(words[5]) == 0                                          # no flag
    assert int(words[4]) == (1 if adaptive else 3)                     # steps counted
    d = np.abs(P.cpu().numpy() - seq.poses[0]).max()
    assert d == 0.0 if np.isinf(lam) else d <= 1e-150
