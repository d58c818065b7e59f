"""The lane layouts of the unicycle rollouts, at the sizes where one gives way
to another and where a lane's steps are cut off: horizons around the multiples
of the steps per lane, rollout counts around the layouts' lines and around the
blocks, with fixed and with constant-velocity obstacles, against the oracle's
rollouts (the bar of the other rollout tests); and batches of such planners,
each member bitwise its single replan."""
import numpy as np
import pytest

import oracle
from paper_2607_06499_amd import workloads as W
from tests import harness as H
from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not H.gpu_ok():
        pytest.skip("no GPU")


SIZES = [(N, K) for N in (1, 2, 3, 15, 16, 17, 31, 32, 33, 34, 48, 61, 62, 63) for K in (7, 65, 300)]
SIZES += [(33, 4096), (33, 4097), (63, 4097), (50, 4111), (5, 16385), (16, 16385), (17, 16385), (31, 16399),
          (32, 16384)]


def _scene(N, K, seed):
    s = W.random_scene(seed, num_samples=K, horizon=N, n_obs=5 + seed % 9)
    if seed % 3 == 1:
        s.spec = s.spec.replace(flags=W.FLAG_OBS_CONST_VEL, ref_mode=W.REF_FIRST_CONTACT)
    return s


@pytest.mark.parametrize("N,K", SIZES)
def test_rollout_layouts_match_oracle(N, K):
    s = _scene(N, K, 200 + N + K)
    pl = P._planner(s.spec)
    P._set_U(pl, s.U0)
    fld = s.field
    before = fld.positions()
    pl.set_history(H.to_dev(before[None]))
    fld.step(s.spec.dt)
    obs = fld.observation()
    r = H.gpu_replan(pl, s.x0, obs)
    o = oracle.replan(s.spec, s.x0, s.U0, obs, np.stack([fld.positions(), before]))
    P._compare_rollouts(r, o, s.spec)
    pl.close()


def test_batch_members_of_every_layout_bitwise():
    from paper_2607_06499_amd import binding as B

    scenes = [_scene(N, K, 900 + i) for i, (N, K) in
              enumerate([(1, 9), (16, 300), (17, 1000), (33, 4096), (33, 4097), (63, 700), (12, 16385), (29, 16400)])]
    a, b = [B.Planner(s.spec) for s in scenes], [B.Planner(s.spec) for s in scenes]
    for s, x, y in zip(scenes, a, b):
        x.set_nominal(H.to_dev(s.U0))
        y.set_nominal(H.to_dev(s.U0))
    xs = [H.to_dev(s.x0) for s in scenes]
    obs = [H.to_dev(s.obstacles) for s in scenes]
    batch = B.Batch(a)
    batch.set_io(xs, obs)
    torch = H.torch_mod()
    for step in range(3):
        if step == 1:
            batch.replan_subset(list(range(len(a))))
        else:
            batch.replan()
        for y, x_t, o in zip(b, xs, obs):
            y.replan(x_t, o)
        torch.cuda.synchronize()
        for i, (x, y) in enumerate(zip(a, b)):
            assert torch.equal(x.U_out, y.U_out) and torch.equal(x.info_buf, y.info_buf), (step, i)
            assert torch.equal(x.debug(B.DBG_COST, x.K), y.debug(B.DBG_COST, y.K)), (step, i)
    batch.close()


@pytest.mark.parametrize("ns,n_obs,N,K,pose", [(1, 1, 7, 33, False), (7, 17, 31, 65, True), (8, 64, 32, 100, False),
                                               (9, 3, 33, 41, True), (16, 64, 40, 50, True), (15, 0, 1, 9, False)])
def test_arm_sphere_groups_match_oracle(ns, n_obs, N, K, pose):
    s = W.random_scene(300 + ns, dynamics=W.ARM6, num_samples=K, horizon=N, n_obs=n_obs)
    kw = dict(n_link_spheres=ns, flags=(W.FLAG_POSE_COST if pose else 0) | W.FLAG_OBS_CONST_VEL)
    if pose:
        kw.update(Q=[10.0, 3.0, 50.0, 0.0, 0.0, 0.0], Qf=[10.0, 3.0, 50.0, 0.0, 0.0, 0.0])
    s.spec = s.spec.replace(**kw)
    pl = P._planner(s.spec)
    P._set_U(pl, s.U0)
    before = s.field.positions()
    if n_obs:
        pl.set_history(H.to_dev(before[None]))
    s.field.step(s.spec.dt)
    obs = s.field.observation()
    r = H.gpu_replan(pl, s.x0, obs)
    hist = np.stack([s.field.positions(), before]) if n_obs else None
    o = oracle.replan(s.spec, s.x0, s.U0, obs, hist)
    P._compare_rollouts(r, o, s.spec)
    pl.close()


# either side of the number of blocks up to which the prologue has a wave of its
# own, for both segment widths (16 rollouts a block for N <= 32, 8 beyond)
@pytest.mark.parametrize("N,K", [(12, 8192), (12, 8193), (32, 8201), (33, 4096), (33, 4097), (63, 4111)])
def test_arm_launch_sizes_match_oracle(N, K):
    s = W.random_scene(500 + N, dynamics=W.ARM6, num_samples=K, horizon=N, n_obs=9)
    pl = P._planner(s.spec)
    P._set_U(pl, s.U0)
    r = H.gpu_replan(pl, s.x0, s.obstacles)
    o = oracle.replan(s.spec, s.x0, s.U0, s.obstacles)
    P._compare_rollouts(r, o, s.spec)
    pl.close()
