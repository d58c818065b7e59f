"""The labelling of a replan's feasible set on the angular windows: feature
sets made through the caller's own rollout records, so that every form of the
pass is reached (no open points; open points and their boundary buckets within
and beyond what a block lists; off-ring points that are core, border or noise
and that join arcs; gaps that need pair tests; more clusters than the chunk
sums hold; sizes around the 1,024-point chunks).

Every result must equal the distance passes' (and the bitmap's where it
exists) bit for bit: labels, counts, cluster statistics, the update and the
info record; and the labels must be DBSCAN of the features by definition.
Three calls in a row on one planner: nothing may be left over between them."""
import math

import numpy as np
import pytest

import oracle
from paper_2607_06499_amd import workloads as W
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not H.gpu_ok():
        pytest.skip("no GPU")


def _dirs(th, r=1.0):
    return np.stack([np.cos(th), np.sin(th)], 1) * np.broadcast_to(r, np.shape(th))[:, None]


def _cases():
    rng = np.random.default_rng(11)
    crit = 2 * math.asin(0.25 / 2)
    beta = 2 * math.pi / 4096
    u = lambda lo, hi, n: rng.uniform(lo, hi, n)  # noqa: E731
    tail = u(2.0, 5.0, 40)
    c = [("dense", _dirs(u(0.0, 1.0, 5000)), 0.25, 20),
         ("outliers", _dirs(np.concatenate([rng.normal(0.0, 0.2, 7000), tail])), 0.25, 20),
         ("all_open", _dirs(u(-math.pi, math.pi, 60)), 0.25, 10),
         ("border_only", _dirs(np.array([0.0, 0.1, 0.2, 0.3, 0.42, 2.0])), 0.25, 4),
         ("one_point", _dirs(np.array([1.0])), 0.25, 1),
         ("more_open_than_listed", _dirs(u(-math.pi, math.pi, 4000)), 0.25, 400),
         ("zone_beyond_list", _dirs(np.concatenate([u(0.0, 0.02, 9000), [crit + 0.01] * 3, u(1.0, 1.2, 30)])), 0.25, 20),
         ("sixty_five_groups", _dirs(np.repeat(np.arange(65) * (2 * math.pi / 65), 20)), 0.03, 5),
         ("ninety_groups", _dirs(np.repeat(np.arange(90) * (2 * math.pi / 90), 20) + rng.normal(0, 0.002, 1800)), 0.03, 5),
         ("sixty_four_groups", _dirs(np.repeat(np.arange(64) * (2 * math.pi / 64), 20)), 0.03, 5)]
    for i, phi in enumerate(np.linspace(crit - 3 * beta, crit + 3 * beta, 7)):
        th = np.concatenate([u(-0.5, 0.0, 150), [0.0], u(phi, phi + 0.5, 150), [phi]]) + u(-3, 3, 1)
        c.append((f"gap_{i}", _dirs(th), 0.25, 5))
    near = lambda n: _dirs(u(0, 2 * math.pi, n), u(1e-8, 5e-7, n))  # noqa: E731  (features well inside the circle)
    rim = lambda th: _dirs(np.asarray(th), 4e-4)  # noqa: E731  (norm about 0.9975)
    arcs = np.concatenate([u(0.0, 0.6, 900), u(1.5, 2.1, 900)])
    c += [("off_noise", np.concatenate([_dirs(arcs), near(1)]), 0.25, 20),
          ("off_core_rim", np.concatenate([_dirs(arcs), rim([0.3, 1.8])]), 0.25, 20),
          ("off_border", np.concatenate([_dirs(u(0.0, 0.05, 30)), rim([0.27, 0.29, -0.21])]), 0.25, 25),
          ("off_bridge", np.concatenate([_dirs(np.concatenate([u(0.0, 0.2, 300), u(0.44, 0.6, 300)])), rim([0.32])]), 0.235, 20),
          ("off_cluster", np.concatenate([near(16), _dirs(arcs)]), 0.25, 10),
          ("off_beyond_list", np.concatenate([_dirs(arcs), near(40), rim([0.3, 1.0, 1.8])]), 0.25, 10),
          ("all_off", near(300), 0.25, 10)]
    for V in (1023, 1024, 1025, 8191, 8193, 12289):
        c.append((f"size_{V}", _dirs(np.concatenate([rng.normal(0.5, 0.3, V - 9), u(2, 6, 9)])), 0.25, 20))
    c.append(("size_65000", _dirs(np.concatenate([rng.normal(0.5, 0.3, 64975), u(2, 6, 25)])), 0.25, 20))
    # K = V + 5 at the ends of the range whose blocks compact for themselves
    for V in (1019, 1020, 2042, 2043, 2044):
        c.append((f"size_{V}", _dirs(np.concatenate([rng.normal(0.5, 0.3, V - 9), u(2, 6, 9)])), 0.25, 20))
    return c


CASES = _cases()


@pytest.mark.parametrize("case", range(len(CASES)), ids=[c[0] for c in CASES])
def test_label_forms(case):
    from paper_2607_06499_amd import binding as B

    name, pts, eps, min_pts = CASES[case]
    rng = np.random.default_rng(100 + case)
    V = len(pts)
    # colliding rollouts among the feasible ones, whose terminal points (the
    # origin) make the reference point
    ncol = 5
    K, N = V + ncol, 4
    col = np.zeros(K, np.int32)
    col[rng.choice(K, ncol, replace=False)] = 1
    p = np.zeros((K, 2), np.float32)
    rec = dict(S=rng.uniform(3, 9, K).astype(np.float32), col=col, first=np.where(col, 0, -1).astype(np.int32),
               p=p, eps=rng.normal(0, 0.3, (K, N, 2)).astype(np.float32))
    spec = W.PlannerSpec(num_samples=K, horizon=N, dbscan_eps=eps, dbscan_min_pts=min_pts, scene_mode=W.DYNAMIC,
                         history_len=3, max_obstacles=1).rounded()
    modes = [B.DBSCAN_WINDOW, B.DBSCAN_TILED] + ([B.DBSCAN_BITMAP] if K <= 16384 else [])
    pls = {m: B.Planner(spec) for m in modes}
    for m, pl in pls.items():
        pl.set_dbscan_mode(m)
        assert pl.dbscan_path() == m
    x = H.to_dev(np.array([-1.0, 0.2, 0.0], np.float32))
    for call in range(3):
        order = rng.permutation(V)
        p[:] = 0.0
        p[col == 0] = pts[order].astype(np.float32)
        obs = H.to_dev(np.array([[0.1 * call, 0.05, 0.2]], np.float32))
        d = {k: H.to_dev(v) for k, v in rec.items()}
        r = {}
        for m, pl in pls.items():
            pl.replan_from_rollouts(x, obs, d["S"], d["col"], d["first"], d["p"], d["p"], d["eps"])
            H.torch_mod().cuda.synchronize()
            r[m] = H.collect_outputs(pl)
        w = r[B.DBSCAN_WINDOW]
        assert w["info"]["n_feasible"] == V and w["info"]["branch"] == 0
        for m in modes[1:]:
            for k in ("label", "z", "c_mean_cost", "c_dir", "c_size", "u_out", "U_new", "U_next"):
                assert np.array_equal(w[k], r[m][k]), (name, call, m, k)
            for k in w["info"]:
                assert np.array_equal(np.asarray(w["info"][k]), np.asarray(r[m]["info"][k])), (name, call, m, k)
        assert H.counts_agree(r[B.DBSCAN_TILED]["ncount"], w["ncount"], min_pts), (name, call)
        if B.DBSCAN_BITMAP in r:
            assert np.array_equal(w["ncount"], r[B.DBSCAN_BITMAP]["ncount"]), (name, call)
        print(f"{name} call {call}: V={V} M={w['info']['n_clusters']} selected={w['info']['selected']}")
        if call == 0 and V <= 16384:
            z64, e32 = w["z"].astype(np.float64), float(np.float32(eps))
            olab = oracle.dbscan(z64, e32, min_pts)[0]
            H.dbscan_check(z64, e32, min_pts, w["ncount"], w["label"], 0.5 * H.STAGE_BAND * e32, exact_ref=olab,
                           tag=name)
    for pl in pls.values():
        pl.close()
