"""Small planners with 3-D features, whose compaction and DBSCAN run in one block:
sizes around its words and its limit, one cluster to more clusters than the chunk
sums hold, more hook trees than a row of the tree graph, points that are all core,
border or noise.  Every result must equal the distance passes' bit for bit, three
calls in a row, and the labels must be DBSCAN of the features by definition."""
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


def _cases():
    rng = np.random.default_rng(21)
    cap = lambda n, s: rng.normal(size=3) + s * rng.normal(size=(n, 3))  # noqa: E731
    every = rng.normal(size=(251, 3))
    c = [(f"size_{K}", np.concatenate([cap((K - 5) // 2, 0.2), cap(K - 5 - (K - 5) // 2, 0.2)]), 0.35, 6)
         for K in (6, 50, 64, 65, 128, 129, 192, 255, 256, 257)]
    c += [("all_noise", every, 0.02, 3), ("all_core", every, 0.02, 1), ("one_cluster", every, 1.9, 4),
          ("border", np.concatenate([cap(20, 0.02), every[:200]]), 0.3, 20),
          ("chains", np.concatenate([every[:125], every[:125] + 0.03]), 0.25, 2),
          ("eighty_groups", np.repeat(every[:80], 3, axis=0) + 0.001 * rng.normal(size=(240, 3)), 0.02, 3)]
    return c


CASES = _cases()


@pytest.mark.parametrize("case", range(len(CASES)), ids=[c[0] for c in CASES])
def test_small_planner(case):
    from paper_2607_06499_amd import binding as B

    name, pts, eps, min_pts = CASES[case]
    rng = np.random.default_rng(300 + case)
    V, ncol = len(pts), 5
    K = V + ncol
    pts = pts / np.linalg.norm(pts, axis=1, keepdims=True)
    s = W.arm6_dynamic(1, K)
    spec = s.spec.replace(dbscan_eps=eps, dbscan_min_pts=min_pts).rounded()
    col = np.zeros(K, np.int32)
    col[rng.choice(K, ncol, replace=False)] = 1
    p = np.zeros((K, 3), np.float32)
    rec = dict(S=rng.uniform(3, 9, K).astype(np.float32), col=col, first=np.where(col, 0, -1).astype(np.int32), p=p,
               eps=rng.normal(0, 0.3, (K, spec.horizon, 6)).astype(np.float32))
    pls = {m: B.Planner(spec) for m in (B.DBSCAN_BITMAP, B.DBSCAN_TILED)}
    for m, pl in pls.items():
        pl.set_dbscan_mode(m)
    x = H.to_dev(np.asarray(s.x0, np.float32))
    for call in range(3):
        p[:] = 0.0
        p[col == 0] = pts[rng.permutation(V)].astype(np.float32)
        obs = H.to_dev(np.asarray(s.obstacles, np.float32) + 0.01 * call)
        d = {k: H.to_dev(v) for k, v in rec.items()}
        r = {}
        for m, pl in pls.items():
            pl.replan_from_rollouts(x, obs, d["S"], d["col"], d["first"], d["p"], d["p"], d["eps"])
            H.torch_mod().cuda.synchronize()
            r[m] = H.collect_outputs(pl)
        a, b = r[B.DBSCAN_BITMAP], r[B.DBSCAN_TILED]
        assert a["info"]["n_feasible"] == V and a["info"]["branch"] == 0
        for k in ("label", "z", "c_mean_cost", "c_dir", "c_size", "u_out", "U_new", "U_next"):
            assert np.array_equal(a[k], b[k]), (name, call, k)
        for k in a["info"]:
            assert np.array_equal(np.asarray(a["info"][k]), np.asarray(b["info"][k])), (name, call, k)
        assert H.counts_agree(b["ncount"], a["ncount"], min_pts), (name, call)
        print(f"{name} call {call}: V={V} M={a['info']['n_clusters']}")
        z64, e32 = a["z"].astype(np.float64), float(np.float32(eps))
        H.dbscan_check(z64, e32, min_pts, a["ncount"], a["label"], 0.5 * H.STAGE_BAND * e32,
                       exact_ref=oracle.dbscan(z64, e32, min_pts)[0], tag=name)
    for pl in pls.values():
        pl.close()
