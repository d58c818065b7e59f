"""Cluster statistics and selection of large planners, whose chunk sums (one per
1,024 points) are requested ahead by the adding threads up to eight chunks and
staged beyond: size, mean cost, minimum cost, direction and the selected cluster
against FP64 sums over the labels, costs and directions that the planner reports.
One to 64 clusters, spread over every chunk or each confined to a few of them."""
import math

import numpy as np
import pytest

from paper_2607_06499_amd import workloads as W
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not H.gpu_ok():
        pytest.skip("no GPU")


@pytest.mark.parametrize("spread", [True, False], ids=["spread", "confined"])
@pytest.mark.parametrize("M", [1, 2, 8, 9, 64])
@pytest.mark.parametrize("V", [8192, 8193, 65000])
def test_chunked_statistics(V, M, spread):
    from paper_2607_06499_amd import binding as B

    rng = np.random.default_rng(V + M)
    group = np.sort(rng.integers(0, M, V))
    if spread:
        group = rng.permutation(group)
    th = group * (2 * math.pi / M) + rng.uniform(-0.01, 0.01, V)
    ncol, N = 5, 4
    K = V + ncol
    col = np.zeros(K, np.int32)
    col[rng.choice(K, ncol, replace=False)] = 1
    p = np.zeros((K, 2), np.float32)  # (the colliding rollouts' points: the reference)
    p[col == 0] = np.stack([np.cos(th), np.sin(th)], 1).astype(np.float32)
    best = (2 * M) // 3
    S = np.full(K, 5.0, np.float32)
    S[col == 0] = (rng.uniform(3, 9, V) + np.where(group == best, 0.0, 2.0 + 0.1 * group)).astype(np.float32)
    rec = dict(S=S, col=col, first=np.where(col, 0, -1).astype(np.int32), p=p,
               eps=rng.normal(0, 0.3, (K, N, 2)).astype(np.float32))
    spec = W.PlannerSpec(num_samples=K, horizon=N, dbscan_eps=0.04, dbscan_min_pts=5, max_obstacles=1).rounded()
    pl = B.Planner(spec)
    x = H.to_dev(np.array([-1.0, 0.2, 0.0], np.float32))
    obs = H.to_dev(np.array([[0.1, 0.05, 0.2]], np.float32))
    d = {k: H.to_dev(v) for k, v in rec.items()}
    pl.replan_from_rollouts(x, obs, d["S"], d["col"], d["first"], d["p"], d["p"], d["eps"])
    r = H.collect_outputs(pl)
    pl.close()
    inf = r["info"]
    assert inf["n_feasible"] == V and inf["n_clusters"] == M
    lab, Sv, g = r["label"], r["S"][r["v_idx"]], r["g"].astype(np.float64)
    # clusters are numbered by their lowest index, and hold the groups
    firsts = [int(np.argmax(group == q)) for q in range(M)]
    assert np.array_equal(lab, np.argsort(np.argsort(firsts))[group])
    mean = np.array([Sv[lab == q].astype(np.float64).mean() for q in range(M)])
    vec = np.stack([g[lab == q].mean(0) for q in range(M)])
    vec /= np.linalg.norm(vec, axis=1, keepdims=True) + float(np.float32(spec.norm_eps))
    assert np.array_equal(r["c_size"], np.bincount(lab, minlength=M))
    assert H.rel_err(r["c_mean_cost"], mean).max() <= 1e-5
    assert np.abs(r["c_dir"] - vec).max() <= 2e-5
    sel = int(np.argmin(mean))
    assert group[np.argmax(lab == sel)] == best
    assert inf["selected"] == sel and inf["selected_size"] == int((lab == sel).sum())
    assert np.float32(inf["s_min"]) == Sv[lab == sel].min()
    if M > 1:
        k = np.sort(mean)
        assert abs(inf["margin"] - (k[1] - k[0])) <= 2e-5 * k[1]
