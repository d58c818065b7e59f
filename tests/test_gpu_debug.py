"""Neighbour counts read through the diagnostics belong to the planner's last
call, whatever its DBSCAN mode is by then, and reading them leaves the planner
as it was: after a replan on the angular windows (also one of a batch) they are
the exact counts, after a stage call that call's."""
import numpy as np
import pytest

from paper_2607_06499_amd import workloads as W
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not H.gpu_ok():
        pytest.skip("no GPU")


def _twins(K, n):
    from paper_2607_06499_amd import binding as B

    s = W.unicycle_static_ahead(3, num_samples=K)
    pls = [B.Planner(s.spec) for _ in range(n)]
    for pl in pls:
        pl.set_nominal(H.to_dev(s.U0))
    return s, pls, H.to_dev(np.asarray(s.x0, np.float32)), H.to_dev(np.asarray(s.obstacles, np.float32))


def _counts(pl, n):
    from paper_2607_06499_amd import binding as B

    return pl.debug(B.DBG_NCOUNT, n).cpu().numpy()


# 2,048 and 2,049: either side of the size to which the labelling compacts
@pytest.mark.parametrize("K", [300, 2048, 2049, 8192])
def test_counts_of_the_last_call(K):
    from paper_2607_06499_amd import binding as B

    torch = H.torch_mod()
    s, (w, bm, bt), x, obs = _twins(K, 3)
    bm.set_dbscan_mode(B.DBSCAN_BITMAP)
    batch = B.Batch([bt])
    batch.set_io([x], [obs])
    w.replan(x, obs)
    bm.replan(x, obs)
    batch.replan()
    torch.cuda.synchronize()
    V = w.info()["n_feasible"]
    assert w.info()["branch"] == 0 and w.info()["n_clusters"] > 0 and V > s.spec.dbscan_min_pts
    exact = _counts(bm, V)
    assert exact.max() > s.spec.dbscan_min_pts
    assert np.array_equal(_counts(w, V), exact)
    # the mode of the next call says nothing about the last one's counts
    for pl in (w, bt):
        pl.set_dbscan_mode(B.DBSCAN_TILED)
        assert np.array_equal(_counts(pl, V), exact)
        pl.set_dbscan_mode(B.DBSCAN_AUTO)
        assert np.array_equal(_counts(pl, V), exact)
    # a stage call's counts and labels, in every mode
    th = np.random.default_rng(K).normal(0.4, 0.5, V - 3)
    z = H.to_dev(np.stack([np.cos(th), np.sin(th)], 1).astype(np.float32))
    for mode in (B.DBSCAN_WINDOW, B.DBSCAN_BITMAP, B.DBSCAN_TILED):
        w.set_dbscan_mode(mode)
        lab, cnt, _ = w.stage_dbscan(z)
        assert np.array_equal(_counts(w, V - 3), cnt.cpu().numpy()), mode
        assert np.array_equal(w.debug(B.DBG_LABEL, V - 3).cpu().numpy(), lab.cpu().numpy()), mode
    # and a replan's again after that
    for pl in (w, bm):
        pl.replan(x, obs)
    torch.cuda.synchronize()
    V = bm.info()["n_feasible"]
    if bm.info()["branch"] == 0:
        assert H.counts_agree(_counts(w, V), _counts(bm, V), s.spec.dbscan_min_pts)  # (the distance passes)
    batch.close()


def test_reading_counts_between_and_beside_replans():
    """Reads before, behind and (from a second stream) beside queued replans are
    accepted and change nothing: every replan equals its twin's."""
    torch = H.torch_mod()
    _, (a, b), x, obs = _twins(8192, 2)
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for call in range(4):
        with torch.cuda.stream(sa):
            torch.cuda._sleep(2_000_000)
            a.replan(x, obs, stream=sa)
        with torch.cuda.stream(sb):
            n = _counts(a, a.K)
        assert n.shape == (a.K,)
        torch.cuda.synchronize()
        b.replan(x, obs)
        torch.cuda.synchronize()
        ra, rb = H.collect_outputs(a), H.collect_outputs(b)
        for k in ("u_out", "U_new", "U_next", "label", "ncount", "z"):
            assert np.array_equal(ra[k], rb[k]), (call, k)
        for k in ra["info"]:
            assert np.array_equal(np.asarray(ra["info"][k]), np.asarray(rb["info"][k])), (call, k)
