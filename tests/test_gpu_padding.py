"""Unused columns of a pass's last tile are nobody's neighbours, whatever the
features and the radius: one feature at a large marker value is noise, and with a
radius whose square overflows FP32 a point has exactly V neighbours.  Through the
allocation-free entry point, the distance and the bitmap passes of a planner, the
small planners' one block and a batch's sorted passes."""
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


def _features(V, p):
    """Three groups and isolated points (non-core columns) on the unit sphere."""
    rng = np.random.default_rng(10 * V + p)
    centre = rng.normal(size=(3, p))
    z = centre[rng.integers(0, 3, V)] + 0.1 * rng.normal(size=(V, p))
    z[::7] = rng.normal(size=(len(z[::7]), p))
    return (z / np.linalg.norm(z, axis=1, keepdims=True)).astype(np.float32)


def _planner(p, V, eps, min_pts):
    from paper_2607_06499_amd import binding as B

    spec = W.PlannerSpec(dynamics=W.UNICYCLE if p == 2 else W.ARM6, num_samples=V, dbscan_eps=eps,
                         dbscan_min_pts=min_pts, dh=W.arm_dh([0.2] * 6)).rounded()
    return B.Planner(spec)


def _each_pass(p, z, eps, min_pts):
    """(name, labels, counts, clusters) of every pass on the features z."""
    from paper_2607_06499_amd import binding as B

    zd = H.to_dev(z)
    yield "noalloc", *[t.cpu().numpy() for t in B.dbscan_noalloc(zd, eps, min_pts)]
    pl = _planner(p, len(z), eps, min_pts)
    for mode in (B.DBSCAN_TILED, B.DBSCAN_BITMAP, B.DBSCAN_AUTO):
        pl.set_dbscan_mode(mode)
        yield f"mode {mode}", *[t.cpu().numpy() for t in pl.stage_dbscan(zd)]
    pl.close()


@pytest.mark.parametrize("marker", [1e30, -1e30, 3e38])
@pytest.mark.parametrize("V", [100, 129, 4095, 5003])
@pytest.mark.parametrize("p", [2, 3])
def test_marker_feature_is_noise(p, V, marker):
    eps, min_pts, at = 0.25, 8, V // 2
    z = _features(V, p)
    z[at] = np.float32(marker)
    z64, e32 = z.astype(np.float64), float(np.float32(eps))
    olab = oracle.dbscan(z64, e32, min_pts)[0]
    assert olab[at] == -1
    for name, lab, cnt, M in _each_pass(p, z, eps, min_pts):
        tag = f"{name} p={p} V={V}"
        # the closed ball holds the point itself, unless its own distance is not a number
        assert lab[at] == -1 and cnt[at] == 1, (tag, lab[at], cnt[at])
        H.dbscan_check(z64, e32, min_pts, cnt, lab, 0.5 * H.STAGE_BAND * e32, exact_ref=olab, tag=tag)
        assert int(M[0]) == int(lab.max()) + 1, tag


@pytest.mark.parametrize("V", [1, 100, 129, 4095, 5003])
@pytest.mark.parametrize("p", [2, 3])
def test_radius_whose_square_overflows(p, V):
    z = _features(V, p)
    for min_pts in (V, V + 20):
        for name, lab, cnt, M in _each_pass(p, z, 1e20, min_pts):
            tag = f"{name} p={p} V={V} min_pts={min_pts}"
            assert np.all(cnt == V), (tag, cnt.min(), cnt.max())
            assert np.all(lab == (0 if min_pts == V else -1)) and int(M[0]) == (1 if min_pts == V else 0), tag


@pytest.mark.parametrize("K", [200, 300])
def test_replans_with_a_radius_whose_square_overflows(K):
    """K = 200: the small planners' block (bitmap), the distance passes and a
    batch's sorted passes; K = 300: the bitmap kernels.  min_pts is one more than
    the feasible rollouts, fewer than the columns of their tiles: no cluster."""
    from paper_2607_06499_amd import binding as B

    torch = H.torch_mod()
    s = P._arm_ahead(1, K)
    x, obs = H.to_dev(np.asarray(s.x0, np.float32)), H.to_dev(np.asarray(s.obstacles, np.float32))

    def planner(mode, min_pts):
        pl = B.Planner(s.spec.replace(dbscan_eps=1e20, dbscan_min_pts=min_pts).rounded())
        pl.set_dbscan_mode(mode)
        pl.set_nominal(H.to_dev(s.U0))
        return pl

    first = H.gpu_replan(planner(B.DBSCAN_TILED, 1), s.x0, s.obstacles)["info"]
    V = first["n_feasible"]
    assert first["branch"] == 0 and first["n_clusters"] == 1 and V % 128
    batch_pl = planner(B.DBSCAN_TILED, V + 1)
    batch = B.Batch([batch_pl])
    batch.set_io([x], [obs])
    batch.replan()
    torch.cuda.synchronize()
    infos = [batch_pl.info()]
    for mode in (B.DBSCAN_TILED, B.DBSCAN_BITMAP):
        pl = planner(mode, V + 1)
        infos.append(H.gpu_replan(pl, s.x0, s.obstacles)["info"])
        assert np.all(pl.debug(B.DBG_NCOUNT, V).cpu().numpy() == V), mode
        pl.close()
    for i in infos:
        assert i["n_feasible"] == V and i["n_clusters"] == 0 and i["selected"] == -1, i
    batch.close()
