"""The launch a planner takes when its caller has not set a mode gives the bits
of both modes, on the chains on either side of the rule (2-D features on the
angular windows, compacting with the labels or before them; the bitmap; 3-D
features), with input and output buffers that change from call to call."""
import numpy as np
import pytest

from paper_2607_06499_amd import workloads as W
from tests import harness as H

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not H.gpu_ok():
        pytest.skip("no GPU")


@pytest.mark.parametrize("mk,bitmap", [(lambda: W.unicycle_dynamic_ahead(5, num_samples=2048), False),
                                       (lambda: W.unicycle_dynamic_ahead(5, num_samples=2049), False),
                                       (lambda: W.unicycle_dynamic_ahead(5, num_samples=1500), True),
                                       (lambda: W.arm6_dynamic(3, 700), False)],
                         ids=["window_2048", "window_2049", "bitmap", "arm"])
def test_unset_mode_agrees(mk, bitmap):
    from paper_2607_06499_amd import binding as B

    torch = H.torch_mod()
    s = mk()
    out = []
    for mode in (None, B.LAUNCH_GRAPH, B.LAUNCH_DIRECT):
        pl = B.Planner(s.spec)
        if mode is not None:
            pl.set_launch_mode(mode)
        if bitmap:
            pl.set_dbscan_mode(B.DBSCAN_BITMAP)
        pl.set_nominal(torch.as_tensor(s.U0).cuda())
        r = []
        for call in range(4):
            # fresh buffers, kept so that no address comes back
            x = H.to_dev(np.asarray(s.x0, np.float32) + 0.01 * call)
            obs = H.to_dev(np.asarray(s.obstacles, np.float32))
            pl.u_out, pl.U_out = torch.zeros_like(pl.u_out), torch.zeros_like(pl.U_out)
            pl.replan(x, obs)
            torch.cuda.synchronize()
            r.append((pl.u_out.cpu().numpy().copy(), pl.U_out.cpu().numpy().copy(),
                      pl.info_buf.cpu().numpy().copy(), x, obs, pl.u_out, pl.U_out))
        out.append(r)
        pl.close()
    for r in out[1:]:
        for a, b in zip(out[0], r):
            for q in range(3):
                assert np.array_equal(a[q], b[q])
