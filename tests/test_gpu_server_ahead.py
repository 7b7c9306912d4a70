"""P sent ahead of a launch (pinned requests admitted to a set that still forms): the results are those of
direct calls, also after cancellations move requests to other places of the set, and with pinned and
pageable requests mixed."""
import numpy as np
import pytest

from paper_2410_03632_amd import blast as B
from paper_2410_03632_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pin", ["all", "none", "odd"])
@pytest.mark.parametrize("drop", [(), (2,), (1, 5, 2)])
def test_ahead_of_the_launch(pin, drop):
    cfg = W.tiny_config(n_ell=6, ell_max=40, n_chi=16, n_R=12, n_cheb=32)
    plan = B.plan_for_config(cfg, precisions=("fp32",))
    srv = B.Server(plan, precision="fp32", p_dtype="fp32", batch=8, n_sets=2, max_g=2, max_s=2, max_wait_ms=300.0)
    try:
        idx = np.arange(plan.n_ell, dtype=np.int32)
        reqs, want = [], []
        for i in range(8):
            inp = W.make_inputs(cfg, W.seed_for(33, i), plan.k_nodes, plan.chi, plan.R, vary=True)
            P = torch.as_tensor(inp.P.astype(np.float32))
            if pin == "all" or (pin == "odd" and i % 2):
                P = P.pin_memory()
            reqs.append((P, inp.Kchi, inp.Kchi2))
            dev = lambda x: torch.as_tensor(np.ascontiguousarray(x)[None]).cuda()
            want.append(plan.forward(P.cuda()[None], dev(inp.Kchi), dev(inp.Kchi2), 2, 2, precision="fp32")[0].cpu().numpy())
        # the first request launches at once; those behind it form the next set until 300 ms have passed (or the
        # first is done)
        tk = [srv.submit(*r, 2, 2, idx) for r in reqs]
        gone = set()
        for d in drop:
            try:
                srv.cancel(tk[d])
                gone.add(d)
            except B.BlastError as e:  # already launched
                assert e.status in (B.E_BUSY, B.E_INVALID)
        for i, t in enumerate(tk):
            if i in gone:
                with pytest.raises(B.BlastError) as e:
                    srv.wait(t)
                assert e.value.status == B.E_CANCELLED
            else:
                assert np.array_equal(srv.wait(t)[0], want[i])
    finally:
        srv.close()
        plan.close()
