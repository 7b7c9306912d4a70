"""FP64 nodal P with rows of no whole padded length, followed in memory by NaN: a read past its last row would meet the
basis' zero columns and make NaN of the last point's sums.  Streamed, fused and w-keeping calls, and the adjoint."""
from contextlib import closing

import numpy as np
import pytest

from paper_2410_03632_amd import blast as B
from paper_2410_03632_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_cheb", [2, 34, 90, 126])
@pytest.mark.parametrize("batch,n_g,n_s,keep", [(1, 2, 1, False), (6, 3, 2, True), (33, 3, 2, False), (33, 3, 2, True),
                                                (70, 3, 2, False), (31, 15, 5, False)])
def test_nan_past_the_end(n_cheb, batch, n_g, n_s, keep):
    cfg = W.tiny_config(n_ell=5, ell_max=30, n_chi=6, n_R=5, n_cheb=n_cheb, n_g=n_g, n_s=n_s)
    with closing(B.plan_for_config(cfg)) as plan:
        g = np.random.default_rng(n_cheb)
        nb = n_g + n_s
        buf = torch.full((batch * 30 * n_cheb + 1024,), float("nan"), dtype=torch.float64, device="cuda")
        P = buf[:batch * 30 * n_cheb].view(batch, 6, 5, n_cheb)
        P.copy_(torch.as_tensor(g.uniform(0.5, 1.5, P.shape)))
        dev = lambda *s: torch.as_tensor(g.uniform(0.5, 1.5, s)).cuda()
        K, K2, dC = dev(batch, nb, 6), dev(batch, nb, 6, 5), dev(batch, B.n_pairs(n_g, n_s), 5)
        w = torch.empty(batch * 30 * plan.rows_pad, dtype=torch.float64, device="cuda") if keep else None
        assert torch.isfinite(plan.forward(P, K, K2, n_g, n_s, w_save=w)).all()
        for d in plan.backward(P, K, K2, n_g, n_s, dC, w_save=w):
            assert torch.isfinite(d).all()
