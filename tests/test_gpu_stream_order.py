"""Small grids, on FP64 with the R nodes summed in ranges by up to two waves per row tile: the order of the sums is the
plan's, so a spectrum is bitwise the same whether the call keeps w, Y, both or neither, in any batch below 32, and
alone or among bins that bring the call past 16 (as the server's bin buckets do)."""
from contextlib import closing

import numpy as np
import pytest

from paper_2410_03632_amd import blast as B
from paper_2410_03632_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# grids of 1 to 16 row tiles that take 1 to 4 ranges, with and without shared tiles, and R nodes that do not divide
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n_ell,n_chi,n_R", [(20, 64, 32), (5, 9, 61), (23, 75, 29), (80, 20, 47), (12, 128, 33)])
def test_bitwise_the_same(n_ell, n_chi, n_R, prec):
    cfg = W.tiny_config(n_ell=n_ell, ell_max=2 * n_ell + 20, n_chi=n_chi, n_R=n_R, n_cheb=32, n_g=4, n_s=3)
    dt = torch.float64 if prec == "fp64" else torch.float32
    with closing(B.plan_for_config(cfg, precisions=("fp64", "fp32"))) as plan:
        g = np.random.default_rng(n_R)
        b = 5
        inp = W.make_inputs(cfg, W.seed_for(41), plan.k_nodes, plan.chi, plan.R)
        dev = lambda x: torch.as_tensor(np.ascontiguousarray(x)).cuda()
        P = dev(inp.P[None] * g.uniform(0.5, 1.5, (b, n_chi, n_R, 1))).to(dt)
        K, K2 = dev(inp.Kchi[None] * g.uniform(0.5, 1.5, (b, 7, 1))), dev(inp.Kchi2[None] * g.uniform(0.5, 1.5, (b, 7, 1, 1)))
        run = lambda *a, **kw: plan.forward(*a, precision=prec, **kw)
        want = run(P, K, K2, 4, 3)
        for kw, ky in ((0, 1), (1, 0), (1, 1)):
            w = torch.empty(b * n_chi * n_R * plan.rows_pad, dtype=dt, device="cuda") if kw else None
            y = torch.empty(plan.y_numel(b, 7), dtype=dt, device="cuda") if ky else None
            assert torch.equal(run(P, K, K2, 4, 3, w_save=w, y_save=y), want), (kw, ky)
        one = run(P[2:3].contiguous(), K[2:3].contiguous(), K2[2:3].contiguous(), 4, 3)
        assert torch.equal(one[0], want[2])
        many = [x.repeat(6, *[1] * (x.dim() - 1))[:27].contiguous() for x in (P, K, K2)]
        assert torch.equal(run(*many, 4, 3)[25], want[0])
        # ten more clustering bins without a kernel: 14 + 3
        put = lambda x: torch.cat([x[:, :4], torch.zeros_like(x[:, :1]).repeat(1, 10, *[1] * (x.dim() - 2)), x[:, 4:]], 1).contiguous()
        got = run(P, put(K), put(K2), 14, 3)
        i4, i14 = np.triu_indices(4), np.triu_indices(14)
        at = {p: k for k, p in enumerate(zip(*map(tuple, i14)))}
        gg = [at[p] for p in zip(*map(tuple, i4))]
        pairs = gg + [105 + 3 * i + j for i in range(4) for j in range(3)] + list(range(105 + 42, 105 + 48))
        assert torch.equal(got[:, pairs], want)
