"""FP64 and FP32 batches of one to four cosmology tiles on basis points large enough that the number of tiles and how
full the last one is decide between streaming the basis and the contraction through w (one grid on each side of
the FP64 rule's 256 KB): the same sums, so every cosmology's spectra are bitwise those of its own call."""
from contextlib import closing

import numpy as np
import pytest

from paper_2410_03632_amd import blast as B
from paper_2410_03632_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ell,n_chi,n_R,n_cheb", [(45, 128, 4, 68), (96, 57, 3, 128)])
@pytest.mark.parametrize("n_g,n_s", [(3, 2), (14, 3)])
def test_as_single_calls(n_ell, n_chi, n_R, n_cheb, n_g, n_s):
    cfg = W.tiny_config(n_ell=n_ell, ell_max=n_ell + 20, n_chi=n_chi, n_R=n_R, n_cheb=n_cheb, n_g=n_g, n_s=n_s)
    with closing(B.plan_for_config(cfg, precisions=("fp64", "fp32"))) as plan:
        g = np.random.default_rng(n_ell)
        inp = W.make_inputs(cfg, W.seed_for(42), plan.k_nodes, plan.chi, plan.R)
        dev = lambda x: torch.as_tensor(np.ascontiguousarray(x)).cuda()
        b = 31
        P = dev(inp.P[None] * g.uniform(0.5, 1.5, (b, n_chi, n_R, 1)))
        K = dev(inp.Kchi[None] * g.uniform(0.5, 1.5, (b, n_g + n_s, 1)))
        K2 = dev(inp.Kchi2[None] * g.uniform(0.5, 1.5, (b, n_g + n_s, 1, 1)))
        for prec, dt in (("fp64", torch.float64), ("fp32", torch.float32)):
            run = lambda n: plan.forward(P[:n].to(dt).contiguous(), K[:n].contiguous(), K2[:n].contiguous(), n_g, n_s,
                                         precision=prec)
            want = torch.cat([plan.forward(P[i:i + 1].to(dt).contiguous(), K[i:i + 1].contiguous(), K2[i:i + 1].contiguous(),
                                           n_g, n_s, precision=prec) for i in range(b)])
            for n in (8, 9, 10, 16, 17, 19, 20, 21, 24, 25, 31):
                assert torch.equal(run(n), want[:n]), (prec, n)
            some = np.arange(n_ell // 3, dtype=np.int32)  # few enough row tiles to stream in any case
            for n in (17, 31):
                got = plan.forward(P[:n].to(dt).contiguous(), K[:n].contiguous(), K2[:n].contiguous(), n_g, n_s,
                                   precision=prec, ell_idx=some)
                assert torch.equal(got, want[:n, :, :n_ell // 3]), (prec, n)
