"""Small FP32 batches whose grid takes six row tiles per work-group: bitwise what the types give alone (few
enough tiles for work-groups of four), and w within the rounding bound u (N + 4) S of numpy's product, u = 2^-24,
S the sum of the magnitudes of its terms."""
from contextlib import closing

import numpy as np
import pytest

from paper_2410_03632_amd import blast as B
from paper_2410_03632_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ell,n_cheb", [(23, 32), (27, 90), (32, 128)])  # 5, 6 and 6 tiles
@pytest.mark.parametrize("batch,n_g,n_s", [(1, 2, 2), (3, 12, 8), (8, 3, 1), (16, 10, 5)])
def test_six_tiles_per_group(n_ell, n_cheb, batch, n_g, n_s):
    n_chi, n_R, nb = 140, 9, n_g + n_s
    g = np.random.default_rng(n_ell + batch)
    c = g.standard_normal((batch, n_chi, n_R, n_cheb))
    dev = [torch.as_tensor(x).cuda() for x in (c, g.uniform(0.1, 1.0, (batch, nb, n_chi)),
                                               g.uniform(-1.0, 1.0, (batch, nb, n_chi, n_R)))]
    cfg = W.tiny_config(n_ell=n_ell, ell_max=40, n_chi=n_chi, n_R=n_R, n_cheb=n_cheb)
    with closing(B.plan_for_config(cfg, precisions=("fp64", "fp32"))) as plan:
        run = lambda **kw: plan.forward(*dev, n_g, n_s, precision="fp32", coef=True, **kw)
        C = run()
        pairs = W.pair_list(n_g, n_s)
        for t in ("gg", "gs", "ss"):
            sel = [p for p, pr in enumerate(pairs) if pr[0] == t]
            assert torch.equal(run(types=(t,)), C[:, sel])
        w = torch.full((batch * n_chi * n_R * plan.rows_pad,), np.nan, dtype=torch.float32, device="cuda")
        assert torch.equal(run(w_save=w), C)
        wk = w.view(batch, n_chi, n_R, -1)[..., :plan.rows].double().cpu().numpy()
        for a in range(0, n_chi, 23):
            T = np.stack([plan.basis_point(a, b) for b in range(n_R)])
            wr, S = np.einsum("brn,zbn->zbr", T, c[:, a]), np.einsum("brn,zbn->zbr", np.abs(T), np.abs(c[:, a]))
            assert np.all(np.abs(wk[:, a] - wr) <= 2.0 ** -24 * (n_cheb + 4) * S)
