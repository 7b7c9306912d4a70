"""FP64 adjoint of the R-quadrature (dK_chi2 from w and dY, dw from dY): with an infinite w, and at a number of R nodes
and multipoles whose padded tables do not fit the LDS of the matrix-core kernel."""
from contextlib import closing

import numpy as np
import pytest

from paper_2410_03632_amd import blast as B
from paper_2410_03632_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _dev(x):
    return torch.as_tensor(np.ascontiguousarray(x)).cuda()


@pytest.mark.parametrize("n_ell", [1, 7, 16])
def test_infinite_w(n_ell):
    """One coefficient of one point is infinite: dK_chi2 there is the sum over the multipoles' rows, infinite where their
    w all have one sign (dY has), and not NaN from the rows that pad the tile."""
    n_chi, n_R = 6, 5
    chi, wchi = B.grid_chi_simpson(n_chi, 200.0, 2000.0)
    R, wR = B.grid_R_fejer(n_R, 0.3)
    ell = np.arange(2, 2 + n_ell)
    with closing(B.Plan(ell, chi, wchi, R, wR, 1e-3, 0.3, 32, types=("gg",))) as plan:
        g = np.random.default_rng(7)
        c = g.uniform(0.5, 1.0, (2, n_chi, n_R, 32))
        K, K2 = g.uniform(0.5, 1.0, (2, 2, n_chi)), g.uniform(0.5, 1.0, (2, 2, n_chi, n_R))
        dC = np.full((2, 3, n_ell), 1.0)

        def run(c):
            w = torch.empty(2 * n_chi * n_R * plan.rows_pad, dtype=torch.float64, device="cuda")
            plan.forward(_dev(c), _dev(K), _dev(K2), 2, 0, coef=True, w_save=w)
            return plan.backward(_dev(c), _dev(K), _dev(K2), 2, 0, _dev(dC), coef=True, w_save=w, want=("K_chi2",))[2].cpu().numpy(), \
                w.view(2, n_chi, n_R, -1)[..., :n_ell].cpu().numpy()
        fine, _ = run(c)
        bad = c.copy()
        bad[1, 2, 3, 0] = np.inf
        got, w = run(bad)
        at = np.zeros(got.shape, bool)
        at[1, :, 2, 3] = True
        assert np.array_equal(got[~at], fine[~at]) and np.isfinite(fine).all()
        inf = w[1, 2, 3]
        assert np.isinf(inf).all()
        if (inf > 0).all() or (inf < 0).all():
            assert np.isinf(got[at]).all(), got[at]
        else:
            assert np.isnan(got[at]).all()


def test_tables_beyond_the_matrix_core_kernel():
    n_chi, n_R, n_ell, n_c, nb = 4, 640, 190, 8, 3
    cfg = W.tiny_config(n_ell=n_ell, ell_max=300, n_chi=n_chi, n_R=n_R, n_cheb=n_c, n_g=2, n_s=1)
    with closing(B.plan_for_config(cfg)) as plan:
        rp, rows = plan.rows_pad, plan.rows
        assert (640 * 18 + 16 * (rp + 2)) * 8 > 160 * 1024 >= (640 * 16 + rp * 17) * 8  # adj_w_kernel's shapes
        g = np.random.default_rng(8)
        c = g.standard_normal((2, n_chi, n_R, n_c))
        K, K2 = g.uniform(0.5, 1.0, (2, nb, n_chi)), g.uniform(-1.0, 1.0, (2, nb, n_chi, n_R))
        dC = g.standard_normal((2, B.n_pairs(2, 1), n_ell))
        w = torch.empty(2 * n_chi * n_R * rp, dtype=torch.float64, device="cuda")
        plan.forward(_dev(c), _dev(K), _dev(K2), 2, 1, coef=True, w_save=w)
        dP, _, dK2 = plan.backward(_dev(c), _dev(K), _dev(K2), 2, 1, _dev(dC), coef=True, w_save=w, want=("P", "K_chi2"))
        l = plan.ell
        norm = 2 / np.pi * np.stack([np.ones_like(l), np.sqrt((l + 2) * (l + 1) * l * (l - 1)),
                                     (l + 2) * (l + 1) * l * (l - 1)])
        dY, mag = np.zeros((2, 3, n_ell, n_chi, nb)), np.zeros((2, 3, n_ell, n_chi, nb))
        Kt = K * (plan.w_chi * plan.chi)
        for p, (t, i, j) in enumerate(W.pair_list(2, 1)):
            t = ("gg", "gs", "ss").index(t)
            d = (norm[t] * dC[:, p])[:, :, None]
            for m, o in ((j, i), (i, j)):
                dY[:, t, :, :, m] += d * Kt[:, o][:, None]
                mag[:, t, :, :, m] += np.abs(d * Kt[:, o][:, None])
        dY, mag = (x.reshape(2, rows, n_chi, nb) for x in (dY, mag))
        u = 2.0 ** -53
        wr = w.view(2, n_chi, n_R, rp)[..., :rows].cpu().numpy()
        want = np.einsum("zabr,zram,b->zmab", wr, dY, plan.w_R, optimize=True)
        S = np.einsum("zabr,zram,b->zmab", np.abs(wr), mag, plan.w_R, optimize=True)
        assert np.all(np.abs(dK2.cpu().numpy() - want) <= u * (rows + 16) * S)
        dw = np.einsum("zmab,zram,b->zabr", K2, dY, plan.w_R, optimize=True)
        dwS = np.einsum("zmab,zram,b->zabr", np.abs(K2), mag, plan.w_R, optimize=True)
        dP = dP.cpu().numpy()
        for a, b in ((0, 0), (1, 639), (3, 317), (2, 16)):
            T = plan.basis_point(a, b)
            assert np.all(np.abs(dP[:, a, b] - dw[:, a, b] @ T) <= u * (rows + 24) * (dwS[:, a, b] @ np.abs(T)))
