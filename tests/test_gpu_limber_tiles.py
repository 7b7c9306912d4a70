"""The Limber kernel at the edges of its tiles (16 multipoles, 64 chi nodes, 16 bins) against the oracle.

Bound: both sides sum n_chi products in FP64, and the extended bracket's third derivative cancels:
its weights sum to about 8 (chi / h)^3 / 6 times nu^-2 against the bracket itself, h the node spacing.
So |dC_ij| <= 64 eps max(n_chi, (chi / h)^3 / nu^2) sqrt(C_ii C_jj), the auto spectra those of the
first-order sum (all its terms positive), with f_t and N_t geometric means over the two legs as well."""
import numpy as np
import pytest

from oracle import limber_approx as L
import oracle as O
from paper_2410_03632_amd import blast as B
from paper_2410_03632_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ell,n_chi,n_g,n_s", [(1, 5, 1, 1), (16, 64, 11, 5), (17, 65, 12, 5), (33, 63, 16, 16),
                                                 (15, 70, 1, 0), (5, 12, 0, 17)])
@pytest.mark.parametrize("order,sub", [(1, False), (2, True)])
def test_limber_tile_edges(n_ell, n_chi, n_g, n_s, order, sub):
    cfg = W.tiny_config(n_ell=n_ell, ell_max=60 if n_ell > 1 else 2, n_chi=n_chi, n_R=2, n_cheb=8, n_g=n_g, n_s=n_s)
    chi, wchi = O.grid_chi(cfg.n_chi, cfg.chi_min, cfg.chi_max)
    plan = B.Plan(cfg.ells(), chi, wchi, *O.grid_R(2, cfg.R_min), cfg.k_min, cfg.k_max, 8)
    try:
        K, _ = W.kernels(W.bins_of(cfg), chi, chi[:, None] * np.ones((1, 2)))
        kl = plan.limber_k()
        P, S = [], []
        for b in range(2):
            cos = W.draw_cosmo(np.random.default_rng(W.seed_for(6, 200 + b)), vary=True)
            S.append(W.p_limber(kl, chi, cos))
            P.append(W.p_limber(kl, chi, cos, nonlinear=True))
        dev = lambda x: torch.as_tensor(np.ascontiguousarray(x)).cuda()
        C = plan.limber(dev(np.stack(P)), dev(np.stack([K, 0.7 * K])), n_g, n_s, order=order,
                        P_sub=dev(np.stack(S)) if sub else None).cpu().numpy()
        types = [t for t, n in (("gg", n_g), ("gs", n_g * n_s), ("ss", n_s)) if n]
        pairs = W.pair_list(n_g, n_s)
        h = (cfg.chi_max - cfg.chi_min) / (n_chi - 1)
        amp = np.maximum(n_chi, (cfg.chi_max / h) ** 3 / (plan.ell + 0.5) ** 2 if order == 2 else 0.0)
        for b in range(2):
            Kb = K * (0.7 if b else 1.0)
            ref = L.cl_limber(plan.ell, chi, wchi, Kb, n_g, n_s, P[b], P_sub=S[b] if sub else None, order=order)
            auto = L.cl_limber(plan.ell, chi, wchi, Kb, n_g, n_s, P[b], order=1)
            diag = {i: auto[p] for p, (t, i, j) in enumerate(pairs) if i == j}
            for p, (t, i, j) in enumerate(pairs):
                tol = 64 * np.finfo(float).eps * amp * np.sqrt(diag[i] * diag[j])
                assert np.all(np.abs(C[b, p] - ref[p]) <= tol), (types, b, p, np.abs(C[b, p] - ref[p]) / tol)
    finally:
        plan.close()
