"""Small batches (contraction and R-quadrature streaming the basis) at the edges of their tiles, against
numpy sums over the plan's own FP64 basis.

P is given as coefficients, so the sums are C = N_t sum_ab (K_i Kt_j + K_j Kt_i) sum_n T_n c_n exactly as
the header states them.  Bound: every product and sum of the path rounds once with unit u (2^-53, or
2^-24 on FP32, whose operands are rounded too), so |dC| <= u (N + n_R + 8) S + 2^-53 (n_chi + 8) S with S
the same sum over the magnitudes of its terms."""
import numpy as np
import pytest

from paper_2410_03632_amd import blast as B
from paper_2410_03632_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

_plans = {}


def _plan(n_cheb, n_ell=7, n_chi=6, n_R=19):
    key = (n_cheb, n_ell, n_chi, n_R)
    if key not in _plans:
        cfg = W.tiny_config(n_ell=n_ell, ell_max=30, n_chi=n_chi, n_R=n_R, n_cheb=n_cheb)
        plan = B.plan_for_config(cfg, precisions=("fp64", "fp32"))
        T = np.stack([[plan.basis_point(a, b) for b in range(n_R)] for a in range(n_chi)])  # [a, b, row, n]
        _plans[key] = plan, T
    return _plans[key]


@pytest.fixture(scope="module", autouse=True)
def _close():
    yield
    for plan, _ in _plans.values():
        plan.close()
    _plans.clear()


def _inputs(plan, batch, nb, seed):
    g = np.random.default_rng(seed)
    c = g.standard_normal((batch, len(plan.chi), len(plan.R), plan.n_cheb))
    K = g.uniform(0.1, 1.0, (batch, nb, len(plan.chi)))
    K2 = g.uniform(-1.0, 1.0, (batch, nb, len(plan.chi), len(plan.R)))
    return c, K, K2


def _reference(plan, T, c, K, K2, ng, ns):
    """(C, S): the sums and the sums of magnitudes, [batch, pair, ell]."""
    out = []
    l = plan.ell
    r = (l + 2) * (l + 1) * l * (l - 1)
    norm = 2 / np.pi * np.stack([np.ones_like(l), np.sqrt(r), r])
    for f in (lambda x: x, np.abs):
        w = np.einsum("abrn,zabn->zabr", f(T), f(c))
        Y = np.einsum("zmab,b,zabr->zmar", f(K2), f(plan.w_R), w).reshape(len(c), ng + ns, len(plan.chi), 3, len(l))
        Kt = f(K * (plan.w_chi * plan.chi))
        rows = []
        for t, i, j in W.pair_list(ng, ns):
            t = ("gg", "gs", "ss").index(t)
            rows.append(norm[t] * (np.einsum("za,zal->zl", Kt[:, i], Y[:, j, :, t]) +
                                   np.einsum("za,zal->zl", Kt[:, j], Y[:, i, :, t])))
        out.append(np.stack(rows, 1))
    return out


def _dev(x, dt=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=dt).cuda()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n_cheb", [5, 32, 64, 90, 128])
@pytest.mark.parametrize("batch,n_g,n_s", [(1, 2, 2), (4, 15, 1), (4, 15, 5), (5, 3, 0), (8, 16, 16), (9, 10, 5),
                                           (16, 1, 3), (17, 4, 4), (31, 10, 10)])
def test_stream_tile_edges(prec, n_cheb, batch, n_g, n_s):
    plan, T = _plan(n_cheb)
    f64 = prec == "fp64"
    c, K, K2 = _inputs(plan, batch, n_g + n_s, 100 * n_cheb + batch)
    ref, S = _reference(plan, T, c, K, K2, n_g, n_s)
    u = 2.0 ** (-53 if f64 else -24)
    tol = u * (plan.n_cheb + len(plan.R) + 8) * S + 2.0 ** -53 * (len(plan.chi) + 8) * S
    args = (_dev(c), _dev(K), _dev(K2), n_g, n_s)
    C = plan.forward(*args, precision=prec, coef=True).cpu().numpy()
    assert np.all(np.abs(C - ref) <= tol), np.max(np.abs(C - ref) / tol)
    # w and Y kept: the same spectra, w the plan's product for every row
    wdt = torch.float64 if f64 else torch.float32
    w = torch.full((batch * len(plan.chi) * len(plan.R) * plan.rows_pad,), np.nan, dtype=wdt, device="cuda")
    y = torch.full((plan.y_numel(batch, n_g + n_s),), np.nan, dtype=wdt, device="cuda")
    C2 = plan.forward(*args, precision=prec, coef=True, w_save=w, y_save=y).cpu().numpy()
    assert np.all(np.abs(C2 - ref) <= tol)
    wk = w.view(batch, len(plan.chi), len(plan.R), plan.rows_pad)[..., :plan.rows].double().cpu().numpy()
    wr, ws = np.einsum("abrn,zabn->zabr", T, c), np.einsum("abrn,zabn->zabr", np.abs(T), np.abs(c))
    assert np.all(np.abs(wk - wr) <= u * (plan.n_cheb + 4) * ws)
    yk = y.view(batch, plan.rows_pad, len(plan.chi), -1)[:, :plan.rows, :, :n_g + n_s].double().cpu().numpy()
    yr, ys = (np.einsum("zmab,b,zabr->zram", k, plan.w_R, x) for k, x in ((K2, wr), (np.abs(K2), ws)))
    assert np.all(np.abs(yk - yr) <= u * (plan.n_cheb + len(plan.R) + 8) * np.abs(ys))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_stream_result_is_the_cosmologys_own(prec):
    """A cosmology's spectra are bitwise the same alone, in any batch and with more bins."""
    plan, T = _plan(64)
    c, K, K2 = _inputs(plan, 31, 9, 3)
    C = plan.forward(_dev(c), _dev(K), _dev(K2), 5, 4, precision=prec, coef=True).cpu().numpy()
    pairs = W.pair_list(5, 4)
    for b0, b1 in ((0, 1), (3, 7), (5, 13), (2, 18), (30, 31)):
        got = plan.forward(_dev(c[b0:b1]), _dev(K[b0:b1]), _dev(K2[b0:b1]), 5, 4, precision=prec, coef=True)
        assert np.array_equal(got.cpu().numpy(), C[b0:b1])
        got = plan.forward(_dev(c[b0:b1]), _dev(K[b0:b1, :5]), _dev(K2[b0:b1, :5]), 5, 0, precision=prec, coef=True,
                           types=("gg",))
        assert np.array_equal(got.cpu().numpy(), C[b0:b1][:, [p for p, pr in enumerate(pairs) if pr[0] == "gg"]])


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("batch", [3, 12])
def test_stream_skips_rows_not_asked_for(prec, batch):
    """Multipole and type subsets (whose other 16-row tiles are not computed) are bitwise slices of the whole:
    with a workspace full of NaN, so that a tile read but not computed would show."""
    plan, T = _plan(32, n_ell=25)
    c, K, K2 = _inputs(plan, batch, 6, 7)
    args = (_dev(c), _dev(K), _dev(K2), 4, 2)
    ws = torch.full((plan.workspace_bytes(batch, prec, 6) // 8,), np.nan, dtype=torch.float64, device="cuda")
    full = plan.forward(*args, precision=prec, coef=True, workspace=ws).cpu().numpy()
    pairs = W.pair_list(4, 2)
    for idx in ([0], [3, 4, 5], [24], list(range(15)), [0, 16, 24]):
        for types in (("gg",), ("ss",), ("gg", "ss"), ("gg", "gs", "ss")):
            sel = [p for p, pr in enumerate(pairs) if pr[0] in types]
            ws.fill_(np.nan)
            got = plan.forward(*args, precision=prec, coef=True, workspace=ws, ell_idx=idx, types=types).cpu().numpy()
            want = full[:, sel][:, :, idx]
            assert np.array_equal(got, want)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n_cheb", [32, 90])
@pytest.mark.parametrize("batch,n_g,n_s", [(32, 3, 1), (33, 10, 5), (40, 16, 4), (100, 2, 2)])
def test_small_grid_large_batch(prec, n_cheb, batch, n_g, n_s):
    """From 32 cosmologies on, grids with few work-groups stream too: within the bound above, and on FP32
    (whose order of summation is the fused kernel's) bitwise what a batch large enough for the fused
    kernel gives the same cosmologies, w and Y included."""
    plan, T = _plan(n_cheb, n_ell=9, n_chi=5, n_R=7)
    nb = n_g + n_s
    c, K, K2 = _inputs(plan, batch, nb, n_cheb + batch)
    ref, S = _reference(plan, T, c, K, K2, n_g, n_s)
    u = 2.0 ** (-53 if prec == "fp64" else -24)
    tol = u * (plan.n_cheb + len(plan.R) + 8) * S + 2.0 ** -53 * (len(plan.chi) + 8) * S
    run = lambda *x, **kw: plan.forward(_dev(x[0]), _dev(x[1]), _dev(x[2]), n_g, n_s, precision=prec, coef=True, **kw)
    C = run(c, K, K2).cpu().numpy()
    assert np.all(np.abs(C - ref) <= tol), np.max(np.abs(C - ref) / tol)
    if prec == "fp32" and nb <= 20:
        many = 16 * (2048 // (5 * 4)) + 32  # past the streaming kernel's waves
        rep = lambda x: np.concatenate([x] * (many // batch + 1))[:many]
        kept = []
        for x in ((c, K, K2), (rep(c), rep(K), rep(K2))):
            n = len(x[0])
            w = torch.zeros(n * 35 * plan.rows_pad, dtype=torch.float32, device="cuda")
            y = torch.zeros(plan.y_numel(n, nb), dtype=torch.float32, device="cuda")
            Cn = run(*x, w_save=w, y_save=y)
            yn = y.view(n, plan.rows_pad, 5, -1)
            # an all-clustering or all-shear row keeps only its own bins' sums on the fused path
            kept.append((Cn[:batch].clone(), w.view(n, -1)[:batch].clone(),
                         yn[:batch, :9, :, :n_g].clone(), yn[:batch, 9:18, :, :nb].clone()))
        for g, h in zip(*kept):
            assert torch.equal(g, h)
        assert np.array_equal(kept[0][0].cpu().numpy(), C)
