"""bench.py's reading of the library's event intervals (no GPU): fused, streamed and unfused calls."""
import os
import sys
import types

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402

CFG = types.SimpleNamespace(n_chi=256, n_R=96, n_cheb=128, n_g=10, n_s=5)
PLAN = types.SimpleNamespace(rows=288, rows_pad=288, n_ell=96)


@pytest.mark.parametrize("prec,batch,ms,kernel,longest", [
    ("fp32", 8, (0.0, 0.004, 0.60, 0.03), "stream_kernel", 0.60),
    ("fp64", 1, (0.0, 0.004, 1.20, 0.02), "stream_kernel", 1.20),
    ("fp64", 17, (0.0, 1.60, 0.40, 0.06), "contract_kernel", 1.60),
    ("fp32", 28, (0.0, 1.00, 0.40, 0.06), "contract_kernel", 1.00),
    ("fp32", 256, (0.0, 0.25, 5.00, 0.29), "contract_quad_kernel", 5.00),
    ("fp64", 256, (0.0, 0.26, 11.5, 0.50), "contract_quad_f64_kernel", 11.5),
    ("fp16x3", 256, (0.0, 0.26, 4.10, 0.30), "contract_quad_wide_kernel", 4.10)])
def test_stages(prec, batch, ms, kernel, longest):
    p = dict(zip(("projection", "contraction", "quad_R", "quad_chi"), ms))
    got, work, kernels = bench.launch_stages(p, PLAN, CFG, prec, batch)
    dom = max((k for k in got if k in work), key=got.get)
    assert dom == "contraction" and got[dom] == longest and kernels[dom] == kernel
    assert 0 < bench.roofline(work[dom], got[dom], prec)["frac"] < 1
    if kernel == "stream_kernel":  # the basis, P, the kernel tables and Y once
        eb = 8 if prec == "fp64" else 4
        NP = 256 * 96
        assert work[dom]["bytes"] == NP * 128 * eb * (288 + batch) + 15 * NP * 8 * batch + 256 * 288 * 16 * eb * batch
        assert "r_weights" not in got and "quad_R" not in got
