"""Dots in pairs: a symmetric R gives two moments per product, any other R one.

Every path decides from R itself, so each case runs a symmetric R and the same
R with one entry changed, which must give the values of the products R v as
they are.  The reference is the plain recurrence in FP64 numpy on the
library's own probes (drawn by the oracle's generator), one moment per product.
FP64 bar 1e-10 relative as in the other parity tests; reduced precision
TOL_F32 / TOL_BF16X3.
"""
import math

import numpy as np
import pytest

import workloads as W
from tolerances import tol_for

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1801_01072_amd as ent  # noqa: E402

DEV = "cuda:0"


def reference(orc, mul, n, method, m, s, seed, dist, u):
    """(moments, per-probe values) of the forward recurrence; mul(V) = R V."""
    G = orc.probe_block(seed, dist, 0, n, s)
    mom = np.zeros((m + 1, s))
    if method == "taylor":
        V = G.copy()
        for k in range(m + 1):
            Y = mul(V) / u
            mom[k] = np.einsum("ij,ij->j", G, Y)
            V = V - Y
        return mom, math.log(1 / u) + u * (mom[1:] / np.arange(1, m + 1)[:, None]).sum(axis=0)
    prev, cur = None, G
    mom[0] = np.einsum("ij,ij->j", G, G)
    for k in range(m):
        X = 2.0 / u * mul(cur) - cur
        prev, cur = cur, X if prev is None else 2 * X - prev
        mom[k + 1] = np.einsum("ij,ij->j", G, cur)
    return mom, -(orc.cheb_coeffs(u, m)[:, None] * mom).sum(axis=0)


def check(orc, R, mul, n, method, m, s, seed, dist, precision, label, **kw):
    u = 0.9 if n > 1 else 1.0
    res, per, mom = ent.entropy_estimate_detail(R, method, m, s, seed, precision=precision, u_fixed=u,
                                                probe_dist=("rademacher", "gaussian")[dist],
                                                flags=ent.FLAG_SKIP_TRACE_CHECK | kw.get("flags", 0))
    rm, rp = reference(orc, mul, n, method, m, s, seed, dist, u)
    em = float(np.max(np.abs(mom - rm) / np.max(np.abs(rm), axis=0)))
    ep = float(np.max(np.abs(per - rp)) / max(np.mean(np.abs(rp)), 1.0))
    print(f"[pairs {label} n={n} s={s} m={m} {method} {precision}] moments {em:.2e} per-probe {ep:.2e}", flush=True)
    assert em <= tol_for(precision) and ep <= tol_for(precision)
    assert res.products == (m if method == "chebyshev" else m + 1)


@pytest.mark.parametrize("precision", ["f64", "f32", "bf16x3"])
@pytest.mark.parametrize("n,s,m", [(1, 1, 2), (2, 3, 1), (63, 17, 2), (64, 64, 3), (65, 65, 4), (130, 128, 9),
                                   (300, 129, 8), (2048, 8, 5), (3000, 20, 6)])
def test_dense(orc, precision, n, s, m):
    R = W.dense_density(W.spectrum_exp(n, max(n / 5.0, 1.0)), 100 + n)
    cases = [("symmetric", R)]
    if n > 1:
        # one entry off in the last row, next to the diagonal, and in the corner
        for (i, j) in ((n - 1, n - 2), (0, n - 1)):
            A = R.copy()
            A[i, j] += 0.05
            cases.append((f"[{i},{j}] changed", A))
    for label, A in cases:
        Ad = torch.from_numpy(A).to(DEV)
        for method in ("chebyshev", "taylor"):
            check(orc, Ad, lambda V, A=A: A @ V, n, method, m, s, 3 + n, 1, precision, label)
    # a NaN is not equal to itself: refused as before
    A = R.copy()
    A[0, 0] = np.nan
    with pytest.raises(ent.EntropyError) as e:
        ent.entropy_estimate(torch.from_numpy(A).to(DEV), "chebyshev", m, s, 1, precision=precision, u_fixed=0.9)
    assert e.value.status in (ent.ENOTDENSITY, ent.ENUMERIC)


def test_dense_strided_storage(orc):
    # the check reads R as it is stored: odd leading dimension, FP32 storage
    n, m, s = 200, 7, 33
    R = W.dense_density(W.spectrum_exp(n, 40.0), 5).astype(np.float32)
    for off in (0.0, 0.05):
        A = R.copy()
        A[150, 3] += off
        big = torch.zeros((n, n + 3), dtype=torch.float32, device=DEV)
        big[:, 1:n + 1] = torch.from_numpy(A).to(DEV)
        A64 = A.astype(np.float64)
        check(orc, big[:, 1:n + 1], lambda V, A=A64: A @ V, n, "chebyshev", m, s, 4, 0, "f64", f"strided {off}")
