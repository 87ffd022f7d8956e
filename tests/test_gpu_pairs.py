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
                                   (300, 129, 8), (2048, 8, 5), (3000, 20, 6), (300, 1500, 4), (1500, 300, 4),
                                   (2100, 130, 5), (128, 16, 31), (129, 33, 6), (192, 40, 7), (193, 40, 7)])
def test_dense(orc, precision, n, s, m):
    # sizes on both sides of the lines between the step kernels: R in registers
    # (up to 192, padded to 64), 16, 32 and 64 probes per workgroup of the
    # small-problem kernel (193 x 40, 3000 x 20, 300 x 129), the tiled kernel whole (300 x 1500) and with K split (1500 x
    # 300, 2100 x 130)
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


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 150, 192, 193])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_small_power_method_and_clenshaw(orc, n, dtype):
    # one launch for every trial and product, and for Clenshaw's schedule
    R = W.dense_density(W.spectrum_exp(n, max(n / 3.0, 1.0)), 7 + n).astype(dtype)
    Rd = torch.from_numpy(R).to(DEV)
    for t, q in ((0, 1), (1, 2), (20, 3)):
        assert ent.power_method(Rd, t, q, 5) == pytest.approx(orc.power_method(R, t, q, 5), rel=1e-12)
    prec = "f64" if dtype == np.float64 else "f32"
    for m, s in ((1, 5), (2, 16), (9, 17)):
        _, per, mom = ent.entropy_estimate_detail(Rd, "chebyshev", m, s, 3, precision=prec, probe_dist="gaussian",
                                                  flags=ent.FLAG_CLENSHAW, trace_tol=1e-4)
        ref = orc.estimate(R, 1, m, s, 3, dist=1)
        e = float(np.max(np.abs(per - ref.per_probe)) / max(np.mean(np.abs(ref.per_probe)), 1.0))
        print(f"[small clenshaw {prec} n={n} m={m} s={s}] per-probe {e:.2e}", flush=True)
        assert e <= tol_for(prec)


def test_small_problem_within_the_workspace_limit():
    """The small-problem kernels need more partial sums than the tiled one: a
    limit that held the estimate before still holds it (on the tiled kernel)."""
    n, m, s = 300, 400, 64
    R = torch.from_numpy(W.dense_density(W.spectrum_exp(n, 60.0), 3)).to(DEV)
    free = ent.entropy_estimate_detail(R, "chebyshev", m, s, 2)
    blocks = 3 * 320 * 64 * 8                # G and two V blocks
    part = (m + 1) * 64 * 8                  # one tile's partials
    ent.release_workspace()
    try:
        ent.set_workspace_limit(blocks + 5 * part + (m + 1) * s * 8 + 200_000)
        held = ent.entropy_estimate_detail(R, "chebyshev", m, s, 2)
        ent.set_workspace_limit(blocks + 5 * part)
        with pytest.raises(ent.EntropyError) as e:
            ent.entropy_estimate(R, "chebyshev", m, s, 2)
        assert e.value.status == ent.ENOMEM
    finally:
        ent.set_workspace_limit(0)
        ent.release_workspace()
    assert held[0].entropy == pytest.approx(free[0].entropy, rel=1e-12)
    assert np.max(np.abs(held[2] - free[2])) <= 1e-10 * float(np.max(free[2]))


def test_dense_strided_storage(orc):
    # the check reads R as it is stored (odd leading dimension, FP32 storage);
    # n is no multiple of the 32 columns a wave takes at a time
    n, m, s = 200, 7, 33
    R = W.dense_density(W.spectrum_exp(n, 40.0), 5).astype(np.float32)
    for off in (0.0, 0.05):
        A = R.copy()
        A[150, 3] += off
        big = torch.zeros((n, n + 3), dtype=torch.float32, device=DEV)
        big[:, 1:n + 1] = torch.from_numpy(A).to(DEV)
        A64 = A.astype(np.float64)
        check(orc, big[:, 1:n + 1], lambda V, A=A64: A @ V, n, "chebyshev", m, s, 4, 0, "f64", f"strided {off}")


def sparse_csr(A, order=None):
    """int64/int32 CSR arrays of a scipy matrix; order: reverses the entries of every row."""
    A = A.tocsr()
    A.sort_indices()
    rp, ci, val = A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data.copy()
    if order == "reversed":
        for i in range(A.shape[0]):
            ci[rp[i]:rp[i + 1]] = ci[rp[i]:rp[i + 1]][::-1].copy()
            val[rp[i]:rp[i + 1]] = val[rp[i]:rp[i + 1]][::-1].copy()
    return rp, ci, val, A.shape[0]


def to_dev(csr, dtype):
    return (torch.from_numpy(csr[0]).to(DEV), torch.from_numpy(csr[1]).to(DEV),
            torch.from_numpy(csr[2].astype(dtype)).to(DEV), csr[3])


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("kind,n,s,m", [("tri", 1, 1, 2), ("tri", 2, 3, 3), ("tri", 65, 100, 4), ("tri", 1000, 130, 21),
                                        ("band", 17, 33, 2), ("band", 300, 64, 5), ("band", 1030, 65, 8),
                                        ("wide", 700, 50, 3), ("wide", 900, 66, 6), ("arrow", 500, 40, 4)])
def test_sparse(orc, kind, n, s, m, dtype):
    """Every sparse form, each with R as it is, with one value or one entry of
    one triangle changed, and with rows whose columns do not ascend (the
    general kernels then keep one moment per product)."""
    import scipy.sparse as sp

    rng = np.random.default_rng(n + m)
    if kind == "tri":
        off = rng.uniform(-1, 1, max(n - 1, 0))
        A = sp.diags([off, rng.uniform(2, 3, n), off], [-1, 0, 1], shape=(n, n))
    elif kind == "band":
        rp, ci, val, _ = W.banded_density_csr(n, 6, seed=n)
        A = sp.csr_matrix((val, ci, rp), shape=(n, n))
    elif kind == "wide":
        B = sp.random(n, n, density=5.0 / n, random_state=rng, format="csr") + sp.eye(n, format="csr")
        A = B @ B.T
    else:  # one long row and column: at most three entries per row on average
        v = rng.uniform(-0.02, 0.02, n - 1)
        A = sp.lil_matrix((n, n))
        A[0, 1:], A[1:, 0] = v, v.reshape(-1, 1)
        A.setdiag(rng.uniform(0.5, 1.0, n))
    A = (A * (0.8 / abs(A).sum(axis=1).max())).astype(dtype).astype(np.float64).tocsr()
    A.sort_indices()
    cases = [("symmetric", A, None, 0)]
    if n > 1:
        V = A.copy()
        V.data[V.indptr[n - 1]] *= 1.5     # last row, leftmost entry
        D = A.tolil()
        row = np.flatnonzero(D[0].toarray().ravel())
        D[0, row[-1]] = 0.0                # first row, rightmost entry
        D = D.tocsr()
        D.eliminate_zeros()
        cases += [("value changed", V, None, 0), ("entry dropped", D, None, 0), ("reversed rows", A, "reversed", 0),
                  ("general", A, None, ent.FLAG_CSR_GENERAL), ("general, changed", V, None, ent.FLAG_CSR_GENERAL)]
    for label, M, order, flags in cases:
        Rd = to_dev(sparse_csr(M, order), dtype)
        for method in ("chebyshev", "taylor"):
            for dist in (0, 1):
                check(orc, Rd, lambda V, M=M: M @ V, n, method, m, s, 7 + n, dist,
                      "f64" if dtype == np.float64 else "f32", f"{kind} {label} {dist}", flags=flags)


@pytest.mark.parametrize("fuse", ["2", "3", "7"])
def test_tridiagonal_launch_splits(orc, monkeypatch, fuse):
    # the moments dealt to several launches, some of one product
    import scipy.sparse as sp

    n, s = 517, 70
    rng = np.random.default_rng(1)
    off = rng.uniform(-1, 1, n - 1)
    A = (sp.diags([off, rng.uniform(2, 3, n), off], [-1, 0, 1]) * 0.15).tocsr()
    monkeypatch.setenv("ENT_TRI_FUSE", fuse)
    for m in (2, 3, 9, 10, 23):
        for method in ("chebyshev", "taylor"):
            for dist in (0, 1):
                check(orc, to_dev(sparse_csr(A), np.float64), lambda V: A @ V, n, method, m, s, 5, dist, "f64",
                      f"tri fuse {fuse}")


@pytest.mark.parametrize("precision", ["f64", "f32", "bf16x3"])
@pytest.mark.parametrize("flags", [0, ent.FLAG_BATCH_STEPWISE])
@pytest.mark.parametrize("changed", [(), (1, 4), (0, 1, 2, 3, 4)])
def test_batch(orc, precision, flags, changed):
    """Each matrix of a batch decides for itself, in every replay: none, some
    or all of them unequal to their transpose (the values are changed in place
    between replays of one graph, and back)."""
    ns, s, seed = [33, 64, 65, 200, 300], 40, 11
    host = [W.dense_density(W.spectrum_exp(n, n / 5.0), 50 + n) for n in ns]
    mats = [torch.from_numpy(R).to(DEV) for R in host]
    for method, m in (("chebyshev", 7), ("taylor", 6)):
        g = ent.Graph(mats, method, m, s, seed, precision=precision, probe_dist="gaussian", u_fixed=0.9, flags=flags)
        for touch in ((), changed, ()):
            for b in touch:
                mats[b][ns[b] - 1, 0] += 0.05
            torch.cuda.synchronize()
            g.launch()
            per = g.per_probe()
            for b in touch:
                mats[b].copy_(torch.from_numpy(host[b]))
            for b, R in enumerate(host):
                A = R.copy()
                if b in touch:
                    A[ns[b] - 1, 0] += 0.05
                _, ref = reference(orc, lambda V, A=A: A @ V, ns[b], method, m, s, seed + b, 1, 0.9)
                e = float(np.max(np.abs(per[b] - ref)) / max(np.mean(np.abs(ref)), 1.0))
                print(f"[pairs batch {precision} {flags} {method} changed {touch}] b={b} per-probe {e:.2e}", flush=True)
                assert e <= tol_for(precision)
        g.destroy()


def hub_csr(n, h, chain, entry=0.0):
    """Laplacian / trace of a star with hub h, and a chain through all vertices
    where `chain` (more than three entries a row); `entry` is added to R[h, n - 1]."""
    A = np.zeros((n, n))
    A[h, :] = A[:, h] = -1.0
    if chain:
        i = np.arange(n - 1)
        A[i, i + 1] = A[i + 1, i] = -0.5
    np.fill_diagonal(A, 0.0)
    np.fill_diagonal(A, -A.sum(axis=1))
    A /= np.trace(A)
    A[h, n - 1] += entry
    return A


@pytest.mark.parametrize("n", [512, 514, 1500])  # hub rows up to, just over and far over a wave's
@pytest.mark.parametrize("chain", [False, True])
@pytest.mark.parametrize("entry", [0.0, 1e-9])
def test_hub_rows(orc, n, chain, entry):
    """One row much longer than the others, at the start, inside and at the end:
    the right values, from half the products exactly where R = R^T."""
    import scipy.sparse as sp

    m, s = 9, 8
    for h in (0, 700 % n, n - 2):
        A = hub_csr(n, h, chain, entry)
        csr = sparse_csr(sp.csr_matrix(A))
        ent.timing_enable(True)
        try:
            check(orc, to_dev(csr, np.float64), lambda V: A @ V, n, "chebyshev", m, s, 3, 0, "f64", f"hub {h}",
                  flags=ent.FLAG_CSR_GENERAL if chain else 0)
            steps = ent.last_timing()["step_launches"]
        finally:
            ent.timing_enable(False)
        assert steps == (m if entry else (m + 1) // 2)


def test_hub_row_costs_no_more_than_it_saves():
    """A star of 200000 vertices, u given: one product for two moments, against
    Clenshaw's three for the same degree, which asks nothing about R^T."""
    import time

    n = 200_000
    i = torch.arange(1, n, device=DEV)
    z, v = torch.zeros_like(i), torch.arange(n, device=DEV)
    rows, cols = torch.cat([i, z, v]), torch.cat([z, i, v])
    d = torch.ones(n, dtype=torch.float64, device=DEV)
    d[0] = n - 1
    vals = torch.cat([torch.full((2 * n - 2,), -1.0, dtype=torch.float64, device=DEV), d]) / (2.0 * (n - 1))
    order = torch.argsort(rows * n + cols)
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(rows, minlength=n), dim=0, out=rp[1:])
    R = (rp, cols[order].to(torch.int32).contiguous(), vals[order].contiguous(), n)

    def best(flags):
        times = []
        for _ in range(4):
            t = time.perf_counter()
            ent.entropy_estimate(R, "chebyshev", 2, 16, 1, u_fixed=1.0, flags=flags)
            times.append(time.perf_counter() - t)
        return min(times)

    pairs, clenshaw = best(0), best(ent.FLAG_CLENSHAW)
    print(f"[hub] pairs {1e3 * pairs:.1f} ms, Clenshaw {1e3 * clenshaw:.1f} ms", flush=True)
    assert pairs < clenshaw


@pytest.mark.parametrize("n,s", [(2048, 256), (1024, 64), (192, 64)])
@pytest.mark.parametrize("changed", [False, True])
def test_moment_sums_in_fp64(orc, n, s, changed):
    """Moments of a diagonal R whose Chebyshev vectors are exact, so that sums alone
    round: R in {0, 1/4, 1/2}, u = 1/2, T_w in {-1, 0, 1}, V_k = T_k g.  A partial sum
    over 16 or 64 rows carries a few half-ulps of its size, independent of each
    other: at most 0.1 n eps over the probes, root mean square, with the doubling of
    a pair; the additions of the partials one by one would carry 0.7 n eps (1.4)."""
    m, seed = 8, 21
    x = np.array([-1.0, 0.0, 1.0])[np.arange(n) % 3]
    R = np.diag((x + 1.0) / 4.0)
    if changed:
        R[0, n - 1] = 2.0 ** -60  # one moment per product, the same vectors to 1e-18
    G = orc.probe_block(seed, 1, 0, n, s)
    _, _, mom = ent.entropy_estimate_detail(torch.from_numpy(R).to(DEV), "chebyshev", m, s, seed, precision="f64",
                                            u_fixed=0.5, probe_dist="gaussian", flags=ent.FLAG_SKIP_TRACE_CHECK)
    g2 = G.astype(np.longdouble) ** 2
    prev, cur = np.ones(n), x
    for w in range(m + 1):
        t = prev if w == 0 else cur
        want = (t[:, None] * g2).sum(axis=0)
        rms = float(np.sqrt(np.mean((mom[w] - want) ** 2)))
        print(f"[sums n={n} w={w}] {rms / (n * 2.0 ** -52):.3f} n eps", flush=True)
        assert rms <= 0.4 * n * 2.0 ** -52
        if w > 0:
            prev, cur = cur, 2.0 * x * cur - prev
