"""Tiles of the dense step at the edges of their chunks and K-splits.

Batches: matrices whose products are fewer, as many or more chunks than a tile
keeps in flight, with and without a ragged last one, in the persistent schedule
(reserved items, R's loads ahead of the wait) and in grouped launches.  Single
matrices: sizes whose K-split is not a power of two, with a ragged last split.
The reference is the plain recurrence in FP64 numpy on the library's own
probes; FP64 bar 1e-10 relative as in the other parity tests, FP32 TOL_F32.
"""
import ctypes

import numpy as np
import pytest

from test_gpu_pairs import check, reference
from tolerances import tol_for

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1801_01072_amd as ent  # noqa: E402

DEV = "cuda:0"


def symmetric(n, seed):
    """Eigenvalues within [0.2, 0.6] for large n, within [0, 0.9] for small n."""
    X = np.random.default_rng(seed).standard_normal((n, n))
    X = X + X.T
    return 0.4 * np.eye(n) + X * (0.2 / max(2.9 * np.sqrt(n), np.linalg.norm(X, 2) if n < 300 else 0.0))


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("flags", [0, ent.FLAG_BATCH_STEPWISE])
@pytest.mark.parametrize("method,m", [("chebyshev", 6), ("taylor", 5)])
def test_batch_chunk_edges(orc, precision, flags, method, m):
    ns, s, seed = [1, 7, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 95, 96, 97, 127, 128, 129, 161, 257], 33, 3
    host = [symmetric(n, n) for n in ns]
    for i in (5, 12, 19):
        host[i][0, ns[i] - 1] += 0.03  # one moment per product
    g = ent.Graph([torch.from_numpy(R).to(DEV) for R in host], method, m, s, seed, precision=precision,
                  probe_dist="gaussian", u_fixed=0.9, flags=flags | ent.FLAG_SKIP_TRACE_CHECK)
    for _ in range(3):
        g.launch()
        per = g.per_probe()
        for b, R in enumerate(host):
            _, ref = reference(orc, lambda V, R=R: R @ V, ns[b], method, m, s, seed + b, 1, 0.9)
            e = float(np.max(np.abs(per[b] - ref)) / max(np.mean(np.abs(ref)), 1.0))
            assert e <= tol_for(precision), (ns[b], e)
    g.destroy()


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("n,s", [(2200, 128), (2500, 200), (3001, 100), (4500, 256), (2111, 130)])
def test_split_counts(orc, precision, n, s):
    R = symmetric(n, n)
    check(orc, torch.from_numpy(R).to(DEV), lambda V: R @ V, n, "chebyshev", 4, s, 7, 1, precision, "splits")


@pytest.mark.parametrize("precision,n", [("f64", 2897), ("f64", 3001), ("f64", 3072), ("f32", 4097), ("f32", 4162),
                                         ("f32", 4224), ("bf16x3", 2433), ("bf16x3", 2560), ("bf16x3", 3001)])
def test_power_method_on_half_of_r(precision, n):
    """A symmetric R read by half against the same R with one entry moved to the
    next number, which is read whole: sums of FP64 products in another order
    (20 products, n eps each: 2e-11 at most) and the moved entry (2^-24 of 1e-2
    relative to the largest eigenvalue)."""
    dtype = np.float64 if precision == "f64" else np.float32
    R = symmetric(n, n).astype(dtype)
    got = []
    for moved in (False, True):
        if moved:
            R[0, n - 1] = np.nextafter(R[0, n - 1], dtype(1))
        got.append(ent.entropy_estimate(torch.from_numpy(R).to(DEV), "chebyshev", 4, 128, 5, precision=precision,
                                        flags=ent.FLAG_SKIP_TRACE_CHECK))
    print(f"[power half {precision} n={n}] u {got[0].u:.15f} whole {got[1].u:.15f}", flush=True)
    assert 0.2 < got[0].u < 2.0 and abs(got[0].u / got[1].u - 1) <= 1e-9


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 63, 64, 255, 511, 512, 513, 700, 1100])
def test_cutoff_coefficients(orc, m):
    """The projection on [lo, u] of every degree, from the moments the call
    reports: cosines to half an ulp and N terms of size <= 1/e added pairwise
    over 64 lanes (oracle: in turn), N eps / e each side, per coefficient; the
    moments of one probe are at most |g|^2 = n each."""
    n, s, lo, u = 24, 3, 1e-3, 0.5
    R = torch.from_numpy(symmetric(n, 5) * 0.5).to(DEV)
    nodes = orc.cutoff_nodes(m)
    a = orc.cheb_interp_coeffs(lo, u, m, nodes)
    bar = 2 * nodes * 2.3e-16 / np.e * (m + 1) * n
    _, per, mom = ent.entropy_estimate_detail(R, "chebyshev", m, s, 2, precision="f64", u_fixed=u, cutoff=lo,
                                              flags=ent.FLAG_SKIP_TRACE_CHECK)
    want = -(a[:, None] * mom).sum(axis=0)
    print(f"[cutoff m={m}] {np.max(np.abs(per - want)):.2e} bar {bar:.2e}", flush=True)
    assert np.max(np.abs(per - want)) <= bar
    got = ent.entropy_estimate_batched([R, R], "chebyshev", m, s, 2, precision="f64", u_fixed=u, cutoff=lo,
                                       flags=ent.FLAG_SKIP_TRACE_CHECK)
    assert abs(got[0].entropy - np.mean(want)) <= bar + 1e-10 * abs(np.mean(want))


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_batch_power_method_on_half(precision):
    """A batch large enough to read half of each symmetric matrix (and both
    halves of any other) against single estimates, which at these sizes read
    all of it: the same FP64 sums in another order, 20 products of n eps each."""
    dtype = np.float64 if precision == "f64" else np.float32
    ns = [1, 2, 63, 127, 128, 129, 255, 257, 384, 1000] + [1160 if precision == "f32" else 808] * 18
    mats = []
    for b, n in enumerate(ns):
        R = symmetric(n, b).astype(dtype)
        if b in (3, 9, 12):
            R[0, n - 1] += dtype(0.01)
        mats.append(torch.from_numpy(R).to(DEV))
    assert sum(M.nbytes for M in mats) >= 96 << 20
    g = ent.Graph(mats, "chebyshev", 3, 20, 9, precision=precision, flags=ent.FLAG_SKIP_TRACE_CHECK)
    for _ in range(3):
        res = g.launch()
        for b, M in enumerate(mats):
            one = ent.entropy_estimate(M, "chebyshev", 3, 20, 9 + b, precision=precision,
                                       flags=ent.FLAG_SKIP_TRACE_CHECK)
            assert abs(res[b].u / one.u - 1) <= 1e-10, (ns[b], res[b].u, one.u)
    g.destroy()


def split_values(R):
    """R as a BF16x3 call multiplies it: the sum of its bf16 parts, in FP32."""
    X = torch.from_numpy(R)
    hi = X.to(torch.bfloat16).float()
    return (hi + (X - hi).to(torch.bfloat16).float()).numpy()


@pytest.mark.parametrize("precision,n", [("f64", 2897), ("f64", 3001), ("f64", 3072), ("f32", 4097), ("f32", 4162),
                                         ("f32", 4224), ("bf16x3", 2433), ("bf16x3", 2560), ("bf16x3", 3001)])
@pytest.mark.parametrize("t", [1, 20])
def test_power_estimate_on_half_of_r(orc, precision, n, t):
    """p~1 itself (u is clamped at 1) of a symmetric R, read by half, and of the
    same R with one entry moved, read whole, against the oracle's power method
    from the same start vector: t + 1 products, n eps each, 2e-11 at most."""
    R = symmetric(n, n).astype(np.float64 if precision == "f64" else np.float32)
    for moved in (0.0, 0.01):
        R[0, n - 1] += R.dtype.type(moved)
        res = ent.entropy_estimate(torch.from_numpy(R).to(DEV), "chebyshev", 4, 128, 5, precision=precision,
                                   power_iters=t, flags=ent.FLAG_SKIP_TRACE_CHECK)
        want = orc.power_method((split_values(R) if precision == "bf16x3" else R).astype(np.float64), t, 1, 5)
        assert abs(res.p1_est / want - 1) <= 2e-11, (moved, res.p1_est, want)


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("t", [1, 20])
def test_batch_power_estimate_on_half(orc, precision, t):
    """p~1 of every matrix of a batch large enough to read half of each symmetric
    one, three of another kind among them, against the oracle's."""
    dtype = np.float64 if precision == "f64" else np.float32
    ns = [1, 2, 63, 127, 128, 129, 255, 257, 384, 1000] + [1160 if precision == "f32" else 808] * 18
    host = []
    for b, n in enumerate(ns):
        R = symmetric(n, b).astype(dtype)
        if b in (3, 7, 9, 12):
            R[0, n - 1] += dtype(0.01)
        host.append(R)
    assert sum(R.nbytes for R in host) >= 96 << 20
    mats = [torch.from_numpy(R).to(DEV) for R in host]
    want = [orc.power_method(R.astype(np.float64), t, 1, 9 + b) for b, R in enumerate(host)]
    g = ent.Graph(mats, "chebyshev", 3, 20, 9, precision=precision, power_iters=t, flags=ent.FLAG_SKIP_TRACE_CHECK)
    for turn in range(3):
        if turn == 2:  # one more of the other kind, and one less, on replay
            for b, d in ((5, 0.02), (9, -0.01)):
                host[b][0, -1] += dtype(d)
                if b == 9:
                    host[b][0, -1] = host[b][-1, 0]
                mats[b].copy_(torch.from_numpy(host[b]))
                want[b] = orc.power_method(host[b].astype(np.float64), t, 1, 9 + b)
        for b, r in enumerate(g.launch()):
            assert abs(r.p1_est / want[b] - 1) <= 2e-11, (turn, ns[b], r.p1_est, want[b])
    g.destroy()


@pytest.mark.parametrize("precision,ns,count", [
    ("f64", [193, 200, 255, 256, 130], 1150), ("f32", [193, 200, 255, 256, 130], 1150),
    ("f64", [1, 64, 65, 511, 512, 513], 110), ("f64", [513, 640, 641], 40),
    ("f32", [127, 769, 770, 895, 896], 55), ("f32", [800, 769], 330)])
def test_batch_power_estimate_of_others(orc, precision, ns, count):
    """The same on both sides of the rule that reads a matrix unequal to its
    transpose by tiles or by rows, and for more than 4096 tiles of 64 rows: one in
    seven of that kind."""
    dtype = np.float64 if precision == "f64" else np.float32
    kinds = [symmetric(n, n).astype(dtype) for n in ns]
    host = [kinds[b % len(ns)].copy() for b in range(count)]
    for R in host[::7]:
        R[0, -1] += dtype(0.01)
    assert sum(R.nbytes for R in host) >= 96 << 20
    want = [orc.power_method(R.astype(np.float64), 2, 1, 9 + b) for b, R in enumerate(host)]
    g = ent.Graph([torch.from_numpy(R).to(DEV) for R in host], "chebyshev", 3, 20, 9, precision=precision,
                  power_iters=2, flags=ent.FLAG_SKIP_TRACE_CHECK)
    for turn in range(2):
        for b, r in enumerate(g.launch()):
            assert abs(r.p1_est / want[b] - 1) <= 2e-11, (turn, b, r.p1_est, want[b])
    g.destroy()


def direct_tiles(n, s):
    """The library's rule: 0 where the tiled kernel runs."""
    f = getattr(ent._lib, "_ZN3ent18dense_direct_tilesEli")
    f.argtypes, f.restype = [ctypes.c_int64, ctypes.c_int32], ctypes.c_int32
    return f(n, s)


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("schedule", ["chebyshev", "taylor", "clenshaw"])
@pytest.mark.parametrize("n,s,split", [(2111, 130, True), (3001, 100, True), (2048, 200, True), (300, 1500, False),
                                       (257, 2100, False)])
@pytest.mark.parametrize("moved", [0.0, 0.01])
def test_every_schedule_on_tiles(orc, precision, schedule, n, s, split, moved):
    """The K-split product with its epilogue, and the whole tile, in each
    schedule: sizes past the small-problem kernels' rule, both kinds of R."""
    m, seed, u = 4, 11, 0.9
    assert n > 192 and direct_tiles(n, s) == 0
    R = symmetric(n, n)
    R[0, n - 1] += moved
    flags = ent.FLAG_SKIP_TRACE_CHECK | (ent.FLAG_CLENSHAW if schedule == "clenshaw" else 0)
    ent.timing_enable(True)
    try:
        _, per, _ = ent.entropy_estimate_detail(torch.from_numpy(R).to(DEV), "taylor" if schedule == "taylor" else "chebyshev",
                                                m, s, seed, precision=precision, u_fixed=u, probe_dist="gaussian",
                                                flags=flags)
        t = ent.last_timing()
    finally:
        ent.timing_enable(False)
    _, want = reference(orc, lambda V: R @ V, n, "taylor" if schedule == "taylor" else "chebyshev", m, s, seed, 1, u)
    e = float(np.max(np.abs(per - want)) / max(np.mean(np.abs(want)), 1.0))
    assert (t["epilogue_launches"] > 0) == split and e <= tol_for(precision), (t, e)


@pytest.mark.parametrize("n", [3000, 4100])  # up to 1128 and 2145 tiles of 64 x 64: all known at the start, and not
@pytest.mark.parametrize("kind", ["rounded", "corner", "equal"])
def test_symmetry_answer_and_trace(n, kind):
    """Products run and the trace for an R that differs from its transpose almost
    everywhere, in one place of the last tile, and nowhere: the trace to n eps of
    its FP64 sum (every term at least 0.4 / n)."""
    g = torch.Generator(device=DEV).manual_seed(n)
    R = torch.randn((n, n), generator=g, dtype=torch.float64, device=DEV) * (0.01 / n ** 1.5)
    R = R + R.T + torch.diag(torch.rand(n, generator=g, dtype=torch.float64, device=DEV) + 0.5) / n
    if kind == "rounded":
        R = R * (1 + (torch.rand((n, n), generator=g, dtype=torch.float64, device=DEV) - 0.5) * 4e-16)
    elif kind == "corner":
        R[n - 1, n - 2] *= 1 + 1e-12
    trace = float(torch.diagonal(R).sum())
    ent.timing_enable(True)
    try:
        for _ in range(3):
            for side in (-1, 1):
                ent.entropy_estimate(R / trace if side < 0 else R, "chebyshev", 6, 8, 1, u_fixed=1.0,
                                     trace_tol=max(abs(trace - 1), 0.0) + n * 2.3e-16 if side > 0 else n * 2.3e-16)
            assert ent.last_timing()["step_launches"] == (3 if kind == "equal" else 6)
    finally:
        ent.timing_enable(False)
    if abs(trace - 1) > 1e-9:
        with pytest.raises(ent.EntropyError, match="trace"):
            ent.entropy_estimate(R, "chebyshev", 6, 8, 1, u_fixed=1.0, trace_tol=abs(trace - 1) - n * 2.3e-16)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_mismatches_everywhere_cost_no_more_than_none(dtype):
    """The check of an R that rounding made unequal to its transpose everywhere,
    against the same R's in Clenshaw, which asks nothing (u given, one step each):
    the check reads R once, less than a power product of the same call does."""
    import time

    n = 8192
    g = torch.Generator(device=DEV).manual_seed(3)
    R = torch.rand((n, n), generator=g, dtype=dtype, device=DEV) / n ** 2
    R = R + R.T + torch.eye(n, dtype=dtype, device=DEV) / n

    def best(M, **kw):
        times = []
        for _ in range(6):
            t = time.perf_counter()
            ent.entropy_estimate(M, "chebyshev", 2, 8, 1, precision="f64" if dtype == torch.float64 else "f32",
                                 u_fixed=1.0, flags=ent.FLAG_SKIP_TRACE_CHECK, **kw)
            times.append(time.perf_counter() - t)
        return min(times)

    equal = best(R)
    A = R * (1 + (torch.rand((n, n), generator=g, dtype=dtype, device=DEV) - 0.5) * (4e-16 if dtype == torch.float64 else 3e-7))
    unequal = best(A)
    one = R.clone()
    one[0, n - 1] *= 1.5
    late = best(one)
    print(f"[check {dtype}] equal {1e6 * equal:.0f} us, everywhere {1e6 * unequal:.0f}, in one place {1e6 * late:.0f}", flush=True)
    assert unequal <= 1.05 * late
