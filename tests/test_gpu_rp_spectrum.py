"""All singular values of a sketch at the edges of the eigenvalue kernels.

sigma^2 are the eigenvalues of the s x s Gram matrix: reduced in registers up to
s = 128, in memory above, each found by its own workgroup.  Against the FP64
oracle: the Gram sums carry n eps lambda_max and the reduction 4 s eps
lambda_max at most.  Spread, equal, few non-zero and tiny eigenvalues; sizes that
split K and that fit one workgroup per tile.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1801_01072_amd as ent  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("s", [1, 2, 3, 4, 15, 16, 17, 63, 64, 65, 127, 128, 129, 200, 256])
@pytest.mark.parametrize("kind", ["spread", "equal", "rank1", "rank3", "tiny"])
def test_all_singular_values(orc, s, kind):
    n, seed = (520 if s % 2 else 300), 11 + s
    p = {"spread": W.spectrum_exp(n, 40.0), "equal": np.full(n, 1.0 / n), "rank1": np.eye(n)[0],
         "rank3": np.eye(n)[0] * 0.5 + np.eye(n)[1] * 0.3 + np.eye(n)[2] * 0.2,
         "tiny": W.spectrum_exp(n, 40.0) * 1e-60}[kind]
    R = np.diag(p) if kind in ("rank1", "rank3", "equal") else W.dense_density(p, n)
    k = min(s, n)
    _, sig, _ = ent.entropy_estimate_detail(torch.from_numpy(R).to(DEV), "randproj", 1, 1, seed, rank_k=k,
                                            sketch_width=s, precision="f64", flags=ent.FLAG_SKIP_TRACE_CHECK)
    _, ref = orc.rp_entropy(R, s, k, seed)
    lam, want = np.asarray(sig) ** 2, np.asarray(ref) ** 2
    err = float(np.max(np.abs(lam - want)) / want.max())
    print(f"[rp spectrum {kind} s={s}] {err:.2e}", flush=True)
    assert np.all(np.diff(sig) <= 0) and err <= (n + 4 * s) * 2.3e-16


@pytest.mark.parametrize("s", [32, 160])
@pytest.mark.parametrize("first", [2, 3, 4])
def test_repeated_values_met_exactly(orc, s, first):
    """A count sketch of a diagonal R on rows of chosen buckets: a Gram matrix
    diag(256 + 1, .., eight 144, ten 143.5, 0, ..) / 2^20 whose 144 the first split
    of [0, 257] into 257 parts meets exactly, eight pivots in turn being zero.
    Every square, sum and point of the split is exact but 143.5's (p^2 within
    2 eps); the bisection ends at 2 ulp."""
    seed, n = 5, 4000
    rows = {}
    for j in range(n):
        rows.setdefault(orc.sketch_bucket(seed, j, s), []).append(j)
    p = np.zeros(n)
    p[rows[0][:2]] = 16.0, 1.0
    for q in range(8):
        p[rows[first + q][0]] = 12.0
    for q in range(10):
        p[rows[first + 8 + q][0]] = np.sqrt(143.5)
    p /= 1024.0
    k = 20
    _, sig, _ = ent.entropy_estimate_detail(torch.from_numpy(np.diag(p)).to(DEV), "randproj", 1, 1, seed, rank_k=k,
                                            sketch_width=s, precision="f64", sketch="count",
                                            flags=ent.FLAG_SKIP_TRACE_CHECK)
    want = np.array([np.sqrt(257.0)] + [12.0] * 8 + [np.sqrt(143.5)] * 10 + [0.0]) / 1024.0
    assert np.allclose(np.asarray(sig), want, rtol=1e-14, atol=1e-12)
