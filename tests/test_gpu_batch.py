"""Batched estimates (grouped launches, hipGraph, autotuned tile shape)
against the FP64 CPU oracle, matrix by matrix and probe by probe."""
import numpy as np
import pytest

import workloads as W
from tolerances import TOL_BF16X3, TOL_F32

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1801_01072_amd as ent  # noqa: E402

DEV = "cuda:0"


def make_batch(ns, seed, dtype=np.float64):
    rng = np.random.default_rng(seed)
    mats, host = [], []
    for i, n in enumerate(ns):
        k = int(rng.integers(max(1, n // 8), n + 1))
        p = W.spectrum_dirichlet(n, k, 0.5, rng)
        R = W.dense_density(p, seed * 1000 + i).astype(dtype)
        host.append(R)
        mats.append(torch.from_numpy(R).to(DEV))
    return mats, host


NS = [33, 64, 100, 129, 200, 257, 300, 511, 700]


@pytest.mark.parametrize("method", ["chebyshev", "taylor"])
def test_batch_fp64_parity(orc, method):
    mats, host = make_batch(NS, 3)
    m, s, seed = 12, 24, 100
    g = ent.Graph(mats, method, m, s, seed, precision="f64", probe_dist="gaussian")
    res = g.launch()
    per = g.per_probe()
    for b, R in enumerate(host):
        ref = orc.estimate(R, 0 if method == "taylor" else 1, m, s, seed + b, dist=1)
        scale = max(np.mean(np.abs(ref.per_probe)), 1e-2)
        err = np.max(np.abs(per[b] - ref.per_probe)) / scale
        print(f"[batch f64 {method}] b={b} n={R.shape[0]} H gpu={res[b].entropy:.12f} "
              f"oracle={ref.entropy:.12f} per-probe err={err:.2e}", flush=True)
        assert err <= 1e-10
        assert res[b].p1_est == pytest.approx(ref.p1_est, rel=1e-12)
    g.destroy()


def test_batch_graph_replays_and_eager_agree():
    mats, host = make_batch(NS, 5, dtype=np.float32)
    g = ent.Graph(mats, "chebyshev", 20, 64, 7, precision="f32")
    eager = ent.entropy_estimate_batched(mats, "chebyshev", 20, 64, 7, precision="f32")
    first = None
    for rep in range(3):
        res = g.launch()
        vals = [r.entropy for r in res]
        if first is None:
            first = vals
        assert vals == first                       # every replay is bitwise identical
        _ = torch.ones(1000, device=DEV).sum().item()   # eager work between replays
    assert first == [r.entropy for r in eager]      # graph == eager run
    _, tm = g.time_eager()
    assert tm["step_launches"] == 20 and tm["steps_ms"] > 0
    g.destroy()


def test_batch_fp32_against_oracle(orc):
    mats, host = make_batch(NS, 7, dtype=np.float32)
    m, s, seed = 20, 64, 11
    g = ent.Graph(mats, "chebyshev", m, s, seed, precision="f32")
    res = g.launch()
    per = g.per_probe()
    for b, R in enumerate(host):
        ref = orc.estimate(R, 1, m, s, seed + b)
        rel = abs(res[b].entropy - ref.entropy) / abs(ref.entropy)
        err = np.max(np.abs(per[b] - ref.per_probe)) / max(np.mean(np.abs(ref.per_probe)), 1e-2)
        print(f"[batch f32] b={b} n={R.shape[0]} rel={rel:.2e} per-probe={err:.2e}", flush=True)
        assert rel <= TOL_F32 and err <= TOL_F32
    g.destroy()


def test_batch_autotune_choice(tmp_path, monkeypatch):
    monkeypatch.setenv("ENT_AUTOTUNE_CACHE", str(tmp_path / "tune.json"))
    mats, host = make_batch([256, 384, 1024, 130], 9, dtype=np.float32)
    g1 = ent.Graph(mats, "chebyshev", 10, 64, 1, precision="f32", flags=ent.FLAG_AUTOTUNE)
    assert g1.tile_rows in (64, 128)
    r1 = g1.launch()
    g2 = ent.Graph(mats, "chebyshev", 10, 64, 1, precision="f32")  # default tile shape
    r2 = g2.launch()
    for a, b in zip(r1, r2):
        assert a.entropy == pytest.approx(b.entropy, rel=1e-5)
    g1.destroy()
    g2.destroy()


def test_batch_errors():
    mats, _ = make_batch([64, 80], 2)
    bad = torch.eye(50, dtype=torch.float64, device=DEV) * 0.5
    with pytest.raises(ent.EntropyError) as e:
        ent.entropy_estimate_batched(mats + [bad], "chebyshev", 5, 8, 0, precision="f64")
    assert e.value.status == ent.ENOTDENSITY and "matrix 2" in e.value.message
    with pytest.raises(ent.EntropyError) as e:
        ent.entropy_estimate_batched(mats, "chebyshev", 5, 300, 0, precision="bf16x3")
    assert e.value.status == ent.EUNSUPPORTED


@pytest.mark.parametrize("method,dtype", [("chebyshev", np.float32), ("taylor", np.float64)])
def test_batch_bf16x3_against_oracle(orc, method, dtype):
    # grouped split / power / GEMM / epilogue: each matrix and probe against
    # the FP64 oracle at the reduced-precision bar
    mats, host = make_batch(NS, 13, dtype=dtype)
    m, s, seed = 16, 40, 21
    g = ent.Graph(mats, method, m, s, seed, precision="bf16x3", probe_dist="gaussian")
    assert g.tile_rows == 128
    res = g.launch()
    per = g.per_probe()
    for b, R in enumerate(host):
        ref = orc.estimate(R.astype(np.float64), 0 if method == "taylor" else 1, m, s, seed + b, dist=1)
        scale = max(np.mean(np.abs(ref.per_probe)), 1e-2)
        err = np.max(np.abs(per[b] - ref.per_probe)) / scale
        rel = abs(res[b].entropy - ref.entropy) / max(abs(ref.entropy), 1e-2)
        print(f"[batch bf16x3 {method}] b={b} n={R.shape[0]} rel={rel:.2e} per-probe={err:.2e}", flush=True)
        assert err <= TOL_BF16X3 and rel <= TOL_BF16X3
        assert res[b].p1_est == pytest.approx(ref.p1_est, rel=1e-6)
    # replays are bitwise identical and equal to the eager sequence
    again = [r.entropy for r in g.launch()]
    assert again == [r.entropy for r in res]
    eager, tm = g.time_eager()
    assert [r.entropy for r in eager] == again
    assert tm["step_launches"] == (m if method == "chebyshev" else m + 1)
    g.destroy()


def test_persistent_schedule_matches_stepwise(orc):
    # the persistent step schedule (default) and one grouped launch per step
    # give bit-identical results (same tile bodies, same reduction order)
    mats, host = make_batch(NS, 19, dtype=np.float32)
    for prec in ("f32", "bf16x3", "f64"):
        gp = ent.Graph(mats, "chebyshev", 14, 64, 5, precision=prec)
        gs = ent.Graph(mats, "chebyshev", 14, 64, 5, precision=prec, flags=ent.FLAG_BATCH_STEPWISE)
        assert gp.window_bytes > 0 and gs.window_bytes == 0
        rp, rs = gp.launch(), gs.launch()
        assert [r.entropy for r in rp] == [r.entropy for r in rs]
        assert np.array_equal(gp.per_probe(), gs.per_probe())
        # replays of the persistent graph stay identical
        _ = torch.ones(1000, device=DEV).sum().item()
        assert [r.entropy for r in gp.launch()] == [r.entropy for r in rp]
        gp.destroy()
        gs.destroy()
    # Taylor through the persistent schedule against the oracle
    g = ent.Graph(mats, "taylor", 9, 32, 3, precision="f64", probe_dist="gaussian")
    res = g.launch()
    per = g.per_probe()
    for b, R in enumerate(host):
        ref = orc.estimate(R.astype(np.float64), 0, 9, 32, 3 + b, dist=1)
        assert np.max(np.abs(per[b] - ref.per_probe)) / max(np.mean(np.abs(ref.per_probe)), 1e-2) <= 1e-10
    g.destroy()


def test_persistent_wait_bound_reports_failure(monkeypatch):
    # a bound of zero polls: a step of a matrix whose previous step is still
    # running gives up at once; the kernel exits normally and the launch
    # reports ENT_EDEVICE (one matrix of 16 row tiles: its step-1 items are
    # taken right after its step-0 items, before those can have finished)
    monkeypatch.setenv("ENT_SCHED_SPIN_LIMIT", "0")
    R = torch.from_numpy(W.dense_density(W.spectrum_exp(2048, 200.0), 3)).to(DEV)
    g = ent.Graph([R], "chebyshev", 12, 64, 1, precision="f32")
    assert g.window_bytes > 0
    with pytest.raises(ent.EntropyError) as ei:
        for _ in range(3):
            g.launch()
    assert ei.value.status == ent.EDEVICE and "bound" in ei.value.message
    g.destroy()
    monkeypatch.delenv("ENT_SCHED_SPIN_LIMIT")
    g = ent.Graph([R], "chebyshev", 12, 64, 1, precision="f32")
    assert np.isfinite(g.launch()[0].entropy)
    g.destroy()


def test_autotune_choices_are_kept_apart(tmp_path, monkeypatch):
    """The step shape and schedule are timed for what runs: each method, and both
    kinds of batch (one matrix unequal to its transpose doubles the steps)."""
    import json

    path = tmp_path / "tune.json"
    monkeypatch.setenv("ENT_AUTOTUNE_CACHE", str(path))

    def keys():
        return set(json.loads(path.read_text()))

    mats = [W.dense_density(W.spectrum_exp(n, n / 5.0), 31 + n) for n in (96, 130, 150)]
    mats = [0.5 * (R + R.T) for R in mats]
    seen = []
    for changed in (False, True):
        if changed:
            mats[1][0, 5] += 1e-3
        dev = [torch.from_numpy(R).to(DEV) for R in mats]
        for method in ("chebyshev", "taylor"):
            for again in (0, 1):
                g = ent.Graph(dev, method, 7, 16, 1, precision="f64",
                              flags=ent.FLAG_AUTOTUNE | ent.FLAG_SKIP_TRACE_CHECK)
                g.launch()
                g.destroy()
                seen.append(keys())
    new = [len(b - a) for a, b in zip(seen, seen[1:])]
    assert new == [0, 1, 0, 1, 0, 1, 0], new
