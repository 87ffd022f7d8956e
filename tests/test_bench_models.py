"""The byte models behind bench.py's roofline figures (algorithmic HBM bytes
per launch of the sparse step kernels) and the split of the recurrence into
multi-step launches, against closed forms written out by hand for the
workloads' shapes: Chebyshev's m steps pass V 3m - 3 times one step per
launch (V_k from step 1, V_{k-1} from step 2, every step writes), Taylor's
m + 1 steps 2m times (no V_{k-1} term, the last step writes nothing), and a
multi-step launch reads V_k and V_{k-1} once and writes two blocks."""
import bench as B


def test_fuse_split():
    assert B.fuse_split(10, 10) == [10]
    assert B.fuse_split(10, 4) == [4, 3, 3]
    assert B.fuse_split(11, 10) == [6, 5]
    assert B.fuse_split(3, 2) == [2, 1]
    assert B.fuse_split(1, 10) == [1]
    for steps in range(1, 64):
        for nf in range(1, 11):
            sz = B.fuse_split(steps, nf)
            assert sum(sz) == steps and max(sz) <= nf and max(sz) - min(sz) <= 1
            assert sz == sorted(sz, reverse=True) and len(sz) == -(-steps // nf)


def test_tridiagonal_models_poisson():
    n, s, m = 10**8, 100, 10
    diag, signs, blk = 4 * 4 * n, n * s / 8, 4 * n * s
    one, steps = B.tri_step_bytes(n, s, m, 4, "chebyshev")
    assert steps == m and one == m * (diag + signs) + (3 * m - 3) * blk
    tay, tsteps = B.tri_step_bytes(n, s, m, 4, "taylor")
    assert tsteps == m + 1 and tay == (m + 1) * (diag + signs) + 2 * m * blk
    # all ten steps in one launch from the sign bits: two blocks written
    tot, launches = B.tri_fused_bytes(n, s, m, 4, "chebyshev", 10)
    assert launches == 1 and tot == diag + signs + 2 * blk
    # launches of 4, 3 and 3 steps (k = 0, 4, 7): the later two read V_k and V_{k-1}
    tot4, l4 = B.tri_fused_bytes(n, s, m, 4, "chebyshev", 4)
    assert l4 == 3 and tot4 == 3 * (diag + signs) + (2 + 4 + 4) * blk
    # FP64 doubles every stored value, not the sign bits
    t64, _ = B.tri_fused_bytes(n, s, m, 8, "chebyshev", 10)
    assert t64 == 2 * diag + signs + 4 * blk
    # Taylor, m + 1 = 11 steps in launches of 6 and 5: the last launch's last step is not written
    tt, lt = B.tri_fused_bytes(n, s, m, 4, "taylor", 10)
    assert lt == 2 and tt == 2 * (diag + signs) + (2 + (1 + 1)) * blk


def test_banded_models_csr1e7():
    n, hp, s, m = 10**7, 16, 64, 40
    slabs = ((n + 15) // 16) * 16 * (16 + 2 * hp) * 4
    signs, blk = n * s / 8, 4 * n * s
    one, steps = B.band_step_bytes(n, hp, s, m, 4, "chebyshev")
    assert steps == m and one == m * (slabs + signs) + (3 * m - 3) * blk
    pair, pairs = B.band_pair_bytes(n, hp, s, m, 4, "chebyshev")
    # 20 launches: the first writes two blocks, the others read two and write two
    assert pairs == 20 and pair == 20 * (slabs + signs) + (2 + 19 * 4) * blk
    # per recurrence step the pairs move about 37% fewer algorithmic bytes
    # (the counters show 26% fewer: the kernel reads each slab twice, once
    # per 32-probe chunk)
    assert 0.60 < (pair / (2 * pairs)) / (one / steps) < 0.66


def test_general_csr_model():
    n, nnz, s, m = 1000, 7000, 64, 8
    csr = (4 + 4) * nnz + 8 * (n + 1)
    one, steps = B.csr_step_bytes(n, nnz, s, m, 4, "chebyshev")
    assert steps == m and one == m * (csr + n * s / 8) + (3 * m - 3) * 4 * n * s


def test_symmetric_estimates_store_nothing_last():
    n, hp, s, m = 10**7, 16, 64, 40
    slabs = ((n + 15) // 16) * 16 * (16 + 2 * hp) * 4
    signs, blk = n * s / 8, 4 * n * s
    # 40 moments from 20 products: ten pairs, the first writes two blocks, the
    # others read two, and all but the last write two
    k, pair, pairs = B.sparse_model(n, 0, hp, s, m, 4, "chebyshev", 2)
    assert k == "band_pair_kernel" and pairs == 10 and pair == 10 * (slabs + signs) + (2 + 8 * 4 + 2) * blk
    # 38 moments from 19 products: nine pairs, and the last product alone (not counted)
    k, pair, pairs = B.sparse_model(n, 0, hp, s, 38, 4, "chebyshev", 2)
    assert pairs == 9 and pair == 9 * (slabs + signs) + (2 + 8 * 4) * blk
    # Taylor, 42 moments from 21 products: ten pairs, one block read by all but the first
    k, pair, pairs = B.sparse_model(n, 0, hp, s, 41, 4, "taylor", 2)
    assert pairs == 10 and pair == 10 * (slabs + signs) + (2 + 9 * 3) * blk
    # Taylor, 40 moments from 20 products: the last pair writes nothing
    k, pair, pairs = B.sparse_model(n, 0, hp, s, 39, 4, "taylor", 2)
    assert pairs == 10 and pair == 10 * (slabs + signs) + (2 + 8 * 3 + 1) * blk
    # one product per launch: the last reads two and writes none
    k, one, steps = B.sparse_model(n, 0, hp, s, m, 4, "chebyshev", 1)
    assert k == "band_step_kernel" and steps == 20 and one == 20 * (slabs + signs) + (3 * 20 - 3 - 1) * blk
    # tridiagonal, ten moments in one launch: nothing but the signs and the diagonals
    k, tri, launches = B.sparse_model(10**8, 0, 1, 100, 10, 4, "chebyshev", 10)
    assert k == "tri_fused_kernel" and launches == 1 and tri == 16 * 10**8 + 10**8 * 100 / 8
    k, csr, steps = B.sparse_model(1000, 7000, 0, 64, 8, 4, "chebyshev", 1)
    assert k == "csr_step_kernel" and steps == 4
    assert csr == 4 * (8 * 7000 + 8 * 1001 + 1000 * 64 / 8) + (3 * 4 - 3 - 1) * 4 * 1000 * 64


def test_dense_kernel_is_the_librarys():
    import ctypes

    import paper_1801_01072_amd as ent

    f = getattr(ent._lib, "_ZN3ent18dense_direct_tilesEli")
    f.argtypes, f.restype = [ctypes.c_int64, ctypes.c_int32], ctypes.c_int32
    for n in (193, 256, 500, 512, 1000, 1024, 1400, 1800, 2048, 3000, 4096, 4100, 8192, 20000):
        for s in (1, 15, 16, 17, 50, 64, 100, 128, 200, 256, 1500):
            want = "dense_direct_kernel" if f(n, s) else "dense_step_kernel"
            assert B.dense_kernel(n, s, "f32", False) == want, (n, s)
    assert B.dense_kernel(192, 50, "f64", False) == "dense_resident_kernel"
    assert B.dense_kernel(8192, 256, "f64", True) == "dense_step_split_kernel"
