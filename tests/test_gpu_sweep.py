"""The sweep kernel: blocks with sides 8 or 16, many rows of X, swept in windows of 1 KiB of a row."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import check, gpu_product

pytestmark = pytest.mark.gpu


def _problem(m, R, C, bs, dtype, out, seed):
    """Block-rows empty, full, of one block and ordinary ones; columns in any order, some stored twice."""
    rng = np.random.default_rng(seed)
    counts = rng.integers(0, max(2, C // 4), size=R)
    counts[0], counts[-1], counts[R // 2] = 0, 1, C
    p = wl.make_problem("sweep", m, C * bs[1], R * bs[0], bs[0], bs[1], dtype, out, ("counts", counts), ("normal", 1.0), ("normal", 1.0), seed)
    for r in range(R):
        a, b = int(p.index_pointer[r]), int(p.index_pointer[r + 1])
        if r % 3 == 1:
            p.block_indices[a:b] = rng.permutation(p.block_indices[a:b])
        if r % 4 == 2 and b - a > 2:
            p.block_indices[a] = p.block_indices[b - 1]
    return p


@pytest.mark.parametrize("dtype,out", [("f32", "f32"), ("f16", "f16"), ("bf16", "bf16"), ("bf16", "f32")])
@pytest.mark.parametrize("bs", [(8, 8), (8, 16), (16, 8), (16, 16)])
@pytest.mark.parametrize("tune", ["variant=6,mt=4,nw=8", "variant=6,mt=4,nw=1", "variant=6,mt=2,nw=4", "variant=6,mt=1,nw=2",
                                  "variant=6,mt=1,nw=4"])
def test_forced_shapes(oracle_mod, monkeypatch, dtype, out, bs, tune):
    """Workgroups of 1, 2 and 4 tiles of rows by 1 to 8 quads, on both sides of a tile's rows; three windows and a ragged
    fourth, one window, a row of one slab; a last quad with one, two and four groups of 16 rows.  An fp32 result is held to
    one quad up to 256 items of 16 x 16 outputs, to two up to 1024, and to four beyond: the last problem, for those only."""
    import paper_2007_13055_amd as lib
    monkeypatch.setenv("BSR_SPMM_TUNE", tune)
    if bs == (16, 16) and dtype == "f32":             # no plan for these
        with pytest.raises(lib.BsrError):
            gpu_product(_problem(16, 4, 4, bs, dtype, out, 700), path=lib.PATH_MFMA)
        return
    cols = 256 if dtype == "f32" else 512
    problems = [(16, cols // bs[1], 80), (65, (3 * cols + 16) // bs[1], 144), (127, 16 // bs[1], 64), (130, (cols + 48) // bs[1], 608)]
    if out == "f32":
        problems.append((530, (2 * cols + 16) // bs[1], 608))
    for i, (m, C, rows) in enumerate(problems):
        p = _problem(m, rows // bs[0], C, bs, dtype, out, 700 + i)
        Yo, So = oracle_mod.bsr_spmm(p.X, p.block_data, p.block_indices, p.index_pointer, p.n)
        Y, W = gpu_product(p, path=lib.PATH_MFMA)
        check(Y, Yo, So, p.tau, f"{bs} {dtype}->{out} m={m} k={p.k} n={p.n} {tune}", out_dtype=out)
        assert np.array_equal(Y, gpu_product(p, path=lib.PATH_MFMA, W=W)[0])


@pytest.mark.parametrize("dtype,out,m,R,sweeps", [("f16", "f16", 15, 501, False), ("f16", "f16", 16, 247, False), ("f16", "f16", 16, 251, True),
                                                  ("bf16", "bf16", 200, 21, True), ("bf16", "f32", 200, 21, False), ("f32", "f32", 400, 67, False)])
@pytest.mark.parametrize("C", [33, 67])
def test_sizes_without_whole_tiles(oracle_mod, dtype, out, m, R, sweeps, C):
    """n or k an odd multiple of 8: the library's own choice on both sides of where it takes the sweep kernel, told by the
    bits of both; what bsr_query_path() answers for a result of W's type is what runs; a caller that asks for the matrix
    cores gets the sweep kernel for these sizes, and is refused for the others."""
    import paper_2007_13055_amd as lib
    p = _problem(m, R, C, (8, 8), dtype, out, 40 + m)
    Yo, So = oracle_mod.bsr_spmm(p.X, p.block_data, p.block_indices, p.index_pointer, p.n)
    Y, W = gpu_product(p)
    check(Y, Yo, So, p.tau, f"{dtype}->{out} m={m} R={R} C={C}", out_dtype=out)
    wave, _ = gpu_product(p, path=lib.PATH_WAVE, W=W)
    assert np.array_equal(Y, wave) == (not sweeps)
    by_name = sweeps or (dtype, out) == ("bf16", "f32")   # where a result of W's type is swept
    assert lib.bsr_query_path(W, m) == (lib.PATH_MFMA if by_name else lib.PATH_WAVE)
    if not by_name:
        with pytest.raises(lib.BsrError):
            gpu_product(p, path=lib.PATH_MFMA, W=W)
        return
    named, _ = gpu_product(p, path=lib.PATH_MFMA, W=W)
    check(named, Yo, So, p.tau, f"by name, {dtype}->{out} m={m} R={R} C={C}", out_dtype=out)
    assert np.array_equal(Y, named) == sweeps


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("bs", [(8, 8), (8, 16), (16, 8)])
def test_infinities_stay_with_their_blocks(oracle_mod, monkeypatch, dtype, bs):
    """Sizes without whole tiles, infinities and NaN in X: an output is not finite exactly where one of its own stored
    blocks reads such an entry, and the others are those of an X without them."""
    import paper_2007_13055_amd as lib
    p = _problem(203, 67, 67, bs, dtype, dtype, 8)
    rng = np.random.default_rng(1)
    bad = np.zeros(p.X.shape, dtype=bool)
    bad[rng.integers(0, p.m, 40), rng.integers(0, p.k, 40)] = True
    bad[202, -1] = bad[0, 0] = True                   # the last row and column, the first
    p.X[bad] = 0.0
    Yo, So = oracle_mod.bsr_spmm(p.X, p.block_data, p.block_indices, p.index_pointer, p.n)
    reads = np.zeros((p.n, p.k), dtype=bool)          # the columns of X that an output's blocks select
    for r in range(67):
        for c in p.block_indices[p.index_pointer[r]:p.index_pointer[r + 1]]:
            reads[r * bs[0]:(r + 1) * bs[0], c * bs[1]:(c + 1) * bs[1]] = True
    hit = (bad.astype(np.int64) @ reads.T.astype(np.int64)) > 0
    p.X[bad] = rng.choice([np.inf, -np.inf, np.nan], size=int(bad.sum()))
    Y, W = gpu_product(p)
    assert np.array_equal(np.isfinite(Y), ~hit)
    check(np.where(hit, Yo, Y), Yo, So, p.tau, f"{bs} {dtype}", out_dtype=dtype)
    wave, _ = gpu_product(p, path=lib.PATH_WAVE, W=W)
    assert np.array_equal(np.isnan(Y), np.isnan(wave))
    monkeypatch.setenv("BSR_SPMM_TUNE", "variant=6")
    assert np.array_equal(Y, gpu_product(p, path=lib.PATH_MFMA)[0], equal_nan=True)   # the sweep kernel did run


@pytest.mark.parametrize("out", ["bf16", "f32"])
def test_tuning_of_sizes_without_whole_tiles(oracle_mod, out):
    """The trials offer the sweep kernel only for results rounded to 16 bits: an fp32 result keeps the wavefront kernels' 64
    partial sums, whatever was remembered."""
    import paper_2007_13055_amd as lib
    from gpu_util import to_device
    p = _problem(400, 67, 67, (8, 8), "bf16", out, 3)
    W = lib.bsr_create(p.n, p.k, p.block_data, p.block_indices, p.index_pointer, dtype="bf16")
    lib.bsr_tune(W, to_device(p.X, "bf16"), y_dtype=out, trials=3)
    r = lib.bsr_tune_result(W, p.m, out)
    assert (r["path"], r["variant"]) == ((lib.PATH_MFMA, 6) if out == "bf16" else (lib.PATH_WAVE, 0))
    Yo, So = oracle_mod.bsr_spmm(p.X, p.block_data, p.block_indices, p.index_pointer, p.n)
    Y, _ = gpu_product(p, W=W)
    check(Y, Yo, So, p.tau, f"tuned {out}", out_dtype=out)


@pytest.mark.parametrize("dtype,R,C,tiles", [("f16", 64, 64, True), ("f32", 64, 64, True), ("f16", 768, 128, False)])
def test_tuning_offers_both_kernels(oracle_mod, dtype, R, C, tiles):
    """Trials of 8-wide blocks: nine settings of the kernel of 16x16 tiles where W has those, and twelve of the sweep kernel."""
    import paper_2007_13055_amd as lib
    from gpu_util import to_device
    p = _problem(100, R, C, (8, 8), dtype, dtype, 4)
    W = lib.bsr_create(p.n, p.k, p.block_data, p.block_indices, p.index_pointer, dtype=dtype)
    tried, _ = lib.bsr_tune(W, to_device(p.X, dtype), trials=2)
    assert tried == (21 if tiles else 12)
    Yo, So = oracle_mod.bsr_spmm(p.X, p.block_data, p.block_indices, p.index_pointer, p.n)
    Y, _ = gpu_product(p, W=W)
    check(Y, Yo, So, p.tau, dtype, out_dtype=dtype)


@pytest.mark.parametrize("dtype,m,R,C,tiles", [("f32", 383, 80, 200, True), ("f32", 384, 80, 200, False), ("f32", 400, 24, 60, True),
                                               ("f16", 64, 64, 64, True), ("f16", 600, 64, 64, False),
                                               ("bf16", 64, 42, 66, True), ("bf16", 600, 42, 66, False)])
def test_which_kernel(oracle_mod, monkeypatch, dtype, m, R, C, tiles):
    """Both sides of the rules between the sweep kernel and the one of 16x16 tiles, told by the bits."""
    import paper_2007_13055_amd as lib
    p = _problem(m, R, C, (8, 8), dtype, "f32", 9)
    Yo, So = oracle_mod.bsr_spmm(p.X, p.block_data, p.block_indices, p.index_pointer, p.n)
    Y, _ = gpu_product(p)
    check(Y, Yo, So, p.tau, f"{dtype} m={m}")
    forced = {}
    for v in (6, 7):
        monkeypatch.setenv("BSR_SPMM_TUNE", f"variant={v}")
        forced[v], _ = gpu_product(p, path=lib.PATH_MFMA)
    assert np.array_equal(Y, forced[7 if tiles else 6])
    assert not np.array_equal(forced[6], forced[7])


@pytest.mark.parametrize("dtype,out", [("f16", "f16"), ("bf16", "f32")])
@pytest.mark.parametrize("m,R,C,count,other,sweeps", [(600, 96, 376, 40, 2, True), (16, 96, 376, 40, 2, False),
                                                      (300, 400, 128, 40, 4, True), (300, 400, 32, 5, 4, False)])
def test_which_kernel_16x16(oracle_mod, monkeypatch, dtype, out, m, R, C, count, other, sweeps):
    """16x16 blocks: both sides of the rules against the k-split and the stripe kernel, told by the bits of fp32 results."""
    import paper_2007_13055_amd as lib
    p = wl.make_problem("which", m, C * 16, R * 16, 16, 16, dtype, out, ("counts", np.full(R, count)), ("normal", 1.0), ("normal", 1.0), 11)
    Yo, So = oracle_mod.bsr_spmm(p.X, p.block_data, p.block_indices, p.index_pointer, p.n)
    Y, _ = gpu_product(p)
    check(Y, Yo, So, p.tau, f"{dtype}->{out} m={m} R={R} C={C}", out_dtype=out)
    monkeypatch.setenv("BSR_SPMM_TUNE", f"variant={6 if sweeps else other}")
    assert np.array_equal(Y, gpu_product(p, path=lib.PATH_MFMA)[0])
    if out == "f32":
        monkeypatch.setenv("BSR_SPMM_TUNE", f"variant={other if sweeps else 6}")
        assert not np.array_equal(Y, gpu_product(p, path=lib.PATH_MFMA)[0])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_too_sparse_to_sweep(oracle_mod, monkeypatch, dtype):
    """A plan of windows would be larger than W by far: no such plan, and the kernel of 16x16 tiles for any m."""
    counts = np.zeros(4096, dtype=np.int64)
    counts[[5, 6, 2000, 4095]] = 16
    p = wl.make_problem("sparse", 400, 1 << 15, 1 << 15, 8, 8, dtype, "f32", ("counts", counts), ("normal", 1.0), ("normal", 1.0), 2)
    Yo, So = oracle_mod.bsr_spmm(p.X, p.block_data, p.block_indices, p.index_pointer, p.n)
    Y, _ = gpu_product(p)
    check(Y, Yo, So, p.tau, dtype)
    for v in (6, 7):
        monkeypatch.setenv("BSR_SPMM_TUNE", f"variant={v}")
        assert np.array_equal(Y, gpu_product(p)[0])
