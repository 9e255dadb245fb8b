"""Products of fewer than 16 rows: which kernel family they take, and that an fp32 result is as exact as before."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import check, gpu_product


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,out", [("f32", "f32"), ("bf16", "f32"), ("f16", "f32"), ("bf16", "bf16")])
@pytest.mark.parametrize("m,R", [(9, 8), (12, 40), (15, 8), (8, 190), (16, 8)])
def test_fp32_results_keep_their_sums_apart(oracle_mod, dtype, out, m, R):
    """One chain per wavefront over all its blocks is up to three times as inexact as 64 partial sums: below 16 rows an
    fp32 result comes from the wavefront-reduction kernels, bit for bit (8 rows of 190 block-rows of 32: 6080 wavefronts,
    from where on 16-bit results take the matrix cores)."""
    import paper_2007_13055_amd as lib
    bs = 32
    p = wl.make_problem("few", m, 60 * bs, R * bs, bs, bs, dtype, out, ("bernoulli", 0.4), ("normal", 1.0), ("normal", 1.0), 400 + m)
    Yo, So = oracle_mod.bsr_spmm(p.X, p.block_data, p.block_indices, p.index_pointer, p.n)
    Y, W = gpu_product(p)
    check(Y, Yo, So, p.tau, f"{dtype}->{out} m={m} R={R}", out_dtype=out)
    wave, _ = gpu_product(p, path=lib.PATH_WAVE, W=W)
    mfma, _ = gpu_product(p, path=lib.PATH_MFMA, W=W)
    if m < 16 and out == "f32":
        assert np.array_equal(Y, wave)
    else:
        assert np.array_equal(Y, mfma)
    assert lib.bsr_query_path(W, m) == (lib.PATH_WAVE if m < 16 and dtype == "f32" else lib.PATH_MFMA)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,m,k", [("bf16", 9, 1 << 26), ("f16", 15, 1 << 26), ("f32", 16, 1 << 25)])
def test_wide_rows_of_x_stay_accepted(oracle_mod, dtype, m, k):
    """Rows of X beyond the k-split kernel's 32-bit offsets: the library's own choice is a kernel that takes them.  Two
    block-rows of one and two blocks; the oracle sees the columns that they name."""
    import torch
    import paper_2007_13055_amd as lib
    from gpu_util import torch_dtype
    bs, C = 16, k // 16
    cols = np.array([C - 1, 0, C // 3], dtype=np.int32)
    ptr = np.array([0, 1, 3], dtype=np.int32)
    rng = np.random.default_rng(m)
    data = wl.round_to_storage(rng.normal(size=(3, bs, bs)).astype(np.float32), dtype)
    Xs = wl.round_to_storage(rng.normal(size=(m, 3 * bs)).astype(np.float32), dtype)
    X = torch.zeros((m, k), dtype=torch_dtype(dtype), device="cuda")
    for j, c in enumerate(cols):
        X[:, int(c) * bs:(int(c) + 1) * bs] = torch.from_numpy(Xs[:, j * bs:(j + 1) * bs]).to("cuda", torch_dtype(dtype))
    Yo, So = oracle_mod.bsr_spmm(Xs, data, np.arange(3, dtype=np.int32), ptr, 2 * bs)
    W = lib.bsr_create(2 * bs, k, data, cols, ptr, dtype=dtype)
    Y = torch.full((m, 2 * bs), float("nan"), dtype=torch_dtype(dtype), device="cuda")
    lib.bsr_spmm(W, X, Y)
    torch.cuda.synchronize()
    check(Y.double().cpu().numpy(), Yo, So, 1e-5, f"{dtype} m={m} k={k}", out_dtype=dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("bs,variant", [(16, 1), (32, 2), (64, 2)])
def test_short_block_rows(oracle_mod, monkeypatch, bs, variant):
    """Three blocks in every second block-row, 1.5 on average: the direct kernel for 16-row blocks, the k-split kernel
    for few items of taller ones; told by the bits of the kernel forced."""
    import paper_2007_13055_amd as lib
    p = wl.make_problem("short", 64, 20 * bs, 64 * bs, bs, bs, "f32", "f32", ("counts", [3, 0] * 32), ("normal", 1.0), ("normal", 1.0), 77)
    Yo, So = oracle_mod.bsr_spmm(p.X, p.block_data, p.block_indices, p.index_pointer, p.n)
    Y, _ = gpu_product(p)
    check(Y, Yo, So, p.tau, f"short rows {bs}")
    forced = {}
    for v in (1, 2):
        monkeypatch.setenv("BSR_SPMM_TUNE", f"variant={v}")
        forced[v], _ = gpu_product(p, path=lib.PATH_MFMA)
    assert not np.array_equal(forced[1], forced[2]) and np.array_equal(Y, forced[variant])
