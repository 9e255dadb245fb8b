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
