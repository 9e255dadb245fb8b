"""The k-split kernel on strips of 16 rows of a block, and small m on the matrix cores."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import check, gpu_product


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,out", [("f32", "f32"), ("f16", "f16"), ("bf16", "f32")])
@pytest.mark.parametrize("bs", [(32, 32), (64, 64), (32, 64), (64, 16)])
@pytest.mark.parametrize("tune", ["", "variant=2,mt=3", "variant=2,mt=3,nw=16,a=1"])
def test_strips_of_blocks(oracle_mod, monkeypatch, dtype, out, bs, tune):
    """Rows of X on both sides of one tile; block-rows empty, of one block, and longer than the descriptor's inline
    list; forced strips with the default and with 16 wavefronts, and whatever the library takes by itself."""
    import paper_2007_13055_amd as lib
    if tune:
        monkeypatch.setenv("BSR_SPMM_TUNE", tune)
    counts = [3, 0, 40, 1, 17]
    for m in (1, 9, 16, 17, 70):
        p = wl.make_problem("strip", m, 40 * bs[1], len(counts) * bs[0], bs[0], bs[1], dtype, out, ("counts", counts),
                            ("normal", 1.0), ("normal", 1.0), 900 + m)
        Yo, So = oracle_mod.bsr_spmm(p.X, p.block_data, p.block_indices, p.index_pointer, p.n)
        Y, W = gpu_product(p, path=lib.PATH_MFMA if tune else lib.PATH_AUTO)
        check(Y, Yo, So, p.tau, f"strips {bs} {dtype}->{out} m={m} {tune}", out_dtype=out)
        Y2, _ = gpu_product(p, path=lib.PATH_MFMA if tune else lib.PATH_AUTO, W=W)
        assert np.array_equal(Y, Y2)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,bs", [("f32", 16), ("f32", 32), ("bf16", 32)])
@pytest.mark.parametrize("longest", [15, 16])
def test_one_long_row_beside_short_ones(oracle_mod, monkeypatch, dtype, bs, longest):
    """Both sides of the rule between the direct and the k-split kernel, told by the bits of fp32 results."""
    import paper_2007_13055_amd as lib
    counts = np.ones(400, dtype=np.int64)
    counts[7] = longest
    p = wl.make_problem("long", 100, 40 * bs, 400 * bs, bs, bs, dtype, "f32", ("counts", counts), ("normal", 1.0), ("normal", 1.0), 5)
    Yo, So = oracle_mod.bsr_spmm(p.X, p.block_data, p.block_indices, p.index_pointer, p.n)
    Y, _ = gpu_product(p)
    check(Y, Yo, So, p.tau, f"{dtype} {bs} longest={longest}", out_dtype="f32")
    forced = {}
    for v in (1, 2):
        monkeypatch.setenv("BSR_SPMM_TUNE", f"variant={v}")
        forced[v], _ = gpu_product(p, path=lib.PATH_MFMA)
    assert np.array_equal(Y, forced[2 if longest >= 16 else 1])
    assert not np.array_equal(forced[1], forced[2])


@pytest.mark.gpu
@pytest.mark.parametrize("R,longest,variant", [(300, 20, 1), (66, 90, 2)])
def test_long_row_of_many_items(oracle_mod, monkeypatch, R, longest, variant):
    """More (block-row, 16 rows) items than a work list holds: both sides of the estimate between the two kernels."""
    import paper_2007_13055_amd as lib
    counts = np.ones(R, dtype=np.int64)
    counts[7] = longest
    p = wl.make_problem("long", 2100, 90 * 16, R * 16, 16, 16, "f32", "f32", ("counts", counts), ("normal", 1.0), ("normal", 1.0), 6)
    Yo, So = oracle_mod.bsr_spmm(p.X, p.block_data, p.block_indices, p.index_pointer, p.n)
    Y, _ = gpu_product(p)
    check(Y, Yo, So, p.tau, f"R={R} longest={longest}")
    for v in (1, 2):
        monkeypatch.setenv("BSR_SPMM_TUNE", f"variant={v}")
        assert np.array_equal(Y, gpu_product(p, path=lib.PATH_MFMA)[0]) == (v == variant)
