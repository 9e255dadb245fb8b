"""fp32 results of the sampled product: no kernel sums the rows in longer chains than a workgroup per block does."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import to_device


def _errors(oracle_mod, monkeypatch, m, R, C, bs, dtype, counts, settings, lends):
    """Root mean square errors against 64 bits, of each (setting, lend)."""
    import torch
    import paper_2007_13055_amd as lib
    p = wl.make_problem("prec", m, C * bs[1], R * bs[0], *bs, dtype, dtype, ("counts", counts), ("normal", 1.0), ("normal", 1.0), 50 + m)
    G = wl.round_to_storage(np.random.default_rng(m).normal(size=(m, p.n)).astype(np.float32), dtype)
    Do, _ = oracle_mod.bsr_sddmm(G, p.X, p.block_indices, p.index_pointer, *bs)
    out = {}
    for sd in settings:
        for lend in lends:
            monkeypatch.setenv("BSR_SPMM_TUNE", f"sd={sd}")
            W = lib.bsr_create(p.n, p.k, p.block_data, p.block_indices, p.index_pointer, dtype=dtype)
            D = lib.bsr_sddmm(W, to_device(G, dtype), to_device(p.X, dtype), d_dtype="f32", lend_scratch=lend)
            torch.cuda.synchronize()
            out[sd, lend] = float(np.sqrt(np.mean((D.double().cpu().numpy().ravel() - Do.ravel()) ** 2)))
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("bs,m", [(bs, m) for bs in ((8, 8), (16, 16), (32, 32), (64, 64)) for m in (97, 530, 2100)
                                  if bs[0] > 8 or m > 500])             # 8-wide blocks take the groups from 256 and 512 rows on
def test_groups_are_as_exact_as_blocks(oracle_mod, monkeypatch, bs, dtype, m):
    """Split (with memory for the partial results) and whole.  The order of additions differs and with it the samples'
    error: 6 % is five times what 10 000 values and more leave to chance; one chain over 2100 rows is 100 % off."""
    R, C = 640 // bs[0], 640 // bs[1]
    e = _errors(oracle_mod, monkeypatch, m, R, C, bs, dtype, [max(1, C // 3)] * R, (1, 2), (True, False))
    for lend in (True, False):
        assert e[2, lend] <= 1.06 * e[1, lend], e


@pytest.mark.gpu
@pytest.mark.parametrize("m", [5, 31, 128, 1500])
@pytest.mark.parametrize("per_row", [50, 110, 270])                     # runs of at most 2, 4 and 8 chunks of 16 blocks
def test_thin_blocks_are_as_exact_whichever_kernel(oracle_mod, monkeypatch, per_row, m):
    """Against the lane kernel (four chains of a quarter of the rows) and, from 32 rows on, the transposed copy (two of
    half of them); 3 % for what chance leaves of 30 000 values and more."""
    e = _errors(oracle_mod, monkeypatch, m, 40, 700, (16, 1), "f32", [per_row] * 40, (1, 2), (True, False))
    for lend in (True, False):
        assert e[2, lend] <= 1.03 * e[1, lend], e
