"""Which kernel the sampled product takes by itself, with memory for its splits and without: told by its bits, which are
those of the kernel forced, and right by the oracle."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import check, to_device

# m, block-rows, block-columns, block, type, stored blocks, kernel with memory, kernel without
RULES = [
    (5000, 32, 32, (32, 32), "bf16", 13, "groups", "block"),         # few blocks, many rows: worth it only split
    (2000, 32, 32, (32, 32), "bf16", 13, "block", "block"),
    (4096, 48, 40, (16, 16), "bf16", 1400, "groups", "groups"),      # many lines: worth it unsplit
    (4000, 32, 32, (32, 32), "f16", 300, "block", "block"),          # 307 MB of lines
    (4000, 32, 32, (32, 32), "f16", 400, "groups", "block"),         # 410 MB
    (300, 20, 30, (8, 8), "bf16", 100, "groups", "groups"),
    (250, 20, 30, (8, 8), "bf16", 100, "block", "block"),
    (3000, 90, 90, (8, 8), "f32", 2400, "block", "block"),           # 1.8 GB of lines
    (3500, 90, 90, (8, 8), "f32", 2400, "groups", "groups"),         # 2.2 GB
    (1600, 20, 20, (64, 64), "f32", 40, "groups", "block"),          # fp32: few blocks, split
    (1100, 60, 60, (32, 32), "f32", 1500, "block", "block"),         # matrix cores busy either way
    (1100, 30, 100, (64, 16), "f32", 1500, "block", "block"),
    (5800, 13, 20, (64, 16), "f32", 75, "groups", "block"),
    (1100, 100, 100, (16, 16), "f32", 4000, "groups", "groups"),     # 1.1 GB of lines
    (3000, 34, 2880, (16, 1), "f32", 4200, "groups", "block"),       # thin: rows split, or a lane per column
    (6, 270, 3264, (16, 1), "f32", 88000, "groups", "groups"),       # no row to split
    (8, 300, 2256, (16, 1), "f32", 15500, "block", "block"),
    (100, 160, 4096, (16, 1), "f32", 33000, "block", "groups"),      # transposed copy, or turned over in LDS
]


def _matrix(rng, R, C, bs, dtype, blocks):
    at = np.sort(rng.choice(R * C, size=blocks, replace=False))
    ptr = np.zeros(R + 1, dtype=np.int32)
    np.cumsum(np.bincount(at // C, minlength=R), out=ptr[1:])
    return np.zeros((blocks, *bs), dtype=np.float32), (at % C).astype(np.int32), ptr


def _run(p, bs, dtype, sd, monkeypatch, G, X, lend):
    import torch
    import paper_2007_13055_amd as lib
    if sd:
        monkeypatch.setenv("BSR_SPMM_TUNE", f"sd={sd}")
    else:
        monkeypatch.delenv("BSR_SPMM_TUNE", raising=False)
    data, idx, ptr = p
    W = lib.bsr_create(G.shape[1], X.shape[1], data, idx, ptr, dtype=dtype)
    D = torch.full((len(idx), *bs), float("nan"), device="cuda")
    lib.bsr_sddmm(W, G, X, D, d_dtype="f32", lend_scratch=lend)
    torch.cuda.synchronize()
    return D.double().cpu().numpy().reshape(len(idx), -1)


@pytest.mark.gpu
@pytest.mark.parametrize("m,R,C,bs,dtype,blocks,lent,alone", RULES)
def test_choice_of_kernel(oracle_mod, monkeypatch, m, R, C, bs, dtype, blocks, lent, alone):
    rng = np.random.default_rng(blocks)
    p = _matrix(rng, R, C, bs, dtype, blocks)
    G, X = (wl.round_to_storage(rng.normal(size=(m, w)).astype(np.float32), dtype) for w in (R * bs[0], C * bs[1]))
    Do, So = oracle_mod.bsr_sddmm(G, X, p[1], p[2], *bs)
    Gd, Xd = to_device(G, dtype), to_device(X, dtype)
    for lend, kernel in ((True, lent), (False, alone)):
        D = _run(p, bs, dtype, 0, monkeypatch, Gd, Xd, lend)
        check(D, Do.reshape(blocks, -1), So.reshape(blocks, -1), 1e-5, f"lend={lend}")
        forced = {"block": _run(p, bs, dtype, 1, monkeypatch, Gd, Xd, lend), "groups": _run(p, bs, dtype, 2, monkeypatch, Gd, Xd, lend)}
        assert not np.array_equal(forced["block"], forced["groups"])
        assert np.array_equal(D, forced[kernel]), f"lend={lend}: not {kernel}"
