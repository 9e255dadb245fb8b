"""The sampled product of 16x1 fp32 blocks: in block-column order (turned over in LDS) and out of it (transposed copy)."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import check, to_device


@pytest.mark.gpu
@pytest.mark.parametrize("density", [0.02, 0.2, 0.45, 0.7])
@pytest.mark.parametrize("ordered", [True, False])
def test_sampled_product_thin_ranges(oracle_mod, monkeypatch, density, ordered):
    """One to three ranges of 256 columns, the last one short; fewer block-rows than a workgroup takes and more; runs
    from none to longer than the accumulators hold (then the other kernel); rows: one, around a step, and split."""
    import torch
    import paper_2007_13055_amd as lib
    monkeypatch.setenv("BSR_SPMM_TUNE", "sd=2")         # that kernel wherever it can take W
    rng = np.random.default_rng(int(density * 100))
    for m, R, C in ((1, 3, 40), (31, 20, 260), (33, 17, 256), (100, 5, 700), (1500, 18, 516)):
        counts = np.minimum(C, rng.poisson(density * C, size=R))
        counts[0] = 0
        counts[-1] = 1
        p = wl.make_problem("sdth", m, C, R * 16, 16, 1, "f32", "f32", ("counts", counts), ("uniform", 1.0), ("uniform", 1.0), 1700 + m)
        idx = p.block_indices.copy()
        a, b = p.index_pointer[1], p.index_pointer[2]
        if b - a > 2:
            idx[a + 1] = idx[a]                        # a column twice
            if not ordered:
                idx[a:b] = idx[a:b][::-1]
        G = rng.normal(size=(m, p.n)).astype(np.float32)
        Do, So = oracle_mod.bsr_sddmm(G, p.X, idx, p.index_pointer, 16, 1)
        W = lib.bsr_create(p.n, p.k, p.block_data, idx, p.index_pointer, dtype="f32")
        outs = []
        for _ in range(2):
            D = torch.full((p.nnzb, 16, 1), float("nan"), device="cuda")
            lib.bsr_sddmm(W, to_device(G, "f32"), to_device(p.X, "f32"), D)
            torch.cuda.synchronize()
            outs.append(D.double().cpu().numpy().reshape(p.nnzb, -1))
        check(outs[0], Do.reshape(p.nnzb, -1), So.reshape(p.nnzb, -1), p.tau, f"thin ranges m={m} {density} {ordered}", out_dtype="f32")
        assert np.array_equal(outs[0], outs[1])
