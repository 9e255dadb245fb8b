"""Few block-rows and many m-tiles: the k-split kernel's work items do not fit a balanced table, which is remembered."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import check, to_device


@pytest.mark.gpu
@pytest.mark.parametrize("R,bs", [(11, 16), (3, 64)])
def test_items_without_a_table(oracle_mod, R, bs):
    """One m without a table (11 x 205 items of 16 rows, 3 x 103 of 32) between two that have one or need none, each twice."""
    import torch
    import paper_2007_13055_amd as lib
    C = 24
    rng = np.random.default_rng(R)
    counts = rng.integers(1, C, size=R)
    W = None
    for m in (300, 3273, 300, 3273, 40):
        p = wl.make_problem("items", m, C * bs, R * bs, bs, bs, "f32", "f32", ("counts", counts), ("uniform", 1.0), ("uniform", 1.0), 77)
        if W is None:
            first = p
            W = lib.bsr_create(p.n, p.k, p.block_data, p.block_indices, p.index_pointer, dtype="f32")
        Yo, So = oracle_mod.bsr_spmm(p.X, first.block_data, first.block_indices, first.index_pointer, p.n)
        Y = lib.bsr_spmm(W, to_device(p.X, "f32"))
        torch.cuda.synchronize()
        check(Y.double().cpu().numpy(), Yo, So, p.tau, f"items m={m}", out_dtype="f32")
