"""The sampled product by groups of blocks that share slabs of G and X, forced, against the oracle."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import check, to_device, torch_dtype


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,out", [("f32", "f32"), ("f16", "f16"), ("bf16", "f32")])
@pytest.mark.parametrize("bs", [(8, 8), (16, 16), (32, 32), (64, 64), (8, 64), (16, 8), (32, 16), (64, 32)])
def test_sampled_product_slab_groups(oracle_mod, monkeypatch, dtype, out, bs):
    """Rows: one, one step of 32 less and more one, several steps, enough for the rows to be split (with the workspace
    the binding lends) and the same without a workspace.  Block-rows from empty to full, unsorted, one block stored
    twice; n and k that end inside a slab and (8-wide blocks) inside a tile."""
    import torch
    import paper_2007_13055_amd as lib
    monkeypatch.setenv("BSR_SPMM_TUNE", "sd=2")
    bs_r, bs_c = bs
    rng = np.random.default_rng(bs_r * 100 + bs_c)
    R, C = 13, 19
    counts = rng.integers(0, C + 1, size=R)
    counts[:3] = [C, 0, 1]
    for m in (1, 31, 33, 160, 1100):
        p = wl.make_problem("slab", m, C * bs_c, R * bs_r, bs_r, bs_c, dtype, dtype, ("counts", counts), ("normal", 1.0),
                            ("normal", 1.0), 2100 + m)
        idx = p.block_indices.copy()
        a, b = p.index_pointer[0], p.index_pointer[1]
        idx[a:b] = rng.permutation(idx[a:b])
        idx[a + 1] = idx[a]
        G = wl.round_to_storage(rng.normal(size=(m, p.n)).astype(np.float32), dtype)
        Do, So = oracle_mod.bsr_sddmm(G, p.X, idx, p.index_pointer, bs_r, bs_c)
        W = lib.bsr_create(p.n, p.k, p.block_data, idx, p.index_pointer, dtype=dtype)
        Gd, Xd = to_device(G, dtype), to_device(p.X, dtype)
        for lent in (True, False):
            D = torch.full((p.nnzb, bs_r, bs_c), float("nan"), dtype=torch_dtype(out), device="cuda")
            if lent:
                lib.bsr_sddmm(W, Gd, Xd, D, d_dtype=out)
            else:
                st = lib.load_library().bsr_sddmm(W.handle, m, Gd.data_ptr(), Xd.data_ptr(), D.data_ptr(),
                                                  {"f32": 0, "f16": 1, "bf16": 2}[out], torch.cuda.current_stream().cuda_stream)
                assert st == 0
            torch.cuda.synchronize()
            check(D.double().cpu().numpy().reshape(p.nnzb, -1), Do.reshape(p.nnzb, -1), So.reshape(p.nnzb, -1), p.tau,
                  f"slabs {bs} {dtype}->{out} m={m} workspace={lent}", out_dtype=out)


@pytest.mark.gpu
def test_sampled_product_captured_first(oracle_mod, monkeypatch):
    """A handle whose first sampled product is recorded into a graph: the copy of its plan runs only with the graph, so an
    eager product before the first replay sends the plan itself; then replays with eager work in between."""
    import torch
    import paper_2007_13055_amd as lib
    monkeypatch.setenv("BSR_SPMM_TUNE", "sd=2")
    m = 1100
    p = wl.make_problem("slab", m, 19 * 16, 13 * 16, 16, 16, "f32", "f32", ("counts", np.full(13, 9)), ("normal", 1.0),
                        ("normal", 1.0), 2190)
    G = np.random.default_rng(5).normal(size=(m, p.n)).astype(np.float32)
    Do, So = oracle_mod.bsr_sddmm(G, p.X, p.block_indices, p.index_pointer, 16, 16)
    W, Gd, Xd = lib.bsr_create(p.n, p.k, p.block_data, p.block_indices, p.index_pointer), to_device(G, "f32"), to_device(p.X, "f32")
    D, E = (torch.full((p.nnzb, 16, 16), float("nan"), device="cuda") for _ in range(2))

    def right(t, what):
        torch.cuda.synchronize()
        check(t.double().cpu().numpy().reshape(p.nnzb, -1), Do.reshape(p.nnzb, -1), So.reshape(p.nnzb, -1), p.tau, what)
        t.fill_(float("nan"))

    W.ensure_scratch(m)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(2):
            lib.bsr_sddmm(W, Gd, Xd, D)
    lib.bsr_sddmm(W, Gd, Xd, E)
    right(E, "eager product before the first replay")
    for replay in range(4):
        g.replay()
        right(D, f"replay {replay}")
        lib.bsr_sddmm(W, Gd, Xd, E)
        right(E, f"eager product after replay {replay}")


@pytest.mark.gpu
def test_debug_mode_checks_the_groups(oracle_mod, monkeypatch):
    """BSR_SPMM_DEBUG=1: a word of the groups' plan damaged in device memory is reported and nothing is stored; repaired,
    the product is the oracle's again."""
    import torch
    import paper_2007_13055_amd as lib
    monkeypatch.setenv("BSR_SPMM_TUNE", "sd=2")
    monkeypatch.setenv("BSR_SPMM_DEBUG", "1")
    m = 300
    p = wl.make_problem("slab", m, 19 * 32, 13 * 32, 32, 32, "f16", "f16", ("counts", np.full(13, 9)), ("normal", 1.0), ("normal", 1.0), 88)
    G = wl.round_to_storage(np.random.default_rng(5).normal(size=(m, p.n)).astype(np.float32), "f16")
    Do, So = oracle_mod.bsr_sddmm(G, p.X, p.block_indices, p.index_pointer, 32, 32)
    W, Gd, Xd = lib.bsr_create(p.n, p.k, p.block_data, p.block_indices, p.index_pointer, dtype="f16"), to_device(G, "f16"), to_device(p.X, "f16")
    D = torch.full((p.nnzb, 32, 32), 7.0, device="cuda")
    words = W._tensors[3].view(torch.int32)
    torch.cuda.synchronize()
    before = words.clone()
    lib.bsr_sddmm(W, Gd, Xd, D, d_dtype="f32")
    torch.cuda.synchronize()
    written = torch.nonzero(words != before).reshape(-1)
    written = written[written >= int(written[-1]) - p.nnzb * 4]          # of those, tile records: the last that were written
    assert written.numel() > 100
    for at in (int(written[0]), int(written[-1])):
        keep = int(words[at])
        words[at] = keep ^ 1
        D.fill_(7.0)
        with pytest.raises(lib.BsrError) as e:
            lib.bsr_sddmm(W, Gd, Xd, D, d_dtype="f32")
        assert e.value.status == 7 and bool((D == 7.0).all())
        words[at] = keep
    lib.bsr_sddmm(W, Gd, Xd, D, d_dtype="f32")
    torch.cuda.synchronize()
    check(D.double().cpu().numpy().reshape(p.nnzb, -1), Do.reshape(p.nnzb, -1), So.reshape(p.nnzb, -1), p.tau, "repaired")
