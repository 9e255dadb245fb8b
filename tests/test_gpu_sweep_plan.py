"""The sweep kernel's plan, which the first product that wants it builds and sends: around graphs, streams and threads."""
import threading

import numpy as np
import pytest

import workloads as wl
from gpu_util import check, to_device, torch_dtype

pytestmark = pytest.mark.gpu

# dtype, result, rows, blocks, block-rows, block-columns, blocks per block-row: products that the sweep kernel takes;
# "created": no other matrix-core kernel for any number of rows, and bsr_create builds the plan
SHAPES = {"16x16": ("f16", "f32", 600, (16, 16), 96, 376, 40), "8x8 fp32": ("f32", "f32", 400, (8, 8), 64, 128, 40),
          "8x8 16-bit": ("bf16", "f32", 203, (8, 8), 66, 68, 20), "created": ("bf16", "f32", 203, (8, 8), 512, 128, 40), "odd sizes": ("f16", "f16", 203, (8, 8), 67, 67, 20)}


def _case(oracle_mod, shape):
    dtype, out, m, bs, R, C, count = SHAPES[shape]
    p = wl.make_problem("plan", m, C * bs[1], R * bs[0], bs[0], bs[1], dtype, out, ("counts", np.full(R, count)), ("normal", 1.0), ("normal", 1.0), 12)
    return p, *oracle_mod.bsr_spmm(p.X, p.block_data, p.block_indices, p.index_pointer, p.n)


def _handle(p):
    import paper_2007_13055_amd as lib
    return lib.bsr_create(p.n, p.k, p.block_data, p.block_indices, p.index_pointer, dtype=p.in_dtype)


def _swept(monkeypatch, p, X):
    """The product by the sweep kernel, of a handle of its own."""
    import paper_2007_13055_amd as lib
    with monkeypatch.context() as mp:
        mp.setenv("BSR_SPMM_TUNE", "variant=6")
        return lib.bsr_spmm_ex(_handle(p), X, y_dtype=p.out_dtype, path=lib.PATH_MFMA)


def _right(Y, Yo, So, p, what):
    import torch
    torch.cuda.synchronize()
    check(Y.double().cpu().numpy(), Yo, So, p.tau, what, out_dtype=p.out_dtype)


@pytest.mark.parametrize("shape", SHAPES)
def test_product_captured_first(oracle_mod, monkeypatch, shape):
    """The first product of a handle goes into a graph (without the plan where another kernel stands in for it), an eager one
    follows before any replay; then another graph, which sweeps, and replays of both with eager work between them."""
    import torch
    import paper_2007_13055_amd as lib
    p, Yo, So = _case(oracle_mod, shape)
    X = to_device(p.X, p.in_dtype)
    want = _swept(monkeypatch, p, X)
    W = _handle(p)
    ys = [torch.empty((p.m, p.n), dtype=torch_dtype(p.out_dtype), device="cuda") for _ in range(2)]
    graphs = []
    for Y in ys:
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            lib.bsr_spmm(W, X, Y, y_dtype=p.out_dtype)
        graphs.append(g)
        assert torch.equal(lib.bsr_spmm(W, X, y_dtype=p.out_dtype), want)
    for replay in range(3):
        for g, Y in zip(graphs, ys):
            Y.fill_(float("nan"))
            torch.cuda.synchronize()
            g.replay()
            _right(Y, Yo, So, p, f"{shape}, replay {replay}")
        assert torch.equal(ys[1], want)
        assert torch.equal(lib.bsr_spmm(W, X, y_dtype=p.out_dtype), want)


@pytest.mark.parametrize("shape", SHAPES)
def test_first_products_of_several_threads(oracle_mod, monkeypatch, shape):
    """Four threads, a stream each, with the first products of one handle."""
    import torch
    import paper_2007_13055_amd as lib
    p, Yo, So = _case(oracle_mod, shape)
    X = to_device(p.X, p.in_dtype)
    want = _swept(monkeypatch, p, X)
    W = _handle(p)
    ys = [torch.full((p.m, p.n), float("nan"), dtype=torch_dtype(p.out_dtype), device="cuda") for _ in range(4)]
    torch.cuda.synchronize()

    def product(Y):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(3):
                lib.bsr_spmm(W, X, Y, y_dtype=p.out_dtype)

    threads = [threading.Thread(target=product, args=(Y,)) for Y in ys]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    _right(want, Yo, So, p, shape)
    assert all(torch.equal(Y, want) for Y in ys)


@pytest.mark.parametrize("shape", ["16x16", "8x8 fp32", "8x8 16-bit", "odd sizes"])
def test_built_by_the_first_product_that_wants_it(oracle_mod, monkeypatch, shape):
    """A handle that only sees few rows has no such plan: a granule that is not there has the place 0xFFFF, which no other
    table holds."""
    import torch
    import paper_2007_13055_amd as lib
    p, Yo, So = _case(oracle_mod, shape)
    X = to_device(p.X, p.in_dtype)
    with monkeypatch.context() as mp:
        mp.setattr(torch, "empty", torch.zeros)       # nothing in the workspace but what the library writes
        W = _handle(p)
    words = W._tensors[3].view(torch.int32)
    for rows, there in ((8, False), (p.m, True)):
        Y = lib.bsr_spmm(W, X[:rows].contiguous(), y_dtype=p.out_dtype)
        _right(Y, Yo[:rows], So[:rows], p, f"{rows} rows")
        assert bool((words == 0xFFFF).any()) == there


@pytest.mark.parametrize("shape", ["8x8 fp32", "created"])
def test_debug_mode_checks_the_plan(oracle_mod, monkeypatch, shape):
    """BSR_SPMM_DEBUG=1: a damaged word of the plan, sent by the first product or by bsr_create, is reported and nothing is
    stored; repaired, the product is the oracle's again."""
    import torch
    import paper_2007_13055_amd as lib
    monkeypatch.setenv("BSR_SPMM_DEBUG", "1")
    p, Yo, So = _case(oracle_mod, shape)
    X = to_device(p.X, p.in_dtype)
    with monkeypatch.context() as mp:
        mp.setattr(torch, "empty", torch.zeros)       # nothing in the workspace but what the library writes
        W = _handle(p)
    words = W._tensors[3].view(torch.int32)
    Y = torch.empty((p.m, p.n), dtype=torch_dtype(p.out_dtype), device="cuda")
    lib.bsr_spmm(W, X, Y, y_dtype=p.out_dtype)
    torch.cuda.synchronize()
    # a word of its records: a granule that is not there has the place 0xFFFF, which no other table holds
    at = int(torch.nonzero(words == 0xFFFF).reshape(-1)[-1])
    keep = int(words[at])
    words[at] = keep ^ 1
    Y.fill_(7.0)
    with pytest.raises(lib.BsrError) as e:
        lib.bsr_spmm(W, X, Y, y_dtype=p.out_dtype)
    assert e.value.status == 7 and bool((Y == 7.0).all())
    words[at] = keep
    lib.bsr_spmm(W, X, Y, y_dtype=p.out_dtype)
    _right(Y, Yo, So, p, "repaired")
