"""The k-split kernel's work lists around graphs: a product recorded first, and graphs that outlive other values of m."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import check, to_device

R, C = 320, 24                                       # 320 block-rows: more items than CUs, so that the kernel wants a list


def _problem(m):
    counts = np.random.default_rng(3).integers(0, 9, size=R)
    return wl.make_problem("list", m, C * 16, R * 16, 16, 16, "f32", "f32", ("counts", counts), ("normal", 1.0), ("normal", 1.0), 31)


def _matrix():
    import paper_2007_13055_amd as lib
    p = _problem(1)
    return lib.bsr_create(p.n, p.k, p.block_data, p.block_indices, p.index_pointer), p


def _inputs(oracle_mod, p, m):
    X = np.random.default_rng(m).normal(size=(m, p.k)).astype(np.float32)
    Yo, So = oracle_mod.bsr_spmm(X, p.block_data, p.block_indices, p.index_pointer, p.n)
    return to_device(X, "f32"), Yo, So


def _right(Y, Yo, So, tau, what):
    import torch
    torch.cuda.synchronize()
    check(Y.double().cpu().numpy(), Yo, So, tau, what)
    Y.fill_(float("nan"))


@pytest.mark.gpu
@pytest.mark.parametrize("m", [12, 40])
def test_product_captured_first(oracle_mod, m):
    """The first product of an m goes into a graph, an eager one follows before any replay; then replays and eager ones."""
    import torch
    import paper_2007_13055_amd as lib
    W, p = _matrix()
    X, Yo, So = _inputs(oracle_mod, p, m)
    Y, E = (torch.full((m, p.n), float("nan"), device="cuda") for _ in range(2))
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(2):
            lib.bsr_spmm_ex(W, X, Y, path=lib.PATH_MFMA)
    for replay in range(4):
        lib.bsr_spmm_ex(W, X, E, path=lib.PATH_MFMA)
        _right(E, Yo, So, p.tau, f"eager product before replay {replay}")
        g.replay()
        _right(Y, Yo, So, p.tau, f"replay {replay}")


@pytest.mark.gpu
def test_graphs_of_several_m(oracle_mod):
    """A graph per m, each after an eager product, more of them than lists are kept; then eager products of further m,
    which replace lists, and every graph again."""
    import torch
    import paper_2007_13055_amd as lib
    W, p = _matrix()
    graphs = []
    for m in (10, 33, 20, 50, 70, 90):
        X, Yo, So = _inputs(oracle_mod, p, m)
        Y = torch.full((m, p.n), float("nan"), device="cuda")
        lib.bsr_spmm_ex(W, X, Y, path=lib.PATH_MFMA)
        _right(Y, Yo, So, p.tau, f"eager product m={m}")
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            lib.bsr_spmm_ex(W, X, Y, path=lib.PATH_MFMA)
        graphs.append((m, g, Y, Yo, So, X))
    for again in range(3):
        for m in (100, 115, 130, 150, 165):
            X, Yo, So = _inputs(oracle_mod, p, m)
            _right(lib.bsr_spmm_ex(W, X, path=lib.PATH_MFMA), Yo, So, p.tau, f"eager product m={m}")
        for m, g, Y, Yo, So, _ in graphs:
            g.replay()
            _right(Y, Yo, So, p.tau, f"replay m={m}, {again}")
