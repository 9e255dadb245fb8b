"""The products' Python entry points: what they accept, return and raise."""
import numpy as np
import pytest


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_entry_points_arguments_and_errors(dtype):
    import torch
    import paper_2007_13055_amd as lib
    from gpu_util import torch_dtype
    T = torch_dtype(dtype)
    data = torch.ones((3, 16, 16), dtype=T, device="cuda")
    W = lib.bsr_create(32, 48, data, np.array([0, 2, 1]), np.array([0, 2, 3]))
    X, G = torch.ones((5, 48), dtype=T, device="cuda"), torch.ones((5, 32), dtype=T, device="cuda")
    want = torch.tensor([32.0] * 16 + [16.0] * 16, device="cuda").expand(5, 32)
    Y, D = torch.empty((5, 32), dtype=T, device="cuda"), torch.empty((3, 16, 16), device="cuda")
    assert lib.bsr_spmm(W, X, Y) is Y and torch.equal(Y.float(), want)
    assert lib.bsr_sddmm(W, G, X, D, d_dtype="f32", lend_scratch=False) is D and bool((D == 5).all())
    new = lib.bsr_spmm_ex(W, X, y_dtype="f32", path=lib.PATH_WAVE)
    assert new.dtype == torch.float32 and new.device == X.device and not new.requires_grad and torch.equal(new, want)
    assert torch.equal(lib.bsr_spmm_ex(W, X, path=1.0).float(), want)                        # whatever int() takes
    new = lib.bsr_sddmm(W=W, G=G, X=X)
    assert new.shape == (3, 16, 16) and new.dtype == T and bool((new == 5).all())
    assert lib.bsr_spmm(W, X[:0]).shape == (0, 32)
    other = torch.float16 if dtype == "f32" else torch.float32
    for call, error in [(lambda: lib.bsr_spmm(W, X[:, :32]), ValueError),                    # k
                        (lambda: lib.bsr_spmm(W, X.reshape(-1)), ValueError),                # rank
                        (lambda: lib.bsr_spmm(W, torch.ones((48, 5), dtype=T, device="cuda").t()), ValueError),   # order
                        (lambda: lib.bsr_spmm(W, X.to(other)), ValueError),                  # type of another W
                        (lambda: lib.bsr_spmm(W, X.double()), KeyError),                     # no such type
                        (lambda: lib.bsr_spmm(W, X, y_dtype="f8"), KeyError),
                        (lambda: lib.bsr_spmm(W, X, Y[:4]), ValueError),
                        (lambda: lib.bsr_spmm(W, X, Y.to(other)), ValueError),
                        (lambda: lib.bsr_sddmm(W, G[:4], X), ValueError),
                        (lambda: lib.bsr_sddmm(W, X, X), ValueError),
                        (lambda: lib.bsr_sddmm(W, G, X, D[:2], d_dtype="f32"), ValueError),
                        (lambda: lib.bsr_spmm_static(W, X.reshape(-1), Y), ValueError),
                        (lambda: lib.bsr_spmm_ex(W, X, path=7), lib.BsrError)]:
        with pytest.raises(error):
            call()
    W.close()
    with pytest.raises(lib.BsrError):
        lib.bsr_spmm(W, X)


def _splitting_product():
    """G, X, W, D of a sampled product whose rows are split, with 6 MB or so of partial results, and the D it has."""
    import torch
    import paper_2007_13055_amd as lib
    g = torch.Generator(device="cuda").manual_seed(3)
    ptr = np.arange(0, 48 * 33, 48)
    W = lib.bsr_create(512, 768, torch.zeros((48 * 32, 16, 16), dtype=torch.bfloat16, device="cuda"), np.tile(np.arange(48), 32), ptr)
    G, X = (torch.randint(-2, 3, (4096, c), generator=g, device="cuda").bfloat16() for c in (512, 768))
    want = (G.float().t() @ X.float()).reshape(32, 16, 48, 16).transpose(1, 2).reshape(-1, 16, 16)   # whole numbers: exact
    return W, G, X, torch.empty((48 * 32, 16, 16), device="cuda"), want


@pytest.mark.gpu
def test_sampled_product_allocates_nothing_unless_lent():
    import torch
    import paper_2007_13055_amd as lib
    W, G, X, D, want = _splitting_product()
    for lend in (False, True):
        torch.cuda.synchronize()
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        lib.bsr_sddmm(W, G, X, D, d_dtype="f32", lend_scratch=lend)
        assert (torch.cuda.max_memory_allocated() > before) == lend        # the case is one that wants memory
        assert torch.equal(D, want)
        D.fill_(float("nan"))


@pytest.mark.gpu
def test_sampled_product_without_memory_for_its_splits():
    import torch
    import paper_2007_13055_amd as lib
    W, G, X, D, want = _splitting_product()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + 4096) / total)
    try:
        rest = []
        with pytest.raises(torch.cuda.OutOfMemoryError):                   # take what is left of the segments in use
            while len(rest) < 1000:
                rest.append(torch.empty(2 << 20, dtype=torch.uint8, device="cuda"))
        lib.bsr_sddmm(W, G, X, D, d_dtype="f32")
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(D, want)


@pytest.mark.gpu
def test_other_threads_run_while_a_plan_is_built():
    """The first sampled product on a pattern builds its plan on the host, tens of ms here: another Python thread goes on
    meanwhile."""
    import threading
    import time
    import torch
    import paper_2007_13055_amd as lib

    def matrix(R, C):
        return lib.bsr_create(8 * R, 8 * C, torch.zeros((R * C, 8, 8), dtype=torch.bfloat16, device="cuda"), np.tile(np.arange(C), R),
                              np.arange(0, R * C + 1, C))

    def inputs(R, C):
        return (torch.ones((512, 8 * c), dtype=torch.bfloat16, device="cuda") for c in (R, C))

    lib.bsr_sddmm(matrix(8, 8), *inputs(8, 8))                             # the kernels are loaded
    W, (G, X) = matrix(1000, 2000), inputs(1000, 2000)
    torch.cuda.synchronize()
    ticks, stop = [], threading.Event()

    def watch():
        while not stop.is_set():
            ticks.append(time.perf_counter())

    t = threading.Thread(target=watch)
    t.start()
    while len(ticks) < 1000:
        time.sleep(0.001)
    start = time.perf_counter()
    lib.bsr_sddmm(W, G, X)
    end = time.perf_counter()
    stop.set()
    t.join()
    inside = [start, *(x for x in ticks if start <= x <= end), end]
    assert end - start > 0.01
    assert max(np.diff(inside)) < 0.3 * (end - start)


@pytest.mark.gpu
def test_results_come_through_the_dispatcher():
    """A dispatch mode sees the results being made, as it saw torch.empty's."""
    import torch
    import paper_2007_13055_amd as lib
    from torch.utils._python_dispatch import TorchDispatchMode

    class Seen(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            made.append((func.overloadpacket.__name__, tuple(args[0])))
            return func(*args, **(kwargs or {}))

    made = []
    W = lib.bsr_create(32, 48, torch.ones((3, 16, 16), device="cuda"), np.array([0, 2, 1]), np.array([0, 2, 3]))
    X, G = torch.ones((5, 48), device="cuda"), torch.ones((5, 32), device="cuda")
    with Seen():
        Y, D = lib.bsr_spmm(W, X), lib.bsr_sddmm(W, G, X)
    assert made == [("empty", (5, 32)), ("empty", (3, 16, 16))]
    assert bool((Y[:, :16] == 32).all()) and bool((D == 5).all())
