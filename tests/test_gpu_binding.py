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
