"""Transposed block values against NumPy, bit for bit."""
import numpy as np
import pytest


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("bs", [(8, 8), (64, 64), (16, 32), (64, 8), (4, 12), (16, 1), (1, 16), (3, 5), (12, 4), (1, 3)])
def test_transposed_values(dtype, bs):
    """Sides that are multiples of what 16 bytes hold, one row or column, and neither; one block and a ragged number."""
    import torch
    import paper_2007_13055_amd as lib
    from gpu_util import torch_dtype
    rng = np.random.default_rng(3)
    for nnzb in (1, 77):
        data = torch.from_numpy(rng.integers(-100, 100, size=(nnzb,) + bs).astype(np.float32)).to("cuda", torch_dtype(dtype))
        perm = rng.permutation(nnzb).astype(np.int32)
        out = torch.full((nnzb, bs[1], bs[0]), 999.0, device="cuda").to(torch_dtype(dtype))
        pd = torch.from_numpy(perm).cuda()
        st = lib.load_library().bsr_transpose_values({"f32": 0, "f16": 1, "bf16": 2}[dtype], bs[0], bs[1], nnzb, pd.data_ptr(),
                                                     data.data_ptr(), out.data_ptr(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert st == 0
        assert np.array_equal(out.float().cpu().numpy(), np.transpose(data.float().cpu().numpy()[perm], (0, 2, 1)))
