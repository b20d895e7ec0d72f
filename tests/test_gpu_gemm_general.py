"""The general product (any strides, either type) around the edges of its 64 x 64 x 32 tiles, with each operand
contiguous along either index, against float64."""
import pytest
import torch

from paper_2312_00752_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (3, 5, 3), (4, 4, 4), (63, 65, 31), (64, 64, 32), (65, 63, 33), (130, 70, 97), (2, 200, 64)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_general_product(M, N, K, dtype):
    g = torch.Generator().manual_seed(M * 1000 + N)

    def stored(rows, cols):   # rows 3 elements further apart than their length, NaN in between
        buf = torch.full((2, rows, cols + 3), float("nan"), dtype=dtype, device=DEV)
        buf[:, :, :cols] = torch.randn((2, rows, cols), generator=g).to(dtype)
        return buf[:, :, :cols]
    for ta in (False, True):
        for tb in (False, True):
            A, X = stored(*((K, M) if ta else (M, K))), stored(*((N, K) if tb else (K, N)))
            a64 = A.cpu().double().transpose(1, 2) if ta else A.cpu().double()
            b64 = X.cpu().double().transpose(1, 2) if tb else X.cpu().double()
            for out, acc in ((torch.float32, False), (dtype, True)):
                C = torch.randn((2, M, N), generator=g).to(out).to(DEV)
                ref = torch.matmul(a64, b64) + (C.cpu().double() if acc else 0.0)
                B.ss_proj_gemm(A, X, C, trans_a=ta, trans_b=tb, accumulate=acc, general=True)
                torch.cuda.synchronize()
                # K roundings of the sum of magnitudes, and one of a bf16 result
                bound = (K + 1) * 2.0 ** -23 * (torch.matmul(a64.abs(), b64.abs()) + ref.abs()) + 2.0 ** -8 * ref.abs() * (out == torch.bfloat16)
                assert ((C.cpu().double() - ref).abs() <= bound + 1e-30).all(), (ta, tb, out)
