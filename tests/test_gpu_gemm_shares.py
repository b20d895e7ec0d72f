"""Products with many output rows whose workgroups take several 16-row tiles each: an odd number of them, a last workgroup with
one, one and four waves per workgroup, the three depths the kernel is built for, whole and ragged."""
import pytest
import torch

from tests import test_gpu_gemm_sizes as sizes

pytestmark = pytest.mark.gpu
BF = torch.bfloat16


# (batch, M, K, N); off whole tiles: 2, 5, 7, 3 and 4 tiles, one wave and (third and last) four, rows of any pitch
@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("nb,M,K,N", [(8, 1610, 25, 259), (8, 1930, 129, 259), (8, 6150, 191, 250), (8, 1930, 96, 129), (4, 4090, 130, 511)])
def test_ragged(nb, M, K, N, pad):
    X = sizes._inside(sizes._rand(nb, K, N, 1), pad)
    W = sizes._inside(sizes._rand(1, M, K, 2), pad)[0]
    sizes._check(W, X, BF, pad=pad)


# whole: 2, 3, 9, 7 and 4 tiles, one wave and, with 9, four; the last one on half of the SIMDs
@pytest.mark.parametrize("nb,M,K,N", [(16, 784, 64, 256), (16, 736, 64, 256), (16, 2176, 128, 256), (2, 2032, 160, 1536), (4, 2064, 128, 192)])
def test_whole(nb, M, K, N):
    sizes._check(sizes._rand(1, M, K, 3)[0], sizes._rand(nb, K, N, 4), BF)
