"""The matrix-core projection products at sizes off every tile: sequences, widths and ranks that are no multiple of
16, 64 or 8, pitches that are not the row length, operands that start at any element.

Every operand lies in a larger buffer of NaNs, so that a value read from outside its rows and used shows in the
result, and nothing around the result may change.
"""
import pytest
import torch

from paper_2312_00752_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BF = torch.bfloat16


def _inside(x, pad):
    """x as a view into a NaN buffer: `pad` elements in front, rows `pad` further apart than their length."""
    nb, rows, cols = x.shape
    buf = torch.full((nb * rows * (cols + pad) + pad,), float("nan"), dtype=x.dtype, device=DEV)
    view = buf[pad:].view(nb, rows, cols + pad)[:, :, :cols] if pad else buf.view(nb, rows, cols)
    view.copy_(x)
    return view


def _rand(nb, rows, cols, seed):
    g = torch.Generator().manual_seed(seed)
    return (torch.randn((nb, rows, cols), generator=g) * 0.5).to(BF).to(DEV)


def _check(A, X, out_dtype, trans_b=False, accumulate=False, workspace=None, pad=0):
    a64, b64 = A.cpu().double(), X.cpu().double()
    ref = torch.matmul(a64, b64.transpose(-1, -2) if trans_b else b64)
    size = a64.abs() @ (b64.transpose(-1, -2) if trans_b else b64).abs()   # bounds every rounding of the sum
    C = _inside(torch.full(ref.shape, float("nan"), dtype=out_dtype, device=DEV), pad)
    if accumulate:
        C.copy_(_rand(*ref.shape, 99))
        ref = ref + C.cpu().double()
    B.ss_proj_gemm(A, X, C, trans_b=trans_b, accumulate=accumulate, workspace=workspace)
    torch.cuda.synchronize()
    got = C.cpu().double()
    # float32 sums: K roundings (or truncations) by 2^-23 of the sum of magnitudes at most; a bf16 result is rounded once more
    K = A.shape[-1]
    bound = K * 2.0 ** -23 * size + (2.0 ** -8 * ref.abs() if out_dtype == BF else 0.0) + 1e-30
    assert torch.isfinite(got).all()
    assert ((got - ref).abs() <= bound).all(), ((got - ref).abs() / bound).max()
    if pad:
        whole = C.as_strided((C.shape[0], C.shape[1], C.shape[2] + pad), C.stride())
        assert torch.isnan(whole[:, :, C.shape[2]:]).all()


# (batch, D, L, R, Mx): the smallest the kernels take; one short of and one past their tiles; more rows of the small
# operand than one launch holds (192); a contraction in two parts
SIZES = [(2, 9, 8, 8, 11), (2, 63, 65, 8, 13), (1, 200, 67, 25, 57), (3, 129, 127, 33, 97), (2, 264, 131, 96, 161),
         (1, 328, 321, 160, 192), (1, 100, 200, 191, 223), (1, 4105, 71, 12, 44)]


@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("nb,D,L,R,Mx", SIZES)
def test_products_of_any_size(nb, D, L, R, Mx, pad):
    u = _inside(_rand(nb, D, L, 1), pad)
    P = _inside(_rand(nb, Mx, L, 2), pad)
    r = P[:, :R]
    W_x, W_dt = _inside(_rand(1, Mx, D, 3), pad)[0], _inside(_rand(1, D, R, 4), pad)[0]
    W_xT, W_dtT = _inside(_rand(1, D, Mx, 5), pad)[0], _inside(_rand(1, R, D, 6), pad)[0]
    ws = torch.full((2 * nb * Mx * L * 4,), 0xFF, dtype=torch.uint8, device=DEV)
    _check(W_x, u, BF, pad=pad)
    _check(W_x, u, BF, workspace=ws, pad=pad)
    _check(W_dtT, u, BF, workspace=ws, pad=pad)
    _check(W_dt, r, BF, pad=pad)
    _check(W_xT, P, BF, accumulate=True, pad=pad)
    _check(u, r, torch.float32, trans_b=True, pad=pad)
    _check(P, u, torch.float32, trans_b=True, pad=pad)


@pytest.mark.parametrize("slabs", [1, 2, 3, 5, 6, 7])
def test_whole_slabs_not_a_multiple_of_the_pipeline(slabs):
    """Aligned operands whose contraction is a whole number of 64-wide slabs but not of four of them."""
    n = 64 * slabs
    X = _rand(2, n, 128, 7)
    _check(_rand(1, 80, n, 8)[0], X, BF)                                    # rows of X contracted
    _check(_rand(2, 128, n, 9), _rand(2, 48, n, 10), torch.float32, trans_b=True)
    _check(_rand(2, 40, n, 11), _rand(2, 192, n, 12), torch.float32, trans_b=True)


@pytest.mark.parametrize("nb,D,L,R,Mx", [(1, 64, 2050, 16, 40), (1, 700, 1000, 8, 24), (2, 2050, 130, 33, 65), (1, 3001, 63, 190, 200)])
@pytest.mark.parametrize("dtype", [BF, torch.float32])
def test_few_tiles_split_the_contraction(nb, D, L, R, Mx, dtype):
    """Products of few tiles and long contractions, with a workspace: up to eight shares per result, the last one ragged."""
    u, P = _rand(nb, D, L, 21).to(dtype), _rand(nb, Mx, L, 22).to(dtype)
    W_x = _rand(1, Mx, D, 23)[0].to(dtype)
    ws = torch.full((8 * nb * max(Mx * L, Mx * D) * 4,), 0xFF, dtype=torch.uint8, device=DEV)
    _check(W_x, u, dtype, workspace=ws)
    _check(u, P[:, :R], torch.float32, trans_b=True, workspace=ws)
    _check(P, u, torch.float32, trans_b=True, workspace=ws)


def test_infinities_and_nan_stay_where_they_belong():
    """A last row or column of infinities reaches the results that contain it and no others."""
    nb, D, L, M = 1, 71, 77, 19
    u, W = _rand(nb, D, L, 13), _rand(1, M, D, 14)[0]
    u[0, D - 1, 5] = float("inf")
    W[:, D - 1] = W[:, D - 1].abs() + 0.1
    C = torch.empty((nb, M, L), dtype=BF, device=DEV)
    B.ss_proj_gemm(W, u, C)
    torch.cuda.synchronize()
    assert (C[0, :, 5] == float("inf")).all()
    C[0, :, 5] = 0
    assert torch.isfinite(C).all()


# float32: (batch, D, L, R, Mx) at the edges of 16-row, 64-column and 16-index steps, of row tiles of 80, of four waves' slabs
F32_SIZES = [(1, 4, 4, 4, 4), (2, 17, 5, 4, 7), (2, 63, 65, 15, 17), (1, 200, 67, 25, 57), (3, 81, 127, 33, 81), (2, 264, 131, 96, 161),
             (1, 260, 321, 160, 192), (1, 1030, 71, 12, 44), (1, 300, 2050, 191, 223)]


@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("nb,D,L,R,Mx", F32_SIZES)
def test_float32_products_of_any_size(nb, D, L, R, Mx, pad):
    f32 = torch.float32
    draw = lambda *a: _inside(_rand(*a).float() * 1.2345678, pad)
    u, P, W_x, W_dt, W_xT = draw(nb, D, L, 1), draw(nb, Mx, L, 2), draw(1, Mx, D, 3)[0], draw(1, D, R, 4)[0], draw(1, D, Mx, 5)[0]
    r = P[:, :R]
    ws = torch.full((8 * nb * max(Mx * L, Mx * D, D * R) * 4,), 0xFF, dtype=torch.uint8, device=DEV)
    _check(W_x, u, f32, pad=pad)
    _check(W_x, u, f32, workspace=ws, pad=pad)
    _check(W_dt, r, f32, pad=pad)
    _check(u, r, f32, trans_b=True, workspace=ws, pad=pad)
    _check(P, u, f32, trans_b=True, workspace=ws, pad=pad)
    # added to the old value: that sum rounds once more
    C = _inside(_rand(nb, D, L, 6).float(), pad)
    old, prod, size = C.cpu().double(), W_xT.cpu().double() @ P.cpu().double(), W_xT.cpu().double().abs() @ P.cpu().double().abs()
    B.ss_proj_gemm(W_xT, P, C, accumulate=True)
    torch.cuda.synchronize()
    assert ((C.cpu().double() - old - prod).abs() <= Mx * 2.0 ** -23 * size + 2.0 ** -24 * (old.abs() + size)).all()


# float32: (batch, M, N, K) of contractions short enough that a wave has row tiles of its own: one to five of them (200 and 130 strips of
# columns are a round of workgroups), the last waves with few rows or none, from the smallest N and K on, and lengths on both sides of the lines
# at which four waves share a tile (48 and 320 indices, along K 16, 88 and 512)
F32_SHORT = [(8, 1030, 259, 25), (4, 777, 511, 191), (8, 1930, 129, 96), (32, 193, 256, 192), (128, 193, 4, 4), (2, 1601, 639, 17),
             (200, 300, 64, 40), (200, 256, 61, 17), (200, 190, 64, 33), (130, 128, 63, 48), (130, 128, 62, 49), (3, 100, 70, 16), (3, 100, 70, 88),
             (3, 100, 70, 89), (1, 70, 300, 12), (2, 300, 7, 30), (4, 700, 640, 320), (4, 700, 640, 321), (40, 260, 250, 19), (260, 300, 66, 8)]


@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("nb,M,N,K", F32_SHORT)
def test_float32_products_of_short_contractions(nb, M, N, K, pad):
    draw = lambda *a: _inside(_rand(*a).float() * 1.2345678, pad)
    W, A, X, XT = draw(1, M, K, 21)[0], draw(nb, M, K, 24), draw(nb, K, N, 22), draw(nb, N, K, 25)
    for a, x, trans_b in ((W, X, False), (A, XT, True), (XT, A, True)):
        _check(a, x, torch.float32, trans_b=trans_b, pad=pad)
        b = (x.transpose(1, 2) if trans_b else x).cpu().double()
        C = _inside(_rand(nb, a.shape[-2], b.shape[-1], 23).float(), pad)
        old, prod, size = C.cpu().double(), a.cpu().double() @ b, a.cpu().double().abs() @ b.abs()
        B.ss_proj_gemm(a, x, C, trans_b=trans_b, accumulate=True)
        torch.cuda.synchronize()
        # as above; the old value's sum rounds once more
        assert ((C.cpu().double() - old - prod).abs() <= K * 2.0 ** -23 * size + 2.0 ** -24 * (old.abs() + size)).all()
        if pad:
            assert torch.isnan(C.as_strided((nb, C.shape[1], C.shape[2] + pad), C.stride())[:, :, C.shape[2]:]).all()


@pytest.mark.parametrize("K", [64, 160, 161, 512, 513])
def test_float32_weight_gradients_on_both_sides_of_the_lines(K):
    for nb, M, N in ((32, 128, 512), (16, 512, 200), (9, 300, 1030)):
        _check(_rand(nb, M, K, 31).float() * 1.2345678, _rand(nb, N, K, 32).float(), torch.float32, trans_b=True)


@pytest.mark.parametrize("K,shared", [(64, 0.842e-7), (200, 1.345e-7), (512, 2.072e-7)])
def test_float32_row_tiles_of_a_wave_round_no_more_than_shared_ones(K, shared):
    """Errors against 64 bits, over the whole result.  `shared`: measured where four waves share a tile, whose chains are a quarter of the
    contraction; one chain through it has 1.44e-7, 2.54e-7 and 4.06e-7.  3 % for the draw."""
    for nb, M, N in ((4, 4096, 256), (4, 288, 4096), (1, 1536, 96)):
        A, X = _rand(nb, M, K, 61).float() * 1.2345678, _rand(nb, N, K, 62).float() * 1.1234567
        C = torch.empty((nb, M, N), dtype=torch.float32, device=DEV)
        B.ss_proj_gemm(A, X, C, trans_b=True)
        ref = torch.matmul(A.double(), X.double().transpose(1, 2).contiguous())
        assert (C.double() - ref).norm() <= 1.03 * shared * ref.norm()


def test_float32_infinities_stay_where_they_belong():
    """The last contraction index, whose step is padded, the last row and the last column hold infinities."""
    u, W = _rand(1, 71, 77, 13).float(), _rand(1, 19, 71, 14)[0].float()
    u[0, 70, 5] = u[0, 3, 76] = float("inf")
    W[:, 70] = W[:, 70].abs() + 0.1
    W[:, 3] = W[:, 3].abs() + 0.1
    for X, kw in ((u, {}), (u.transpose(1, 2).contiguous(), {"trans_b": True})):
        C = torch.empty((1, 19, 77), dtype=torch.float32, device=DEV)
        B.ss_proj_gemm(W, X, C, **kw)
        torch.cuda.synchronize()
        assert (C[0, :, 5] == float("inf")).all() and (C[0, :, 76] == float("inf")).all()
        C[0, :, 5] = C[0, :, 76] = 0
        assert torch.isfinite(C).all()
