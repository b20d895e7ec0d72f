// The layer's projections (Algorithm 2 with the selection functions of Section 3.2: s_B, s_C linear in
// the input; s_Delta in the low-rank form Linear_D(Linear_R(x)) of Section 3.6) and their gradients, as
// this library's own kernels.  All of them are "skinny" products: one side of each is the (D, L) matrix
// of a batch entry (u, delta, d delta, du), the other has R or R + 2N (8..192) rows, so they are
// bound by reading or writing a (B, D, L) tensor once, not by arithmetic, and are built around that:
// the big operand is read (or the big result written) exactly once, in 128-byte row pieces, and the
// small operand is shared through LDS or the L2.
//
//   gemm():  C[i] (M x N) = op(A[i]) (M x K)  op(B[i]) (K x N)  [+ C[i]],  strides in elements, float accumulation.
//
// bf16 products of the three shapes the layer needs go to v_mfma_f32_16x16x32_bf16 kernels (lane l
// supplies row, resp. column, l % 16 of an operand at the 8 contraction indices from 8 * (l / 16);
// accumulator element i is row 4 * (l / 16) + i, column l % 16):
//   gemm_nt_kernel    C = A B^T with both operands contiguous along the contraction index (the
//                     weight gradients: contraction over L).  A workgroup takes 64 rows of the big
//                     operand, staged in 64-wide slabs through LDS, against up to 192 rows of the
//                     small one, whose fragments each wave takes straight from the L2.
//   gemm_rows_kernel  few output rows, long contraction over the ROWS of the (K, N) operand
//                     ([r;B;C] = W_x u, dr = W_dt^T ddelta): that operand is contiguous along N, not
//                     along the contraction index, so two rows at a time are interleaved into 32-bit
//                     pairs on their way into LDS and a fragment is four such pairs.
//   gemm_cols_kernel  many output rows, short contraction (delta = W_dt r, du += W_x^T d[r;B;C]): a
//                     wave keeps its 64 columns of the small (K, N) operand in registers and walks
//                     the rows of the other; the product is formed transposed, so that a lane holds
//                     consecutive columns of the result.  With a result that is added to, gemm_cols_add_kernel: 64 x 64
//                     tiles through LDS.
// float32 products of these shapes go to gemm_f32_kernel; gemm_generic_kernel takes every other stride and dtype (64 x 64
// tiles through LDS, float MFMAs): sizes below 8, and below 4 in float32.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <type_traits>

#include "ss_device.h"
#include "ss_kernels.h"

namespace ss {

namespace {

template <typename T> __device__ __forceinline__ float ld(const T* p);
template <> __device__ __forceinline__ float ld<float>(const float* p) { return *p; }
template <> __device__ __forceinline__ float ld<bf16_t>(const bf16_t* p) { return bf16_to_f32(*p); }
template <typename T> __device__ __forceinline__ void st(T* p, float v);
template <> __device__ __forceinline__ void st<float>(float* p, float v) { *p = v; }
template <> __device__ __forceinline__ void st<bf16_t>(bf16_t* p, float v) { *p = bf16_t(f32_to_bf16_bits(v)); }

// Out[b][m][n] = sum over the parts of Part[part][b][m][n], in their order; one thread per element.
template <typename TC>
__global__ void __launch_bounds__(256) parts_reduce_kernel(const float* __restrict__ Part, int parts, TC* __restrict__ Out, long ldc,
                                                           long c_batch, int M, int N, long items)
{
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;   // over batch * M * N = the elements of a part
    if (idx >= items) return;
    float v = Part[idx];
    for (int z = 1; z < parts; ++z) v += Part[z * items + idx];
    const long bm = idx / N;
    st(Out + bm / M * c_batch + bm % M * ldc + idx % N, v);
}
template <typename TC>
void reduce_parts(const GemmArgs& g, int parts, TC* C, int M, int N, hipStream_t stream)
{
    const long items = (long)g.batch * M * N;
    hipLaunchKernelGGL((parts_reduce_kernel<TC>), dim3((unsigned)((items + 255) / 256)), dim3(256), 0, stream,
                       static_cast<const float*>(g.split_ws), parts, C, g.ldc, g.c_batch, M, N, items);
}

constexpr int SMAX = 192;   // rows of the small operand in one launch of a matrix-core kernel; they are built for 64, 128 and 192 of them
constexpr int GT = 64;   // tile edge
constexpr int GK = 32;   // contraction indices per step
constexpr int GP = GT + 4;   // LDS pitch (floats) of a contraction index's 64 rows or columns

// One operand of the general kernel: element (r, k) at p + r * s_r + k * s_k, R rows (or columns), K contraction indices.
// A thread moves two pieces of four consecutive elements per step, along whichever index is contiguous; a piece is
// read whole from inside the matrix (clamped) and only the last tile or step, a uniform case, takes its elements
// one by one.  Neither index contiguous, or fewer than four of it: always one by one.
template <typename T>
struct gemm_operand {
    const T* p;
    long s_r, s_k;
    int R, K, r0, mode;   // mode 0: k contiguous, 1: r contiguous, 2: elements one by one
    typedef uint32_t raw_t __attribute__((ext_vector_type(sizeof(T))));   // four elements
    raw_t x[2];
    __device__ __forceinline__ gemm_operand(const T* p_, long s_r_, long s_k_, int R_, int K_, int r0_)
        : p(p_), s_r(s_r_), s_k(s_k_), R(R_), K(K_), r0(r0_),
          mode(s_k_ == 1 && K_ >= 4 ? 0 : (s_r_ == 1 && R_ >= 4 ? 1 : 2)) {}
    // piece e of this thread: first row and index within the tile
    __device__ __forceinline__ void place(int e, int& r, int& k) const
    {
        const int i = (int)threadIdx.x + 256 * e;
        if (mode == 1) { k = i >> 4; r = (i & 15) * 4; } else { r = i >> 3; k = (i & 7) * 4; }
    }
    __device__ __forceinline__ void load(int k0)
    {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            int r, k;
            place(e, r, k);
            const long rr = mode == 1 ? min(r0 + r, R - 4) : min(r0 + r, R - 1), kk = mode == 0 ? min(k0 + k, K - 4) : min(k0 + k, K - 1);
            if (mode != 2) x[e] = load_any<raw_t>(p + rr * s_r + kk * s_k, 0u);
        }
    }
    __device__ __forceinline__ void store(int k0, float (*dst)[GP])
    {
        const bool single = mode == 2 || k0 + GK > K || (mode == 1 && r0 + GT > R);   // uniform
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            int r, k;
            place(e, r, k);
            float v[4];
            if (single) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int ri = r0 + r + (mode == 1 ? i : 0), ki = k0 + k + (mode == 1 ? 0 : i);
                    v[i] = ri < R && ki < K ? ld(p + ri * s_r + ki * s_k) : 0.0f;
                }
            } else if constexpr (sizeof(T) == 2) {
                v[0] = bf16_lo(x[e][0]); v[1] = bf16_hi(x[e][0]); v[2] = bf16_lo(x[e][1]); v[3] = bf16_hi(x[e][1]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = __uint_as_float(x[e][i]);
            }
            if (mode == 1) {
                *reinterpret_cast<float4*>(&dst[k][r]) = make_float4(v[0], v[1], v[2], v[3]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) dst[k + i][r] = v[i];
            }
        }
    }
};

// Any strides, either type: 64 x 64 tiles through LDS as floats, a step ahead in registers, 32 x 32 outputs per wave
// on v_mfma_f32_16x16x4_f32 (lane l supplies row, resp. column, l % 16 at contraction index l / 16; float products
// and sums, as on the vector ALU).
template <typename T, typename TC>
__global__ void __launch_bounds__(256) gemm_generic_kernel(const GemmArgs g)
{
    __shared__ __attribute__((aligned(16))) float As[2][GK][GP];
    __shared__ __attribute__((aligned(16))) float Bs[2][GK][GP];
    const int tid = threadIdx.x, lane = tid & 63, kg = lane >> 4, j = lane & 15;
    const int wm = (tid >> 7) * 32, wn = ((tid >> 6) & 1) * 32;
    const int m0 = blockIdx.y * GT, n0 = blockIdx.x * GT;
    const long bi = blockIdx.z % g.batch;
    // parts > 1: this workgroup's part of the contraction, its float32 share left for parts_reduce_kernel
    const int part = blockIdx.z / g.batch, parts = gridDim.z / g.batch;
    const int per_part = ((g.K + GK - 1) / GK + parts - 1) / parts * GK;
    const int k_begin = part * per_part, k_end = min(g.K, k_begin + per_part);
    gemm_operand<T> A(static_cast<const T*>(g.A) + bi * g.a_batch, g.a_m, g.a_k, g.M, g.K, m0);
    gemm_operand<T> B(static_cast<const T*>(g.B) + bi * g.b_batch, g.b_n, g.b_k, g.N, g.K, n0);
    TC* __restrict__ C = static_cast<TC*>(g.C) + bi * g.c_batch;
    f32x4_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) acc[i][0] = acc[i][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (k_begin < k_end) {
        A.load(k_begin);
        B.load(k_begin);
        A.store(k_begin, As[0]);
        B.store(k_begin, Bs[0]);
    }
    __syncthreads();
    int buf = 0;
    for (int k0 = k_begin; k0 < k_end; k0 += GK, buf ^= 1) {
        const bool more = k0 + GK < k_end;   // uniform
        if (more) {
            A.load(k0 + GK);
            B.load(k0 + GK);
        }
#pragma unroll
        for (int k = 0; k < GK; k += 4) {
            const float* a = &As[buf][k + kg][wm + j];
            const float* b = &Bs[buf][k + kg][wn + j];
            const float a0 = a[0], a1 = a[16], b0 = b[0], b1 = b[16];
            acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b0, acc[0][0], 0, 0, 0);
            acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b1, acc[0][1], 0, 0, 0);
            acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b0, acc[1][0], 0, 0, 0);
            acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b1, acc[1][1], 0, 0, 0);
        }
        if (more) {
            A.store(k0 + GK, As[buf ^ 1]);
            B.store(k0 + GK, Bs[buf ^ 1]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int n = n0 + wn + 16 * c + j;
            if (n >= g.N) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm + 16 * i + 4 * kg + r;
                if (m >= g.M) continue;
                float v = acc[i][c][r];
                if (parts > 1) {
                    static_cast<float*>(g.split_ws)[(((long)part * g.batch + bi) * g.M + m) * g.N + n] = v;
                    continue;
                }
                TC* dst = C + (long)m * g.ldc + n;
                if (g.accumulate) v += ld(dst);
                st(dst, v);
            }
        }
}

// Parts of a contraction of K that goes over `tiles` workgroups: one, unless that leaves half of the 256 compute units
// or more idle; then as many, up to eight, as give each unit a workgroup and each workgroup 256 contraction
// indices, if the workspace holds the shares.  Rounded so that none is empty when dealt out in steps of `step`.
int parts_for(const GemmArgs& g, long tiles, int K, int step, size_t share)
{
    if (!g.split_ws || g.accumulate || tiles > 128) return 1;
    int parts = 1;
    while (parts < 8 && tiles * parts * 2 <= 256 && K / (parts * 2) >= 256 && (size_t)(parts * 2) * share <= g.split_ws_bytes) parts *= 2;
    const int steps = (K + step - 1) / step, per = (steps + parts - 1) / parts;
    return (steps + per - 1) / per;
}

template <typename T, typename TC>
int launch_generic(const GemmArgs& g, hipStream_t stream)
{
    const long tm = (g.M + GT - 1) / GT, tn = (g.N + GT - 1) / GT;
    int parts = g.K > 0 ? parts_for(g, tm * tn * g.batch, g.K, GK, (size_t)g.batch * g.M * g.N * sizeof(float)) : 1;
    if ((long)parts * g.batch > 65535) parts = 1;
    const dim3 grid((unsigned)tn, (unsigned)tm, (unsigned)(g.batch * parts));
    hipLaunchKernelGGL((gemm_generic_kernel<T, TC>), grid, dim3(256), 0, stream, g);
    if (parts > 1) reduce_parts<TC>(g, parts, static_cast<TC*>(g.C), g.M, g.N, stream);
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_LAUNCH;
}

// ---- float32 operands -------------------------------------------------------------------------------
// C (M x N) = A B with A contiguous along the contraction index and B along either: the six products of the float32
// layer.  Its floor is the float matrix rate (128 multiply-adds per clock and CU), so what matters is that every SIMD has a wave that
// issues MFMAs back to back: a wave owns 16 MT rows x 64 columns of the result, whose operands it loads straight into the
// fragments' registers, AHEAD (two to four) slabs of 16 contraction indices ahead, without LDS or barriers.  A lane's 16-byte piece of an
// operand that is contiguous along the contraction index holds indices 4 g .. 4 g + 3 of the slab (g = lane / 16); the i-th
// MFMA of a slab contracts over element i of the four groups, so with B contiguous along N the lane reads row 4 g + i, columns
// 4 j .. 4 j + 3 (j = lane % 16), one for each of its four column tiles: rows of 256 bytes, and the lane's results are
// four consecutive columns.
// KW = 4: the workgroup's waves share a tile and deal out its slabs; their sums are added through LDS in the order of the
// waves.  Long contractions, where tiles are few.  KW = 1: four tiles one below the other, for short contractions (see f32_own_tiles).
// CHAIN: one chain of multiply-adds through the contraction.  Otherwise every slab is summed by itself and then added, so that the error is
// no larger than with the shorter chains of four waves: 4 x 4096 x 256 over 64 / 512 indices, relative to 64 bits, in one chain 1.44e-7 / 4.06e-7,
// shared 0.84e-7 / 2.07e-7, by slabs 0.84e-7 / 1.29e-7.
// BK: B contiguous along the contraction index; out_t: the result is stored transposed (the operand with more rows is B then).
// Through LDS, 64 x 64 per workgroup and one step ahead (gemm_generic_kernel), a launch had one wave per SIMD that
// waited for LDS, barrier and memory in turn.  us per call, that kernel / this one: W_x u 2 x 4096 x 1024, R = 128 (18 at the peak
// rate) 114 / 35, 1 x 2560 x 300, R = 80 26.0 / 13.9; W_dt r 1 x 5120 x 3001, R = 160 83 / 64; dW_x 8 x 768 x 4096, R = 24 121 / 47; with
// shorter chains the error against 64 bits is the same or smaller (W_x u, D = 5120: 1.3e-6 / 4.6e-7).
template <bool BK, int MT, int KW, bool CHAIN = KW == 4>
__global__ void __launch_bounds__(256, KW == 1 ? 2 : 1) gemm_f32_kernel(const GemmArgs g, const int out_t)
{
    constexpr int AHEAD = MT <= 2 ? 4 : (KW == 1 && MT == 5 ? 2 : 3);   // with two, two waves of five row tiles of their own fit a SIMD (up to 20 bytes a lane wait in scratch, outside the loop)
    __shared__ f32x4_t red[KW == 4 ? 3 * 4 * 4 * 64 : 1];
    const int lane = threadIdx.x & 63, kg = lane >> 4, j = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = blockIdx.x * 64, m0 = (KW == 4 ? blockIdx.y : blockIdx.y * 4 + wave) * 16 * MT;
    if (KW == 1 && m0 >= g.M) return;   // uniform; no barriers in this form
    const long bi = blockIdx.z % g.batch;
    const int part = blockIdx.z / g.batch, parts = gridDim.z / g.batch;
    const int slabs = (g.K + 15) / 16, per_part = (slabs + parts - 1) / parts;
    const int s_end = min(slabs, (part + 1) * per_part);
    const int s_begin = part * per_part + (KW == 4 ? wave : 0);
    const float* __restrict__ A = static_cast<const float*>(g.A) + bi * g.a_batch;
    const float* __restrict__ B = static_cast<const float*>(g.B) + bi * g.b_batch;
    const int M = g.M, N = g.N, K = g.K;
    // byte offsets within a batch entry's operand (the launch checks that they fit)
    uint32_t a_row[MT], b_row[BK ? 4 : 1];
    const uint32_t b_step = BK ? 0u : (uint32_t)(g.b_k * 4);
    const int n_at = BK ? n0 + 4 * j : min(n0 + 4 * j, N - 4);   // first of the lane's four columns
#pragma unroll
    for (int t = 0; t < MT; ++t) a_row[t] = (uint32_t)(min(m0 + 16 * t + j, M - 1) * g.a_m * 4);
    if constexpr (BK) {
#pragma unroll
        for (int c = 0; c < 4; ++c) b_row[c] = (uint32_t)(min(n_at + c, N - 1) * g.b_n * 4);
    } else {
        b_row[0] = (uint32_t)n_at * 4u;
    }
    u32x4 a[AHEAD][MT], b[AHEAD][4];
    f32x4_t acc[MT][4];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[t][c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto load = [&](auto slot, int s) {   // past the last slab: that one again
        constexpr int S = decltype(slot)::value;
        const int k = 16 * min(s, s_end - 1) + 4 * kg;
        const uint32_t ka = (uint32_t)row_piece(k, 4, K) * 4u;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if constexpr (BK) b[S][c] = load_any<u32x4>(B, b_row[c] + ka);
            else b[S][c] = load_any<u32x4>(B, b_row[0] + (uint32_t)min(k + c, K - 1) * b_step);
        }
#pragma unroll
        for (int t = 0; t < MT; ++t) a[S][t] = load_any<u32x4>(A, a_row[t] + ka);
    };
    f32x4_t wait[4] = {};   // without CHAIN: the last row tile's sum of the slab before
    auto multiply = [&](auto slot, int s) {
        constexpr int S = decltype(slot)::value;
        if (16 * (s + 1) > K) {   // uniform: the last slab, zeros past K in both operands
            const int k = 16 * s + 4 * kg;
            using piece_f = tile_mma<float>;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if constexpr (BK) b[S][c] = piece_f::cut(b[S][c], k, K);
                else if (k + c >= K) b[S][c] = u32x4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int t = 0; t < MT; ++t) a[S][t] = piece_f::cut(a[S][t], k, K);
        }
        auto mfma = [&](int t, int c, int i, f32x4_t sum) {
            return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[S][t][i]), __uint_as_float(BK ? b[S][c][i] : b[S][i][c]), sum, 0, 0, 0);
        };
        if constexpr (CHAIN) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int t = 0; t < MT; ++t)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[t][c] = mfma(t, c, i, acc[t][c]);
        } else {
            // a row tile's sum is added up between the instructions of the next one's (all sixteen behind their own: a sixth more time)
#pragma unroll
            for (int t = 0; t < MT; ++t) {
                f32x4_t sum[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        sum[c] = mfma(t, c, i, i == 0 ? f32x4_t{0.f, 0.f, 0.f, 0.f} : sum[c]);
                        acc[(t + MT - 1) % MT][c][i] += wait[c][i];
                    }
#pragma unroll
                for (int c = 0; c < 4; ++c) wait[c] = sum[c];
            }
        }
    };
    if (s_begin < s_end) {   // uniform
        load(std::integral_constant<int, 0>{}, s_begin);
        load(std::integral_constant<int, 1>{}, s_begin + KW);
        if constexpr (AHEAD >= 3) load(std::integral_constant<int, 2>{}, s_begin + 2 * KW);
        if constexpr (AHEAD == 4) load(std::integral_constant<int, 3>{}, s_begin + 3 * KW);
        for (int s = s_begin; s < s_end; s += AHEAD * KW) {
            auto turn = [&](auto slot) {
                constexpr int S = decltype(slot)::value;
                if (s + S * KW < s_end) multiply(slot, s + S * KW);   // uniform
                load(slot, s + (S + AHEAD) * KW);
            };
            turn(std::integral_constant<int, 0>{});
            turn(std::integral_constant<int, 1>{});
            if constexpr (AHEAD >= 3) turn(std::integral_constant<int, 2>{});
            if constexpr (AHEAD == 4) turn(std::integral_constant<int, 3>{});
        }
    }
    // a tile's results: element r of v[c] is row m_tile + 4 g + r, column n_at + c
    const bool share = parts > 1;   // this part's share, left for parts_reduce_kernel
    float* __restrict__ C = share ? static_cast<float*>(g.split_ws) + ((long)part * g.batch + bi) * M * N : static_cast<float*>(g.C) + bi * g.c_batch;
    const long ldc = share ? (out_t ? M : N) : g.ldc;
    auto store = [&](const f32x4_t (&v)[4], int m_tile) {
        const int m = m_tile + 4 * kg;
        if (out_t) {   // uniform; the launch never asks for it with a result that is added to
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float* row = C + (long)(n_at + c) * ldc + m;
                if (n_at + c < n0 + 4 * j || n_at + c >= N) continue;
                if (m + 4 <= M) store_any(row, 0u, v[c]);
                else
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (m + r < M) row[r] = v[c][r];
            }
            return;
        }
        const bool whole = n_at == n0 + 4 * j && n_at + 4 <= N;
        f32x4_t x[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = f32x4_t{v[0][r], v[1][r], v[2][r], v[3][r]};
        if (g.accumulate) {   // uniform; all requested before one is waited for, past the end the last row and column (not used)
            f32x4_t old[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float* row = C + (long)min(m + r, M - 1) * ldc;
                if (whole) old[r] = load_any<f32x4_t>(row + n_at, 0u);
                else
#pragma unroll
                    for (int c = 0; c < 4; ++c) old[r][c] = row[min(n_at + c, N - 1)];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] += old[r];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (m + r >= M) continue;
            float* row = C + (long)(m + r) * ldc + n_at;
            if (whole) store_any(row, 0u, x[r]);
            else
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (n_at + c >= n0 + 4 * j && n_at + c < N) row[c] = x[r][c];
        }
    };
    if constexpr (KW == 1) {
        if constexpr (!CHAIN) {
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[MT - 1][c] += wait[c];
        }
#pragma unroll
        for (int t = 0; t < MT; ++t) store(acc[t], m0 + 16 * t);
    } else {
        // four 16-row tiles at a time: wave w adds up the w-th, its own share in the place of its number
#pragma unroll
        for (int t0 = 0; t0 < MT; t0 += 4) {
            if (t0 > 0) __syncthreads();   // the tiles before have been read
#pragma unroll
            for (int tt = 0; tt < 4; ++tt)
                if (t0 + tt < MT && tt != wave) {
                    const int slot = wave < tt ? wave : wave - 1;
#pragma unroll
                    for (int c = 0; c < 4; ++c) red[((slot * 4 + tt) * 4 + c) * 64 + lane] = acc[t0 + tt < MT ? t0 + tt : 0][c];
                }
            __syncthreads();
            if (t0 + wave < MT) {   // uniform
                f32x4_t v[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    f32x4_t own = acc[t0][c];
#pragma unroll
                    for (int tt = 1; tt < 4; ++tt)
                        if (t0 + tt < MT && tt == wave) own = acc[t0 + tt < MT ? t0 + tt : 0][c];
                    f32x4_t others[3];
#pragma unroll
                    for (int slot = 0; slot < 3; ++slot) others[slot] = red[((slot * 4 + wave) * 4 + c) * 64 + lane];
                    v[c] = wave == 0 ? own : others[0];
                    v[c] += wave == 1 ? own : (wave == 0 ? others[0] : others[1]);
                    v[c] += wave == 2 ? own : (wave < 2 ? others[1] : others[2]);
                    v[c] += wave == 3 ? own : others[2];
                }
                store(v, m0 + 16 * (t0 + wave));
            }
        }
    }
}

// Row tiles of a wave that has them to itself (KW = 1): of one to five (two waves a SIMD), the number with the least rounds of 256
// workgroups times what a slab of the tile loads and multiplies (the four pieces of B cost a row tile if they are rows, two along K).
// us, 1 / 2 / 3 / 4 / 5: W_dt r 16 x 1536 x 64, K = 96 9.5 / 9.6 / 11.1 / 13.2 / 15.0, 16 x 4096 x 64, K = 96 16.6 / 15.3 / 17.6 / 14.5 / 18.1,
// 16 x 1536 x 1024, K = 96 69 / 64 / 55.1 / 55.8 / 56.2; dW_x 4 x 288 x 4096, K = 64 24.7 / 20.3 / 19.0 / 21.4 / 14.0.
int f32_row_tiles(const GemmArgs& g, long strips, bool bk)
{
    int best = 1;
    double least = 0.0;
    for (int mt = 1; mt <= 5; ++mt) {
        const long wgs = strips * g.batch * ((g.M + 64L * mt - 1) / (64L * mt));
        const double cost = (wgs <= 512 ? (double)((wgs + 255) / 256) : (double)wgs / 256) * (mt + (bk ? 2 : 1));
        if (mt == 1 || cost <= least) { least = cost; best = mt; }
    }
    return best;
}
// Whether a wave has row tiles of its own, by measurement, us, own / shared by four waves.  With B contiguous along N for up to 48 contraction
// indices (1 x 200 x 4, K = 24 4.9 / 7.2), and up to 320 if that gives 160 workgroups (1 x 1536 x 700, K = 192, 132 of them: 12.9 / 11.5).  With B
// along K four waves that share a tile have a slab each up to 64 indices, and only a long contraction pays for adding up their sums: own tiles up to
// 88 indices (but not a single slab of few row tiles, 1 x 1536 x 96, K = 16 6.5 / 5.6), of four and more row tiles up to 512.  dW_dt 16 x 4096 x 256,
// K = 64 41.0 / 79.9, 200 73.8 / 95.9, 512 148 / 174; 1 x 1536 x 96, K = 64 7.3 / 8.1, 96 9.4 / 8.1.
bool f32_own_tiles(const GemmArgs& g, long strips, bool bk, int mt)
{
    if (bk) return mt >= 4 ? g.K <= 512 : g.K > 16 && g.K <= 88;
    return g.K <= 48 || (g.K <= 320 && g.M > SMAX && strips * g.batch * ((g.M + 64L * mt - 1) / (64L * mt)) >= 160);
}
// The float32 kernel for this product, if it is one of its forms; SS_ERR_UNSUPPORTED otherwise (nothing enqueued).
int launch_f32(const GemmArgs& g0, hipStream_t stream)
{
    GemmArgs g = g0;
    const bool bk = g.b_k == 1;
    if (g.a_k != 1 || g.K < 4 || g.a_m < 0 || g.b_k < 0 || g.b_n < 0 || !(bk || (g.b_n == 1 && g.N >= 4))) return SS_ERR_UNSUPPORTED;
    const int out_t = bk && g.M > g.N && !g.accumulate;
    if (out_t) {
        std::swap(g.M, g.N);
        std::swap(g.A, g.B);
        std::swap(g.a_m, g.b_n);
        std::swap(g.a_batch, g.b_batch);
    }
    // 32-bit byte offsets within a batch entry
    const double limit = 4294967296.0;
    if (4.0 * ((double)g.M * g.a_m + g.K) >= limit || 4.0 * (bk ? (double)g.N * g.b_n + g.K : (double)g.K * g.b_k + g.N) >= limit) return SS_ERR_UNSUPPORTED;
    const long strips = (g.N + 63) / 64;
    const int own = f32_row_tiles(g, strips, bk);
    if (f32_own_tiles(g, strips, bk, own)) {
        const long rows = (g.M + 64L * own - 1) / (64L * own);
        if (rows > 65535) return SS_ERR_UNSUPPORTED;
        const dim3 grid((unsigned)strips, (unsigned)rows, (unsigned)g.batch);
        // many tiles of many rows over up to 192 indices in one chain, which takes 6 to 8 % less (16 x 4096 x 64, K = 192 19.3 / 21.2)
        const bool chain = !bk && g.K <= SMAX && g.M > SMAX && strips * g.batch * ((g.M + 255) / 256) >= 128;
#define SS_LAUNCH_F32(MT)                                                                                                  \
    case MT:                                                                                                               \
        if (bk) hipLaunchKernelGGL((gemm_f32_kernel<true, MT, 1>), grid, dim3(256), 0, stream, g, out_t);                   \
        else if (chain) hipLaunchKernelGGL((gemm_f32_kernel<false, MT, 1, true>), grid, dim3(256), 0, stream, g, 0);        \
        else hipLaunchKernelGGL((gemm_f32_kernel<false, MT, 1>), grid, dim3(256), 0, stream, g, 0);                         \
        break
        switch (own) {
            SS_LAUNCH_F32(1); SS_LAUNCH_F32(2); SS_LAUNCH_F32(3); SS_LAUNCH_F32(4); SS_LAUNCH_F32(5);
        }
#undef SS_LAUNCH_F32
        return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_LAUNCH;
    }
    const int tiles = (g.M + 79) / 80, mt = ((g.M + tiles - 1) / tiles + 15) / 16;   // row tiles of up to 80 (two waves per SIMD), of even height
    const long my = (g.M + 16 * mt - 1) / (16 * mt);
    if (my > 65535) return SS_ERR_UNSUPPORTED;
    // parts of the contraction: two workgroups per CU, while each wave keeps four slabs
    const size_t items = (size_t)g.batch * g.M * g.N;
    int parts = 1;
    if (g.split_ws && !g.accumulate)
        while (parts < 8 && strips * my * g.batch * parts * 2 <= 512 && g.K / (parts * 2) >= 256 && parts * 2 * items * sizeof(float) <= g.split_ws_bytes) parts *= 2;
    const int slabs = (g.K + 15) / 16, per = (slabs + parts - 1) / parts;
    parts = (slabs + per - 1) / per;   // none empty
    if ((long)parts * g.batch > 65535) parts = 1;
    const dim3 grid((unsigned)strips, (unsigned)my, (unsigned)(g.batch * parts));
#define SS_LAUNCH_F32(MT)                                                                                                  \
    case MT:                                                                                                               \
        if (bk) hipLaunchKernelGGL((gemm_f32_kernel<true, MT, 4>), grid, dim3(256), 0, stream, g, out_t);                   \
        else hipLaunchKernelGGL((gemm_f32_kernel<false, MT, 4>), grid, dim3(256), 0, stream, g, 0);                         \
        break
    switch (mt) {
        SS_LAUNCH_F32(1); SS_LAUNCH_F32(2); SS_LAUNCH_F32(3); SS_LAUNCH_F32(4); SS_LAUNCH_F32(5);
    }
#undef SS_LAUNCH_F32
    if (parts > 1) reduce_parts<float>(g, parts, static_cast<float*>(g.C), out_t ? g.N : g.M, out_t ? g.M : g.N, stream);
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_LAUNCH;
}

// ---- matrix-core kernels (bf16) -------------------------------------------------------------------
// Each exists twice.  The plain form takes operands made of whole 16-byte pieces (pitches and batch strides
// multiples of 8 elements, 16-byte aligned, contraction and columns whole slabs and tiles).  The RAG form takes
// any size from 8 up and any pitch: pieces are read in one access at element alignment from inside the row
// (row_piece), and only the last slab or tile, a uniform case, shifts the piece that reaches past the end into
// place with zeros behind it; rows past the end re-read the last one and what comes of them is not stored.
// Such sizes (sequences that are not a multiple of 64, widths that are not a multiple of 512 and so ranks that
// are not a multiple of 16) used to take the general kernel: [r;B;C] and delta of 4 x 4096 x 1531 338 us each.
using mma = tile_mma<bf16_t>;
constexpr int KSLAB = 64;          // contraction indices per step
constexpr int KP = KSLAB + 8;      // LDS pitch of a slab row (bf16): 144 bytes, 16-byte aligned, off the banks
constexpr int XPITCH = 64 + 4;     // LDS pitch of a row of pairs (32-bit)

__device__ __forceinline__ f32x4_t mfma_bf16(uint4 a, uint4 b, f32x4_t c)
{
    return mma::step(u32x4{a.x, a.y, a.z, a.w}, u32x4{b.x, b.y, b.z, b.w}, c);
}

// Eight consecutive elements from index k of a row of n; native vectors, not the uint4 struct: a copy of that
// struct is a memcpy, and registers that are only ever memcpy'd into and out of stay in scratch memory.
template <bool RAG>
__device__ __forceinline__ u32x4 piece(const bf16_t* __restrict__ row, int k, int n)
{
    if constexpr (RAG) return load_any<u32x4>(row + row_piece(k, 8, n), 0u);
    else return *reinterpret_cast<const u32x4*>(row + k);
}
// The same with the non-temporal hint.
template <bool RAG>
__device__ __forceinline__ uint4 piece_stream(const bf16_t* __restrict__ row, int k, int n)
{
    typedef u32x4 any_t __attribute__((aligned(2)));
    u32x4 v;
    if constexpr (RAG) v = __builtin_nontemporal_load(reinterpret_cast<const any_t*>(row + row_piece(k, 8, n)));
    else v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(row + k));
    return make_uint4(v.x, v.y, v.z, v.w);
}
// A piece read so, from index k on, zeros past the row's end.
__device__ __forceinline__ u32x4 cut(u32x4 v, int k, int n) { return drop_front<16>(v, k - row_piece(k, 8, n)); }
__device__ __forceinline__ uint4 cut(uint4 v, int k, int n)
{
    const u32x4 x = cut(u32x4{v.x, v.y, v.z, v.w}, k, n);
    return make_uint4(x[0], x[1], x[2], x[3]);
}

// 16-byte pieces of an (S rows) x (64 columns) slab of a row-major bf16 matrix: piece p -> row p / 8,
// columns 8 * (p % 8) ..+7; thread t takes pieces t, t + 256, ... (NST / 2 of them cover 16 NST rows).  Pieces
// past row S - 1 re-read the last row and land in LDS rows whose products are not stored.
template <int NST>
__device__ __forceinline__ void slab_load(u32x4 (&x)[NST / 2], const bf16_t* __restrict__ src, long ld, int S, int k0, int tid)
{
#pragma unroll
    for (int e = 0; e < NST / 2; ++e) {
        const int p = tid + 256 * e, row = min(p >> 3, S - 1);
        x[e] = *reinterpret_cast<const u32x4*>(src + (long)row * ld + k0 + (p & 7) * 8);
    }
}
template <int NST>
__device__ __forceinline__ void slab_store(const u32x4 (&x)[NST / 2], bf16_t (*dst)[KP], int tid)
{
#pragma unroll
    for (int e = 0; e < NST / 2; ++e) {
        const int p = tid + 256 * e;
        *reinterpret_cast<u32x4*>(&dst[p >> 3][(p & 7) * 8]) = x[e];
    }
}

// Two rows (contraction indices 2p and 2p + 1) of a (K, N) operand that is contiguous along N,
// eight columns each, interleaved into eight 32-bit pairs {row 2p (low half), row 2p + 1 (high half)}.
__device__ __forceinline__ void pair_rows(uint4 lo, uint4 hi, uint4& out0, uint4& out1)
{
    const uint32_t l[4] = {lo.x, lo.y, lo.z, lo.w}, h[4] = {hi.x, hi.y, hi.z, hi.w};
    uint32_t o[8];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        o[2 * m] = (l[m] & 0xffffu) | (h[m] << 16);
        o[2 * m + 1] = (l[m] >> 16) | (h[m] & 0xffff0000u);
    }
    out0 = make_uint4(o[0], o[1], o[2], o[3]);
    out1 = make_uint4(o[4], o[5], o[6], o[7]);
}

// The kernels below walk the contraction index in 64-wide slabs and keep PD slabs in flight: the
// requests for slab s + PD go out at the start of step s into registers (slot s % PD, named at compile
// time: the loop is unrolled PD times), step s multiplies out of LDS buffer s % 2, and slab s + 1
// moves from its registers into the other LDS buffer before the step's one barrier.  The operand that
// streams from HBM is loaded with the non-temporal hint so that it does not push the small one out
// of the L2.  Requests past the last slab re-read the last slab (never used) instead of branching, so
// that the compiler's wait counts stay those of the steady state; the up to PD - 1 slabs left over are written
// out behind the loop.
// In gemm_nt_kernel and gemm_rows_kernel only the streamed operand goes through LDS, where all four waves read it.
// The small operand's 16-row tiles are dealt out to the waves (tile w + 4 i), and a wave takes its fragments straight
// from the L2: no two waves want the same ones.  Rows past S re-read the last one, and what comes of them is not
// stored.  (With the small operand in LDS and a 16-row fragment of the big one per wave, every wave read the whole
// slab, 100 KB of LDS traffic per step and workgroup against 40: dW_dt and dW_x of 8 x 4096 x 2048 55 and 58 us,
// now 48 and 58; of 8 x 1536 x 2047 44 and 45, now 30 and 44; of 2 x 5120 x 4096 74 and 89, now 52 and 63.)
constexpr int PD = 4;
constexpr long ROWS_MIN_WGS = 512;   // two workgroups of gemm_rows_kernel fit on each of the 256 CUs
constexpr int ROWS_MIN_SPLIT_K = 4096;   // shorter contractions lose more to the second launch than they gain (K = 1536: 21 -> 25 us)

// A wave's fragments of the small operand for one slab: tiles w + 4 i, contraction halves ks.
template <int NTW> struct small_frags { u32x4 f[NTW][2]; };
template <bool RAG, int NTW, bool SKIP>
__device__ __forceinline__ void load_frags(small_frags<NTW>& x, const bf16_t* __restrict__ src, long ld, int S, int w, int lane, int k0, int K)
{
#pragma unroll
    for (int i = 0; i < NTW; ++i) {
        if (SKIP && i == NTW - 1 && 16 * (w + 4 * i) >= S) continue;   // uniform: this wave has no such tile (gemm_rows_kernel: slower, 73 -> 97 us)
        const bf16_t* row = src + (long)min(16 * (w + 4 * i) + (lane & 15), S - 1) * ld;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) x.f[i][ks] = piece<RAG>(row, k0 + 32 * ks + 8 * (lane >> 4), K);
    }
}
template <int NTW>
__device__ __forceinline__ void cut_frags(small_frags<NTW>& x, int lane, int k0, int K)
{
#pragma unroll
    for (int i = 0; i < NTW; ++i)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) x.f[i][ks] = cut(x.f[i][ks], k0 + 32 * ks + 8 * (lane >> 4), K);
}

// C[big][small] (or, OUT_T, C[small][big]), float32, = sum_k Big[big][k] Small[small][k] per batch entry.
// grid (M big rows / 64 rounded up, batch, parts).  S <= 64 NTW.  Plain: K % 64 == 0, M % 64 == 0, ldc and c_batch % 4 == 0.
// With parts > 1 workgroup (., ., z) contracts over the z-th part of K and C is one share after another, part_stride apart.
template <bool OUT_T, bool RAG, int NTW>
__global__ void __launch_bounds__(256, 2) gemm_nt_kernel(const bf16_t* __restrict__ Big, long big_ld, long big_batch,
                                                       const bf16_t* __restrict__ Small, long small_ld, long small_batch,
                                                       float* __restrict__ C, long ldc, long c_batch, long part_stride, int M, int S,
                                                       int K, int vec_c)
{
    __shared__ __attribute__((aligned(16))) bf16_t Bs[2][64][KP];
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, j = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int d0 = blockIdx.x * 64;
    const long b = blockIdx.y;
    const int br = tid >> 3, bk = (tid & 7) * 8;   // this thread's pieces of the big operand's slab: rows br and br + 32
    // this part's slabs: rows and contraction counted from its first one
    const int slabs = (K + KSLAB - 1) / KSLAB, per_part = (slabs + (int)gridDim.z - 1) / (int)gridDim.z;
    const int k_first = blockIdx.z * per_part * KSLAB, nsteps = min(slabs - (int)blockIdx.z * per_part, per_part);
    K -= k_first;
    const bf16_t* __restrict__ brow0 = Big + k_first + b * big_batch + (long)(RAG ? min(d0 + br, M - 1) : d0 + br) * big_ld;
    const bf16_t* __restrict__ brow1 = Big + k_first + b * big_batch + (long)(RAG ? min(d0 + br + 32, M - 1) : d0 + br + 32) * big_ld;
    const bf16_t* __restrict__ sm = Small + k_first + b * small_batch;
    f32x4_t acc[4][NTW];
#pragma unroll
    for (int rt = 0; rt < 4; ++rt)
#pragma unroll
        for (int i = 0; i < NTW; ++i) acc[rt][i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // one named set of registers per slot, and the step written out per slot (a macro), so that every
    // register set is addressed statically
    small_frags<NTW> sf0, sf1, sf2, sf3;
    uint4 br0[2], br1[2], br2[2], br3[2];
#define SS_NT_ISSUE(s_, SF, BR)                                          \
    {                                                                    \
        const int k0_ = min((s_), nsteps - 1) * KSLAB;                   \
        BR[0] = piece_stream<RAG>(brow0, k0_ + bk, K);                   \
        BR[1] = piece_stream<RAG>(brow1, k0_ + bk, K);                   \
        load_frags<RAG, NTW, true>(SF, sm, small_ld, S, w, lane, k0_, K);\
    }
#define SS_NT_FILL(s_, BUF, BR)                                          \
    {                                                                    \
        if (RAG && ((s_) + 1) * KSLAB > K) {                     \
            BR[0] = cut(BR[0], (s_) * KSLAB + bk, K);          \
            BR[1] = cut(BR[1], (s_) * KSLAB + bk, K);          \
        }                                                                \
        *reinterpret_cast<uint4*>(&Bs[BUF][br][bk]) = BR[0];             \
        *reinterpret_cast<uint4*>(&Bs[BUF][br + 32][bk]) = BR[1];        \
    }
    // step s_ out of LDS buffer BUF; this slot's registers are free again (its slab went into LDS a
    // step ago, its fragments are copied out first), the next slot's slab moves into the other buffer
#define SS_NT_STEP(s_, BUF, SF, BR, BRN)                                                                              \
    {                                                                                                                 \
        small_frags<NTW> cur = SF;                                                                                    \
        if (RAG && ((s_) + 1) * KSLAB > K) cut_frags<NTW>(cur, lane, (s_) * KSLAB, K);              \
        SS_NT_ISSUE((s_) + PD, SF, BR)                                                                                \
        _Pragma("unroll") for (int ks = 0; ks < 2; ++ks)                                                              \
            _Pragma("unroll") for (int rt = 0; rt < 4; ++rt)                                                          \
            {                                                                                                         \
                const u32x4 bf = *reinterpret_cast<const u32x4*>(&Bs[BUF][16 * rt + j][32 * ks + 8 * g]);             \
                _Pragma("unroll") for (int i = 0; i < NTW; ++i) acc[rt][i] = mma::step(bf, cur.f[i][ks], acc[rt][i]); \
            }                                                                                                         \
        if ((s_) + 1 < nsteps) SS_NT_FILL((s_) + 1, (BUF) ^ 1, BRN)                                                   \
        __syncthreads();                                                                                              \
    }
    SS_NT_ISSUE(0, sf0, br0)
    __builtin_amdgcn_sched_barrier(0);
    SS_NT_ISSUE(1, sf1, br1)
    __builtin_amdgcn_sched_barrier(0);
    SS_NT_ISSUE(2, sf2, br2)
    __builtin_amdgcn_sched_barrier(0);
    SS_NT_ISSUE(3, sf3, br3)
    __builtin_amdgcn_sched_barrier(0);
    SS_NT_FILL(0, 0, br0)
    __syncthreads();
    int s0 = 0;
    for (; s0 + PD <= nsteps; s0 += PD) {
        SS_NT_STEP(s0, 0, sf0, br0, br1)
        SS_NT_STEP(s0 + 1, 1, sf1, br1, br2)
        SS_NT_STEP(s0 + 2, 0, sf2, br2, br3)
        SS_NT_STEP(s0 + 3, 1, sf3, br3, br0)
    }
    if (s0 < nsteps) SS_NT_STEP(s0, 0, sf0, br0, br1)
    if (s0 + 1 < nsteps) SS_NT_STEP(s0 + 1, 1, sf1, br1, br2)
    if (s0 + 2 < nsteps) SS_NT_STEP(s0 + 2, 0, sf2, br2, br3)
#undef SS_NT_STEP
#undef SS_NT_FILL
#undef SS_NT_ISSUE
    float* __restrict__ c = C + blockIdx.z * part_stride + b * c_batch;
#pragma unroll
    for (int rt = 0; rt < 4; ++rt)
#pragma unroll
        for (int t = 0; t < NTW; ++t) {
            const int row = d0 + 16 * rt + 4 * g, col = 16 * (w + 4 * t) + j;
            if (col >= S) continue;
            if (OUT_T && vec_c) {
                if (row < M) *reinterpret_cast<float4*>(c + (long)col * ldc + row) = make_float4(acc[rt][t][0], acc[rt][t][1], acc[rt][t][2], acc[rt][t][3]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (!RAG || row + i < M) c[OUT_T ? (long)col * ldc + row + i : (long)(row + i) * ldc + col] = acc[rt][t][i];
            }
        }
}

// Out (S x N per batch entry, bf16) = W (S x K, contiguous along K) X (K x N, contiguous along N).
// grid (N / 64 rounded up, batch, parts).  S <= 64 NTW; any K and N >= 8, any pitch (RAG).
// With parts > 1 workgroup (., ., z) contracts over the z-th part of K (none of them empty) and leaves its float32
// share in Part[z][batch entry][S][N] for rows_reduce_kernel: a product with few columns would otherwise put a single
// workgroup on a CU, with nothing to run while that one waits at its barrier.
template <int NTW>
__global__ void __launch_bounds__(256, 2) gemm_rows_kernel(const bf16_t* __restrict__ W, long w_ld, long w_batch,
                                                         const bf16_t* __restrict__ X, long x_ld, long x_batch,
                                                         bf16_t* __restrict__ Out, long o_ld, long o_batch, int S, int N, int K,
                                                         float* __restrict__ Part)
{
    __shared__ __attribute__((aligned(16))) uint32_t Xp[2][KSLAB / 2][XPITCH];
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, j = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = blockIdx.x * 64;
    const long b = blockIdx.y;
    const int slabs = (K + KSLAB - 1) / KSLAB, per_part = (slabs + (int)gridDim.z - 1) / (int)gridDim.z;
    const int first = blockIdx.z * per_part, nsteps = min(slabs - first, per_part);   // this part's slabs
    const bf16_t* __restrict__ wm = W + b * w_batch;
    const int xp = tid >> 3, xo = tid & 7;   // pair of rows, group of eight columns
    const bf16_t* __restrict__ xcol = X + b * x_batch;
    f32x4_t acc[NTW][4];
#pragma unroll
    for (int i = 0; i < NTW; ++i)
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) acc[i][ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    small_frags<NTW> wf0, wf1, wf2, wf3;   // one named set of registers per slot, steps written out (see gemm_nt_kernel)
    uint4 xr0[2], xr1[2], xr2[2], xr3[2];
#define SS_ROWS_ISSUE(s_, WF, XR)                                                          \
    {                                                                                      \
        const int k0_ = (first + min((s_), nsteps - 1)) * KSLAB, x0_ = k0_ + 2 * xp;       \
        XR[0] = piece_stream<true>(xcol + (long)min(x0_, K - 1) * x_ld, n0 + 8 * xo, N);         \
        XR[1] = piece_stream<true>(xcol + (long)min(x0_ + 1, K - 1) * x_ld, n0 + 8 * xo, N); \
        load_frags<true, NTW, false>(WF, wm, w_ld, S, w, lane, k0_, K);                            \
    }
#define SS_ROWS_FILL(s_, BUF, XR)                                                          \
    {                                                                                      \
        const int k0_ = (first + (s_)) * KSLAB;                                            \
        if (n0 + 64 > N) {                                                          \
            XR[0] = cut(XR[0], n0 + 8 * xo, N);                                            \
            XR[1] = cut(XR[1], n0 + 8 * xo, N);                                            \
        }                                                                                  \
        if (k0_ + KSLAB > K) {                                                      \
            if (k0_ + 2 * xp >= K) XR[0] = make_uint4(0u, 0u, 0u, 0u);                     \
            if (k0_ + 2 * xp + 1 >= K) XR[1] = make_uint4(0u, 0u, 0u, 0u);                 \
        }                                                                                  \
        uint4 o0_, o1_;                                                                    \
        pair_rows(XR[0], XR[1], o0_, o1_);                                                 \
        *reinterpret_cast<uint4*>(&Xp[BUF][xp][8 * xo]) = o0_;                             \
        *reinterpret_cast<uint4*>(&Xp[BUF][xp][8 * xo + 4]) = o1_;                         \
    }
#define SS_ROWS_STEP(s_, BUF, WF, XR, XRN)                                                                            \
    {                                                                                                                 \
        small_frags<NTW> cur = WF;                                                                                    \
        if ((first + (s_) + 1) * KSLAB > K) cut_frags<NTW>(cur, lane, (first + (s_)) * KSLAB, K);              \
        SS_ROWS_ISSUE((s_) + PD, WF, XR) /* this slot's slab went into LDS a step ago */                              \
        _Pragma("unroll") for (int ks = 0; ks < 2; ++ks)                                                              \
            _Pragma("unroll") for (int ct = 0; ct < 4; ++ct)                                                          \
            {                                                                                                         \
                const uint32_t* xq = &Xp[BUF][16 * ks + 4 * g][16 * ct + j];                                          \
                const u32x4 bf = {xq[0], xq[XPITCH], xq[2 * XPITCH], xq[3 * XPITCH]};                                 \
                _Pragma("unroll") for (int i = 0; i < NTW; ++i) acc[i][ct] = mma::step(cur.f[i][ks], bf, acc[i][ct]); \
            }                                                                                                         \
        if ((s_) + 1 < nsteps) SS_ROWS_FILL((s_) + 1, (BUF) ^ 1, XRN)                                                 \
        __syncthreads();                                                                                              \
    }
    SS_ROWS_ISSUE(0, wf0, xr0)
    __builtin_amdgcn_sched_barrier(0);
    SS_ROWS_ISSUE(1, wf1, xr1)
    __builtin_amdgcn_sched_barrier(0);
    SS_ROWS_ISSUE(2, wf2, xr2)
    __builtin_amdgcn_sched_barrier(0);
    SS_ROWS_ISSUE(3, wf3, xr3)
    __builtin_amdgcn_sched_barrier(0);
    SS_ROWS_FILL(0, 0, xr0)
    __syncthreads();
    int s0 = 0;
    for (; s0 + PD <= nsteps; s0 += PD) {
        SS_ROWS_STEP(s0, 0, wf0, xr0, xr1)
        SS_ROWS_STEP(s0 + 1, 1, wf1, xr1, xr2)
        SS_ROWS_STEP(s0 + 2, 0, wf2, xr2, xr3)
        SS_ROWS_STEP(s0 + 3, 1, wf3, xr3, xr0)
    }
    if (s0 < nsteps) SS_ROWS_STEP(s0, 0, wf0, xr0, xr1)
    if (s0 + 1 < nsteps) SS_ROWS_STEP(s0 + 1, 1, wf1, xr1, xr2)
    if (s0 + 2 < nsteps) SS_ROWS_STEP(s0 + 2, 0, wf2, xr2, xr3)
#undef SS_ROWS_STEP
#undef SS_ROWS_FILL
#undef SS_ROWS_ISSUE
    const bool split = gridDim.z > 1;
    float* __restrict__ pp = Part + ((long)blockIdx.z * gridDim.y + b) * S * N;
    bf16_t* __restrict__ o = Out + b * o_batch;
#pragma unroll
    for (int t = 0; t < NTW; ++t)
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
            const int row = 16 * (w + 4 * t) + 4 * g, col = n0 + 16 * ct + j;
            if (col >= N) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (row + i >= S) continue;
                if (split) pp[(long)(row + i) * N + col] = acc[t][ct][i];
                else o[(long)(row + i) * o_ld + col] = bf16_t(f32_to_bf16_bits(acc[t][ct][i]));
            }
        }
}

// The same product for operands of whole pieces (K % 64 == 0, N % 64 == 0, S <= 16 NST), the weights through LDS too.
// Against fragments from the L2 that is the faster form for a large X, us, this kernel / gemm_rows_kernel:
//   8 x 4096 x 2048, S = 160: 58 / 74, S = 128: 52 / 61      2 x 5120 x 16384, S = 192: 119 / 150, S = 160: 103 / 138
//   32 x 2048 x 2048, S = 96: 77 / 89, S = 64: 69 / 71
// and the slower one by 4 to 25 % for a smaller one (both forms would be needed for that line):
//   8 x 1536 x 2048, S = 80: 18.9 / 18.0      8 x 3072 x 2048, S = 128: 48 / 36      4 x 2560 x 4096, S = 112: 38 / 29
//   2 x 5120 x 4096, S = 192: 54 / 49         4 x 4096 x 1536, S = 128: 36 / 28      1 x 4096 x 2048, S = 160: 20.8 / 21.1
// grid (N / 64, batch, parts).
template <int NST>
__global__ void __launch_bounds__(256, 2) gemm_rows_lds_kernel(const bf16_t* __restrict__ W, long w_ld, long w_batch,
                                                         const bf16_t* __restrict__ X, long x_ld, long x_batch,
                                                         bf16_t* __restrict__ Out, long o_ld, long o_batch, int S, int N, int K,
                                                         float* __restrict__ Part)
{
    __shared__ __attribute__((aligned(16))) bf16_t Ws[2][NST * 16][KP];
    __shared__ __attribute__((aligned(16))) uint32_t Xp[2][KSLAB / 2][XPITCH];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, g = lane >> 4, j = lane & 15;
    const int n0 = blockIdx.x * 64;
    const long b = blockIdx.y;
    const int slabs = (K + KSLAB - 1) / KSLAB, per_part = (slabs + (int)gridDim.z - 1) / (int)gridDim.z;
    const int first = blockIdx.z * per_part, nsteps = min(slabs - first, per_part);   // this part's slabs
    const bf16_t* __restrict__ wm = W + b * w_batch;
    const int xp = tid >> 3, xo = tid & 7;   // pair of rows, group of eight columns
    const bf16_t* __restrict__ xcol = X + b * x_batch;
    const int ST = (S + 15) >> 4;
    // The four waves split the S x 64 tile two by two: wave (wv, wc) has half of the output's row tiles and
    // column tiles 2 wc, 2 wc + 1, so that every weight fragment read from LDS feeds two MFMAs (with a wave
    // per column tile each wave read the whole weight slab and LDS was the limit: 78 -> 68 us).
    const int wv = w >> 1, wc = w & 1;
    const int RH = (ST + 1) >> 1;
    constexpr int MAXRH = NST / 2;
    f32x4_t acc[MAXRH][2];
#pragma unroll
    for (int ri = 0; ri < MAXRH; ++ri) acc[ri][0] = acc[ri][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    u32x4 wr0[NST / 2], wr1[NST / 2], wr2[NST / 2], wr3[NST / 2];   // one named set of registers per slot, steps written out (see gemm_nt_kernel)
    uint4 xr0[2], xr1[2], xr2[2], xr3[2];
#define SS_ROWS_ISSUE(s_, WR, XR)                                                          \
    {                                                                                      \
        const int k0_ = (first + min((s_), nsteps - 1)) * KSLAB, x0_ = k0_ + 2 * xp;       \
        XR[0] = piece_stream<false>(xcol + (long)x0_ * x_ld, n0 + 8 * xo, N);         \
        XR[1] = piece_stream<false>(xcol + (long)(x0_ + 1) * x_ld, n0 + 8 * xo, N); \
        slab_load<NST>(WR, wm, w_ld, S, k0_, tid);                                         \
    }
#define SS_ROWS_FILL(BUF, WR, XR)                                                          \
    {                                                                                      \
        slab_store<NST>(WR, Ws[BUF], tid);                                                 \
        uint4 o0_, o1_;                                                                    \
        pair_rows(XR[0], XR[1], o0_, o1_);                                                 \
        *reinterpret_cast<uint4*>(&Xp[BUF][xp][8 * xo]) = o0_;                             \
        *reinterpret_cast<uint4*>(&Xp[BUF][xp][8 * xo + 4]) = o1_;                         \
    }
#define SS_ROWS_STEP(s_, BUF, WR, XR, WRN, XRN)                                                                       \
    {                                                                                                                 \
        SS_ROWS_ISSUE((s_) + PD, WR, XR) /* this slot's slab went into LDS a step ago */                              \
        _Pragma("unroll") for (int ks = 0; ks < 2; ++ks)                                                              \
        {                                                                                                             \
            const uint32_t* xq = &Xp[BUF][16 * ks + 4 * g][32 * wc + j];                                              \
            const uint4 bf0 = make_uint4(xq[0], xq[XPITCH], xq[2 * XPITCH], xq[3 * XPITCH]);                          \
            const uint4 bf1 = make_uint4(xq[16], xq[XPITCH + 16], xq[2 * XPITCH + 16], xq[3 * XPITCH + 16]);          \
            _Pragma("unroll") for (int ri = 0; ri < MAXRH; ++ri) if (ri < RH && wv * RH + ri < ST)                    \
            {                                                                                                         \
                const uint4 af = *reinterpret_cast<const uint4*>(&Ws[BUF][16 * (wv * RH + ri) + j][32 * ks + 8 * g]); \
                acc[ri][0] = mfma_bf16(af, bf0, acc[ri][0]);                                                          \
                acc[ri][1] = mfma_bf16(af, bf1, acc[ri][1]);                                                          \
            }                                                                                                         \
        }                                                                                                             \
        if ((s_) + 1 < nsteps) SS_ROWS_FILL((BUF) ^ 1, WRN, XRN)                                                      \
        __syncthreads();                                                                                              \
    }
    SS_ROWS_ISSUE(0, wr0, xr0)
    __builtin_amdgcn_sched_barrier(0);
    SS_ROWS_ISSUE(1, wr1, xr1)
    __builtin_amdgcn_sched_barrier(0);
    SS_ROWS_ISSUE(2, wr2, xr2)
    __builtin_amdgcn_sched_barrier(0);
    SS_ROWS_ISSUE(3, wr3, xr3)
    __builtin_amdgcn_sched_barrier(0);
    SS_ROWS_FILL(0, wr0, xr0)
    __syncthreads();
    int s0 = 0;
    for (; s0 + PD <= nsteps; s0 += PD) {
        SS_ROWS_STEP(s0, 0, wr0, xr0, wr1, xr1)
        SS_ROWS_STEP(s0 + 1, 1, wr1, xr1, wr2, xr2)
        SS_ROWS_STEP(s0 + 2, 0, wr2, xr2, wr3, xr3)
        SS_ROWS_STEP(s0 + 3, 1, wr3, xr3, wr0, xr0)
    }
    if (s0 < nsteps) SS_ROWS_STEP(s0, 0, wr0, xr0, wr1, xr1)
    if (s0 + 1 < nsteps) SS_ROWS_STEP(s0 + 1, 1, wr1, xr1, wr2, xr2)
    if (s0 + 2 < nsteps) SS_ROWS_STEP(s0 + 2, 0, wr2, xr2, wr3, xr3)
#undef SS_ROWS_STEP
#undef SS_ROWS_FILL
#undef SS_ROWS_ISSUE
    const bool split = gridDim.z > 1;
    float* __restrict__ pp = Part + ((long)blockIdx.z * gridDim.y + b) * S * N;
    bf16_t* __restrict__ o = Out + b * o_batch;
#pragma unroll
    for (int ri = 0; ri < MAXRH; ++ri)
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2) {
            const int row = 16 * (wv * RH + ri) + 4 * g, col = n0 + 32 * wc + j + 16 * c2;
            if (ri >= RH) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (row + i >= S) continue;
                if (split) pp[(long)(row + i) * N + col] = acc[ri][c2][i];
                else o[(long)(row + i) * o_ld + col] = bf16_t(f32_to_bf16_bits(acc[ri][c2][i]));
            }
        }
}

// Out[b][row][8 c ..+7] (bf16) = sum over the parts of Part[part][b][row][8 c ..+7]; one thread per eight columns.
__global__ void __launch_bounds__(256) rows_reduce_kernel(const float* __restrict__ Part, int parts, long part_stride,
                                                           bf16_t* __restrict__ Out, long o_ld, long o_batch, int S, int ncols,
                                                           long items)
{
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= items) return;
    const int per_row = ncols >> 3;
    const int c8 = (int)(idx % per_row);
    const long br = idx / per_row;
    const int row = (int)(br % S);
    const long b = br / S;
    const float* __restrict__ src = Part + br * ncols + 8 * c8;
    float4 lo = *reinterpret_cast<const float4*>(src), hi = *reinterpret_cast<const float4*>(src + 4);
    for (int z = 1; z < parts; ++z) {
        const float4 l2 = *reinterpret_cast<const float4*>(src + z * part_stride);
        const float4 h2 = *reinterpret_cast<const float4*>(src + z * part_stride + 4);
        lo.x += l2.x; lo.y += l2.y; lo.z += l2.z; lo.w += l2.w;
        hi.x += h2.x; hi.y += h2.y; hi.z += h2.z; hi.w += h2.w;
    }
    uint4 o;
    o.x = f32_to_bf16_bits(lo.x) | ((uint32_t)f32_to_bf16_bits(lo.y) << 16);
    o.y = f32_to_bf16_bits(lo.z) | ((uint32_t)f32_to_bf16_bits(lo.w) << 16);
    o.z = f32_to_bf16_bits(hi.x) | ((uint32_t)f32_to_bf16_bits(hi.y) << 16);
    o.w = f32_to_bf16_bits(hi.z) | ((uint32_t)f32_to_bf16_bits(hi.w) << 16);
    *reinterpret_cast<uint4*>(Out + b * o_batch + (long)row * o_ld + 8 * c8) = o;
}

// Out (M x N per batch entry, bf16) = W (M x K, contiguous along K) Y (K x N, contiguous along N).
// Workgroups of one or four waves, of 64 columns each; grid (columns / those of a workgroup, M / (16 * mtiles), batch) rounded up,
// mtiles = 16-row tiles of the result per workgroup; every wave has columns.  K <= 32 NKS.  Plain: K % 32 == 0, N % 64 == 0,
// M % 16 == 0, whole 16-byte pieces.
// Bound by writing Out once, if little else moves.  A wave owns 64 columns and walks the row tiles by itself, without LDS and
// without a barrier; four waves of a workgroup are neighbours along N, so that the weights, the same for all four, come
// from the L2 once per 256 columns (with 64 columns per workgroup they were 256 MB at 8 x 4096 x 2048 against the 134 of Out).
// The wave's part of Y stays in registers as first operands of the transposed product, whose row r is a column of Y and
// may be any: a lane reads four columns at eight contraction indices, and a byte permute takes column c's pairs out of
// them, so row r of product c is column strip_col(r) + c.  With strip_col as below a lane's results of all four products
// are two runs of eight columns, and each of the two stores that write them covers 64 contiguous bytes of sixteen rows.
// us, before (64 x 64 tiles through LDS, a column strip per workgroup) / now: 8 x 4096 x 2048, K = 128: 58 / 43; 2 x 5120 x 4096, K = 160:
// 45 / 30; 4 x 2560 x 2048, K = 80: 19 / 15; 8 x 1536 x 2047, K = 48: 22 / 21; 4 x 4096 x 1531, K = 128: 36 / 33.
__device__ __forceinline__ int strip_col(int r) { return 32 * ((r >> 1) & 1) + 8 * (r >> 2) + 4 * (r & 1); }
template <bool RAG, int NKS>
__global__ void __launch_bounds__(256, 2) gemm_cols_kernel(const bf16_t* __restrict__ W, long w_ld, const bf16_t* __restrict__ Y,
                                                           long y_ld, long y_batch, bf16_t* __restrict__ Out, long o_ld, long o_batch,
                                                           int M, int N, int K, int mtiles)
{
    const int lane = threadIdx.x & 63, g = lane >> 4, j = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = blockIdx.x * blockDim.x + 64 * w;
    if (n0 >= N) return;   // uniform; no barrier below
    const long b = blockIdx.z;
    const int KS = (K + 31) >> 5;   // 32-wide contraction steps (<= NKS)
    const int t_begin = blockIdx.y * mtiles, t_end = min((M + 15) / 16, t_begin + mtiles);
    auto load_w = [&](u32x4 (&f)[NKS], int t) {
        const int m = 16 * min(t, t_end - 1) + j;
        const bf16_t* __restrict__ wrow = W + (long)(RAG ? min(m, M - 1) : m) * w_ld;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
            if (ks < KS) f[ks] = piece<RAG>(wrow, 32 * ks + 8 * g, K);
    };
    constexpr int AHEAD = 2;   // tiles requested ahead
    u32x4 wf[AHEAD][NKS];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) load_w(wf[i], t_begin + i);
    // the columns of Y: row r of the products, see above
    u32x4 yf[NKS][4];
    {
        const int col = n0 + strip_col(j), ycol = RAG ? row_piece(col, 4, N) : col;
        const bf16_t* __restrict__ y = Y + b * y_batch + ycol;
        u32x2 raw[NKS][8];
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
            if (ks < KS)
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const int k = 32 * ks + 8 * g + r;
                    raw[ks][r] = load_any<u32x2>(y + (long)(RAG ? min(k, K - 1) : k) * y_ld, 0u);
                }
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
            if (ks < KS) {
                if constexpr (RAG) {
                    const int sh = 16 * min(col - ycol, 4);   // a piece that ended past the row; whole pieces past it are not stored
#pragma unroll
                    for (int r = 0; r < 8; ++r) {
                        const uint64_t v = (uint64_t(raw[ks][r][1]) << 32) | raw[ks][r][0];
                        const uint64_t x = sh >= 64 || 32 * ks + 8 * g + r >= K ? 0ull : v >> sh;
                        raw[ks][r] = u32x2{(uint32_t)x, (uint32_t)(x >> 32)};
                    }
                }
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        yf[ks][c][q] = __builtin_amdgcn_perm(raw[ks][2 * q + 1][c >> 1], raw[ks][2 * q][c >> 1], c & 1 ? 0x07060302u : 0x05040100u);
            }
    }
    // a lane's results: row 16 t + j, columns n0 + 32 h + 8 g ..+7 for h = 0, 1
    bf16_t* __restrict__ o = Out + b * o_batch;
    const int oc = n0 + 8 * g;
    auto do_tile = [&](int t, auto slot_tag) {
        constexpr int SLOT = decltype(slot_tag)::value;
        f32x4_t acc[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
            if (ks < KS) {
                u32x4 x = wf[SLOT][ks];
                if (RAG && 32 * (ks + 1) > K) x = cut(x, 32 * ks + 8 * g, K);   // the last step
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[c] = mma::step(yf[ks][c], x, acc[c]);
            }
        load_w(wf[SLOT], t + AHEAD);
        const int m = 16 * t + j;
        bf16_t* __restrict__ row = o + (long)m * o_ld;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float r[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) r[i] = acc[i & 3][2 * h + (i >> 2)];
            const uint4 x = io8<bf16_t>::pack(r);
            if constexpr (!RAG) *reinterpret_cast<uint4*>(row + oc + 32 * h) = x;
            else if (n0 + 64 <= N && 16 * t + 16 <= M) store_row16(row + oc + 32 * h, u32x4{x.x, x.y, x.z, x.w});   // uniform
            else if (m < M && oc + 32 * h < N) io8<bf16_t>::store_elem(row + oc + 32 * h, 0u, x, N - (oc + 32 * h));
        }
    };
    for (int t = t_begin; t < t_end; t += AHEAD) {
        do_tile(t, std::integral_constant<int, 0>{});
        if (t + 1 < t_end) do_tile(t + 1, std::integral_constant<int, 1>{});
    }
}

// Out += W Y, of the same operands.  A result that is also read is the faster for leaving through LDS in whole rows of 128
// bytes, 64 of them per workgroup: in the layer's backward pass, us, this kernel / the one above with the old values
// requested two tiles ahead: 8 x 4096 x 2048, K = 160, 77 / 84, 8 x 1536 x 2047, K = 80, 42 / 47.
// grid (N / 64, M / (64 * mtiles), batch) rounded up, mtiles = 64-row tiles of the result per workgroup (the small
// operand is prepared once for all of them).  K <= 32 NKS.  Plain: K % 32 == 0, N % 64 == 0, M % (64 * mtiles) == 0.
template <bool RAG, int NKS>
__global__ void __launch_bounds__(256) gemm_cols_add_kernel(const bf16_t* __restrict__ W, long w_ld, const bf16_t* __restrict__ Y,
                                                         long y_ld, long y_batch, bf16_t* __restrict__ Out, long o_ld, long o_batch,
                                                         int M, int N, int K, int mtiles)
{
    __shared__ __attribute__((aligned(16))) uint32_t Yp[NKS * 16][XPITCH];         // pairs of contraction indices x 64 columns
    __shared__ __attribute__((aligned(16))) float Os[64][64 + 4];                 // a tile of the result on its way out (two of them, one barrier per tile: slower, 71 -> 76 us)
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, g = lane >> 4, j = lane & 15;
    const int n0 = blockIdx.x * 64;
    const int m_base = blockIdx.y * 64 * mtiles;
    const long b = blockIdx.z;
    const bf16_t* __restrict__ y = Y + b * y_batch;
    const int KS = (K + 31) >> 5;   // 32-wide contraction steps (<= NKS)
    // the small operand, paired and into LDS: item p -> pair of rows p / 8, eight columns from 8 * (p % 8)
    for (int p = tid; p < KS * 16 * 8; p += 256) {
        const int pr = p >> 3, po = p & 7;
        u32x4 lo = piece<RAG>(y + (long)(RAG ? min(2 * pr, K - 1) : 2 * pr) * y_ld, n0 + 8 * po, N);
        u32x4 hi = piece<RAG>(y + (long)(RAG ? min(2 * pr + 1, K - 1) : 2 * pr + 1) * y_ld, n0 + 8 * po, N);
        if constexpr (RAG) {
            const u32x4 zero = {0u, 0u, 0u, 0u};
            lo = 2 * pr < K ? cut(lo, n0 + 8 * po, N) : zero;
            hi = 2 * pr + 1 < K ? cut(hi, n0 + 8 * po, N) : zero;
        }
        uint4 o0, o1;
        pair_rows(make_uint4(lo[0], lo[1], lo[2], lo[3]), make_uint4(hi[0], hi[1], hi[2], hi[3]), o0, o1);
        *reinterpret_cast<uint4*>(&Yp[pr][8 * po]) = o0;
        *reinterpret_cast<uint4*>(&Yp[pr][8 * po + 4]) = o1;
    }
    __syncthreads();
    // ... and from there into registers as fragments: first operand of the transposed product,
    // row = column 16 ct + j of Y, contraction indices 32 ks + 8 g ..+7
    uint4 yf[4][NKS];
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
            if (ks < KS) {
                const uint32_t* q = &Yp[16 * ks + 4 * g][16 * ct + j];
                yf[ct][ks] = make_uint4(q[0], q[XPITCH], q[2 * XPITCH], q[3 * XPITCH]);
            }
    const bf16_t* __restrict__ wcol = W;
    auto load_w = [&](uint4 (&f)[NKS], int m0) {
        const bf16_t* __restrict__ wrow = wcol + (long)(RAG ? min(m0 + 16 * w + j, M - 1) : m0 + 16 * w + j) * w_ld;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
            if (ks < KS) {
                const u32x4 x = piece<RAG>(wrow, 32 * ks + 8 * g, K);
                f[ks] = make_uint4(x[0], x[1], x[2], x[3]);
            }
    };
    uint4 wf[NKS];
    load_w(wf, m_base);
    bf16_t* __restrict__ o = Out + b * o_batch;
    for (int mt = 0; mt < mtiles; ++mt) {
        const int m0 = m_base + 64 * mt;
        if (RAG && m0 >= M) break;   // uniform
        uint4 wc[NKS];
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
            wc[ks] = wf[ks];
            if (RAG && ks < KS && 32 * (ks + 1) > K) wc[ks] = cut(wc[ks], 32 * ks + 8 * g, K);   // the last step
        }
        if (mt + 1 < mtiles) load_w(wf, m0 + 64);
        // earlier values of this tile: requested before the arithmetic
        u32x4 prev[2];
        uint32_t last[2];   // RAG: see load_row16
        auto prev_at = [&](int e) {
            const int idx = tid + 256 * e, row = idx >> 3, pc = idx & 7;
            return o + (long)(RAG ? min(m0 + row, M - 1) : m0 + row) * o_ld + (RAG ? row_piece(n0 + 8 * pc, 8, N) : n0 + 8 * pc);
        };
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if constexpr (RAG) load_row16(prev_at(e), Out, prev[e], last[e]);
            else prev[e] = *reinterpret_cast<const u32x4*>(prev_at(e));
        }
        f32x4_t acc[4];
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
            acc[ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks)
                if (ks < KS) acc[ct] = mfma_bf16(yf[ct][ks], wc[ks], acc[ct]);   // (Y^T W^T): row 16 ct + 4 g + i of Y^T, column 16 w + j of W^T
        }
        if (mt > 0) __syncthreads();   // the previous tile has left Os
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
            *reinterpret_cast<float4*>(&Os[16 * w + j][16 * ct + 4 * g]) = make_float4(acc[ct][0], acc[ct][1], acc[ct][2], acc[ct][3]);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int idx = tid + 256 * e, row = idx >> 3, pc = idx & 7;
            const float4 lo = *reinterpret_cast<const float4*>(&Os[row][8 * pc]);
            const float4 hi = *reinterpret_cast<const float4*>(&Os[row][8 * pc + 4]);
            float r[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
            if constexpr (RAG) {
                prev[e] = shift_row16(prev_at(e), Out, prev[e], last[e]);
                if (n0 + 64 > N) prev[e] = cut(prev[e], n0 + 8 * pc, N);
            }
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                r[2 * m] += bf16_lo(prev[e][m]);
                r[2 * m + 1] += bf16_hi(prev[e][m]);
            }
            bf16_t* dst = o + (long)(m0 + row) * o_ld + n0 + 8 * pc;
            if constexpr (RAG) {
                const uint4 x = io8<bf16_t>::pack(r);
                if (n0 + 64 <= N && m0 + 64 <= M) store_row16(dst, u32x4{x.x, x.y, x.z, x.w});   // uniform
                else if (m0 + row < M) io8<bf16_t>::store_elem(dst, 0u, x, N - (n0 + 8 * pc));
            } else {
                *reinterpret_cast<uint4*>(dst) = io8<bf16_t>::pack(r);
            }
        }
    }
}

inline bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
inline bool mult8(long x) { return x % 8 == 0; }
inline unsigned tiles64(int n) { return (unsigned)((n + 63) / 64); }

// One launch each (the small operand has at most SMAX rows).
template <bool OUT_T, bool RAG>
void launch_nt(const GemmArgs& g, const bf16_t* big, long big_ld, long big_batch, const bf16_t* small, long small_ld, long small_batch,
               float* C, int M, int S, hipStream_t stream)
{
    // parts go to the workspace, each as a dense (batch, rows, columns) block, and are added up from there
    const int parts = parts_for(g, (long)tiles64(M) * g.batch, g.K, KSLAB, (size_t)g.batch * M * S * sizeof(float));
    float* const dst = parts > 1 ? static_cast<float*>(g.split_ws) : C;
    const long ldc = parts > 1 ? (OUT_T ? M : S) : g.ldc, c_batch = parts > 1 ? (long)M * S : g.c_batch, part_stride = (long)g.batch * M * S;
    const dim3 grid(tiles64(M), (unsigned)g.batch, (unsigned)parts);
    const int vec_c = M % 4 == 0 && ldc % 4 == 0 && c_batch % 4 == 0 && al16(dst);   // four rows of the big operand are one aligned store (OUT_T)
#define SS_LAUNCH_NT(NTW) hipLaunchKernelGGL((gemm_nt_kernel<OUT_T, RAG, NTW>), grid, dim3(256), 0, stream, big, big_ld, big_batch, \
                                             small, small_ld, small_batch, dst, ldc, c_batch, part_stride, M, S, g.K, vec_c)
    if (S <= 64) SS_LAUNCH_NT(1); else if (S <= 128) SS_LAUNCH_NT(2); else SS_LAUNCH_NT(3);
#undef SS_LAUNCH_NT
    if (parts > 1) reduce_parts<float>(g, parts, C, OUT_T ? S : M, OUT_T ? M : S, stream);
}
template <bool RAG>
void launch_rows(const GemmArgs& g, const bf16_t* A, bf16_t* C, int S, int parts, hipStream_t stream)
{
    const dim3 grid(tiles64(g.N), (unsigned)g.batch, (unsigned)parts);
    const bf16_t* B = static_cast<const bf16_t*>(g.B);
    float* ws = static_cast<float*>(g.split_ws);
#define SS_LAUNCH_ROWS(KERN) hipLaunchKernelGGL(KERN, grid, dim3(256), 0, stream, A, g.a_m, g.a_batch, B, g.b_k, g.b_batch, C, \
                                                g.ldc, g.c_batch, S, g.N, g.K, ws)
    if constexpr (RAG) {
        if (S <= 64) SS_LAUNCH_ROWS(gemm_rows_kernel<1>); else if (S <= 128) SS_LAUNCH_ROWS(gemm_rows_kernel<2>); else SS_LAUNCH_ROWS(gemm_rows_kernel<3>);
    } else {
        if (S <= 96) SS_LAUNCH_ROWS(gemm_rows_lds_kernel<6>); else if (S <= 160) SS_LAUNCH_ROWS(gemm_rows_lds_kernel<10>); else SS_LAUNCH_ROWS(gemm_rows_lds_kernel<12>);
    }
#undef SS_LAUNCH_ROWS
    if (parts > 1) {
        if constexpr (RAG) {
            reduce_parts<bf16_t>(g, parts, C, S, g.N, stream);
        } else {
            const long items = (long)g.batch * S * (g.N / 8);
            hipLaunchKernelGGL(rows_reduce_kernel, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, stream, ws, parts,
                               (long)g.batch * S * g.N, C, g.ldc, g.c_batch, S, g.N, items);
        }
    }
}
// gemm_cols_kernel: 16-row tiles per workgroup, and waves of one.  All waves run at once, at most two per SIMD (2048), since a
// round more costs what all before it do (4 x 4096 x 1531 in 528 workgroups of four, where 512 fit: 33.4 us, in 480: 28.3); and one per
// SIMD, for the longest contractions one on every other, where that leaves a wave few tiles, since each wave lays out its columns of Y
// first.  us, waves on half of the SIMDs / one / two per SIMD: K = 128, 1 x 4096 x 256 (2 tiles) 3.7 / 4.4 / -, 1 x 4096 x 1024 - / 6.9 / 8.4,
// 64 x 4096 x 64 (one: 16 tiles) - / 15.8 / 16.5, off whole lines 64 x 4096 x 16 - / 17.8 / 15.1; K = 48, 4 x 1536 x 512 (one: 3 tiles)
// - / 5.0 / 5.1, 64 x 1536 x 64 (6) - / 7.2 / 6.7.
// One wave to a workgroup balances better (1 x 5120 x 256 5.0 / 4.4 us); four together, where the strips of 64 columns come in whole fours,
// if the weights are read often or rows of the result share cache lines (8 x 4096 x 250 12.2 / 13.4).
// (Counted in workgroups of four before, empty waves included, us, before / now: 64 x 1536 x 64 9.9 / 6.8, 1 x 5120 x 256 6.7 / 4.4,
// 2 x 4096 x 1531 23.4 / 19.4; but 64 x 4096 x 128 23.6 / 24.2.)
void cols_shares(const GemmArgs& g, int& mtiles, int& waves)
{
    const long strips = tiles64(g.N), mt = (g.M + 15) / 16;
    const bool whole_lines = g.N % 64 == 0 && g.ldc % 64 == 0;
    auto share = [&](long most) {
        const long parts = std::max(1L, most / (strips * g.batch));   // of the row tiles, per 64 columns
        return (mt + parts - 1) / parts;
    };
    const long few = g.K <= 32 ? 1 : (g.K <= 96 ? 3 : (whole_lines ? 16 : 6));
    long tiles = share(1024);
    if (g.K > 96 && share(512) <= 4) tiles = share(512);
    else if (tiles > few) tiles = share(2048);
    mtiles = (int)std::min(64L, tiles);
    waves = strips % 4 == 0 && (!whole_lines || mtiles > 8) ? 4 : 1;
}
template <bool RAG>
void launch_cols(const GemmArgs& g, int mtiles, int waves, hipStream_t stream)
{
    const dim3 grid((unsigned)(tiles64(g.N) / waves), (unsigned)(((g.M + 15) / 16 + mtiles - 1) / mtiles), (unsigned)g.batch);
    const dim3 grid_add(tiles64(g.N), (unsigned)((tiles64(g.M) + mtiles - 1) / mtiles), (unsigned)g.batch);
    const int KS = (g.K + 31) / 32;
    const bf16_t *A = static_cast<const bf16_t*>(g.A), *B = static_cast<const bf16_t*>(g.B);
#define SS_LAUNCH_COLS(NKS)                                                                                                                  \
    if (g.accumulate)                                                                                                                        \
        hipLaunchKernelGGL((gemm_cols_add_kernel<RAG, NKS>), grid_add, dim3(256), 0, stream, A, g.a_m, B, g.b_k, g.b_batch,                    \
                           static_cast<bf16_t*>(g.C), g.ldc, g.c_batch, g.M, g.N, g.K, mtiles);                                               \
    else                                                                                                                                     \
        hipLaunchKernelGGL((gemm_cols_kernel<RAG, NKS>), grid, dim3(64 * waves), 0, stream, A, g.a_m, B, g.b_k, g.b_batch,                     \
                           static_cast<bf16_t*>(g.C), g.ldc, g.c_batch, g.M, g.N, g.K, mtiles)
    if (KS <= 3) { SS_LAUNCH_COLS(3); } else if (KS <= 5) { SS_LAUNCH_COLS(5); } else { SS_LAUNCH_COLS(6); }
#undef SS_LAUNCH_COLS
}

// The matrix-core kernel for this product, if there is one; SS_ERR_UNSUPPORTED otherwise (nothing enqueued).
int launch_fast(const GemmArgs& g, hipStream_t stream)
{
    if (!g.bf16) return launch_f32(g, stream);
    if (g.K < 8 || g.M / 64 > 65535 || g.N / 64 > 65535) return SS_ERR_UNSUPPORTED;
    const bf16_t* A = static_cast<const bf16_t*>(g.A);
    const bf16_t* B = static_cast<const bf16_t*>(g.B);
    const bool whole = al16(g.A) && al16(g.B) && al16(g.C) && mult8(g.a_batch) && mult8(g.b_batch);   // operands made of aligned 16-byte pieces
    if (g.a_k == 1 && g.b_k == 1 && g.c_float && !g.accumulate) {
        // C = A B^T: the operand with more rows is split over workgroups and waves, the other one, up to SMAX rows at a time,
        // is read straight from the L2
        float* C = static_cast<float*>(g.C);
        const bool out_t = g.M < g.N;
        const int big = out_t ? g.N : g.M, small = out_t ? g.M : g.N;
        const bool rag = !(whole && g.K % KSLAB == 0 && big % 64 == 0 && mult8(g.a_m) && mult8(g.b_n) && g.ldc % 4 == 0 && g.c_batch % 4 == 0);
        for (int s0 = 0; s0 < small; s0 += SMAX) {
            const int S = small - s0 < SMAX ? small - s0 : SMAX;
            if (out_t) {
                auto f = rag ? launch_nt<true, true> : launch_nt<true, false>;
                f(g, B, g.b_n, g.b_batch, A + (long)s0 * g.a_m, g.a_m, g.a_batch, C + (long)s0 * g.ldc, big, S, stream);
            } else {
                auto f = rag ? launch_nt<false, true> : launch_nt<false, false>;
                f(g, A, g.a_m, g.a_batch, B + (long)s0 * g.b_n, g.b_n, g.b_batch, C + s0, big, S, stream);
            }
        }
        return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_LAUNCH;
    }
    if (g.a_k == 1 && g.b_n == 1 && !g.c_float && g.N >= 8) {
        const bool whole_c = whole && g.N % 64 == 0 && mult8(g.a_m) && mult8(g.b_k) && mult8(g.ldc) && mult8(g.c_batch);
        if (g.K <= SMAX && g.a_batch == 0) {
            const bool plain = whole_c && g.K % 32 == 0 && g.M % (g.accumulate ? 64 : 16) == 0;
            int mtiles = 1, waves = 1;
            if (g.accumulate) {
                // as many 64-row tiles per workgroup as fit, up to 16, while the launch keeps >= 1024 workgroups
                const long cols = (long)tiles64(g.N) * g.batch, mt = tiles64(g.M);
                for (int c = 16; c > 1; c >>= 1)
                    if (mt % c == 0 && cols * (mt / c) >= 1024) { mtiles = c; break; }
            } else {
                cols_shares(g, mtiles, waves);
            }
            if (plain) launch_cols<false>(g, mtiles, waves, stream);
            else launch_cols<true>(g, mtiles, waves, stream);
            return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_LAUNCH;
        }
        if (!g.accumulate) {
            bf16_t* C = static_cast<bf16_t*>(g.C);
            const bool rag = !(whole_c && g.K % KSLAB == 0);
            // fewer than two workgroups per CU: two parts if the workspace holds two float32 shares (headline shape: 66 -> 57 us both launches together; four parts measured slower)
            const long wgs = (long)tiles64(g.N) * g.batch;
            const size_t share = (size_t)g.batch * g.M * g.N * sizeof(float);
            int parts = parts_for(g, wgs, g.K, KSLAB, share);
            if (parts == 1 && wgs < ROWS_MIN_WGS && g.K >= ROWS_MIN_SPLIT_K && g.split_ws && 2 * share <= g.split_ws_bytes) parts = 2;
            for (int s0 = 0; s0 < g.M; s0 += SMAX) {   // in stream order: the shares of one launch are added up before the next overwrites them
                const int S = g.M - s0 < SMAX ? g.M - s0 : SMAX;
                const bf16_t* a = A + (long)s0 * g.a_m;
                bf16_t* c = C + (long)s0 * g.ldc;
                if (rag) launch_rows<true>(g, a, c, S, parts, stream); else launch_rows<false>(g, a, c, S, parts, stream);
            }
            return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_LAUNCH;
        }
    }
    return SS_ERR_UNSUPPORTED;
}

}  // namespace

int gemm(const GemmArgs& g, hipStream_t stream)
{
    if (g.M <= 0 || g.N <= 0 || g.batch <= 0) return SS_OK;
    if (g.K < 0 || !g.C || (g.K > 0 && (!g.A || !g.B))) return SS_ERR_NULL;   // K = 0: an empty sum, operands not read
    if ((g.M + GT - 1) / GT > 65535 || g.batch > 65535) return SS_ERR_UNSUPPORTED;
    if (!g.general) {
        const int rc = launch_fast(g, stream);
        if (rc != SS_ERR_UNSUPPORTED) return rc;
    }
    if (g.bf16) return g.c_float ? launch_generic<bf16_t, float>(g, stream) : launch_generic<bf16_t, bf16_t>(g, stream);
    return launch_generic<float, float>(g, stream);
}

}  // namespace ss
