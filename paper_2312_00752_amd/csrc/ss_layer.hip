// Selective SSM layer: conv -> SiLU -> projections -> scan -> gate, forward and backward
// with recomputation (see include/ss_layer.h).
//
// The scan, the convolution and the projections are all this library's own kernels (ss::gemm for
// the projections and their gradients).  Everything is laid out so that no product needs a
// transposed copy of a (B, D, L) tensor: with the sequence axis last, a batch entry of u is a
// (D, L) row-major matrix, [r;B;C] = W_x @ u lands directly in the (B, N, L) layout the scan reads
// (B and C are rows R.. of the result: the scan is told the batch stride), and
// delta_raw = W_dt @ r lands in the (B, D, L) layout of the scan's step-size input.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ss_device.h"
#include "ss_kernels.h"
#include "ss_layer.h"

namespace {

inline bool aligned_to(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }
inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// C[i] (M x N) = op(A[i]) (M x K) @ op(B[i]) (K x N) + beta * C[i] (beta 0 or 1), all ROW-major with
// row pitches lda/ldb/ldc of the stored matrices and element strides sA/sB/sC between batch
// entries; C is float32 if c_float, else in the io dtype.
bool gemm_rm(hipStream_t st, bool tA, bool tB, int M, int N, int K, const void* A, int lda, long sA,
             const void* B, int ldb, long sB, float beta, void* C, int ldc, long sC, int batch, bool bf16, bool c_float = false,
             void* split_ws = nullptr, size_t split_ws_bytes = 0)
{
    ss::GemmArgs g{};
    g.M = M; g.N = N; g.K = K; g.batch = batch;
    g.A = A; g.a_m = tA ? 1 : lda; g.a_k = tA ? lda : 1; g.a_batch = sA;
    g.B = B; g.b_k = tB ? 1 : ldb; g.b_n = tB ? ldb : 1; g.b_batch = sB;
    g.C = C; g.ldc = ldc; g.c_batch = sC;
    g.bf16 = bf16; g.c_float = c_float || !bf16; g.accumulate = beta != 0.0f;
    g.split_ws = split_ws; g.split_ws_bytes = split_ws_bytes;
    return ss::gemm(g, st) == SS_OK;
}

// ---- small kernels around the GEMMs -----------------------------------------------------------
// out[i] = sum_b part[b][i], accumulation in batch order, for the partial results of two weight gradients.
__global__ void sum_partials_kernel(const float* __restrict__ part0, long n0, float* __restrict__ out0, const float* __restrict__ part1,
                                    long n1, float* __restrict__ out1, int nb)
{
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n0 + n1) return;
    const bool second = i >= n0;
    const float* __restrict__ part = second ? part1 : part0;
    const long n = second ? n1 : n0;
    if (second) i -= n0;
    float acc = 0.0f;
    for (int b = 0; b < nb; ++b) acc += part[b * n + i];
    (second ? out1 : out0)[i] = acc;
}

// ---- decode: [r;B;C]_t = u_t @ W_x^T on the matrix cores --------------------------------------------
// P (nb, nm) float32 = u (nb, D) @ W (nm, D)^T, both operands with the contraction index contiguous, which is
// exactly how the matrix cores want their fragments (tile_mma): one 16-byte load each, no staging, at element
// alignment, so any D that holds a whole piece will do; the step that reaches past D cuts its pieces.  The
// product is tiny (64 x 160 x 4096 for the headline layer) and bound by the latency of getting W and u on
// chip, so it is spread thin: workgroup (x, y, z) owns the 16 x 16 tile (x, y) of P over the z-th part of the
// contraction index and spreads that part over its eight waves (four steps' loads in flight per wave); the waves'
// accumulators are added through LDS in a fixed order and written to the z-th partial result, P + z * nb * nm.
// The consumer adds the few partial results, again in a fixed order, so the outcome does not depend on timing
// (atomics across workgroups would make it so).  RAG: D is not a whole number of steps.
constexpr int XP_WAVES = 8;
constexpr int XP_NPARTS = ss::STEP_NPARTS;   // partial results (fixed, so that the consumer can unroll over them)

template <typename T, bool RAG>
__global__ void __launch_bounds__(64 * XP_WAVES) xproj_decode_kernel(const T* __restrict__ u, const T* __restrict__ W,
                                                                     float* __restrict__ P, int nb, int nm, int D)
{
    using mma = ss::tile_mma<T>;
    using ss::f32x4_t;
    __shared__ f32x4_t part[XP_WAVES - 1][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row0 = blockIdx.x * 16, col0 = blockIdx.y * 16;   // tile of P; its columns are rows of W
    const int urow = min(row0 + (lane & 15), nb - 1);           // rows past the end shadow the last one
    const int wrow = min(col0 + (lane & 15), nm - 1);
    const int ksub = mma::E * (lane >> 4);
    const T* up = u + (size_t)urow * D;
    const T* wp = W + (size_t)wrow * D;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    constexpr int STRIDE = mma::K * XP_WAVES;
    const int kpart = ((D + XP_NPARTS - 1) / XP_NPARTS + mma::K - 1) / mma::K * mma::K;   // contraction elements per part
    const int kend = min(D, (int)(blockIdx.z + 1) * kpart);
    auto load = [&](const T* row, int k) {
        if constexpr (RAG) return mma::load(row, k + ksub, D);
        else return *reinterpret_cast<const ss::u32x4*>(row + k + ksub);
    };
    auto step = [&](ss::u32x4 a, ss::u32x4 b, int k) {
        if (RAG && k + mma::K > D) {   // uniform
            a = mma::cut(a, k + ksub, D);
            b = mma::cut(b, k + ksub, D);
        }
        acc = mma::step(a, b, acc);
    };
    int k = blockIdx.z * kpart + mma::K * wave;
    for (; k + 3 * STRIDE < kend; k += 4 * STRIDE) {   // four steps' loads in flight together
        ss::u32x4 a[4], b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[i] = load(up, k + i * STRIDE);
            b[i] = load(wp, k + i * STRIDE);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) step(a[i], b[i], k + i * STRIDE);
    }
    for (; k < kend; k += STRIDE) step(load(up, k), load(wp, k), k);
    if (wave > 0) part[wave - 1][lane] = acc;
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int w = 0; w < XP_WAVES - 1; ++w) acc += part[w][lane];
        // accumulator element r of lane l is row 4 * (l / 16) + r, column l % 16 of the tile
        const int col = col0 + (lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = row0 + 4 * (lane >> 4) + r;
            if (row < nb && col < nm) P[((size_t)blockIdx.z * nb + row) * nm + col] = acc[r];
        }
    }
}
template <typename T>
int launch_xproj_decode(const void* u, const void* W, float* P, int nb, int nm, int D, hipStream_t st)
{
    const dim3 grid((unsigned)((nb + 15) / 16), (unsigned)((nm + 15) / 16), (unsigned)XP_NPARTS), block(64 * XP_WAVES);
    const T *up = static_cast<const T*>(u), *wp = static_cast<const T*>(W);
    if (D % ss::tile_mma<T>::K == 0) hipLaunchKernelGGL((xproj_decode_kernel<T, false>), grid, block, 0, st, up, wp, P, nb, nm, D);
    else hipLaunchKernelGGL((xproj_decode_kernel<T, true>), grid, block, 0, st, up, wp, P, nb, nm, D);
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_LAUNCH;
}

// The same product with the convolution in front of it (width 4, whole pairs of channels): u = SiLU(conv(window, x)) of
// the tile's entries and the part's channels is formed in LDS, two channels per thread and every entry of the tile, so that
// taps are read once per workgroup; the workgroups of the first column tile also leave u in memory for the step
// kernel.  The window is only read: other column tiles form the same u, so the step kernel, the next launch, slides it.  What
// the column tiles repeat is a few multiply-adds and reads from the L2; what it saves is a launch that the product waits for.  That
// pays where a call is launches and latency (conv_in_xproj).  us per call from Python, D 4096 bf16, batch 1, three launches / two:
// 15.7 / 12.9; replayed from a HIP graph, batch 1, 2, 4: D 4096 bf16 9.8 / 8.7, 11.2 / 10.5, 12.2 / 11.3, D 1536 8.3 / 7.2, 8.7 / 7.9,
// 9.8 / 9.0; but batch 8: 12.6 / 13.6, 64: 18.3 / 18.7.
// Values, and the order of every sum, are those of three launches.  ROWS: entries a thread's loads are issued for together.
constexpr int CX_BATCH = 4;
template <typename T> constexpr int CX_COLS = 3072 / (int)sizeof(T);   // channels staged at a time: 49 KB of LDS
template <typename T, bool RAG, int ROWS>
__global__ void __launch_bounds__(64 * XP_WAVES) conv_xproj_decode_kernel(const T* __restrict__ win, const T* __restrict__ x,
                                                                          const float* __restrict__ cw, const float* __restrict__ cb,
                                                                          T* __restrict__ u, const T* __restrict__ W,
                                                                          float* __restrict__ P, int nb, int nm, int D)
{
    using mma = ss::tile_mma<T>;
    using ss::f32x4_t;
    using ss::u32x2;
    using ss::u32x4;
    constexpr int COLS = CX_COLS<T>, PAD = 16 / (int)sizeof(T), STEPS = COLS / mma::K / XP_WAVES;   // STEPS: of a wave
    __shared__ __attribute__((aligned(16))) T s_u[16][COLS + PAD];
    __shared__ f32x4_t part[XP_WAVES - 1][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = blockIdx.x * 16, col0 = blockIdx.y * 16;
    const int rows = min(16, nb - row0);
    const int wrow = min(col0 + (lane & 15), nm - 1);
    const int ksub = mma::E * (lane >> 4);
    const T* wp = W + (size_t)wrow * D;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    const int kpart = ((D + XP_NPARTS - 1) / XP_NPARTS + mma::K - 1) / mma::K * mma::K;
    const int kend = min(D, (int)(blockIdx.z + 1) * kpart);
    for (int c0 = blockIdx.z * kpart; c0 < kend; c0 += COLS) {
        const int n = min(COLS, kend - c0), steps = (n + mma::K - 1) / mma::K;   // n is even
        u32x4 wf[STEPS];   // requested before anything else; read at element alignment from inside the row
#pragma unroll
        for (int i = 0; i < STEPS; ++i)
            if (wave + XP_WAVES * i < steps) wf[i] = mma::load(wp, c0 + mma::K * (wave + XP_WAVES * i) + ksub, D);   // uniform
        for (int p = tid; p < n / 2; p += 64 * XP_WAVES) {
            const int d = c0 + 2 * p;
            const u32x4 k0 = ss::load_any<u32x4>(cw + (size_t)d * 4, 0u), k1 = ss::load_any<u32x4>(cw + (size_t)d * 4, 16u);
            const u32x2 bb = ss::load_any<u32x2>(cb + d, 0u);
            const float ka[4] = {__uint_as_float(k0[0]), __uint_as_float(k0[1]), __uint_as_float(k0[2]), __uint_as_float(k0[3])};
            const float kb[4] = {__uint_as_float(k1[0]), __uint_as_float(k1[1]), __uint_as_float(k1[2]), __uint_as_float(k1[3])};
            for (int r0 = 0; r0 < rows; r0 += ROWS) {
                T s[ROWS][6], xn[ROWS][2];   // the two channels' windows, one after the other, and new samples
#pragma unroll
                for (int r = 0; r < ROWS; ++r) {
                    const size_t at = (size_t)(row0 + min(r0 + r, rows - 1)) * D + d;
                    const T* sp = win + at * 3;
                    const u32x2 w01 = ss::load_any<u32x2>(sp, 0u);
                    if constexpr (sizeof(T) == 2) {
                        const uint32_t w2 = ss::load_any<uint32_t>(sp, 8u), w3 = ss::load_any<uint32_t>(x + at, 0u);
                        s[r][0] = T(w01[0]); s[r][1] = T(w01[0] >> 16); s[r][2] = T(w01[1]); s[r][3] = T(w01[1] >> 16);
                        s[r][4] = T(w2); s[r][5] = T(w2 >> 16);
                        xn[r][0] = T(w3); xn[r][1] = T(w3 >> 16);
                    } else {
                        const u32x4 w2 = ss::load_any<u32x4>(sp, 8u);
                        const u32x2 w3 = ss::load_any<u32x2>(x + at, 0u);
                        s[r][0] = __uint_as_float(w01[0]); s[r][1] = __uint_as_float(w01[1]);
#pragma unroll
                        for (int i = 0; i < 4; ++i) s[r][2 + i] = __uint_as_float(w2[i]);
                        xn[r][0] = __uint_as_float(w3[0]); xn[r][1] = __uint_as_float(w3[1]);
                    }
                }
#pragma unroll
                for (int r = 0; r < ROWS; ++r) {
                    T o[2];
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const float xs[4] = {ss::io_to_f32<T>(s[r][3 * i]), ss::io_to_f32<T>(s[r][3 * i + 1]),
                                             ss::io_to_f32<T>(s[r][3 * i + 2]), ss::io_to_f32<T>(xn[r][i])};
                        const float v = ss::conv_at(i ? kb : ka, __uint_as_float(bb[i]), xs);
                        o[i] = ss::f32_to_io<T>(v * ss::sigmoid_fast(v));
                    }
                    const int rr = min(r0 + r, rows - 1);
                    typedef T pair_t __attribute__((ext_vector_type(2)));
                    *reinterpret_cast<pair_t*>(&s_u[rr][2 * p]) = pair_t{o[0], o[1]};
                    if (blockIdx.y == 0) *reinterpret_cast<pair_t*>(u + (size_t)(row0 + rr) * D + d) = pair_t{o[0], o[1]};   // uniform
                }
            }
        }
        if (RAG && n % mma::K != 0)   // the product's last step: zeros past D
            for (int i = tid; i < 16 * mma::K; i += 64 * XP_WAVES) {
                const int c = steps * mma::K - 1 - i / 16;
                if (c >= n) s_u[i % 16][c] = ss::f32_to_io<T>(0.0f);
            }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < STEPS; ++i)
            if (wave + XP_WAVES * i < steps) {   // uniform
                const int k = mma::K * (wave + XP_WAVES * i);
                u32x4 b = wf[i];
                if (RAG && c0 + k + mma::K > D) b = mma::cut(b, c0 + k + ksub, D);   // uniform
                acc = mma::step(*reinterpret_cast<const u32x4*>(&s_u[lane & 15][k + ksub]), b, acc);
            }
        if (c0 + COLS < kend) __syncthreads();   // s_u is rewritten
    }
    if (wave > 0) part[wave - 1][lane] = acc;
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int w = 0; w < XP_WAVES - 1; ++w) acc += part[w][lane];
        const int col = col0 + (lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = row0 + 4 * (lane >> 4) + r;
            if (row < nb && col < nm) P[((size_t)blockIdx.z * nb + row) * nm + col] = acc[r];
        }
    }
}
template <typename T, int ROWS>
int launch_conv_xproj_rows(const ss_layer_step_params* p, void* u, float* P, hipStream_t st)
{
    const int nb = p->batch, D = p->dim, nm = p->dt_rank + 2 * p->dstate;
    const dim3 grid((unsigned)((nb + 15) / 16), (unsigned)((nm + 15) / 16), (unsigned)XP_NPARTS), block(64 * XP_WAVES);
    const T *win = static_cast<const T*>(p->conv_state), *x = static_cast<const T*>(p->x_t), *W = static_cast<const T*>(p->W_x);
    if (D % ss::tile_mma<T>::K == 0)
        hipLaunchKernelGGL((conv_xproj_decode_kernel<T, false, ROWS>), grid, block, 0, st, win, x, p->conv_w, p->conv_b, static_cast<T*>(u), W, P, nb, nm, D);
    else
        hipLaunchKernelGGL((conv_xproj_decode_kernel<T, true, ROWS>), grid, block, 0, st, win, x, p->conv_w, p->conv_b, static_cast<T*>(u), W, P, nb, nm, D);
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_LAUNCH;
}
// Whether it is taken: width 4, an even number of channels and up to CX_BATCH entries, up to one and a half rounds of staging (3 KB of a
// part's channels; the second waits for the first): float32 D <= 4608, 16-bit 9216, one entry alone 5120 and 10240.  Above, a launch
// less no longer pays even for a caller that is bound by its launches.  us, three launches / two, called from Python (14.4 to 16
// for three, from host to host): float32, batch 2, D 3584 14.4 / 13.4, D 4608 14.4 to 16.0 / 14.4, D 5120 16.0 / 16.6; bf16, batch 4,
// D 6400 14.4 / 13.2, D 8192 14.5 to 16.3 / 14.8; from a HIP graph: float32, batch 2, D 3072 13.0 / 11.9, D 4096 14.8 / 15.1, D 8192
// 18.2 / 21.7; bf16, batch 4, D 6144 13.2 / 12.7, D 8192 13.9 / 14.3; batch 1, float32 D 5120 14.3 / 13.7, D 6400 13.8 / 14.8, bf16 D 8192
// 12.3 / 11.9.
template <typename T>
bool conv_in_xproj(const ss_layer_step_params* p)
{
    const size_t part = ((size_t)p->dim + XP_NPARTS - 1) / XP_NPARTS * sizeof(T);
    return p->conv_width == 4 && p->dim % 2 == 0 && p->batch <= CX_BATCH && part <= (p->batch == 1 ? 5120 : 4608);
}
template <typename T>
int launch_conv_xproj(const ss_layer_step_params* p, void* u, float* P, hipStream_t st)
{
    if (p->batch == 1) return launch_conv_xproj_rows<T, 1>(p, u, P, st);
    return launch_conv_xproj_rows<T, 4>(p, u, P, st);
}

// r (the first R rows of each batch entry of P, (B, Mx, L) in rows ld apart) transposed and zero-padded to
// (B, Lp, Rp), for the delta projection inside the scan kernel (see FwdArgs::rT).  32 x 32 tiles
// through LDS; block (32, 8), grid (Lp / 32, Rp / 32, B).
__global__ void transpose_r_kernel(const ss::bf16_t* __restrict__ P, long bstride, int ld, ss::bf16_t* __restrict__ rT, int R, int L,
                                   int Lp, int Rp)
{
    __shared__ ss::bf16_t tile[32][33];
    const int t0 = blockIdx.x * 32, r0 = blockIdx.y * 32, b = blockIdx.z;
    const int tx = threadIdx.x, ty = threadIdx.y;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = r0 + ty + 8 * i, t = t0 + tx;
        tile[ty + 8 * i][tx] = (r < R && t < L) ? P[(size_t)b * bstride + (size_t)r * ld + t] : ss::bf16_t(0);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int t = t0 + ty + 8 * i, r = r0 + tx;
        rT[((size_t)b * Lp + t) * Rp + r] = tile[tx][ty + 8 * i];
    }
}

// What the backward pass needs before its first kernel, in one launch (as launches of their own these four were 5 us each, one
// after the other): the weights W_dt and W_x transposed, (rows, cols) -> (cols, rows), a 32 x 32 tile through LDS per workgroup of
// (32, 8) threads, and zeros where the scan's and the convolution's kernels add up dB and dC, and the tap and bias gradients.
struct BeginArgs {
    const void* src[2];
    void* dst[2];
    int rows[2], cols[2], tiles[2];
    float* zero[4];
    long n[4];
    int zero_blocks;
};
template <typename T>
__global__ void __launch_bounds__(256) bwd_begin_kernel(const BeginArgs a)
{
    __shared__ T tile[32][33];
    int blk = blockIdx.x;
    if (blk >= a.tiles[0] + a.tiles[1]) {   // uniform
        blk -= a.tiles[0] + a.tiles[1];
        const long first = (long)blk * 256 + threadIdx.y * 32 + threadIdx.x, step = (long)a.zero_blocks * 256;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            for (long i = first; i < a.n[k]; i += step) a.zero[k][i] = 0.0f;
        return;
    }
    const int m = blk >= a.tiles[0];
    if (m) blk -= a.tiles[0];
    const T* __restrict__ src = static_cast<const T*>(a.src[m]);
    T* __restrict__ dst = static_cast<T*>(a.dst[m]);
    const int rows = a.rows[m], cols = a.cols[m], across = (cols + 31) / 32;
    const int c0 = blk % across * 32, r0 = blk / across * 32;
    const int tx = threadIdx.x, ty = threadIdx.y;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = r0 + ty + 8 * i, c = c0 + tx;
        if (r < rows && c < cols) tile[ty + 8 * i][tx] = src[(size_t)r * cols + c];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = c0 + ty + 8 * i, r = r0 + tx;
        if (r < rows && c < cols) dst[(size_t)c * rows + r] = tile[tx][ty + 8 * i];
    }
}

// ---- buffers -------------------------------------------------------------------------------------
struct Shape {
    size_t B, D, L, N, R, Mx, esz;
};
Shape shape_of(const ss_layer_params* p)
{
    Shape s;
    s.B = p->batch; s.D = p->dim; s.L = p->seqlen; s.N = p->dstate; s.R = p->dt_rank;
    s.Mx = s.R + 2 * s.N;
    s.esz = p->io_dtype == SS_BF16 ? 2 : 4;
    return s;
}

ss_fwd_params scan_params(const ss_layer_params* p)
{
    ss_fwd_params f{};
    f.batch = p->batch; f.dim = p->dim; f.seqlen = p->seqlen; f.dstate = p->dstate;
    f.io_dtype = p->io_dtype;
    f.flags = SS_DELTA_SOFTPLUS | SS_HAS_DELTA_BIAS | SS_HAS_D | SS_HAS_Z;
    return f;
}

// Elements between the rows of the layer's own tensors: u, [r;B;C], delta, their gradients and the saved y.  Every other row of an odd number of 16-bit elements
// starts off a 32-bit word, where wide accesses are much slower; rows of these are a whole number of 16-byte pieces apart.
// us, rows of L / this: training 8 x 1536 x 2047 951 / 835, 2 x 2560 x 4095 896 / 771, prefill 4 x 4096 x 1531 266 / 247 (the nt products of
// the first 46 and 31 / 23 and 20, since a wave reads its fragments of [r;B;C] straight from memory).  From 32 steps on: prefill 64 x 1536 x 63
// 114.9 / 112.9, x 33 104.9 / 106.0 (training 370 / 362), x 25 91.8 / 93.7 (334 / 340), x 9 89.5 / 91.2.
int own_pitch(const ss_layer_params* p)
{
    return p->io_dtype == SS_BF16 && p->seqlen % 2 != 0 && p->seqlen >= 32 && p->seqlen < (1 << 22) ? (p->seqlen + 7) / 8 * 8 : p->seqlen;
}

// saved:   [P = [r;B;C] (B, Mx, own_pitch) io][workspace of the scan]
struct SavedLayout { size_t P_off, scan_off, scan_bytes, total; };
SavedLayout saved_layout(const ss_layer_params* p)
{
    const Shape s = shape_of(p);
    const ss_fwd_params f = scan_params(p);
    SavedLayout w{};
    w.P_off = 0;
    w.scan_off = round_up(s.B * s.Mx * own_pitch(p) * s.esz, 256);
    w.scan_bytes = ss::scan_workspace_bytes(&f, 1, own_pitch(p));
    w.total = w.scan_off + round_up(w.scan_bytes, 256);
    return w;
}

// scratch: forward  [u][delta][P and the scan's split scratch, used if nothing is saved][r transposed and padded, bf16]
//          backward [u][delta][du][ddelta][dP (B, Mx, own_pitch) io][dB, dC (B,N,L) f32]
//                   [partials of dW_dt (B,D,R) f32][partials of dW_x (B,Mx,D) f32]
//                   [W_dt transposed (R,D) io][W_x transposed (D,Mx) io]
//          both     [float32 shares of a projection whose contraction is split across workgroups: two of (B,Mx,L), or up to
//                    eight of the largest small product]
struct ScratchLayout { size_t u, delta, P, scan_ws, scan_ws_bytes, rT, du, ddelta, dP, dB, dC, part_dt, part_x, WdtT, WxT, gsplit, gsplit_bytes, total; };
ScratchLayout scratch_layout(const ss_layer_params* p, bool bwd)
{
    const Shape s = shape_of(p);
    ScratchLayout w{};
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t at = off; off += round_up(bytes, 256); return at; };
    // The (B,D,L) buffers start 65 KiB (a multiple of 256 bytes) further apart than their size: the scan
    // touches all of them at the same row and step, and with rows a large power of two of bytes apart equal
    // starting offsets into the memory channels' interleave would put all of that on one channel.
    constexpr size_t SKEW = 66560;
    const size_t T = s.B * s.D * own_pitch(p) * s.esz + SKEW;
    w.u = take(T);
    w.delta = take(T);
    if (!bwd) {
        w.P = take(s.B * s.Mx * own_pitch(p) * s.esz);
        const ss_fwd_params f = scan_params(p);
        w.scan_ws_bytes = ss::scan_workspace_bytes(&f, 0, own_pitch(p));
        w.scan_ws = take(w.scan_ws_bytes);
        w.rT = take(s.B * round_up(s.L, 32) * round_up(s.R, 32) * s.esz);
    } else {
        w.du = take(T);
        w.ddelta = take(T);
        w.dP = take(s.B * s.Mx * own_pitch(p) * s.esz);
        w.dB = take(s.B * s.N * s.L * sizeof(float));
        w.dC = take(s.B * s.N * s.L * sizeof(float));
        w.part_dt = take(s.B * s.D * s.R * sizeof(float));
        w.part_x = take(s.B * s.Mx * s.D * sizeof(float));
        w.WdtT = take(s.R * s.D * s.esz);
        w.WxT = take(s.D * s.Mx * s.esz);
    }
    // two shares of [r;B;C], or the up to 256 64-wide tiles a small product of at most Mx rows is cut into (see parts_for)
    const size_t two = 2 * s.B * s.Mx * s.L * sizeof(float);
    const size_t columns = s.B * (bwd && s.D > s.L ? s.D : s.L), eight = 8 * columns * s.Mx * sizeof(float), most = (size_t)256 * 64 * s.Mx * sizeof(float);
    w.gsplit_bytes = std::max(two, std::min(eight, most));
    w.gsplit = take(w.gsplit_bytes);
    w.total = off;
    return w;
}

bool shape_ok(const ss_layer_params* p)
{
    return p->batch >= 1 && p->dim >= 1 && p->seqlen >= 1 && p->dstate >= 1 && p->dt_rank >= 1 && p->conv_width >= 1;
}

int check_layer(const ss_layer_params* p, bool bwd)
{
    if (!p) return SS_ERR_NULL;
    if (!shape_ok(p)) return SS_ERR_SHAPE;
    if (p->dstate > SS_MAX_DSTATE || p->conv_width > SS_CONV_MAX_WIDTH) return SS_ERR_UNSUPPORTED;
    if (p->io_dtype != SS_F32 && p->io_dtype != SS_BF16) return SS_ERR_UNSUPPORTED;
    if (p->flags != 0) return SS_ERR_UNSUPPORTED;
    // the projections take 32-bit sizes
    if ((long)p->dim * p->dt_rank >= 0x7fffffffL || (long)p->dim * (p->dt_rank + 2 * p->dstate) >= 0x7fffffffL)
        return SS_ERR_UNSUPPORTED;
    if (!p->x || !p->z || !p->conv_w || !p->conv_b || !p->W_x || !p->W_dt || !p->dt_bias || !p->A || !p->Dskip)
        return SS_ERR_NULL;
    if (!bwd && !p->out) return SS_ERR_NULL;
    if (!bwd && ((p->h_last && !aligned_to(p->h_last, 4)) || (p->conv_state && !aligned_to(p->conv_state, 2))))
        return SS_ERR_ALIGN;
    const void* io[] = {p->x, p->z, p->W_x, p->W_dt, bwd ? nullptr : p->out};
    for (const void* q : io)
        if (q && !aligned_to(q, 16)) return SS_ERR_ALIGN;
    const void* f32[] = {p->conv_w, p->conv_b, p->dt_bias, p->A, p->Dskip};
    for (const void* q : f32)
        if (!aligned_to(q, 4)) return SS_ERR_ALIGN;
    if (bwd || p->saved) {
        if (!p->saved || p->saved_bytes < saved_layout(p).total) return SS_ERR_WORKSPACE;
        if (!aligned_to(p->saved, 256)) return SS_ERR_ALIGN;
    }
    if (!p->scratch || p->scratch_bytes < scratch_layout(p, bwd).total) return SS_ERR_WORKSPACE;
    if (!aligned_to(p->scratch, 256)) return SS_ERR_ALIGN;
    return SS_OK;
}

ss_conv_params conv_params(const ss_layer_params* p, void* u)
{
    ss_conv_params c{};
    c.batch = p->batch; c.dim = p->dim; c.seqlen = p->seqlen; c.width = p->conv_width;
    c.io_dtype = p->io_dtype;
    c.flags = SS_CONV_SILU | SS_CONV_HAS_BIAS;
    c.x = p->x; c.w = p->conv_w; c.bias = p->conv_b;
    c.out = u;
    return c;
}

}  // namespace

extern "C" {

size_t ss_layer_saved_bytes(const ss_layer_params* p)
{
    if (!p || !shape_ok(p)) return 0;
    return saved_layout(p).total;
}

size_t ss_layer_scratch_bytes(const ss_layer_params* p, int for_backward)
{
    if (!p || !shape_ok(p)) return 0;
    return scratch_layout(p, for_backward != 0).total;
}

int ss_layer_fwd(const ss_layer_params* p, void* stream)
{
    int rc = check_layer(p, false);
    if (rc != SS_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Shape s = shape_of(p);
    const bool bf16 = p->io_dtype == SS_BF16;
    const ScratchLayout sc = scratch_layout(p, false);
    const SavedLayout sv = saved_layout(p);
    char* scratch = static_cast<char*>(p->scratch);
    char* saved = static_cast<char*>(p->saved);
    char* u = scratch + sc.u;
    char* delta = scratch + sc.delta;
    char* P = saved ? saved + sv.P_off : scratch + sc.P;
    const int B = p->batch, D = p->dim, L = p->seqlen, N = p->dstate, R = p->dt_rank, Mx = R + 2 * N, Ld = own_pitch(p);

    ss_conv_params c = conv_params(p, u);
    if (p->conv_state && p->conv_width > 1) {
        c.flags |= SS_CONV_WRITE_STATE;
        c.state_out = p->conv_state;
    }
    if ((rc = ss::conv_fwd_pitched(&c, Ld, stream)) != SS_OK) return rc;
    // [r;B;C] = W_x @ u
    if (!gemm_rm(st, false, false, Mx, L, D, p->W_x, D, 0, u, Ld, (long)D * Ld, 0.0f, P, Ld, (long)Mx * Ld, B, bf16, false,
                 scratch + sc.gsplit, sc.gsplit_bytes))
        return SS_ERR_LAUNCH;
    ss_fwd_params f = scan_params(p);
    f.u = u; f.delta = delta; f.z = p->z;
    f.Bmat = P + (size_t)R * Ld * s.esz;
    f.Cmat = P + (size_t)(R + N) * Ld * s.esz;
    f.A = p->A; f.Dskip = p->Dskip; f.delta_bias = p->dt_bias;
    f.out = p->out;
    if (p->h_last) {
        f.flags |= SS_WRITE_H_LAST;
        f.h_last = p->h_last;
    }
    if (saved) {
        f.flags |= SS_SAVE_FOR_BWD;
        f.workspace = saved + sv.scan_off;
        f.workspace_bytes = sv.scan_bytes;
    } else if (sc.scan_ws_bytes) {
        f.workspace = scratch + sc.scan_ws;   // lets a long sequence with few rows be split
        f.workspace_bytes = sc.scan_ws_bytes;
    }
    // bf16: delta_raw = W_dt r is formed inside the scan kernel where that variant applies
    if (ss::scan_fwd_fusable(&f, Ld, R)) {
        ss::bf16_t* rT = reinterpret_cast<ss::bf16_t*>(scratch + sc.rT);
        const int Lp = (L + 31) / 32 * 32, Rp = (R + 31) / 32 * 32;
        hipLaunchKernelGGL(transpose_r_kernel, dim3((unsigned)(Lp / 32), (unsigned)(Rp / 32), (unsigned)B), dim3(32, 8), 0, st,
                           reinterpret_cast<const ss::bf16_t*>(P), (long)Mx * Ld, Ld, rT, R, L, Lp, Rp);
        if (hipGetLastError() != hipSuccess) return SS_ERR_LAUNCH;
        rc = ss::scan_fwd_fused(&f, (long)Mx * Ld, Ld, p->W_dt, R, rT, stream);
        if (rc != SS_ERR_UNSUPPORTED) return rc;   // otherwise nothing was enqueued: take the general path
    }
    // delta_raw = W_dt @ r
    if (!gemm_rm(st, false, false, D, L, R, p->W_dt, R, 0, P, Ld, (long)Mx * Ld, 0.0f, delta, Ld, (long)D * Ld, B, bf16, false,
                 scratch + sc.gsplit, sc.gsplit_bytes))
        return SS_ERR_LAUNCH;
    return ss::scan_fwd_strided(&f, (long)Mx * Ld, Ld, stream);
}

int ss_layer_bwd(const ss_layer_bwd_params* q, void* stream)
{
    if (!q) return SS_ERR_NULL;
    const ss_layer_params* p = &q->fwd;
    int rc = check_layer(p, true);
    if (rc != SS_OK) return rc;
    if (!q->dout || !q->dx || !q->dz || !q->dconv_w || !q->dconv_b || !q->dW_x || !q->dW_dt || !q->ddt_bias ||
        !q->dA || !q->dD)
        return SS_ERR_NULL;
    if (!aligned_to(q->dout, 16) || !aligned_to(q->dx, 16) || !aligned_to(q->dz, 16)) return SS_ERR_ALIGN;
    const void* f32[] = {q->dconv_w, q->dconv_b, q->dW_x, q->dW_dt, q->ddt_bias, q->dA, q->dD};
    for (const void* g : f32)
        if (!aligned_to(g, 4)) return SS_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Shape s = shape_of(p);
    const bool bf16 = p->io_dtype == SS_BF16;
    const ScratchLayout sc = scratch_layout(p, true);
    const SavedLayout sv = saved_layout(p);
    char* scratch = static_cast<char*>(p->scratch);
    char* saved = static_cast<char*>(p->saved);
    char *u = scratch + sc.u, *delta = scratch + sc.delta, *du = scratch + sc.du, *ddelta = scratch + sc.ddelta;
    char* dP = scratch + sc.dP;
    float* dB = reinterpret_cast<float*>(scratch + sc.dB);
    float* dC = reinterpret_cast<float*>(scratch + sc.dC);
    char* P = saved + sv.P_off;
    const int B = p->batch, D = p->dim, L = p->seqlen, N = p->dstate, R = p->dt_rank, Mx = R + 2 * N, Ld = own_pitch(p);

    // The two products with a transposed weight take it from a transposed copy (a megabyte each), so
    // that their first operand is contiguous along the contraction index like everywhere else.
    char *WdtT = scratch + sc.WdtT, *WxT = scratch + sc.WxT;
    {
        BeginArgs g{};
        auto weight = [&](int m, const void* src, void* dst, int rows, int cols) {
            g.src[m] = src; g.dst[m] = dst; g.rows[m] = rows; g.cols[m] = cols;
            g.tiles[m] = (rows + 31) / 32 * ((cols + 31) / 32);   // below 2^31: dim * rows of W_x is (check_layer)
        };
        weight(0, p->W_dt, WdtT, D, R);
        weight(1, p->W_x, WxT, Mx, D);
        auto zeros = [&](int k, float* dst, long n) { g.zero[k] = dst; g.n[k] = n; };
        const long nbc = (long)B * N * L;
        zeros(0, dB, nbc);
        zeros(1, dC, nbc);
        zeros(2, q->dconv_w, (long)D * p->conv_width);
        zeros(3, q->dconv_b, D);
        g.zero_blocks = (int)std::min(1024L, (std::max(nbc, (long)D * p->conv_width) + 255) / 256);
        const dim3 grid((unsigned)(g.tiles[0] + g.tiles[1] + g.zero_blocks)), block(32, 8);
        if (bf16) hipLaunchKernelGGL(bwd_begin_kernel<ss::bf16_t>, grid, block, 0, st, g);
        else hipLaunchKernelGGL(bwd_begin_kernel<float>, grid, block, 0, st, g);
        if (hipGetLastError() != hipSuccess) return SS_ERR_LAUNCH;
    }
    // recompute the two cheap intermediates
    ss_conv_params c = conv_params(p, u);
    if ((rc = ss::conv_fwd_pitched(&c, Ld, stream)) != SS_OK) return rc;
    if (!gemm_rm(st, false, false, D, L, R, p->W_dt, R, 0, P, Ld, (long)Mx * Ld, 0.0f, delta, Ld, (long)D * Ld, B, bf16, false,
                 scratch + sc.gsplit, sc.gsplit_bytes))
        return SS_ERR_LAUNCH;

    // the weight gradients of each batch entry; of a single one they are the result
    float* part_dt = B == 1 ? q->dW_dt : reinterpret_cast<float*>(scratch + sc.part_dt);
    float* part_x = B == 1 ? q->dW_x : reinterpret_cast<float*>(scratch + sc.part_x);

    // the scan
    ss_bwd_params b{};
    b.fwd = scan_params(p);
    b.fwd.u = u; b.fwd.delta = delta; b.fwd.z = p->z;
    b.fwd.Bmat = P + (size_t)R * Ld * s.esz;
    b.fwd.Cmat = P + (size_t)(R + N) * Ld * s.esz;
    b.fwd.A = p->A; b.fwd.Dskip = p->Dskip; b.fwd.delta_bias = p->dt_bias;
    b.fwd.workspace = saved + sv.scan_off;
    b.fwd.workspace_bytes = sv.scan_bytes;
    b.dout = q->dout;
    b.du = du; b.ddelta = ddelta; b.dz = q->dz;
    b.dB = dB; b.dC = dC;
    b.dA = q->dA; b.dD = q->dD; b.ddelta_bias = q->ddt_bias;
    // ... which leaves dB and dC next to where dr will be as well: rows R.. of dP
    const ss::BwdSide side = {true, dP + (size_t)R * Ld * s.esz, Ld, (long)Mx * Ld};
    if ((rc = ss::scan_bwd_strided(&b, (long)Mx * Ld, Ld, &side, stream)) != SS_OK) return rc;

    // delta_raw = W_dt @ r:  dr = W_dt^T @ ddelta  (rows 0..R-1 of dP),  dW_dt = sum_b ddelta r^T
    if (!gemm_rm(st, false, false, R, L, D, WdtT, D, 0, ddelta, Ld, (long)D * Ld, 0.0f, dP, Ld, (long)Mx * Ld, B, bf16, false,
                 scratch + sc.gsplit, sc.gsplit_bytes))
        return SS_ERR_LAUNCH;
    if (!gemm_rm(st, false, true, D, R, L, ddelta, Ld, (long)D * Ld, P, Ld, (long)Mx * Ld, 0.0f, part_dt, R, (long)D * R, B, bf16, true,
                 scratch + sc.gsplit, sc.gsplit_bytes))
        return SS_ERR_LAUNCH;
    // [r;B;C] = W_x @ u:  du += W_x^T @ dP,  dW_x = sum_b dP u^T
    if (!gemm_rm(st, false, false, D, L, Mx, WxT, Mx, 0, dP, Ld, (long)Mx * Ld, 1.0f, du, Ld, (long)D * Ld, B, bf16))
        return SS_ERR_LAUNCH;
    if (!gemm_rm(st, false, true, Mx, D, L, dP, Ld, (long)Mx * Ld, u, Ld, (long)D * Ld, 0.0f, part_x, D, (long)Mx * D, B, bf16, true,
                 scratch + sc.gsplit, sc.gsplit_bytes))
        return SS_ERR_LAUNCH;
    if (B > 1) {
        const long n_dt = (long)D * R, n_x = (long)Mx * D;
        hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)((n_dt + n_x + 255) / 256)), dim3(256), 0, st,
                           part_dt, n_dt, q->dW_dt, part_x, n_x, q->dW_x, B);
        if (hipGetLastError() != hipSuccess) return SS_ERR_LAUNCH;
    }
    // u = SiLU(conv(x))
    ss_conv_bwd_params cb{};
    cb.fwd = conv_params(p, nullptr);
    cb.dout = du; cb.dx = q->dx; cb.dw = q->dconv_w; cb.dbias = q->dconv_b;
    return ss::conv_bwd_pitched(&cb, Ld, true, stream);
}

size_t ss_layer_step_scratch_bytes(const ss_layer_step_params* p)
{
    if (!p || p->batch < 1 || p->dim < 1 || p->dstate < 1 || p->dt_rank < 1) return 0;
    const size_t esz = p->io_dtype == SS_BF16 ? 2 : 4;
    const size_t B = p->batch, D = p->dim, Mx = (size_t)p->dt_rank + 2 * (size_t)p->dstate;
    // u_t, delta_t, [r;B;C]_t in the io dtype, and the float32 partial results of the bf16 path's projection
    return 2 * round_up(B * D * esz, 256) + round_up(B * Mx * esz, 256) + round_up(XP_NPARTS * B * Mx * sizeof(float), 256);
}

int ss_layer_step(const ss_layer_step_params* p, void* stream)
{
    if (!p) return SS_ERR_NULL;
    if (p->batch < 1 || p->dim < 1 || p->dstate < 1 || p->dt_rank < 1 || p->conv_width < 1) return SS_ERR_SHAPE;
    if (p->dstate > SS_MAX_DSTATE || p->conv_width > SS_CONV_MAX_WIDTH) return SS_ERR_UNSUPPORTED;
    if (p->io_dtype != SS_F32 && p->io_dtype != SS_BF16) return SS_ERR_UNSUPPORTED;
    if (p->flags != 0) return SS_ERR_UNSUPPORTED;
    if (!p->h || !p->x_t || !p->z_t || !p->conv_w || !p->conv_b || !p->W_x || !p->W_dt || !p->dt_bias || !p->A ||
        !p->Dskip || !p->out_t || (p->conv_width > 1 && !p->conv_state))
        return SS_ERR_NULL;
    const bool bf16 = p->io_dtype == SS_BF16;
    const size_t esz = bf16 ? 2 : 4;
    // all that any of the launches would refuse: a call that is refused has touched neither h nor conv_state
    if (!aligned_to(p->W_x, 16) || !aligned_to(p->W_dt, 16) || !aligned_to(p->h, 16)) return SS_ERR_ALIGN;
    if (!aligned_to(p->z_t, esz) || !aligned_to(p->out_t, esz)) return SS_ERR_ALIGN;
    if (!aligned_to(p->dt_bias, 4) || !aligned_to(p->A, 4) || !aligned_to(p->Dskip, 4)) return SS_ERR_ALIGN;
    if (!p->scratch || p->scratch_bytes < ss_layer_step_scratch_bytes(p)) return SS_ERR_WORKSPACE;
    if (!aligned_to(p->scratch, 256)) return SS_ERR_ALIGN;
    if (!aligned_to(p->x_t, esz) || !aligned_to(p->conv_state, esz) || !aligned_to(p->conv_w, 4) || !aligned_to(p->conv_b, 4)) return SS_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int B = p->batch, D = p->dim, N = p->dstate, R = p->dt_rank, Mx = R + 2 * N;
    char* scratch = static_cast<char*>(p->scratch);
    char* u_t = scratch;
    char* delta_t = u_t + round_up((size_t)B * D * esz, 256);
    char* P_t = delta_t + round_up((size_t)B * D * esz, 256);

    float* P_acc = reinterpret_cast<float*>(P_t + round_up((size_t)B * Mx * esz, 256));

    ss_conv_step_params c{};
    c.batch = B; c.dim = D; c.width = p->conv_width; c.io_dtype = p->io_dtype;
    c.flags = SS_CONV_SILU | SS_CONV_HAS_BIAS;
    c.state = p->conv_state; c.x_t = p->x_t; c.w = p->conv_w; c.bias = p->conv_b; c.out_t = u_t;
    ss_step_params s{};
    s.batch = B; s.dim = D; s.dstate = N; s.io_dtype = p->io_dtype;
    s.flags = SS_DELTA_SOFTPLUS | SS_HAS_DELTA_BIAS | SS_HAS_D | SS_HAS_Z;
    s.h = p->h; s.u_t = u_t; s.z_t = p->z_t;
    s.A = p->A; s.Dskip = p->Dskip; s.delta_bias = p->dt_bias;
    s.out_t = p->out_t;

    // both projections on the matrix cores, delta_t = W_dt r_t inside the state-update kernel, no atomics: two launches with the
    // convolution inside the first projection (conv_in_xproj), three otherwise
    if (D >= 8 && R >= 8 && R <= 256 && N <= 16) {
        if ((long)B * D >= 0x7fffffffL) return SS_ERR_UNSUPPORTED;
        if (bf16 ? conv_in_xproj<ss::bf16_t>(p) : conv_in_xproj<float>(p)) {
            const int rc = bf16 ? launch_conv_xproj<ss::bf16_t>(p, u_t, P_acc, st) : launch_conv_xproj<float>(p, u_t, P_acc, st);
            if (rc != SS_OK) return rc;
            return ss::step_projected(&s, P_acc, p->W_dt, R, Mx, p->conv_state, p->x_t, stream);
        }
        int rc = ss_conv_step(&c, stream);
        if (rc != SS_OK) return rc;
        rc = bf16 ? launch_xproj_decode<ss::bf16_t>(u_t, p->W_x, P_acc, B, Mx, D, st)
                  : launch_xproj_decode<float>(u_t, p->W_x, P_acc, B, Mx, D, st);
        if (rc != SS_OK) return rc;
        return ss::step_projected(&s, P_acc, p->W_dt, R, Mx, nullptr, nullptr, stream);
    }

    int rc = ss_conv_step(&c, stream);
    if (rc != SS_OK) return rc;
    // [r;B;C]_t (B, Mx) = u_t (B, D) @ W_x^T;   delta_t (B, D) = r_t (B, R) @ W_dt^T
    if (!gemm_rm(st, false, true, B, Mx, D, u_t, D, 0, p->W_x, D, 0, 0.0f, P_t, Mx, 0, 1, bf16)) return SS_ERR_LAUNCH;
    if (!gemm_rm(st, false, true, B, D, R, P_t, Mx, 0, p->W_dt, R, 0, 0.0f, delta_t, D, 0, 1, bf16)) return SS_ERR_LAUNCH;
    s.delta_t = delta_t;
    s.B_t = P_t + (size_t)R * esz;
    s.C_t = P_t + (size_t)(R + N) * esz;
    return ss::step_strided(&s, Mx, stream);
}

int ss_proj_gemm(const ss_gemm_params* p, void* stream)
{
    if (!p) return SS_ERR_NULL;
    if (p->M < 0 || p->N < 0 || p->K < 0 || p->batch < 0) return SS_ERR_SHAPE;
    if (p->io_dtype != SS_F32 && p->io_dtype != SS_BF16) return SS_ERR_UNSUPPORTED;
    if (p->flags & ~(SS_GEMM_C_FLOAT | SS_GEMM_ACCUMULATE | SS_GEMM_GENERAL)) return SS_ERR_UNSUPPORTED;
    if (p->M == 0 || p->N == 0 || p->batch == 0) return SS_OK;
    if (!p->C || (p->K > 0 && (!p->A || !p->B))) return SS_ERR_NULL;   // K = 0: an empty sum, A and B are not read
    ss::GemmArgs g{};
    g.M = p->M; g.N = p->N; g.K = p->K; g.batch = p->batch;
    g.A = p->A; g.a_m = p->a_m; g.a_k = p->a_k; g.a_batch = p->a_batch;
    g.B = p->B; g.b_k = p->b_k; g.b_n = p->b_n; g.b_batch = p->b_batch;
    g.C = p->C; g.ldc = p->ldc; g.c_batch = p->c_batch;
    g.bf16 = p->io_dtype == SS_BF16;
    g.c_float = (p->flags & SS_GEMM_C_FLOAT) || !g.bf16;
    g.accumulate = p->flags & SS_GEMM_ACCUMULATE;
    g.general = p->flags & SS_GEMM_GENERAL;
    if (p->workspace && aligned_to(p->workspace, 256)) {
        g.split_ws = p->workspace;
        g.split_ws_bytes = p->workspace_bytes;
    }
    return ss::gemm(g, static_cast<hipStream_t>(stream));
}

size_t ss_proj_gemm_workspace_bytes(const ss_gemm_params* p)
{
    if (!p || p->M < 0 || p->N < 0 || p->batch < 0) return 0;
    return 2 * (size_t)p->batch * (size_t)p->M * (size_t)p->N * sizeof(float);
}

}  // extern "C"
