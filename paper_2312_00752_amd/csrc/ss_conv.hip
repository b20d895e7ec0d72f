// Short causal per-channel convolution (+ SiLU): forward, backward and single-token step
// for gfx950, with their C-ABI entry points (see include/ss_conv.h).
//
// The operation moves 2-3 tensors of (B,D,L) elements and does about ten flops per
// element, so it is bound by HBM and the kernels are organised around 16-byte accesses:
// a lane owns 8 consecutive steps of one (b,d) row, a wave owns a "piece" of 512 steps.
// The W-1 samples in front of a lane's slice are fetched with one extra 8- or 16-byte load
// that hits the line the neighbouring lane has just brought in.  Taps are kept
// right-aligned in four slots (slot j multiplies x[t-3+j]; unused leading slots are zero),
// so one code path serves every width up to 4.
#include <hip/hip_runtime.h>
#include <type_traits>

#include "ss_conv.h"
#include "ss_device.h"
#include "ss_kernels.h"

namespace ss {

constexpr int TAPS = SS_CONV_MAX_WIDTH;  // 4
constexpr int HALO = TAPS - 1;           // 3
constexpr int PIECE = WAVE * 8;          // steps one wave covers per pass

struct ConvArgs {
    int B, D, L, W;
    int Lo;   // elements between the rows of out (forward) or dout (backward): L, or in 16-bit at an odd L a multiple of 8.  Read by the forms that such
              // rows reach only: the others took 1 to 6 % longer with it (backward 256 x 1536 x 5 float32 151.9 / 143.3 us, 8 x 1536 x 2048 35.0 / 34.3)
    unsigned flags;
    const void *x, *state_in, *dout;
    const float *w, *bias;
    void *out, *state_out, *dx;
    float *dw, *dbias;
};

// How the rows of a call are read and written: one element at a time (fewer than 8 steps), in whole aligned
// 16-byte pieces (L a multiple of 8), or in pieces at element alignment (any other length: the piece that
// reaches past the end is read from inside the row and shifted into place, see row_piece), which for an odd number of
// 16-bit elements can be laid on whole words (see row_phase).  The last two are for an odd number of 16-bit elements whose out
// (ROWS_SHIFT, forward) or dout (ROWS_ODD_ONE, backward) has rows of whole 16-byte pieces, as in the layer: the other tensor's rows are read
// from the word a slice lies on and put in place in registers, so that nothing is accessed off a word.
enum { ROWS_SHORT, ROWS_WHOLE, ROWS_ANY, ROWS_ODD, ROWS_SHIFT, ROWS_ODD_ONE };
__host__ __device__ constexpr bool starts_early(int kind) { return kind == ROWS_ODD || kind == ROWS_ODD_ONE; }
// Pieces of 512 steps that a row is dealt out in.  An odd number of steps leaves room in the last one for the step that
// ROWS_ODD begins early.
__host__ __device__ __forceinline__ int row_pieces(int L) { return (L + PIECE - 1) / PIECE; }


__device__ __forceinline__ void load_taps(const float* __restrict__ w, int d, int W, float (&k4)[TAPS])
{
#pragma unroll
    for (int j = 0; j < TAPS; ++j) {
        const int k = j - (TAPS - W);
        k4[j] = k >= 0 ? w[(size_t)d * W + k] : 0.0f;
    }
}

// Sample of the sequence before its start: index t in [-(W-1), -1] comes from state_in.
template <typename T>
__device__ __forceinline__ float before_start(const T* __restrict__ state_row, int t, int W)
{
    const int idx = t + (W - 1);
    return (state_row != nullptr && idx >= 0) ? io_to_f32<T>(state_row[idx]) : 0.0f;
}

// xs[0..2] = x[t0-3..t0-1], xs[3..10] = x[t0..t0+7] (zero past the end of the row); one element at a time.
template <typename T>
__device__ __forceinline__ void load_window(const T* __restrict__ row, const T* __restrict__ state_row, int t0,
                                            int L, int W, float (&xs)[HALO + 8])
{
    const int nvalid = min(max(L - t0, 0), 8);
    float cur[8];
    io8<T>::unpack(io8<T>::template load<false>(row + t0, nvalid), cur);
#pragma unroll
    for (int j = 0; j < 8; ++j) xs[HALO + j] = cur[j];
#pragma unroll
    for (int j = 0; j < HALO; ++j) {
        const int t = t0 - HALO + j;
        xs[j] = (nvalid == 0) ? 0.0f : (t >= 0 ? io_to_f32<T>(row[t]) : before_start<T>(state_row, t, W));
    }
}

// The same for rows of 8 steps and more, in two halves so that all the loads of a unit are issued back to
// back and waited for once, where the form above waits for each conditional load in turn.  Rows of whole
// slices (L a multiple of 8): branch-free buffer loads (an offset out of range returns zeros); others: loads
// at element alignment from clamped places, shifted and masked when unpacked.  `next` additionally fetches
// the 4 samples after the slice.
template <typename T>
struct window_raw {
    typename io8<T>::raw cur;
    typename io4<T>::raw halo, next;
    uint32_t st[HALO];
};
template <typename T>
__device__ __forceinline__ uint32_t row_bytes(int L) { return (uint32_t)L * (uint32_t)sizeof(T); }   // rows below 2^31 bytes (checked by the host)
// ROWS_ODD: how many elements a row starts off a whole 32-bit word.  Slices start that many steps earlier, the
// first one of such a row before the row, so that every access lies on words: off them the hardware takes wide accesses much
// more slowly, and of an odd number of steps every other row is.  (Uniform: a wave works on one row.)
template <typename T, int KIND>
__device__ __forceinline__ int row_phase(const T* row)
{
    if constexpr (starts_early(KIND)) return (int)((reinterpret_cast<uintptr_t>(row) >> 1) & 1);
    else return 0;
}
template <int KIND>
__device__ __forceinline__ bool before_row(int t0) { return starts_early(KIND) && t0 < 0; }
template <int KIND>
__device__ __forceinline__ int slice_start(int t0) { return starts_early(KIND) ? max(t0, 0) : t0; }
template <typename T, int KIND, bool NEXT>
__device__ __forceinline__ window_raw<T> issue_window_any(const T* row, const T* state_row, int t0, int L, int W)
{
    window_raw<T> r;
    const uint32_t esz = (uint32_t)sizeof(T);
    r.cur = io8<T>::load_elem(row, (uint32_t)row_piece(slice_start<KIND>(t0), 8, L) * esz);
    r.halo = io4<T>::load_elem(row, (uint32_t)row_piece(max(t0 - 4, 0), 4, L) * esz);
    if (NEXT) r.next = io4<T>::load_elem(row, (uint32_t)row_piece(t0 + 8, 4, L) * esz);
    // The window of W - 1 samples: behind a branch it is waited for by itself, so every lane reads it, and without one the row's start (of
    // at least 8).  The waves of ROWS_ODD are rarely a row's first and do without.
    if constexpr (starts_early(KIND)) {
#pragma unroll
        for (int j = 0; j < HALO; ++j) r.st[j] = 0u;
        if (state_row && t0 <= 0) {
#pragma unroll
            for (int j = 0; j < HALO; ++j) r.st[j] = state_row[max(min(j - (TAPS - W), W - 2), 0)];
        }
    } else {
        const T* const st = state_row ? state_row : row;
#pragma unroll
        for (int j = 0; j < HALO; ++j) {
            const T v = st[max(min(j - (TAPS - W), W - 2), 0)];
            if constexpr (sizeof(T) == 2) r.st[j] = v; else r.st[j] = __float_as_uint(v);
        }
    }
    return r;
}
// One step earlier: what was read from the row's start moves up by one, behind v0.
template <int N>
__device__ __forceinline__ void shift_up(float (&v)[N], float v0)
{
#pragma unroll
    for (int j = N - 1; j > 0; --j) v[j] = v[j - 1];
    v[0] = v0;
}
// The slice from t0 of a row, of which t < 0 and t >= L are not stored.
template <typename T, int KIND>
__device__ __forceinline__ void store_slice_any(T* row, int t0, const float (&o)[8], int nvalid)
{
    if (before_row<KIND>(t0)) {   // the first lane of a row off a word
#pragma unroll
        for (int j = 1; j < 8; ++j)
            if (j < nvalid) row[j - 1] = f32_to_io<T>(o[j]);
    } else {
        io8<T>::store_elem(row, (uint32_t)t0 * (uint32_t)sizeof(T), io8<T>::pack(o), nvalid);
    }
}
// after issue_window_any: shifts the pieces into place and clears what lies outside the row
template <typename T, int KIND, bool NEXT>
__device__ __forceinline__ void settle_window(window_raw<T>& r, bool has_state, int t0, int L, int W)
{
    if (t0 + 12 > L) {   // only the last lanes of a row
        if (!before_row<KIND>(t0)) io8<T>::drop(r.cur, t0 - row_piece(t0, 8, L));
        if (t0 > 0) io4<T>::drop(r.halo, t0 - 4 - row_piece(t0 - 4, 4, L));
        if (NEXT) io4<T>::drop(r.next, t0 + 8 - row_piece(t0 + 8, 4, L));
    }
#pragma unroll
    for (int j = 0; j < HALO; ++j) r.st[j] = has_state && j >= TAPS - W ? r.st[j] : 0u;
}
template <typename T, bool NEXT>
__device__ __forceinline__ window_raw<T> issue_window(rsrc_t brow, rsrc_t bstate, int t0, int L, int W)
{
    window_raw<T> r;
    const uint32_t esz = (uint32_t)sizeof(T);
    r.cur = io8<T>::load_buf(brow, t0 < L ? (uint32_t)t0 * esz : BUF_OFF);
    // t0 is a multiple of 8, so the four samples in front of the slice are aligned
    r.halo = io4<T>::load_buf(brow, (t0 > 0 && t0 < L) ? (uint32_t)(t0 - 4) * esz : BUF_OFF);
    if (NEXT) r.next = io4<T>::load_buf(brow, t0 + 8 < L ? (uint32_t)(t0 + 8) * esz : BUF_OFF);
#pragma unroll
    for (int j = 0; j < HALO; ++j) {   // the window handed over from before the sequence, for the row's first slice
        const int idx = j - (TAPS - W);
        r.st[j] = buf_load_elem<T>(bstate, (t0 == 0 && idx >= 0) ? (uint32_t)idx * esz : BUF_OFF);
    }
    return r;
}
template <typename T>
__device__ __forceinline__ float raw_to_f32(uint32_t bits)
{
    if constexpr (sizeof(T) == 2) return bf16_to_f32(bf16_t(bits)); else return __uint_as_float(bits);
}
// xs as load_window; xn[0..3] = x[t0+8..t0+11] if fetched
template <typename T, bool NEXT>
__device__ __forceinline__ void unpack_window(const window_raw<T>& r, int t0, float (&xs)[HALO + 8], float (&xn)[4])
{
    float cur[8], h[4];
    io8<T>::unpack(r.cur, cur);
    io4<T>::unpack(r.halo, h);
#pragma unroll
    for (int j = 0; j < 8; ++j) xs[HALO + j] = cur[j];
#pragma unroll
    for (int j = 0; j < HALO; ++j) xs[j] = t0 > 0 ? h[j + 1] : raw_to_f32<T>(r.st[j]);
    if (NEXT) io4<T>::unpack(r.next, xn);
}

// ROWS_SHIFT: xs[0 .. 10] = x[t0 - 3 .. t0 + 7] of a row that may start off a word (uniform), t0 a multiple of eight: the 16 elements
// from the word of t0 - 4 on, of which the row's own phase picks eleven.  A row off a word is not the tensor's first, so
// the element in front of it is memory of the tensor (and is not used).
template <typename T>
__device__ __forceinline__ void load_shifted(const T* row, const T* state_row, int t0, int L, int W, float (&xs)[HALO + 8])
{
    const int s = (int)((reinterpret_cast<uintptr_t>(row) >> 1) & 1), tb = t0 - s;
    const int at_cur = row_piece(tb, 8, L), at_halo = t0 > 0 ? row_piece(tb - 4, 4, L) : 0, at_next = row_piece(tb + 8, 4, L);
    typename io8<T>::raw cur = io8<T>::load_elem(row + at_cur, 0u);
    typename io4<T>::raw halo = io4<T>::load_elem(row + at_halo, 0u), next = io4<T>::load_elem(row + at_next, 0u);
    float st[HALO] = {0.f, 0.f, 0.f};
    if (t0 == 0) {   // the window handed over from before the sequence
#pragma unroll
        for (int j = 0; j < HALO; ++j) st[j] = before_start<T>(state_row, j - HALO, W);
    }
    if (t0 + 12 > L) {   // only the last lanes of a row
        io8<T>::drop(cur, tb - at_cur);
        if (t0 > 0) io4<T>::drop(halo, tb - 4 - at_halo);
        io4<T>::drop(next, tb + 8 - at_next);
    }
    float h[4], c[8], n[4];
    io4<T>::unpack(halo, h);
    io8<T>::unpack(cur, c);
    io4<T>::unpack(next, n);
    auto elem = [&](int i) { return i < 4 ? h[i < 4 ? i : 0] : (i < 12 ? c[i >= 4 && i < 12 ? i - 4 : 0] : n[i >= 12 ? i - 12 : 0]); };
#pragma unroll
    for (int j = 0; j < HALO + 8; ++j) xs[j] = s ? elem(j + 2) : elem(j + 1);
#pragma unroll
    for (int j = 0; j < HALO; ++j) xs[j] = t0 > 0 ? xs[j] : st[j];
}

// ---- forward --------------------------------------------------------------------------------
// One wave per (row, piece); grid = ceil(B*D*pieces / NWAVES) workgroups.
// Bound by HBM.  In the layer at 8 x 1536 x 2047 bf16, us, ROWS_ANY / ROWS_ODD: 26.0 / 24.8 (2048 steps: 21); its backward kernel
// 57.8 / 48.0 (2048 steps: 34; part of its window still goes through 6 KB of LDS, because window_raw is passed by value).
template <typename T, int KIND, bool SILU>
__global__ __launch_bounds__(THREADS) void conv_fwd_kernel(const ConvArgs a)
{
    const int lane = threadIdx.x & (WAVE - 1);
    const int pieces = row_pieces(a.L);
    const long unit = (long)blockIdx.x * NWAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (unit >= (long)a.B * a.D * pieces) return;
    const long r = unit / pieces;                 // row b*D + d
    const int piece = int(unit - r * pieces);
    const int d = int(r % a.D);
    const T* row = static_cast<const T*>(a.x) + (size_t)r * a.L;
    const int t0 = piece * PIECE + lane * 8 - row_phase<T, KIND>(row);
    if (t0 >= a.L) return;

    const T* state_row = (a.flags & SS_CONV_HAS_STATE) ? static_cast<const T*>(a.state_in) + (size_t)r * (a.W - 1) : nullptr;
    float k4[TAPS];
    load_taps(a.w, d, a.W, k4);
    const float bias = (a.flags & SS_CONV_HAS_BIAS) ? a.bias[d] : 0.0f;

    float xs[HALO + 8];
    if constexpr (KIND == ROWS_SHIFT) {
        load_shifted<T>(row, state_row, t0, a.L, a.W, xs);
    } else if constexpr (KIND == ROWS_ANY || KIND == ROWS_ODD) {
        float unused[4];
        window_raw<T> wr = issue_window_any<T, KIND, false>(row, state_row, t0, a.L, a.W);
        settle_window<T, KIND, false>(wr, state_row != nullptr, t0, a.L, a.W);
        unpack_window<T, false>(wr, t0, xs, unused);
        if (before_row<KIND>(t0)) shift_up(xs, 0.0f);
    } else if constexpr (KIND == ROWS_WHOLE) {
        const rsrc_t brow = make_rsrc(row, row_bytes<T>(a.L));
        const rsrc_t bstate = make_rsrc(state_row ? state_row : row, state_row ? (uint32_t)(a.W - 1) * (uint32_t)sizeof(T) : 0u);
        float unused[4];
        unpack_window<T, false>(issue_window<T, false>(brow, bstate, t0, a.L, a.W), t0, xs, unused);
    } else {
        load_window<T>(row, state_row, t0, a.L, a.W, xs);
    }
    float o[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const float v = conv_at(k4, bias, xs + j);
        o[j] = SILU ? v * sigmoid_fast(v) : v;
    }
    const int nvalid = min(a.L - t0, 8);
    T* const orow = static_cast<T*>(a.out) + (size_t)r * (KIND == ROWS_SHIFT ? a.Lo : a.L);
    if constexpr (KIND == ROWS_SHIFT) {   // whole: what lies past the end is the space between the rows
        io8<T>::store_elem(orow + t0, 0u, io8<T>::pack(o), 8);
    } else if constexpr (KIND == ROWS_ANY || KIND == ROWS_ODD) {
        store_slice_any<T, KIND>(orow, t0, o, nvalid);
    } else {
        io8<T>::template store<KIND == ROWS_WHOLE>(orow + t0, o, nvalid);
    }

    if ((a.flags & SS_CONV_WRITE_STATE) && t0 + 8 >= a.L) {  // the lane that holds the last sample
        T* so = static_cast<T*>(a.state_out) + (size_t)r * (a.W - 1);
        for (int j = 0; j < a.W - 1; ++j) {
            const int i = a.L - (a.W - 1) + j - (t0 - HALO);    // position in xs, 0..10
            float v = 0.0f;
#pragma unroll
            for (int q = 0; q < HALO + 8; ++q) v = (q == i) ? xs[q] : v;
            so[j] = f32_to_io<T>(v);
        }
    }
}

// seqlen == 0: the window does not move.
template <typename T>
__global__ void conv_state_copy_kernel(const T* __restrict__ in, T* __restrict__ out, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = in ? in[i] : T(0);
}

// ---- backward -------------------------------------------------------------------------------
// dx[t] = sum_j k4[j] * dv[t+3-j], dv = dout * SiLU'(v);  dk4[j] = sum_{b,t} dv[t] x[t-3+j].
// grid = (D, nsplit): the waves of column d share out its B*pieces (row, piece) units, keep
// the tap and bias gradients in registers and add them to dw/dbias once at the end.
template <typename T, int KIND, bool SILU>
__global__ __launch_bounds__(THREADS) void conv_bwd_kernel(const ConvArgs a)
{
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int d = blockIdx.x;
    const int pieces = row_pieces(a.L);
    const int units = a.B * pieces;
    const int stride = gridDim.y * NWAVES;

    float k4[TAPS];
    load_taps(a.w, d, a.W, k4);
    const float bias = (a.flags & SS_CONV_HAS_BIAS) ? a.bias[d] : 0.0f;
    float gk[TAPS] = {0.f, 0.f, 0.f, 0.f}, gb = 0.0f;

    for (int unit = blockIdx.y * NWAVES + wave; unit < units; unit += stride) {
        const int b = unit / pieces, piece = unit - b * pieces;
        const size_t r = (size_t)b * a.D + d;
        const T* row = static_cast<const T*>(a.x) + r * a.L;
        const int t0 = piece * PIECE + lane * 8 - row_phase<T, KIND>(row);
        const T* grow = static_cast<const T*>(a.dout) + r * (KIND == ROWS_ODD_ONE || KIND == ROWS_ANY ? a.Lo : a.L);
        const T* state_row = (a.flags & SS_CONV_HAS_STATE) ? static_cast<const T*>(a.state_in) + r * (a.W - 1) : nullptr;
        const int nvalid = min(max(a.L - t0, 0), 8);

        float xs[HALO + 8], g[8], dv[8 + HALO];
        float xn[4] = {0.f, 0.f, 0.f, 0.f}, gn[4] = {0.f, 0.f, 0.f, 0.f};   // x and dout of the 4 steps after the slice (8 steps and more)
        if constexpr (KIND == ROWS_ODD_ONE) {
            // dout's rows are on words, so a slice that starts early in x starts off one in them: from the element in front of it (of a first
            // slice, in the space behind the previous row: a row off a word is not the first), and one element on in registers
            window_raw<T> wr = issue_window_any<T, KIND, true>(row, state_row, t0, a.L, a.W);
            const int s = row_phase<T, KIND>(row), tg = t0 - s, at_g = row_piece(tg, 8, a.L), at_n = row_piece(tg + 8, 4, a.L);
            typename io8<T>::raw rg = io8<T>::load_elem(grow + at_g, 0u);
            typename io4<T>::raw rgn = io4<T>::load_elem(grow + at_n, 0u);
            settle_window<T, KIND, true>(wr, state_row != nullptr, t0, a.L, a.W);
            if (t0 + 12 > a.L) {
                io8<T>::drop(rg, tg - at_g);
                io4<T>::drop(rgn, tg + 8 - at_n);
            }
            unpack_window<T, true>(wr, t0, xs, xn);
            float c[8], n[4];
            io8<T>::unpack(rg, c);
            io4<T>::unpack(rgn, n);
            auto elem = [&](int i) { return i < 8 ? c[i < 8 ? i : 0] : n[i >= 8 ? i - 8 : 0]; };
#pragma unroll
            for (int j = 0; j < 8; ++j) g[j] = s ? elem(j + 1) : elem(j);
#pragma unroll
            for (int j = 0; j < HALO; ++j) gn[j] = s ? elem(j + 9) : elem(j + 8);
            if (before_row<KIND>(t0)) {
                shift_up(xs, 0.0f);
                g[0] = 0.0f;
            }
        } else if constexpr (KIND == ROWS_ANY || KIND == ROWS_ODD) {
            const uint32_t esz = (uint32_t)sizeof(T);
            window_raw<T> wr = issue_window_any<T, KIND, true>(row, state_row, t0, a.L, a.W);
            typename io8<T>::raw rg = io8<T>::load_elem(grow, (uint32_t)row_piece(slice_start<KIND>(t0), 8, a.L) * esz);
            typename io4<T>::raw rgn = io4<T>::load_elem(grow, (uint32_t)row_piece(t0 + 8, 4, a.L) * esz);
            settle_window<T, KIND, true>(wr, state_row != nullptr, t0, a.L, a.W);
            if (t0 + 12 > a.L) {
                if (!before_row<KIND>(t0)) io8<T>::drop(rg, t0 - row_piece(t0, 8, a.L));
                io4<T>::drop(rgn, t0 + 8 - row_piece(t0 + 8, 4, a.L));
            }
            unpack_window<T, true>(wr, t0, xs, xn);
            io8<T>::unpack(rg, g);
            io4<T>::unpack(rgn, gn);
            if (before_row<KIND>(t0)) { shift_up(xs, 0.0f); shift_up(g, 0.0f); }
        } else if constexpr (KIND == ROWS_WHOLE) {
            const rsrc_t brow = make_rsrc(row, row_bytes<T>(a.L));
            const rsrc_t bgrow = make_rsrc(grow, row_bytes<T>(a.L));
            const rsrc_t bstate = make_rsrc(state_row ? state_row : row, state_row ? (uint32_t)(a.W - 1) * (uint32_t)sizeof(T) : 0u);
            const uint32_t esz = (uint32_t)sizeof(T);
            const window_raw<T> wr = issue_window<T, true>(brow, bstate, t0, a.L, a.W);
            const typename io8<T>::raw rg = io8<T>::load_buf(bgrow, t0 < a.L ? (uint32_t)t0 * esz : BUF_OFF);
            const typename io4<T>::raw rgn = io4<T>::load_buf(bgrow, t0 + 8 < a.L ? (uint32_t)(t0 + 8) * esz : BUF_OFF);
            unpack_window<T, true>(wr, t0, xs, xn);
            io8<T>::unpack(rg, g);
            io4<T>::unpack(rgn, gn);
        } else {
            load_window<T>(row, state_row, t0, a.L, a.W, xs);
            io8<T>::unpack(io8<T>::template load<false>(grow + t0, nvalid), g);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (SILU) {
                const float v = conv_at(k4, bias, xs + j);
                const float s = sigmoid_fast(v);
                dv[j] = g[j] * s * fmaf(v, 1.0f - s, 1.0f);
            } else {
                dv[j] = g[j];
            }
        }
        // dv of the three steps after the slice: the next lane's first three, except for
        // the last lane of the wave, which works them out from global memory.
#pragma unroll
        for (int j = 0; j < HALO; ++j) {
            const float nb = __shfl_down(dv[j], 1);
            dv[8 + j] = (lane < WAVE - 1 && t0 + 8 + j < a.L) ? nb : 0.0f;
        }
        if (lane == WAVE - 1 && t0 + 8 < a.L) {
            float xe[2 * HALO];   // x[t0+5 .. t0+10]
#pragma unroll
            for (int j = 0; j < 2 * HALO; ++j) {
                if constexpr (KIND != ROWS_SHORT) xe[j] = j < HALO ? xs[HALO + 5 + j] : xn[j - HALO];
                else xe[j] = (t0 + 5 + j < a.L) ? io_to_f32<T>(row[t0 + 5 + j]) : 0.0f;
            }
#pragma unroll
            for (int j = 0; j < HALO; ++j) {
                float gj;
                if constexpr (KIND != ROWS_SHORT) gj = gn[j];
                else gj = (t0 + 8 + j < a.L) ? io_to_f32<T>(grow[t0 + 8 + j]) : 0.0f;
                if (SILU) {
                    const float v = conv_at(k4, bias, xe + j);
                    const float s = sigmoid_fast(v);
                    dv[8 + j] = gj * s * fmaf(v, 1.0f - s, 1.0f);
                } else {
                    dv[8 + j] = gj;
                }
            }
        }
        float o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            o[j] = fmaf(k4[0], dv[j + 3], fmaf(k4[1], dv[j + 2], fmaf(k4[2], dv[j + 1], k4[3] * dv[j])));
            if (j == 0 && before_row<KIND>(t0)) continue;   // no step of the row: dout is zero there, but the window need not be finite
            gb += dv[j];
#pragma unroll
            for (int i = 0; i < TAPS; ++i) gk[i] = fmaf(dv[j], xs[j + i], gk[i]);
        }
        if constexpr (KIND == ROWS_ANY || starts_early(KIND)) store_slice_any<T, KIND>(static_cast<T*>(a.dx) + r * a.L, t0, o, nvalid);
        else io8<T>::template store<KIND == ROWS_WHOLE>(static_cast<T*>(a.dx) + r * a.L + t0, o, nvalid);
    }

#pragma unroll
    for (int m = WAVE / 2; m >= 1; m >>= 1) {
        gb += __shfl_xor(gb, m);
#pragma unroll
        for (int i = 0; i < TAPS; ++i) gk[i] += __shfl_xor(gk[i], m);
    }
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < TAPS; ++i) {
            const int k = i - (TAPS - a.W);
            if (k >= 0) atomicAdd(a.dw + (size_t)d * a.W + k, gk[i]);
        }
        if (a.flags & SS_CONV_HAS_BIAS) atomicAdd(a.dbias + d, gb);
    }
}

__global__ void conv_zero_kernel(float* __restrict__ p, size_t n, float* __restrict__ q, size_t m)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0f;
    if (q && i < m) q[i] = 0.0f;
}

// ---- one token --------------------------------------------------------------------------------
template <typename T, bool SILU>
__global__ void conv_step_kernel(T* __restrict__ state, const T* __restrict__ x_t, const float* __restrict__ w,
                                 const float* __restrict__ bias, T* __restrict__ out_t, int rows, int D, int W)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= rows) return;
    const int d = r % D;
    // Everything is requested up front, from clamped (valid) addresses and with no arithmetic on a
    // loaded value in between; masked afterwards.  Written with a test per load, the compiler
    // waited for each in turn, and the window was shifted through memory: seven round trips.
    const int lead = TAPS - W;             // unused leading slots of the right-aligned window
    T* s = state + (size_t)r * (W - 1);
    float kr[TAPS];
    T sr[HALO];
#pragma unroll
    for (int j = 0; j < TAPS; ++j) kr[j] = w[(size_t)d * W + max(j - lead, 0)];
    const T xt = x_t[r];
    const float braw = (bias ? bias : w)[bias ? d : 0];
    if (W > 1) {
#pragma unroll
        for (int j = 0; j < HALO; ++j) sr[j] = s[max(j - lead, 0)];
    } else {
#pragma unroll
        for (int j = 0; j < HALO; ++j) sr[j] = xt;
    }
    float k4[TAPS], win[TAPS];   // win[3] is the new sample
#pragma unroll
    for (int j = 0; j < TAPS; ++j) k4[j] = j >= lead ? kr[j] : 0.0f;
#pragma unroll
    for (int j = 0; j < HALO; ++j) win[j] = j >= lead ? io_to_f32<T>(sr[j]) : 0.0f;
    win[3] = io_to_f32<T>(xt);
    const float v = conv_at(k4, bias ? braw : 0.0f, win);
    out_t[r] = f32_to_io<T>(SILU ? v * sigmoid_fast(v) : v);
    // the window slides by one sample: slot j takes slot j + 1, the last slot the new sample
#pragma unroll
    for (int j = 0; j < HALO; ++j)
        if (j >= lead) s[j - lead] = j == HALO - 1 ? xt : sr[j + 1 < HALO ? j + 1 : j];
}

// The same for width 4, two neighbouring channels of an entry per thread (an even dim): their windows, taps and samples are contiguous, and
// read and written in words where one channel per thread touches every window of three elements with six accesses.  us, one / two / four
// channels a thread: 256 x 5120 bf16 10.7 / 5.9 / 7.0, float32 12.2 / 8.6 / 9.4, 64 x 4096 bf16 4.2 / 4.0 / 3.8.
template <typename T, bool SILU>
__global__ void __launch_bounds__(256) conv_step_pair_kernel(T* __restrict__ state, const T* __restrict__ x_t, const float* __restrict__ w,
                                                              const float* __restrict__ bias, T* __restrict__ out_t, int pairs, int D)
{
    constexpr int C = 2;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= pairs) return;
    const size_t r = (size_t)i * C;   // first of the thread's rows b * D + d
    const int d = (int)(r % D);
    typedef uint32_t raw_x __attribute__((ext_vector_type(C * sizeof(T) / 4)));
    constexpr int SW = 3 * C * (int)sizeof(T) / 4;   // words of the windows
    T* const s = state + r * 3;
    uint32_t sw[SW];
    u32x4 k[C];
    float bv[C];
#pragma unroll
    for (int j = 0; j < SW; j += 2) {
        if (SW - j >= 2) {
            const u32x2 v = load_any<u32x2>(s, 4u * j);
            sw[j] = v[0]; sw[j + 1 < SW ? j + 1 : j] = v[1];
        } else {
            sw[j] = load_any<uint32_t>(s, 4u * j);
        }
    }
    const raw_x xr = load_any<raw_x>(x_t + r, 0u);
#pragma unroll
    for (int c = 0; c < C; ++c) k[c] = load_any<u32x4>(w + (size_t)d * 4, 16u * c);
#pragma unroll
    for (int c = 0; c < C; ++c) bv[c] = (bias ? bias : w)[bias ? d + c : 0];
    // element e of the windows, of the samples
    T win[3 * C], x[C], o[C], next[3 * C];
#pragma unroll
    for (int e = 0; e < 3 * C; ++e) {
        if constexpr (sizeof(T) == 2) win[e] = T(sw[e / 2] >> (16 * (e & 1))); else win[e] = __uint_as_float(sw[e]);
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
        if constexpr (sizeof(T) == 2) x[c] = T(xr[c / 2] >> (16 * (c & 1))); else x[c] = __uint_as_float(xr[c]);
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const float k4[4] = {__uint_as_float(k[c][0]), __uint_as_float(k[c][1]), __uint_as_float(k[c][2]), __uint_as_float(k[c][3])};
        const float xs[4] = {io_to_f32<T>(win[3 * c]), io_to_f32<T>(win[3 * c + 1]), io_to_f32<T>(win[3 * c + 2]), io_to_f32<T>(x[c])};
        const float v = conv_at(k4, bias ? bv[c] : 0.0f, xs);
        o[c] = f32_to_io<T>(SILU ? v * sigmoid_fast(v) : v);
        next[3 * c] = win[3 * c + 1]; next[3 * c + 1] = win[3 * c + 2]; next[3 * c + 2] = x[c];
    }
    raw_x orow;
#pragma unroll
    for (int j = 0; j < C * (int)sizeof(T) / 4; ++j) {
        if constexpr (sizeof(T) == 2) orow[j] = uint32_t(o[2 * j]) | (uint32_t(o[2 * j + 1]) << 16); else orow[j] = __float_as_uint(o[j]);
    }
    store_any(out_t + r, 0u, orow);
#pragma unroll
    for (int j = 0; j < SW; ++j) {
        if constexpr (sizeof(T) == 2) sw[j] = uint32_t(next[2 * j]) | (uint32_t(next[2 * j + 1]) << 16); else sw[j] = __float_as_uint(next[j]);
    }
#pragma unroll
    for (int j = 0; j < SW; j += 2) {
        if (SW - j >= 2) store_any(s, 4u * j, u32x2{sw[j], sw[j + 1 < SW ? j + 1 : j]});
        else store_any(s, 4u * j, sw[j]);
    }
}

// ---- host ---------------------------------------------------------------------------------------
template <typename T, int KIND>
hipError_t launch_conv_fwd_t(const ConvArgs& a, hipStream_t st)
{
    const long pieces = row_pieces(a.L);
    const long units = (long)a.B * a.D * pieces;
    const dim3 grid((unsigned)((units + NWAVES - 1) / NWAVES));
    if (a.flags & SS_CONV_SILU) hipLaunchKernelGGL((conv_fwd_kernel<T, KIND, true>), grid, dim3(THREADS), 0, st, a);
    else hipLaunchKernelGGL((conv_fwd_kernel<T, KIND, false>), grid, dim3(THREADS), 0, st, a);
    return hipGetLastError();
}

template <typename T, int KIND>
hipError_t launch_conv_bwd_t(const ConvArgs& a, hipStream_t st)
{
    const long pieces = row_pieces(a.L);
    const long units = (long)a.B * pieces;
    // enough waves to keep every SIMD streaming, but no more splits than there are units
    long nsplit = (8192 + (long)a.D * NWAVES - 1) / ((long)a.D * NWAVES);
    const long most = (units + NWAVES - 1) / NWAVES;
    nsplit = nsplit < most ? nsplit : most;
    nsplit = nsplit < 1 ? 1 : (nsplit > 65535 ? 65535 : nsplit);
    const dim3 grid((unsigned)a.D, (unsigned)nsplit);
    if (a.flags & SS_CONV_SILU) hipLaunchKernelGGL((conv_bwd_kernel<T, KIND, true>), grid, dim3(THREADS), 0, st, a);
    else hipLaunchKernelGGL((conv_bwd_kernel<T, KIND, false>), grid, dim3(THREADS), 0, st, a);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_conv_t(const ConvArgs& a, bool bwd, hipStream_t st)
{
    // ROWS_ODD from two pieces a row: below, the lane that starts early costs more than the words give (us, ROWS_ANY / ROWS_ODD, buffers
    // not in a cache, forward: 8 x 4096 x 101 14.5 / 15.3, 16 x 2048 x 515 28.5 / 29.1, 4 x 4096 x 1531 28.9 / 28.8, 8 x 1536 x 2047
    // 27.1 / 23.8; backward: 8 x 4096 x 101 36.3 / 38.6, 4 x 4096 x 1531 48.6 / 44.0, 8 x 1536 x 2047 48.9 / 43.5).
    const bool odd = sizeof(T) == 2 && a.L % 2 == 1 && a.L > 2 * PIECE;
    const int kind = a.L % 8 == 0 ? ROWS_WHOLE : (a.L < 8 ? ROWS_SHORT : (odd ? ROWS_ODD : ROWS_ANY));
    if constexpr (sizeof(T) == 2) {
        if (a.Lo != a.L) return !bwd ? launch_conv_fwd_t<T, ROWS_SHIFT>(a, st) : (odd ? launch_conv_bwd_t<T, ROWS_ODD_ONE>(a, st) : launch_conv_bwd_t<T, ROWS_ANY>(a, st));
        if (kind == ROWS_ODD) return bwd ? launch_conv_bwd_t<T, ROWS_ODD>(a, st) : launch_conv_fwd_t<T, ROWS_ODD>(a, st);
    }
    if (kind == ROWS_WHOLE) return bwd ? launch_conv_bwd_t<T, ROWS_WHOLE>(a, st) : launch_conv_fwd_t<T, ROWS_WHOLE>(a, st);
    if (kind == ROWS_ANY) return bwd ? launch_conv_bwd_t<T, ROWS_ANY>(a, st) : launch_conv_fwd_t<T, ROWS_ANY>(a, st);
    return bwd ? launch_conv_bwd_t<T, ROWS_SHORT>(a, st) : launch_conv_fwd_t<T, ROWS_SHORT>(a, st);
}

}  // namespace ss

namespace {

constexpr uint32_t kConvFlags = SS_CONV_SILU | SS_CONV_HAS_BIAS | SS_CONV_HAS_STATE | SS_CONV_WRITE_STATE;
inline bool aligned_to(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

int check_conv(const ss_conv_params* p, bool for_bwd)
{
    if (!p) return SS_ERR_NULL;
    if (p->batch < 1 || p->dim < 1 || p->seqlen < 0 || p->width < 1) return SS_ERR_SHAPE;
    if (p->width > SS_CONV_MAX_WIDTH) return SS_ERR_UNSUPPORTED;
    if (p->io_dtype != SS_F32 && p->io_dtype != SS_BF16) return SS_ERR_UNSUPPORTED;
    if (p->flags & ~kConvFlags) return SS_ERR_UNSUPPORTED;
    const size_t esz = p->io_dtype == SS_BF16 ? 2 : 4;
    const bool empty = p->seqlen == 0;
    if (!p->w) return SS_ERR_NULL;
    if ((p->flags & SS_CONV_HAS_BIAS) && !p->bias) return SS_ERR_NULL;
    if (!empty && (!p->x || (!for_bwd && !p->out))) return SS_ERR_NULL;
    const bool windowed = p->width > 1;
    if (windowed && (p->flags & SS_CONV_HAS_STATE) && !p->state_in) return SS_ERR_NULL;
    if (!for_bwd && windowed && (p->flags & SS_CONV_WRITE_STATE) && !p->state_out) return SS_ERR_NULL;
    if ((p->x && !aligned_to(p->x, 16)) || (!for_bwd && p->out && !aligned_to(p->out, 16))) return SS_ERR_ALIGN;
    if ((p->state_in && !aligned_to(p->state_in, esz)) || (p->state_out && !aligned_to(p->state_out, esz))) return SS_ERR_ALIGN;
    if (!aligned_to(p->w, 4) || (p->bias && !aligned_to(p->bias, 4))) return SS_ERR_ALIGN;
    // rows are addressed through buffer resources with 31-bit offsets
    if ((size_t)p->seqlen * sizeof(float) >= ((size_t)1 << 31)) return SS_ERR_UNSUPPORTED;
    // the forward grid is one-dimensional
    const long pieces = ((long)p->seqlen + ss::PIECE - 1) / ss::PIECE;
    if ((long)p->batch * p->dim * pieces / ss::NWAVES >= 0x7fffffffL) return SS_ERR_UNSUPPORTED;
    if ((long)p->batch * pieces >= 0x7fffffffL) return SS_ERR_UNSUPPORTED;
    return SS_OK;
}

ss::ConvArgs make_conv_args(const ss_conv_params* p)
{
    ss::ConvArgs a{};
    a.B = p->batch; a.D = p->dim; a.L = p->seqlen; a.W = p->width;
    a.flags = p->flags;
    if (p->width == 1) a.flags &= ~(unsigned)(SS_CONV_HAS_STATE | SS_CONV_WRITE_STATE);
    a.x = p->x; a.state_in = p->state_in; a.w = p->w; a.bias = p->bias;
    a.out = p->out; a.state_out = p->state_out;
    a.Lo = p->seqlen;
    return a;
}
bool pitch_ok(const ss_conv_params* p, int pitch)
{
    return pitch == p->seqlen || (p->io_dtype == SS_BF16 && p->seqlen >= 8 && p->seqlen % 2 == 1 && pitch % 8 == 0 && pitch > p->seqlen);
}

}  // namespace

namespace ss {

int conv_fwd_pitched(const ss_conv_params* p, int pitch, void* stream)
{
    const int rc = check_conv(p, false);
    if (rc != SS_OK) return rc;
    if (!pitch_ok(p, pitch)) return SS_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    ss::ConvArgs a = make_conv_args(p);
    a.Lo = pitch;
    hipError_t e = hipSuccess;
    if (a.L == 0) {
        if (a.flags & SS_CONV_WRITE_STATE) {
            const size_t n = (size_t)a.B * a.D * (a.W - 1);
            const void* in = (a.flags & SS_CONV_HAS_STATE) ? a.state_in : nullptr;
            const dim3 grid((unsigned)((n + 255) / 256));
            if (p->io_dtype == SS_BF16)
                hipLaunchKernelGGL(ss::conv_state_copy_kernel<ss::bf16_t>, grid, dim3(256), 0, st,
                                   static_cast<const ss::bf16_t*>(in), static_cast<ss::bf16_t*>(a.state_out), n);
            else
                hipLaunchKernelGGL(ss::conv_state_copy_kernel<float>, grid, dim3(256), 0, st,
                                   static_cast<const float*>(in), static_cast<float*>(a.state_out), n);
            e = hipGetLastError();
        }
    } else {
        e = p->io_dtype == SS_BF16 ? ss::launch_conv_t<ss::bf16_t>(a, false, st) : ss::launch_conv_t<float>(a, false, st);
    }
    return e == hipSuccess ? SS_OK : SS_ERR_LAUNCH;
}

int conv_bwd_pitched(const ss_conv_bwd_params* p, int pitch, bool cleared, void* stream)
{
    if (!p) return SS_ERR_NULL;
    const int rc = check_conv(&p->fwd, true);
    if (rc != SS_OK) return rc;
    if (!pitch_ok(&p->fwd, pitch)) return SS_ERR_UNSUPPORTED;
    const bool empty = p->fwd.seqlen == 0;
    if (!p->dw) return SS_ERR_NULL;
    if ((p->fwd.flags & SS_CONV_HAS_BIAS) && !p->dbias) return SS_ERR_NULL;
    if (!empty && (!p->dout || !p->dx)) return SS_ERR_NULL;
    if ((p->dout && !aligned_to(p->dout, 16)) || (p->dx && !aligned_to(p->dx, 16))) return SS_ERR_ALIGN;
    if (!aligned_to(p->dw, 4) || (p->dbias && !aligned_to(p->dbias, 4))) return SS_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    ss::ConvArgs a = make_conv_args(&p->fwd);
    a.dout = p->dout; a.dx = p->dx; a.dw = p->dw;
    a.Lo = pitch;
    a.dbias = (a.flags & SS_CONV_HAS_BIAS) ? p->dbias : nullptr;
    const size_t nw = (size_t)a.D * a.W, nb = a.dbias ? (size_t)a.D : 0;
    if (!cleared) hipLaunchKernelGGL(ss::conv_zero_kernel, dim3((unsigned)((nw + 255) / 256)), dim3(256), 0, st, a.dw, nw, a.dbias, nb);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && !empty)
        e = p->fwd.io_dtype == SS_BF16 ? ss::launch_conv_t<ss::bf16_t>(a, true, st) : ss::launch_conv_t<float>(a, true, st);
    return e == hipSuccess ? SS_OK : SS_ERR_LAUNCH;
}

}  // namespace ss

extern "C" {

int ss_conv_fwd(const ss_conv_params* p, void* stream) { return ss::conv_fwd_pitched(p, p ? p->seqlen : 0, stream); }

int ss_conv_bwd(const ss_conv_bwd_params* p, void* stream) { return ss::conv_bwd_pitched(p, p ? p->fwd.seqlen : 0, false, stream); }

int ss_conv_step(const ss_conv_step_params* p, void* stream)
{
    if (!p) return SS_ERR_NULL;
    if (p->batch < 1 || p->dim < 1 || p->width < 1) return SS_ERR_SHAPE;
    if (p->width > SS_CONV_MAX_WIDTH) return SS_ERR_UNSUPPORTED;
    if (p->io_dtype != SS_F32 && p->io_dtype != SS_BF16) return SS_ERR_UNSUPPORTED;
    if (p->flags & ~(uint32_t)(SS_CONV_SILU | SS_CONV_HAS_BIAS)) return SS_ERR_UNSUPPORTED;
    if (!p->x_t || !p->w || !p->out_t || (p->width > 1 && !p->state)) return SS_ERR_NULL;
    if ((p->flags & SS_CONV_HAS_BIAS) && !p->bias) return SS_ERR_NULL;
    const size_t esz = p->io_dtype == SS_BF16 ? 2 : 4;
    if (!aligned_to(p->x_t, esz) || !aligned_to(p->out_t, esz) || (p->state && !aligned_to(p->state, esz)) ||
        !aligned_to(p->w, 4) || (p->bias && !aligned_to(p->bias, 4)))
        return SS_ERR_ALIGN;
    const long rows = (long)p->batch * p->dim;
    if (rows >= 0x7fffffffL) return SS_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const float* bias = (p->flags & SS_CONV_HAS_BIAS) ? p->bias : nullptr;
    const bool silu = p->flags & SS_CONV_SILU;
    auto launch = [&](auto* s) {
        typedef typename std::remove_pointer<decltype(s)>::type T;
        const T* x = static_cast<const T*>(p->x_t);
        T* o = static_cast<T*>(p->out_t);
        const bool pairs = p->width == 4 && p->dim % 2 == 0;
        const int n = (int)(pairs ? rows / 2 : rows);
        const dim3 grid((unsigned)((n + 255) / 256)), block(256);
        if (pairs) {
            if (silu) hipLaunchKernelGGL((ss::conv_step_pair_kernel<T, true>), grid, block, 0, st, s, x, p->w, bias, o, n, p->dim);
            else hipLaunchKernelGGL((ss::conv_step_pair_kernel<T, false>), grid, block, 0, st, s, x, p->w, bias, o, n, p->dim);
        } else {
            if (silu) hipLaunchKernelGGL((ss::conv_step_kernel<T, true>), grid, block, 0, st, s, x, p->w, bias, o, n, p->dim, p->width);
            else hipLaunchKernelGGL((ss::conv_step_kernel<T, false>), grid, block, 0, st, s, x, p->w, bias, o, n, p->dim, p->width);
        }
    };
    if (p->io_dtype == SS_BF16) launch(static_cast<ss::bf16_t*>(p->state));
    else launch(static_cast<float*>(p->state));
    return hipGetLastError() == hipSuccess ? SS_OK : SS_ERR_LAUNCH;
}

}  // extern "C"
