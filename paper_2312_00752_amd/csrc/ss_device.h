// Device-side helpers shared by the selective-scan kernels (gfx950 only).
//
// Work decomposition used by every scan kernel in this library.  A workgroup of NWAVES
// waves owns ROWS (b,d) rows of one batch entry and walks the sequence in chunks of
// CHUNK_T steps.  In the "state view" lane l of every wave is row l, and wave w carries
// states 4w..4w+3 of that row in registers: the recurrence of Eq. 2a runs as a plain
// sequential loop with the minimum per-(t,n) work (one exp, three multiply-adds), no scan
// re-association overhead, and -- because all lanes of a wave share b, t and n -- B and C
// are wave-uniform and come through the scalar data path instead of LDS.  In the
// "pointwise view" thread i is (row i/4, 8-step slice i%4): it does the per-(b,d,t) work
// (softplus, gate, conversions) on coalesced 16-byte global accesses.  The two views
// exchange data through LDS tiles of ROWS x CHUNK_T floats.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ss {

constexpr int WAVE = 64;
constexpr int STATES_PER_LANE = 4;
constexpr int NWAVES = 4;                              // covers N <= 16
constexpr int ROWS = WAVE;                             // rows per workgroup
constexpr int THREADS = NWAVES * WAVE;                 // 256
constexpr int NPAD = STATES_PER_LANE * NWAVES;         // 16
constexpr int CHUNK_T = 32;                            // steps per forward chunk
constexpr int CKPT_T = 16;                             // == SS_CHECKPOINT_STEPS
constexpr int SLICE = CHUNK_T * ROWS / THREADS;        // 8 steps per thread in the pointwise view
constexpr int SLICES = CHUNK_T / SLICE;                // 4 threads per row in the pointwise view
constexpr int TPAD = CHUNK_T + 4;                      // LDS row pitch (floats) of (row, t) tiles

// State held by slot k of wave w, and state stored at position 4w + k of a 16-float workspace
// record: 4w + k, or 4k + w when the states are dealt out to the waves in turn (FwdArgs::il).
__host__ __device__ __forceinline__ int slot_state(int w, int k, int il) { return il ? k * NWAVES + w : w * STATES_PER_LANE + k; }
__host__ __device__ __forceinline__ int position_state(int pos, int il) { return slot_state(pos / STATES_PER_LANE, pos % STATES_PER_LANE, il); }
// slots per lane a kernel is built for when the states are dealt out: 1, 2 or 4
__host__ __device__ __forceinline__ int slots_for(int N, int il) { return !il ? STATES_PER_LANE : (N <= NWAVES ? 1 : (N <= 2 * NWAVES ? 2 : STATES_PER_LANE)); }

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

typedef uint16_t bf16_t;  // storage only; arithmetic is always float
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float log2_fast(float x) { return __builtin_amdgcn_logf(x); }
__device__ __forceinline__ float rcp_fast(float x) { return __builtin_amdgcn_rcpf(x); }

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(uint32_t(v) << 16); }

// float -> bf16 with the hardware converter of gfx950 (round to nearest even, NaN kept)
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));  // v_cvt_pk_bf16_f32
}
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) { return pack_bf16x2(f, 0.0f) & 0xffffu; }

// softplus(r) = log(1 + e^r) and sigmoid(r), sharing one exponential and one reciprocal.
// With w = fl(1 + e) and c = e - (w - 1), the exact rounding error of that sum,
// log(1 + e) = log(w) + log(1 + c / w) = log(w) + c / w to float precision: accurate for every
// e, however small, with no case split (w = 1 gives e itself).  Above r = 20 softplus(r) = r to
// float precision (and e^r may overflow, which the select discards); the exponent is capped
// so that the sigmoid comes out as 1 there instead of inf * 0.  The cap keeps a NaN (fminf would
// not), so that a step size without a value is one in every kernel; it costs what fminf does.
__device__ __forceinline__ void softplus_sigmoid(float r, float& sp, float& sg)
{
    const float e = exp2_fast(__builtin_elementwise_minimum(r * LOG2E, 64.0f));
    const float w = 1.0f + e;
    const float inv = rcp_fast(w);                 // 1 / (1 + e^r)
    const float c = e - (w - 1.0f);
    const float lp = fmaf(log2_fast(w), LN2, c * inv);
    sp = (r > 20.0f) ? r : lp;
    sg = e * inv;                                  // e^r / (1 + e^r)
}
// softplus alone, where no derivative is asked for: max(r, 0) + log(1 + e) with e = e^-|r| <= 1.  w lies between 1 and 2, so
// 1 / w in the correction c / w (|c| <= 2^-24) may be 1 - e / 2, off by less than a tenth: no reciprocal, no overflow to
// cap and no case split.  Eleven instructions, two of them transcendental, against twelve with three; its error is that of
// the form above below r = 0 and no larger above (float32 emulation over 0..20: worst 1.6e-7 / 1.8e-7, rms 2.3e-8 / 4.0e-8).
__device__ __forceinline__ float softplus(float r)
{
    const float e = exp2_fast(fabsf(r) * -LOG2E);
    const float w = 1.0f + e;
    const float c = e - (w - 1.0f);
    return fmaf(c, fmaf(e, -0.5f, 1.0f), log2_fast(w) * LN2) + fmaxf(r, 0.0f);
}
template <typename T> __device__ __forceinline__ float io_to_f32(T v);
template <> __device__ __forceinline__ float io_to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float io_to_f32<bf16_t>(bf16_t v) { return bf16_to_f32(v); }
template <typename T> __device__ __forceinline__ T f32_to_io(float v);
template <> __device__ __forceinline__ float f32_to_io<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t f32_to_io<bf16_t>(float v) { return bf16_t(f32_to_bf16_bits(v)); }

// The short convolution at one step: taps right-aligned in four slots, xs the four samples up to the step.
__device__ __forceinline__ float conv_at(const float (&k4)[4], float bias, const float* xs)
{
    return fmaf(k4[3], xs[3], fmaf(k4[2], xs[2], fmaf(k4[1], xs[1], fmaf(k4[0], xs[0], bias))));
}

// Exact zero-order hold (Eq. 4): phi(dt, A) = (exp(dt A) - 1) / A multiplies B u in the
// state update (dt itself where A == 0), and d phi / d A = (x e^x - (e^x - 1)) / A^2 with
// x = dt A (dt^2 / 2 where A == 0).  Both differences cancel for small x, where the Taylor
// series is used instead (|x| < 1/8: truncation error below 1e-8 relative).
struct zoh_terms { float phi, dphi_dA; };
__device__ __forceinline__ zoh_terms zoh_phi(float dt, float A, float invA, float abar, bool want_dA)
{
    const float x = dt * A;
    const bool small = fabsf(x) < 0.125f;
    const float em1_series = x * fmaf(x, fmaf(x, fmaf(x, fmaf(x, 1.0f / 120.0f, 1.0f / 24.0f), 1.0f / 6.0f), 0.5f), 1.0f);
    const float em1 = small ? em1_series : abar - 1.0f;
    zoh_terms r;
    r.phi = (A == 0.0f) ? dt : em1 * invA;
    r.dphi_dA = 0.0f;
    if (want_dA) {
        // x e^x - (e^x - 1) = sum_{k>=2} (k-1)/k! x^k
        const float x2 = x * x;
        const float num_series = x2 * fmaf(x, fmaf(x, fmaf(x, fmaf(x, 1.0f / 144.0f, 1.0f / 30.0f), 0.125f), 1.0f / 3.0f), 0.5f);
        const float num = small ? num_series : fmaf(x, abar, -em1);
        r.dphi_dA = (A == 0.0f) ? 0.5f * dt * dt : num * invA * invA;
    }
    return r;
}

// The same phi for the kernels that are short of registers and issue slots, from what the recurrence has
// anyway (x2 = dt A log2 e, abar = 2^x2) and inv_A = 1/A (0 for A = 0): dt (1 + x/2 + x^2/6) for
// |dt A| < 2^-7 (relative error < 3e-8; covers A = 0), (abar - 1)/A beyond (relative error of the
// exponential's last bit over |dt A|, < 2e-5).
constexpr float ZOH_SMALL_X2 = 0.0078125f * LOG2E;   // the threshold on dt * A * log2(e)
constexpr float ZOH_SMALL_X2_GRAD = 0.0625f * LOG2E;  // the same for the gradient term that carries dphi/dA (backward pass)
// |x| < limit ? small : large, as a compare and a select.  Written out: from the conditional expression the
// compiler builds a divergent branch per state and step (both sides under execution masks), which breaks an
// unrolled sweep into hundreds of basic blocks and spills hundreds of registers.
__device__ __forceinline__ float select_small(float x, float limit, float small, float large)
{
    float r;
    asm("v_cmp_lt_f32_e64 vcc, |%1|, %2\n\t"
        "v_cndmask_b32_e32 %0, %4, %3, vcc"
        : "=v"(r) : "v"(x), "s"(limit), "v"(small), "v"(large) : "vcc");
    return r;
}
__device__ __forceinline__ float zoh_phi_fast(float dt, float x2, float abar, float inv_A)
{
    const float series = dt * fmaf(x2, fmaf(x2, LN2 * LN2 / 6.0f, LN2 / 2.0f), 1.0f);
    return select_small(x2, ZOH_SMALL_X2, series, (abar - 1.0f) * inv_A);
}

// Complex decay factor of one step, abar = exp(dt (Ar + i Ai)) = (re, im): the magnitude from
// the exponential unit, the rotation from the hardware sine / cosine, which take their
// argument in revolutions (the fraction is taken first; they are specified for |x| <= 256).
struct cplx { float re, im; };
constexpr float INV_2PI = 0.15915494309189535f;
__device__ __forceinline__ cplx complex_decay(float dt, float Ar_log2e, float Ai)
{
    const float mag = exp2_fast(dt * Ar_log2e);
    const float rev = __builtin_amdgcn_fractf(dt * Ai * INV_2PI);
    cplx r;
    r.re = mag * __builtin_amdgcn_cosf(rev);
    r.im = mag * __builtin_amdgcn_sinf(rev);
    return r;
}

__device__ __forceinline__ float sigmoid_fast(float z)
{
    return rcp_fast(1.0f + exp2_fast(-z * LOG2E));
}

// A 16-byte load of data the kernel reads exactly once, with the streaming (non-temporal)
// hint.  When the row pitch is a large power of two, the rows a wave reads at the same
// step fall into the same set of the vector L1 and evict each other; streaming loads do
// not suffer from that (measured: 20 % on the forward pass of the 2^20-step workload, and
// no change where the pitch is small).  The 8-byte bf16 loads of the backward kernel keep
// the default policy: two of them share a 16-byte neighbourhood and do profit from the L1.
__device__ __forceinline__ uint4 load16_once(const void* p)
{
    const u32x4 x = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return make_uint4(x.x, x.y, x.z, x.w);
}

// ---- workgroup numbering ---------------------------------------------------------------
// The dispatcher hands consecutive workgroup indices to the chip's eight XCDs in turn, and each
// XCD has an L2 of its own.  Renumbered like this, XCD x works on indices [x*n/8, (x+1)*n/8):
// neighbours in the index (row groups of one batch entry) share an L2.  A bijection on [0, n)
// whenever it applies (n a multiple of 8); the identity otherwise.
__device__ __forceinline__ unsigned xcd_contiguous(unsigned i, unsigned n)
{
    return (n % 8u == 0u) ? (i % 8u) * (n / 8u) + i / 8u : i;
}

// ---- buffer-addressed accesses ---------------------------------------------------------
// Memory operations retire in order and the compiler can let younger ones stay outstanding
// across a wait only if it can count them: a store or load inside an `if` counts as "maybe
// zero", and a wait for an older load then degenerates to "wait for everything", i.e. for
// the acknowledgement of stores issued a moment ago.  The hot loops therefore use buffer
// instructions, which are issued unconditionally: the hardware drops a store, and returns
// zero for a load, whose offset lies at or beyond the resource's size, so a lane (or a whole
// access) is switched off with an out-of-range offset (or a size of zero) instead of a
// branch.  Resources are built per workgroup (64 rows), which keeps offsets far below 2^31.
using rsrc_t = __amdgpu_buffer_rsrc_t;
constexpr uint32_t BUF_OFF = 0x80000000u;   // an offset beyond any resource built here
__device__ __forceinline__ rsrc_t make_rsrc(const void* p, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ uint4 buf_load16_once(rsrc_t r, uint32_t off)   // streaming hint, as load16_once
{
    const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 2);
    return make_uint4(x.x, x.y, x.z, x.w);
}
__device__ __forceinline__ void buf_store16(rsrc_t r, uint32_t off, uint4 v)
{
    const u32x4 x = {v.x, v.y, v.z, v.w};
    __builtin_amdgcn_raw_buffer_store_b128(x, r, (int)off, 0, 0);
}

__device__ __forceinline__ uint4 buf_load16(rsrc_t r, uint32_t off)
{
    const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
    return make_uint4(x.x, x.y, x.z, x.w);
}
typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint2 buf_load8(rsrc_t r, uint32_t off)
{
    const u32x2v x = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
    return make_uint2(x.x, x.y);
}
// one io element as raw bits (zero if off is out of range)
template <typename T>
__device__ __forceinline__ uint32_t buf_load_elem(rsrc_t r, uint32_t off)
{
    if constexpr (sizeof(T) == 2) return (uint32_t)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r, (int)off, 0, 0);
    else return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0);
}

// ---- rows of any length: accesses aligned to an element only ---------------------------------
// The widest loads and stores at an address that is a multiple of the element size.  The hardware takes
// them in one instruction (the compiler's default access mode on this target), so a row that is not a
// whole number of 16-byte pieces costs the same instructions as one that is; what it loses is the
// out-of-range rule of the buffer resources, so offsets are clamped into the row instead (row_piece).
template <typename V, int A> struct elem_aligned { typedef V type __attribute__((aligned(A))); };
template <typename V, typename T>
__device__ __forceinline__ V load_any(const T* base, uint32_t byte_off)
{
    return *reinterpret_cast<const typename elem_aligned<V, (int)sizeof(T)>::type*>(reinterpret_cast<const char*>(base) + byte_off);
}
template <typename V, typename T>
__device__ __forceinline__ void store_any(T* base, uint32_t byte_off, V v)
{
    *reinterpret_cast<typename elem_aligned<V, (int)sizeof(T)>::type*>(reinterpret_cast<char*>(base) + byte_off) = v;
}
// Off a whole 32-bit word (half of the rows of an odd number of 16-bit elements) the hardware takes such an access
// much more slowly: the 50 MB of 8 x 1536 rows of 2047, written 29 us against 17 for 2046, read and written 45 against 26.  So the whole
// words among eight such elements go in one access and the odd ends in one each (22 and 31 us).
__device__ __forceinline__ bool off_word(const bf16_t* p) { return (reinterpret_cast<uintptr_t>(p) & 2) != 0; }
__device__ __forceinline__ void store_row16(bf16_t* p, u32x4 v)
{
    typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
    if (!off_word(p)) {
        *reinterpret_cast<elem_aligned<u32x4, 4>::type*>(p) = v;
    } else {
        p[0] = bf16_t(v[0]);
        *reinterpret_cast<elem_aligned<u32x3, 4>::type*>(p + 1) = u32x3{__builtin_amdgcn_alignbit(v[1], v[0], 16), __builtin_amdgcn_alignbit(v[2], v[1], 16),
                                                                        __builtin_amdgcn_alignbit(v[3], v[2], 16)};
        p[7] = bf16_t(v[3] >> 16);
    }
}
// Eight elements from p, in two halves so that nothing waits between the request and the use: the four words from the one
// that p lies in, and the eighth element; shift_row16 puts them in place.  The word holds p's predecessor, which must be
// memory of the same tensor: at the tensor's first element the words are read from p itself, off a word.
__host__ __device__ __forceinline__ uintptr_t row16_words(uintptr_t p, uintptr_t first) { return (p & ~uintptr_t(3)) > first ? (p & ~uintptr_t(3)) : first; }
__device__ __forceinline__ void load_row16(const bf16_t* p, const bf16_t* first, u32x4& d, uint32_t& last)
{
    d = *reinterpret_cast<const elem_aligned<u32x4, 2>::type*>(row16_words(reinterpret_cast<uintptr_t>(p), reinterpret_cast<uintptr_t>(first)));
    last = p[7];
}
__device__ __forceinline__ u32x4 shift_row16(const bf16_t* p, const bf16_t* first, u32x4 d, uint32_t last)
{
    const bool shifted = off_word(p) && p != first;
    const uint32_t s = shifted ? 16u : 0u;
    return u32x4{__builtin_amdgcn_alignbit(d[1], d[0], s), __builtin_amdgcn_alignbit(d[2], d[1], s), __builtin_amdgcn_alignbit(d[3], d[2], s),
                 shifted ? __builtin_amdgcn_alignbit(last, d[3], 16) : d[3]};
}
// A piece of `len` steps starting at t of a row of L >= len steps: where to read it so that the access stays
// inside the row.  A piece that ends past the row is read from L - len; dropping its first t - row_piece(t)
// elements (drop_front) leaves the piece's own, followed by zeros.
__device__ __forceinline__ int row_piece(int t, int len, int L) { return min(t, L - len); }
// v without its first n elements of ELEM_BITS bits, zeros moving in at the end (n >= 0; the whole vector or more: zeros)
template <int ELEM_BITS>
__device__ __forceinline__ u32x4 drop_front(u32x4 v, int n)
{
    const uint64_t lo = (uint64_t(v[1]) << 32) | v[0], hi = (uint64_t(v[3]) << 32) | v[2];
    const int s = n * ELEM_BITS;
    uint64_t a = 0, b = 0;
    if (s < 64) { a = s == 0 ? lo : (lo >> s) | (hi << (64 - s)); b = hi >> s; }
    else if (s < 128) a = hi >> (s - 64);
    return u32x4{(uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32)};
}

// ---- 16 x 16 products on the matrix cores, either io type ----------------------------------------------
// One 16-byte piece per lane and operand: lane l holds row (column) l % 16 at the E consecutive contraction
// indices from E * (l / 16); accumulator element i of lane l is row 4 * (l / 16) + i, column l % 16.  bf16: one
// 16x16x32 MFMA.  float: four 16x16x4 MFMAs, the i-th of which contracts over element i of the four lane groups.
typedef float f32x4_t __attribute__((ext_vector_type(4)));
template <typename T>
struct tile_mma {
    static constexpr int E = 16 / (int)sizeof(T), K = 4 * E;   // elements per piece, contraction indices per step
    static __device__ __forceinline__ f32x4_t step(u32x4 a, u32x4 b, f32x4_t c)
    {
        if constexpr (sizeof(T) == 2) {
            typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
            return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[i]), __uint_as_float(b[i]), c, 0, 0, 0);
            return c;
        }
    }
    // the piece from index k of a row of n >= E elements, at element alignment from inside the row, and shifted into place
    static __device__ __forceinline__ u32x4 load(const T* row, int k, int n) { return load_any<u32x4>(row + row_piece(k, E, n), 0u); }
    static __device__ __forceinline__ u32x4 cut(u32x4 v, int k, int n) { return drop_front<8 * (int)sizeof(T)>(v, k - row_piece(k, E, n)); }
};

// ---- 8 consecutive io elements <-> 8 floats -------------------------------------------
// VEC: every row starts 16-byte aligned and L is a multiple of 8, so a slice is either
// whole (nvalid == 8, one or two 16-byte accesses) or empty.  Otherwise the `nvalid`
// leading elements are accessed one by one; the rest read as zero / are not written.
template <typename T> struct io8;

template <> struct io8<float> {
    struct raw { float4 a, b; };
    template <bool VEC>
    static __device__ __forceinline__ raw load(const float* p, int nvalid)
    {
        raw r;
        if (VEC) {  // nvalid is 0 or 8
            r.a = r.b = make_float4(0.f, 0.f, 0.f, 0.f);
            if (nvalid == 8) {
                const uint4 x = load16_once(p), y = load16_once(p + 4);
                r.a = make_float4(__uint_as_float(x.x), __uint_as_float(x.y), __uint_as_float(x.z), __uint_as_float(x.w));
                r.b = make_float4(__uint_as_float(y.x), __uint_as_float(y.y), __uint_as_float(y.z), __uint_as_float(y.w));
            }
        } else {
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = (j < nvalid) ? p[j] : 0.0f;
            r.a = make_float4(v[0], v[1], v[2], v[3]);
            r.b = make_float4(v[4], v[5], v[6], v[7]);
        }
        return r;
    }
    static __device__ __forceinline__ raw load_buf(rsrc_t rs, uint32_t off)   // whole slice, or zeros if off is out of range
    {
        const uint4 x = buf_load16_once(rs, off), y = buf_load16_once(rs, off + 16);
        raw r;
        r.a = make_float4(__uint_as_float(x.x), __uint_as_float(x.y), __uint_as_float(x.z), __uint_as_float(x.w));
        r.b = make_float4(__uint_as_float(y.x), __uint_as_float(y.y), __uint_as_float(y.z), __uint_as_float(y.w));
        return r;
    }
    static __device__ __forceinline__ raw load_elem(const float* p, uint32_t off)   // eight elements at element alignment
    {
        const u32x4 x = load_any<u32x4>(p, off), y = load_any<u32x4>(p, off + 16);
        raw r;
        r.a = make_float4(__uint_as_float(x[0]), __uint_as_float(x[1]), __uint_as_float(x[2]), __uint_as_float(x[3]));
        r.b = make_float4(__uint_as_float(y[0]), __uint_as_float(y[1]), __uint_as_float(y[2]), __uint_as_float(y[3]));
        return r;
    }
    static __device__ __forceinline__ void drop(raw& r, int n)   // the first n elements; zeros move in
    {
        float v[8], o[8];
        unpack(r, v);
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = 0.0f;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (n == k) {
#pragma unroll
                for (int j = 0; j + k < 8; ++j) o[j] = v[j + k];
            }
        r.a = make_float4(o[0], o[1], o[2], o[3]);
        r.b = make_float4(o[4], o[5], o[6], o[7]);
    }
    struct packed { uint4 a, b; };   // eight elements as stored
    static __device__ __forceinline__ void store_elem(float* p, uint32_t off, const packed& x, int n)   // the first n elements
    {
        if (n >= 8) {
            store_any(p, off, u32x4{x.a.x, x.a.y, x.a.z, x.a.w});
            store_any(p, off + 16, u32x4{x.b.x, x.b.y, x.b.z, x.b.w});
        } else {
            const uint32_t w[8] = {x.a.x, x.a.y, x.a.z, x.a.w, x.b.x, x.b.y, x.b.z, x.b.w};
#pragma unroll
            for (int j = 0; j < 7; ++j)
                if (j < n) store_any(p, off + 4u * j, w[j]);
        }
    }
    static __device__ __forceinline__ packed pack(const float (&v)[8])
    {
        return {make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])),
                make_uint4(__float_as_uint(v[4]), __float_as_uint(v[5]), __float_as_uint(v[6]), __float_as_uint(v[7]))};
    }
    static __device__ __forceinline__ void store_packed(rsrc_t rs, uint32_t off, const packed& x)   // dropped if off is out of range
    {
        buf_store16(rs, off, x.a);
        buf_store16(rs, off + 16, x.b);
    }
    static __device__ __forceinline__ void store_buf(rsrc_t rs, uint32_t off, const float (&v)[8]) { store_packed(rs, off, pack(v)); }
    static __device__ __forceinline__ void unpack(const raw& r, float (&v)[8])
    {
        v[0] = r.a.x; v[1] = r.a.y; v[2] = r.a.z; v[3] = r.a.w;
        v[4] = r.b.x; v[5] = r.b.y; v[6] = r.b.z; v[7] = r.b.w;
    }
    template <bool VEC>
    static __device__ __forceinline__ void store(float* p, const float (&v)[8], int nvalid)
    {
        if (VEC) {
            if (nvalid == 8) {
                *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
                *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (j < nvalid) p[j] = v[j];
        }
    }
};

template <> struct io8<bf16_t> {
    struct raw { uint4 w; };
    template <bool VEC>
    static __device__ __forceinline__ raw load(const bf16_t* p, int nvalid)
    {
        raw r;
        if (VEC) {  // nvalid is 0 or 8
            r.w = make_uint4(0u, 0u, 0u, 0u);
            if (nvalid == 8) r.w = load16_once(p);
        } else {
            uint32_t v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = (j < nvalid) ? uint32_t(p[j]) : 0u;
            r.w = make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16),
                             v[6] | (v[7] << 16));
        }
        return r;
    }
    static __device__ __forceinline__ raw load_buf(rsrc_t rs, uint32_t off)   // whole slice, or zeros if off is out of range
    {
        raw r;
        r.w = buf_load16_once(rs, off);
        return r;
    }
    static __device__ __forceinline__ raw load_elem(const bf16_t* p, uint32_t off)   // eight elements at element alignment
    {
        const u32x4 x = load_any<u32x4>(p, off);
        raw r;
        r.w = make_uint4(x[0], x[1], x[2], x[3]);
        return r;
    }
    static __device__ __forceinline__ void drop(raw& r, int n)   // the first n elements; zeros move in
    {
        const u32x4 x = drop_front<16>(u32x4{r.w.x, r.w.y, r.w.z, r.w.w}, n);
        r.w = make_uint4(x[0], x[1], x[2], x[3]);
    }
    typedef uint4 packed;   // eight elements as stored
    static __device__ __forceinline__ void store_elem(bf16_t* p, uint32_t off, packed x, int n)   // the first n elements
    {
        if (n >= 8) {
            store_any(p, off, u32x4{x.x, x.y, x.z, x.w});
        } else {
            const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int j = 0; j < 7; ++j)
                if (j < n) store_any(p, off + 2u * j, bf16_t(w[j >> 1] >> (16 * (j & 1))));
        }
    }
    static __device__ __forceinline__ packed pack(const float (&v)[8])
    {
        return make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
    }
    static __device__ __forceinline__ void store_packed(rsrc_t rs, uint32_t off, packed x) { buf_store16(rs, off, x); }   // dropped if off is out of range
    static __device__ __forceinline__ void store_buf(rsrc_t rs, uint32_t off, const float (&v)[8]) { store_packed(rs, off, pack(v)); }
    static __device__ __forceinline__ void unpack(const raw& r, float (&v)[8])
    {
        v[0] = bf16_lo(r.w.x); v[1] = bf16_hi(r.w.x);
        v[2] = bf16_lo(r.w.y); v[3] = bf16_hi(r.w.y);
        v[4] = bf16_lo(r.w.z); v[5] = bf16_hi(r.w.z);
        v[6] = bf16_lo(r.w.w); v[7] = bf16_hi(r.w.w);
    }
    template <bool VEC>
    static __device__ __forceinline__ void store(bf16_t* p, const float (&v)[8], int nvalid)
    {
        if (VEC) {
            if (nvalid == 8)
                *reinterpret_cast<uint4*>(p) = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                                          pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (j < nvalid) p[j] = bf16_t(f32_to_bf16_bits(v[j]));
        }
    }
};

// ---- 4 consecutive io elements <-> 4 floats (same VEC contract: whole or empty) ----------
template <typename T> struct io4;

template <> struct io4<float> {
    struct raw { float4 a; };
    template <bool VEC>
    static __device__ __forceinline__ raw load(const float* p, int nvalid)
    {
        raw r;
        if (VEC) {
            r.a = make_float4(0.f, 0.f, 0.f, 0.f);
            if (nvalid == 4) {
                const uint4 x = load16_once(p);
                r.a = make_float4(__uint_as_float(x.x), __uint_as_float(x.y), __uint_as_float(x.z), __uint_as_float(x.w));
            }
        } else {
            r.a = make_float4(0 < nvalid ? p[0] : 0.f, 1 < nvalid ? p[1] : 0.f, 2 < nvalid ? p[2] : 0.f,
                              3 < nvalid ? p[3] : 0.f);
        }
        return r;
    }
    static __device__ __forceinline__ raw load_buf(rsrc_t rs, uint32_t off)   // whole slice, or zeros if off is out of range
    {
        const uint4 x = buf_load16(rs, off);
        raw r;
        r.a = make_float4(__uint_as_float(x.x), __uint_as_float(x.y), __uint_as_float(x.z), __uint_as_float(x.w));
        return r;
    }
    static __device__ __forceinline__ raw load_elem(const float* p, uint32_t off)   // four elements at element alignment
    {
        const u32x4 x = load_any<u32x4>(p, off);
        raw r;
        r.a = make_float4(__uint_as_float(x[0]), __uint_as_float(x[1]), __uint_as_float(x[2]), __uint_as_float(x[3]));
        return r;
    }
    static __device__ __forceinline__ void drop(raw& r, int n)   // the first n elements; zeros move in
    {
        const u32x4 x = drop_front<32>(u32x4{__float_as_uint(r.a.x), __float_as_uint(r.a.y), __float_as_uint(r.a.z), __float_as_uint(r.a.w)}, n);
        r.a = make_float4(__uint_as_float(x[0]), __uint_as_float(x[1]), __uint_as_float(x[2]), __uint_as_float(x[3]));
    }
    typedef uint4 packed;   // four elements as stored
    static __device__ __forceinline__ void store_elem(float* p, uint32_t off, packed x, int n)   // the first n elements
    {
        if (n >= 4) {
            store_any(p, off, u32x4{x.x, x.y, x.z, x.w});
        } else {
            const uint32_t w[3] = {x.x, x.y, x.z};
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (j < n) store_any(p, off + 4u * j, w[j]);
        }
    }
    static __device__ __forceinline__ packed pack(const float (&v)[4])
    {
        return make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3]));
    }
    static __device__ __forceinline__ void store_packed(rsrc_t rs, uint32_t off, packed x) { buf_store16(rs, off, x); }   // dropped if off is out of range
    static __device__ __forceinline__ void store_buf(rsrc_t rs, uint32_t off, const float (&v)[4]) { store_packed(rs, off, pack(v)); }
    static __device__ __forceinline__ void unpack(const raw& r, float (&v)[4])
    {
        v[0] = r.a.x; v[1] = r.a.y; v[2] = r.a.z; v[3] = r.a.w;
    }
    template <bool VEC>
    static __device__ __forceinline__ void store(float* p, const float (&v)[4], int nvalid)
    {
        if (VEC) {
            if (nvalid == 4) *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j < nvalid) p[j] = v[j];
        }
    }
};

template <> struct io4<bf16_t> {
    struct raw { uint2 w; };
    template <bool VEC>
    static __device__ __forceinline__ raw load(const bf16_t* p, int nvalid)
    {
        raw r;
        if (VEC) {
            r.w = make_uint2(0u, 0u);
            if (nvalid == 4) r.w = *reinterpret_cast<const uint2*>(p);
        } else {
            uint32_t v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = (j < nvalid) ? uint32_t(p[j]) : 0u;
            r.w = make_uint2(v[0] | (v[1] << 16), v[2] | (v[3] << 16));
        }
        return r;
    }
    static __device__ __forceinline__ raw load_buf(rsrc_t rs, uint32_t off)   // whole slice, or zeros if off is out of range
    {
        raw r;
        r.w = buf_load8(rs, off);
        return r;
    }
    static __device__ __forceinline__ raw load_elem(const bf16_t* p, uint32_t off)   // four elements at element alignment
    {
        const u32x2 x = load_any<u32x2>(p, off);
        raw r;
        r.w = make_uint2(x[0], x[1]);
        return r;
    }
    static __device__ __forceinline__ void drop(raw& r, int n)   // the first n elements; zeros move in
    {
        const u32x4 x = drop_front<16>(u32x4{r.w.x, r.w.y, 0u, 0u}, n);
        r.w = make_uint2(x[0], x[1]);
    }
    typedef uint2 packed;   // four elements as stored
    static __device__ __forceinline__ void store_elem(bf16_t* p, uint32_t off, packed x, int n)   // the first n elements
    {
        if (n >= 4) {
            store_any(p, off, u32x2{x.x, x.y});
        } else {
            const uint32_t w[2] = {x.x, x.y};
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (j < n) store_any(p, off + 2u * j, bf16_t(w[j >> 1] >> (16 * (j & 1))));
        }
    }
    static __device__ __forceinline__ packed pack(const float (&v)[4]) { return make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])); }
    static __device__ __forceinline__ void store_packed(rsrc_t rs, uint32_t off, packed p)   // dropped if off is out of range
    {
        const u32x2v x = {p.x, p.y};
        __builtin_amdgcn_raw_buffer_store_b64(x, rs, (int)off, 0, 0);
    }
    static __device__ __forceinline__ void store_buf(rsrc_t rs, uint32_t off, const float (&v)[4]) { store_packed(rs, off, pack(v)); }
    static __device__ __forceinline__ void unpack(const raw& r, float (&v)[4])
    {
        v[0] = bf16_lo(r.w.x); v[1] = bf16_hi(r.w.x);
        v[2] = bf16_lo(r.w.y); v[3] = bf16_hi(r.w.y);
    }
    template <bool VEC>
    static __device__ __forceinline__ void store(bf16_t* p, const float (&v)[4], int nvalid)
    {
        if (VEC) {
            if (nvalid == 4)
                *reinterpret_cast<uint2*>(p) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j < nvalid) p[j] = bf16_t(f32_to_bf16_bits(v[j]));
        }
    }
};

// A thread's slice of eight steps of a chunk in the quad-broadcast kernels.  bf16: eight consecutive steps, 16 bytes.  float:
// four steps from each half of the chunk, so that every access of the four threads of a row covers 64 bytes of it without gaps.
// Rows of any length gain nothing from it and keep eight steps (layer prefill 1 x 3936 x 4649 342 us, by fours 347).
// (Eight consecutive steps are two accesses of 16 bytes, 32 apart, to the same lines, and half-filled writes: float32
// forward + backward 8 x 4096 x 2048 1110 -> 1075 us, 2 x 5120 x 16384 3730 -> 3680, 1 x 256 x 2^20 8670 -> 7830.)
template <typename T, bool RAG> __host__ __device__ constexpr int slice_pieces() { return sizeof(T) == 4 && !RAG ? 2 : 1; }
template <typename T, int PC> struct slice_io : io8<T> {};
template <> struct slice_io<float, 2> : io4<float> {};
template <typename IO, int PC>
__device__ __forceinline__ void unpack_slice(const typename IO::raw (&r)[PC], float (&v)[8])
{
#pragma unroll
    for (int p = 0; p < PC; ++p) {
        float x[8 / PC];
        IO::unpack(r[p], x);
#pragma unroll
        for (int j = 0; j < 8 / PC; ++j) v[p * (8 / PC) + j] = x[j];
    }
}
template <typename IO, int PC>
__device__ __forceinline__ void pack_slice(const float (&v)[8], typename IO::packed (&r)[PC])
{
#pragma unroll
    for (int p = 0; p < PC; ++p) {
        float x[8 / PC];
#pragma unroll
        for (int j = 0; j < 8 / PC; ++j) x[j] = v[p * (8 / PC) + j];
        r[p] = IO::pack(x);
    }
}

__device__ __forceinline__ float f4_get(const float4& v, int j)
{
    return j == 0 ? v.x : (j == 1 ? v.y : (j == 2 ? v.z : v.w));
}

// ---- wave-uniform fetch of B or C for one state over a group of GROUP_T steps ------------
// The address depends only on the block, the wave index and loop counters, so the load
// and the bf16 widening are done by the scalar unit and the values reach the vector ALU
// as scalar operands.  Groups are kept small (4 steps: 8 or 16 bytes) so that two groups
// of all 8 (state, B|C) rows fit the scalar register file and the next group can be in
// flight while the current one is consumed.
constexpr int GROUP_T = 4;
typedef __attribute__((address_space(4))) const u32x2 const_u32x2;  // constant address space
typedef __attribute__((address_space(4))) const u32x4 const_u32x4;

template <typename T> struct bc_group;
template <> struct bc_group<float> {
    uint32_t w[4];
    __device__ __forceinline__ float get(int j) const { return __uint_as_float(w[j]); }
};
template <> struct bc_group<bf16_t> {
    uint32_t w[2];
    __device__ __forceinline__ float get(int j) const { return (j & 1) ? bf16_hi(w[j >> 1]) : bf16_lo(w[j >> 1]); }
};

// Whether a kernel takes rows FwdArgs::Li and Lb apart: those the layer has for an odd number of 16-bit steps.  The kernels that the layer
// does not launch so are built without (exact zero-order hold, bf16, us: 8 x 1536 x 2047 874 / 862, 16 x 768 x 333 211 / 207).
template <typename T, bool RAG, bool ZOH>
constexpr bool own_rows() { return RAG && !ZOH && sizeof(T) == 2; }

// Rows that the kernels off the quad-broadcast ones read element by element (SHORT): those that do not hold a slice (8 steps forward, 4 backward),
// and float32 ones of little more, where there is too little to gain for what shifting the last slice into place costs.  Forward + backward, us, by
// elements / slices: 64 x 768, fixed B, bf16 x 2 52.5 / 59.3, x 7 61.7 / 58.2 (4 in the backward pass), float32 x 9 51.1 / 54.8, x 15 54.2 / 57.5,
// complex x 17 98.2 / 101.6, 8 x 4096 x 21 63.8 / 64.4.
template <typename T>
constexpr bool short_rows(int L, int slice) { return L < (sizeof(T) == 4 ? 20 : slice); }

// Slices of 8 and of 4 steps of a row for the kernels that take rows of any length (VEC: of whole slices; SHORT: see above; otherwise of at least
// E steps): those from t, in one access.  Element by element, each behind a branch, complex state 2 x 1536 x 2047 bf16 took 1056 us forward +
// backward, now 598 (2048 steps: 300), fixed B 4 x 1536 x 2047 970, now 590.  on: false reads as zeros.
template <typename T, bool VEC, bool SHORT, template <typename> class IO, int E>
__device__ __forceinline__ typename IO<T>::raw load_slice(const T* __restrict__ row, int t, int L, bool on)
{
    const int n = on ? min(max(L - t, 0), E) : 0;
    if constexpr (VEC || SHORT) {
        return IO<T>::template load<VEC>(row + t, n);
    } else {
        const int tp = row_piece(t, E, L);
        typename IO<T>::raw r = IO<T>::load_elem(row + tp, 0u);
        if (n < E) IO<T>::drop(r, on ? t - tp : E);
        return r;
    }
}
template <typename T, bool VEC, bool SHORT> __device__ __forceinline__ typename io8<T>::raw load_slice8(const T* row, int t, int L, bool on) { return load_slice<T, VEC, SHORT, io8, 8>(row, t, L, on); }
template <typename T, bool VEC, bool SHORT> __device__ __forceinline__ typename io4<T>::raw load_slice4(const T* row, int t, int L, bool on) { return load_slice<T, VEC, SHORT, io4, 4>(row, t, L, on); }
template <typename T, bool VEC, bool SHORT, template <typename> class IO, int E>
__device__ __forceinline__ void store_slice(T* p, const float (&v)[E], int n)   // the first n elements
{
    if constexpr (VEC || SHORT) IO<T>::template store<VEC>(p, v, n);
    else IO<T>::store_elem(p, 0u, IO<T>::pack(v), n);
}

// p: start of the (b,n) row; t: first step of the group; L: row length.
// MASKED: `state_ok` false (padding state) reads as zero.
template <typename T, bool VEC, bool MASKED, bool SHORT>
__device__ __forceinline__ bc_group<T> load_bc(const T* __restrict__ p, int t, int L, bool state_ok)
{
    bc_group<T> g;
    if (VEC) {
        // Rows are 16-byte aligned and L is a multiple of 8, so a group is whole or lies
        // entirely past the end; the latter is redirected to the last whole group (its
        // values are never used: those steps run with dt = 0 and are not stored).  B and
        // C are never written by the kernels, so reading them through the constant address
        // space is sound; with the wave-uniform address it selects the scalar load path.
        const int tc = min(t, L - GROUP_T);
        if constexpr (sizeof(T) == 2) {
            const u32x2 v = *(const_u32x2*)(p + tc);
            g.w[0] = v.x; g.w[1] = v.y;
        } else {
            const u32x4 v = *(const_u32x4*)(p + tc);
            g.w[0] = v.x; g.w[1] = v.y; g.w[2] = v.z; g.w[3] = v.w;
        }
        if (MASKED) {
#pragma unroll
            for (int i = 0; i < int(sizeof(g.w) / 4); ++i) g.w[i] = state_ok ? g.w[i] : 0u;
        }
    } else if (sizeof(T) == 2 && !SHORT) {   // a row of any length: in one access, from inside the row, and shifted into place at its
        // end.  (Float elements are words, which the scalar path reads one by one: complex state 2 x 1536 x 2047 603 us, in one access 665.)
        const int tp = row_piece(t, GROUP_T, L), n = t - tp;
        const u32x2 v = load_any<u32x2>(p + tp, 0u);
        uint64_t x = (uint64_t(v[1]) << 32) | v[0];
        if (n > 0) x = n < GROUP_T ? x >> (16 * n) : 0;   // uniform
        if (MASKED) x = state_ok ? x : 0;
        g.w[0] = (uint32_t)x; g.w[1] = (uint32_t)(x >> 32);
    } else {
        uint32_t e[GROUP_T];
#pragma unroll
        for (int j = 0; j < GROUP_T; ++j) {
            const bool ok = (!MASKED || state_ok) && (t + j < L);
            if constexpr (sizeof(T) == 2) e[j] = ok ? uint32_t(p[t + j]) : 0u;
            else e[j] = ok ? __float_as_uint(p[t + j]) : 0u;
        }
        if constexpr (sizeof(T) == 2) { g.w[0] = e[0] | (e[1] << 16); g.w[1] = e[2] | (e[3] << 16); }
        else { g.w[0] = e[0]; g.w[1] = e[1]; g.w[2] = e[2]; g.w[3] = e[3]; }
    }
    return g;
}

// The same from the staged, wave-packed copy (see stage_bc_kernel): everything a wave needs of
// B and C for one group of steps is one contiguous piece, element (which * 4 + k) * 4 + j for
// B (which = 0) or C (1), the wave's state k and step j.  One or two scalar loads, no clamp,
// no mask, one base address per wave.
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(4))) const u32x16 const_u32x16;
constexpr int STAGE_GROUP = 2 * STATES_PER_LANE * GROUP_T;   // elements per wave and group
template <typename T> struct bcs_group;
template <> struct bcs_group<float> {
    uint32_t w[STAGE_GROUP];
    __device__ __forceinline__ float B(int k, int j) const { return __uint_as_float(w[k * GROUP_T + j]); }
    __device__ __forceinline__ float C(int k, int j) const { return __uint_as_float(w[(STATES_PER_LANE + k) * GROUP_T + j]); }
};
template <> struct bcs_group<bf16_t> {
    uint32_t w[STAGE_GROUP / 2];
    __device__ __forceinline__ float get(int e) const { return (e & 1) ? bf16_hi(w[e >> 1]) : bf16_lo(w[e >> 1]); }
    __device__ __forceinline__ float B(int k, int j) const { return get(k * GROUP_T + j); }
    __device__ __forceinline__ float C(int k, int j) const { return get((STATES_PER_LANE + k) * GROUP_T + j); }
};
template <typename T>
__device__ __forceinline__ bcs_group<T> load_bcs(const T* __restrict__ p)
{
    bcs_group<T> g;
    const u32x16 v = *(const_u32x16*)p;
#pragma unroll
    for (int i = 0; i < 16; ++i) g.w[i] = v[i];
    if constexpr (sizeof(T) == 4) {
        const u32x16 v2 = *(const_u32x16*)(p + 16);
#pragma unroll
        for (int i = 0; i < 16; ++i) g.w[16 + i] = v2[i];
    }
    return g;
}

// The scalar loads above are issued only one group (4 steps) ahead, which hides an L2 hit
// but not a trip to HBM.  When B and C are not already L2-resident (one batch entry, long
// sequence), the wave therefore touches the lines it will need one chunk later with
// ordinary vector loads: lanes 0..3 one element of each of its B rows, lanes 4..7 of its C
// rows, at step t.  The value is only handed to `consume_touch` an iteration later.
template <typename T>
__device__ __forceinline__ uint32_t touch_bc(const void* Bm, const void* Cm, int b, long bstride, int N, int L, int w,
                                              int lane, int t)
{
    // the raw bits, untouched: any arithmetic on the value would make the wave wait for it here
    uint32_t v = 0u;
    if (lane < 2 * STATES_PER_LANE && t >= 0 && t < L) {
        const int n = min(w * STATES_PER_LANE + (lane & 3), N - 1);
        const T* p = static_cast<const T*>(lane < STATES_PER_LANE ? Bm : Cm) + (long)b * bstride + (long)n * L + t;
        if constexpr (sizeof(T) == 2) v = *p; else v = __float_as_uint(*p);
    }
    return v;
}
// Rows of the pointwise view.  Four lanes share a row (one 16-byte piece of it each, or two), so sixteen
// consecutive lanes - what the LDS serves together - hold four rows.  With consecutive rows and the padded
// pitches that keep the one-lane-per-row view free of bank conflicts (five or nine pieces per row), those
// sixteen lanes collided two-way (3-4 % of the backward kernel's time); with the rows picked as below they
// touch sixteen different 16-byte slots.  A wave still owns sixteen consecutive rows, and the four lanes of
// a row stay adjacent, so global accesses do not change.
//   pitch 5, one piece per lane  (slot = 5 r + q):      rows r, r + 4, r + 8, r + 12
//   pitch 9, pieces 2 q, 2 q + 1 (slot = 9 r + 2 q):    rows r, r + 1, r + 8, r + 9   (r even)
__device__ __forceinline__ int pointwise_row_pitch5(int tid)
{
    return (tid >> 6) * 16 + ((tid >> 2) & 3) * 4 + ((tid >> 4) & 3);
}
__device__ __forceinline__ int pointwise_row_pitch9(int tid)
{
    const int m = (tid >> 2) & 3;
    return (tid >> 6) * 16 + 2 * ((tid >> 4) & 3) + (m & 1) + 8 * (m >> 1);
}
__device__ __forceinline__ void consume_touch(uint32_t v) { asm volatile("" ::"v"(v)); }

// ---- B and C as quad-broadcast operands ---------------------------------------------------
// A register that holds, in every group of four lanes, B (or C) of a wave's four state slots (slot k
// in lane k) can be the first operand of a multiply or multiply-add with the DPP control
// quad_perm [k,k,k,k]: every lane then reads slot k's value.  The compiler folds such a broadcast
// into a multiply only now and then and never into a multiply-add with an accumulator, so these
// instruction groups are written out.

// The input term of Eq. 2a for a lane's SPL states: bu[k] = B_k * du, with Bq holding B of the
// wave's states in every group of four lanes (slot k in lane k).  Written out for the same
// reason as adjoint_step_dpp, with the same leading wait state.
#define SS_QP(k) " quad_perm:[" #k "," #k "," #k "," #k "] row_mask:0xf bank_mask:0xf"
template <int SPL>
__device__ __forceinline__ void input_step_dpp(float (&bu)[STATES_PER_LANE], float Bq, float du)
{
    if constexpr (SPL == 4)
        asm("s_nop 1\n\t"
            "v_mul_f32_dpp %0, %4, %5" SS_QP(0) "\n\t"
            "v_mul_f32_dpp %1, %4, %5" SS_QP(1) "\n\t"
            "v_mul_f32_dpp %2, %4, %5" SS_QP(2) "\n\t"
            "v_mul_f32_dpp %3, %4, %5" SS_QP(3)
            : "=&v"(bu[0]), "=&v"(bu[1]), "=&v"(bu[2]), "=&v"(bu[3]) : "v"(Bq), "v"(du));
    else if constexpr (SPL == 2)
        asm("s_nop 1\n\t"
            "v_mul_f32_dpp %0, %2, %3" SS_QP(0) "\n\t"
            "v_mul_f32_dpp %1, %2, %3" SS_QP(1)
            : "=&v"(bu[0]), "=&v"(bu[1]) : "v"(Bq), "v"(du));
    else
        asm("s_nop 1\n\t"
            "v_mul_f32_dpp %0, %1, %2" SS_QP(0)
            : "=&v"(bu[0]) : "v"(Bq), "v"(du));
}

// The same for four slots as one matrix instruction.  v_mfma_f32_4x4x1 is sixteen independent outer products, one per
// group of four lanes: D[i][j] = A[i] x B[j] with A[i] in lane i, B[j] in lane j and D[i][j] in register i of lane j.
// With A = Bq (slot i's operand in lane i) and B = du that is bu[k] = B_k du for every row, exact products as before, in
// one issue slot instead of four and without the wait states of a DPP read.  The compiler must see what reads the result (it
// knows the wait a matrix instruction needs): not for a value that inline assembly takes next.
template <int SPL>
__device__ __forceinline__ void input_step_mfma(float (&bu)[STATES_PER_LANE], float Bq, float du)
{
    if constexpr (SPL == 4) {
        const f32x4_t x = __builtin_amdgcn_mfma_f32_4x4x1f32(Bq, du, f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
        for (int k = 0; k < 4; ++k) bu[k] = x[k];
    } else {
        input_step_dpp<SPL>(bu, Bq, du);
    }
}

// One step of the adjoint recurrence for a lane's SPL states.  On entry g[k] = abar+ g+ of slot k;
// Cq / Bq hold C / B of the wave's states in every group of four lanes (slot k in lane k).
//     g[k] += C_k dy            (the gradient reaching h_t)          sb = sum_k B_k g[k]
// The leading wait state covers a DPP operand the compiler might have copied with a vector move
// just before (a DPP read needs two wait states after a vector write of the same register).
template <int SPL>
__device__ __forceinline__ void adjoint_step_dpp(f32x4_t& g, float& sb, float Cq, float Bq, float dy)
{
    float g0 = g[0], g1 = g[1], g2 = g[2], g3 = g[3];
    if constexpr (SPL == 4)
        asm("s_nop 1\n\t"
            "v_fmac_f32_dpp %0, %5, %7" SS_QP(0) "\n\t"
            "v_fmac_f32_dpp %1, %5, %7" SS_QP(1) "\n\t"
            "v_fmac_f32_dpp %2, %5, %7" SS_QP(2) "\n\t"
            "v_fmac_f32_dpp %3, %5, %7" SS_QP(3) "\n\t"
            "v_mul_f32_dpp %4, %6, %0" SS_QP(0) "\n\t"
            "v_fmac_f32_dpp %4, %6, %1" SS_QP(1) "\n\t"
            "v_fmac_f32_dpp %4, %6, %2" SS_QP(2) "\n\t"
            "v_fmac_f32_dpp %4, %6, %3" SS_QP(3)
            : "+v"(g0), "+v"(g1), "+v"(g2), "+v"(g3), "=&v"(sb) : "v"(Cq), "v"(Bq), "v"(dy));
    else if constexpr (SPL == 2)
        asm("s_nop 1\n\t"
            "v_fmac_f32_dpp %0, %3, %5" SS_QP(0) "\n\t"
            "v_fmac_f32_dpp %1, %3, %5" SS_QP(1) "\n\t"
            "v_mul_f32_dpp %2, %4, %0" SS_QP(0) "\n\t"
            "v_fmac_f32_dpp %2, %4, %1" SS_QP(1)
            : "+v"(g0), "+v"(g1), "=&v"(sb) : "v"(Cq), "v"(Bq), "v"(dy));
    else
        asm("s_nop 1\n\t"
            "v_fmac_f32_dpp %0, %2, %4" SS_QP(0) "\n\t"
            "v_mul_f32_dpp %1, %3, %0" SS_QP(0)
            : "+v"(g0), "=&v"(sb) : "v"(Cq), "v"(Bq), "v"(dy));
    g[0] = g0; g[1] = g1; g[2] = g2; g[3] = g3;
}
// The first half of adjoint_step_dpp alone (for the adjoint aggregate of a segment): g[k] += C_k dy.
template <int SPL>
__device__ __forceinline__ void adjoint_input_dpp(float (&g)[STATES_PER_LANE], float Cq, float dy)
{
    if constexpr (SPL == 4)
        asm("s_nop 1\n\t"
            "v_fmac_f32_dpp %0, %4, %5" SS_QP(0) "\n\t"
            "v_fmac_f32_dpp %1, %4, %5" SS_QP(1) "\n\t"
            "v_fmac_f32_dpp %2, %4, %5" SS_QP(2) "\n\t"
            "v_fmac_f32_dpp %3, %4, %5" SS_QP(3)
            : "+v"(g[0]), "+v"(g[1]), "+v"(g[2]), "+v"(g[3]) : "v"(Cq), "v"(dy));
    else if constexpr (SPL == 2)
        asm("s_nop 1\n\t"
            "v_fmac_f32_dpp %0, %2, %3" SS_QP(0) "\n\t"
            "v_fmac_f32_dpp %1, %2, %3" SS_QP(1)
            : "+v"(g[0]), "+v"(g[1]) : "v"(Cq), "v"(dy));
    else
        asm("s_nop 1\n\t"
            "v_fmac_f32_dpp %0, %1, %2" SS_QP(0)
            : "+v"(g[0]) : "v"(Cq), "v"(dy));
}

// The read-out of Eq. 2b for a lane's SPL states: y = sum_k C_k h[k], Cq holding C like Bq above.
template <int SPL>
__device__ __forceinline__ void readout_step_dpp(float& y, float Cq, const float (&h)[STATES_PER_LANE])
{
    if constexpr (SPL == 4)
        asm("s_nop 1\n\t"
            "v_mul_f32_dpp %0, %1, %2" SS_QP(0) "\n\t"
            "v_fmac_f32_dpp %0, %1, %3" SS_QP(1) "\n\t"
            "v_fmac_f32_dpp %0, %1, %4" SS_QP(2) "\n\t"
            "v_fmac_f32_dpp %0, %1, %5" SS_QP(3)
            : "=&v"(y) : "v"(Cq), "v"(h[0]), "v"(h[1]), "v"(h[2]), "v"(h[3]));
    else if constexpr (SPL == 2)
        asm("s_nop 1\n\t"
            "v_mul_f32_dpp %0, %1, %2" SS_QP(0) "\n\t"
            "v_fmac_f32_dpp %0, %1, %3" SS_QP(1)
            : "=&v"(y) : "v"(Cq), "v"(h[0]), "v"(h[1]));
    else
        asm("s_nop 1\n\t"
            "v_mul_f32_dpp %0, %1, %2" SS_QP(0)
            : "=&v"(y) : "v"(Cq), "v"(h[0]));
}
// The read-outs of a group of four steps together: y[j] = sum_k C_k(j) h[j][k], Cq the group's four steps.  One wait for
// all of them, and four sums side by side instead of one dependent chain after another.
__device__ __forceinline__ void readout_group_dpp(float (&y)[4], const float4& Cq, const float (&h)[4][STATES_PER_LANE])
{
    asm("s_nop 1\n\t"
        "v_mul_f32_dpp %0, %4, %8" SS_QP(0) "\n\t"
        "v_mul_f32_dpp %1, %5, %12" SS_QP(0) "\n\t"
        "v_mul_f32_dpp %2, %6, %16" SS_QP(0) "\n\t"
        "v_mul_f32_dpp %3, %7, %20" SS_QP(0) "\n\t"
        "v_fmac_f32_dpp %0, %4, %9" SS_QP(1) "\n\t"
        "v_fmac_f32_dpp %1, %5, %13" SS_QP(1) "\n\t"
        "v_fmac_f32_dpp %2, %6, %17" SS_QP(1) "\n\t"
        "v_fmac_f32_dpp %3, %7, %21" SS_QP(1) "\n\t"
        "v_fmac_f32_dpp %0, %4, %10" SS_QP(2) "\n\t"
        "v_fmac_f32_dpp %1, %5, %14" SS_QP(2) "\n\t"
        "v_fmac_f32_dpp %2, %6, %18" SS_QP(2) "\n\t"
        "v_fmac_f32_dpp %3, %7, %22" SS_QP(2) "\n\t"
        "v_fmac_f32_dpp %0, %4, %11" SS_QP(3) "\n\t"
        "v_fmac_f32_dpp %1, %5, %15" SS_QP(3) "\n\t"
        "v_fmac_f32_dpp %2, %6, %19" SS_QP(3) "\n\t"
        "v_fmac_f32_dpp %3, %7, %23" SS_QP(3)
        : "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2]), "=&v"(y[3])
        : "v"(Cq.x), "v"(Cq.y), "v"(Cq.z), "v"(Cq.w), "v"(h[0][0]), "v"(h[0][1]), "v"(h[0][2]), "v"(h[0][3]), "v"(h[1][0]),
          "v"(h[1][1]), "v"(h[1][2]), "v"(h[1][3]), "v"(h[2][0]), "v"(h[2][1]), "v"(h[2][2]), "v"(h[2][3]), "v"(h[3][0]),
          "v"(h[3][1]), "v"(h[3][2]), "v"(h[3][3]));
}
#undef SS_QP

// ---- segments of a split sequence --------------------------------------------------------------
// What enters a segment from the n segments before it, for a lane's four slots: c = loc(0), then
// c = exp(A sum_dt(i)) c + loc(i) for i = 1 .. n-1, where loc(i) / sum_dt(i) are segment i's own end state and sum
// of step sizes (counted from the far end).  Up to CARRY_INLINE segments every workgroup works this out
// for itself at its start: a few hundred bytes per row from the L2, loads of eight segments at a time in flight,
// instead of a launch between the two passes that depend on each other (9 us forward and 5 us backward at
// 8 x 1536 x 2048; the chain itself is below 2 us).  Longer chains, which every workgroup would repeat, keep the
// kernel of their own.
constexpr int CARRY_INLINE = 16;
template <typename LOC, typename SUM>
__device__ __forceinline__ f32x4_t chain_segments(int n, const float (&A2)[STATES_PER_LANE], LOC loc, SUM sum_dt)
{
    constexpr int BATCH = 8;
    f32x4_t c = loc(0);
    for (int i0 = 1; i0 < n; i0 += BATCH) {
        f32x4_t l[BATCH];
        float sd[BATCH];
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            const int i = min(i0 + j, n - 1);
            l[j] = loc(i);
            sd[j] = sum_dt(i);
        }
#pragma unroll
        for (int j = 0; j < BATCH; ++j)
            if (i0 + j < n) {   // uniform
#pragma unroll
                for (int k = 0; k < STATES_PER_LANE; ++k) c[k] = fmaf(exp2_fast(A2[k] * sd[j]), c[k], l[j][k]);
            }
    }
    return c;
}

}  // namespace ss
