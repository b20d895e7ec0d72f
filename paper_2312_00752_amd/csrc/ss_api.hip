// C-ABI entry points: host-side validation and dispatch only (see include/ss_scan.h).
#include <hip/hip_runtime.h>

#include <atomic>

#include "ss_device.h"
#include "ss_kernels.h"
#include "ss_layer.h"
#include "ss_scan.h"

// Scratch of ss_scan_fwd_static: lives in the library's device image, one copy per GPU.  In host
// code this name is only a handle for hipGetSymbolAddress; the device address it yields is what
// every kernel argument below uses.
static __device__ __align__(256) unsigned char scratch[SS_STATIC_SCRATCH_BYTES];

namespace {

constexpr uint32_t kFwdFlags = SS_DELTA_SOFTPLUS | SS_HAS_DELTA_BIAS | SS_HAS_D | SS_HAS_Z |
                               SS_HAS_H0 | SS_WRITE_H_LAST | SS_SAVE_FOR_BWD | SS_EXACT_ZOH_B |
                               SS_B_FIXED | SS_C_FIXED | SS_COMPLEX_STATE;
constexpr uint32_t kStepFlags = SS_DELTA_SOFTPLUS | SS_HAS_DELTA_BIAS | SS_HAS_D | SS_HAS_Z | SS_EXACT_ZOH_B |
                                SS_B_FIXED | SS_C_FIXED | SS_COMPLEX_STATE;

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }
inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
// Real numbers per state vector: a complex state is a (re, im) pair of slots, and everything
// below the validation works on slots.
inline int slots(const ss_fwd_params* p) { return p->dstate * ((p->flags & SS_COMPLEX_STATE) ? 2 : 1); }
inline int slots(const ss_step_params* p) { return p->dstate * ((p->flags & SS_COMPLEX_STATE) ? 2 : 1); }

// Split of the sequence across workgroups.  The scan kernels run one workgroup per 64 rows
// of a batch entry; when that fills the chip badly and the sequence is long, L is cut into
// segments (multiples of 64 steps) that are scanned
// concurrently and stitched with a carry pass (Appendix D: the scan continues from the
// state the previous chunk ended in; here the chunks run in parallel from aggregates).
struct SegPlan {
    int nseg, seg_len;
};
// Modelled duration (in steps of one unsplit workgroup running alone on its compute unit) of a
// launch of n equal workgroups of len steps each.  Two workgroups fit a compute unit and then
// take `pair` times what one takes alone (selective B and C 4/3: 256 workgroups of 2048 steps
// take 1.01 ms, 512 take 1.35 ms), so the chip takes workgroups in rounds of 512.  A workgroup's
// set-up, pipeline fill and final stores cost about as much as 32 more steps (fitted to sweeps of
// the segment count at 160 x 16384, 192 x 2048 and 4 x 2^20 workgroups x steps).  The fits are of the main passes and of
// aggregate passes that ran two workgroups per unit as well.  The aggregate kernels have since come to run four; what
// they take per step is now 0.35 (4 x 2^20), 0.40 (160 x 16384) and 0.44 (192 x 2048) of a main pass, and neither the
// rounds nor AGG_COST have been fitted again.
constexpr double AGG_COST = 0.36;   // an aggregate pass, per step of a main pass (over forward + backward)
double launch_cost(long n, long len, double pair = 1.0 / 0.75)
{
    const double fixed = 32.0;
    const long full = n / 512, rest = n % 512;
    return ((double)len + fixed) * ((double)full * pair + (rest == 0 ? 0.0 : (rest <= 256 ? 1.0 : pair)));
}

long segment_length(int L, long nseg)
{
    // whole pairs of 32-step chunks: the forward kernel issues the traffic of an even chunk and the
    // odd one after it together
    long len = ((L + nseg - 1) / nseg + 63) / 64 * 64;
    // A segment length that is a large power of two makes every workgroup walk the memory
    // channels in lockstep (all segment starts alias); an odd multiple of 64 steps staggers them
    // (measured: 7-12 % on the 2^20-step workload).  Short segments are staggered only when
    // there are hundreds of them; otherwise the shorter last segment costs more than the
    // aliasing does (measured on 8K- and 64K-step sequences).
    if (nseg > 1 && len % 256 == 0) len += len >= 2048 ? 192 : (nseg >= 256 ? 64 : 0);
    return len;
}

SegPlan plan_segments(int B, int D, int L)
{
    const long wgs = (long)B * ((D + 63) / 64);
    SegPlan s{1, (L + 31) / 32 * 32};
    if (s.seg_len == 0) s.seg_len = 32;
    if (L < 128) return s;
    // Pick the number of segments that the model says finishes first: the main pass over
    // wgs * nseg workgroups plus the aggregate pass over wgs * (nseg - 1) of them.  Segments stay
    // at least 64 steps long (two forward chunks), and a launch within 8192 workgroups, which
    // bounds the aggregates' workspace.
    double best = launch_cost(wgs, s.seg_len);
    long best_n = 1;
    const long fit = 8192 / wgs > 2 ? 8192 / wgs : 2;
    const long longest = L / 64 < 4096 ? L / 64 : 4096;
    const long most = longest < fit ? longest : fit;
    for (long want = 2; want <= most; ++want) {
        const long len = segment_length(L, want);
        const long n = (L + len - 1) / len;   // what that length really gives
        if (n < 2) continue;
        const double c = launch_cost(wgs * n, len) + AGG_COST * launch_cost(wgs * (n - 1), len);
        if (c < best * 0.97) { best = c; best_n = want; }   // more segments only for a clear gain
    }
    if (best_n > 1) {
        s.seg_len = (int)segment_length(L, best_n);
        s.nseg = (L + s.seg_len - 1) / s.seg_len;
    }
    return s;
}

// Whether that plan pays with a time-invariant B and / or C, whose kernels are others: forward + backward of 72 grids of 64 to 2112 row
// groups x 128 to 8192 steps in the 18 forms of B and C, state, rule and dtype, whole and in this plan, by the model above with what two
// workgroups of a unit take (pair) and what the launches of a split call cost beside (launches, in steps) fitted for each form.  Where it
// keeps a split that does not pay, that costs 6 % at most (256 x 2048 float32 C 840 / 891).  us, whole / split, refused: exact zero-order hold, whose backward
// kernels have a unit to themselves, 256 x 2048 bf16 B and C 1339 / 1539; B and C in registers, float32 256 x 2048 665 / 889, bf16
// 256 x 512 175 / 192; grids that share units as they are, 320 x 2048 float32 C 1 / 1.04.  Kept: 64 x 2048 bf16 B 777 / 230, with the
// exact hold 1576 / 512, 320 x 2048 1 / 0.84; 256 x 2048 bf16 B 790 / 689.
bool fixed_split_pays(const ss_fwd_params* p, const SegPlan& s)
{
    const bool both = (p->flags & SS_B_FIXED) && (p->flags & SS_C_FIXED), zoh = p->flags & SS_EXACT_ZOH_B;
    const bool f32 = p->io_dtype != SS_BF16, cplx = p->flags & SS_COMPLEX_STATE, whole_slices = p->seqlen % 8 == 0;
    const long wgs = (long)p->batch * ((p->dim + 63) / 64);
    if (!zoh && ((wgs > 256 && wgs <= 512) || (both && p->seqlen < 256))) return false;   // 64 x 200 B and C, float32: 77.7 / 84.1
    double pair = 1.3, launches = wgs <= 64 ? 28.0 : 30.0;   // 128 steps, C, bf16, whole / split: 1 x 4096 60.4 / 58.4, 2 x 4096 1 / 1.05
    if (zoh) {
        pair = both ? 1.35 : 1.25;
        launches = 0.0;
    } else if (both) {
        pair = whole_slices ? (f32 ? 1.95 : 1.55) : (f32 ? 1.8 : 1.4);
        if (!whole_slices) launches = f32 ? 0.0 : 40.0;
    } else if (f32 && whole_slices) {
        if (cplx || (p->flags & SS_B_FIXED)) pair = cplx ? 1.5 : 1.55;
    } else if (f32 && (p->flags & SS_B_FIXED)) {
        pair = cplx ? 1.65 : 1.4;
        launches = cplx ? 0.0 : 40.0;
    }
    auto main_pass = [&](long n, long len) {
        const double shared = launch_cost(n, len, pair);
        return zoh ? 0.4 * shared + 0.6 * (double)(len + 32) * (double)((n + 255) / 256) : shared;   // forward + backward
    };
    return main_pass(wgs * s.nseg, s.seg_len) + AGG_COST * launch_cost(wgs * (s.nseg - 1), s.seg_len, pair) + launches <
           main_pass(wgs, (p->seqlen + 31) / 32 * 32);
}

inline bool fixed_bc(const ss_fwd_params* p) { return p->flags & (SS_B_FIXED | SS_C_FIXED); }
// a forward call with a time-invariant B or C that keeps nothing asks for no scratch, and is not split
inline int split_steps(const ss_fwd_params* p, bool for_bwd) { return for_bwd || !fixed_bc(p) ? p->seqlen : 0; }
SegPlan plan_of(const ss_fwd_params* p, bool for_bwd)
{
    const SegPlan s = plan_segments(p->batch, p->dim, split_steps(p, for_bwd));
    return s.nseg > 1 && fixed_bc(p) && !fixed_split_pays(p, s) ? plan_segments(p->batch, p->dim, 0) : s;
}

// Workspace layouts, each block 256-byte aligned.
//   forward only:  [io pre-gate y B*D*L, only with a gate and more than 16 states]
//                  [float seg_h nseg*B*D*16][float seg_sumdt nseg*B*D]        (only when split)
//   with backward: [float checkpoints groups*nck*B*D*16][io pre-gate y B*D*L, only with a gate]
//                  [seg_h][seg_sumdt][float seg_g nseg*B*D*16]                 (only when split)
//                  [float dA partials nseg*B*D*16][float dD partials nseg*B*D][float dbias partials nseg*B*D]
//                  [float dB partials nseg*B*D*16][float dC partials nseg*B*D*16]    (only for a time-invariant B / C)
//   both end with: [io staged B and C, B * ceil16(slots) * Lp * 2]    (only for a real state with selective B and C)
// where Lp is L rounded up to a whole 32-step chunk.  The staged copy is written and read by the kernels for fewer than
// 8 or at least 2^23 steps only (FwdArgs::dpp_ok false); the size of a workspace does not depend on that, so that a
// caller's allocations do not change with the path.
struct WsLayout {
    size_t ckpt_off, ckpt_group, y_off, segh_off, segdt_off, segg_off, dA_off, dD_off, db_off, dBf_off, dCf_off;
    size_t bcs_off, total;
    int Lp;
    SegPlan plan;
};
// Whether the call has operands that can be repacked: a real state's selective B and C.
inline bool stageable(const ss_fwd_params* p)
{
    return !(p->flags & (SS_B_FIXED | SS_C_FIXED | SS_COMPLEX_STATE)) && p->seqlen > 0;
}
WsLayout ws_layout(const ss_fwd_params* p, bool for_bwd, int pitch, const SegPlan& plan)
{
    const size_t nck = ((size_t)p->seqlen + SS_CHECKPOINT_STEPS - 1) / SS_CHECKPOINT_STEPS;
    const size_t rows = (size_t)p->batch * p->dim;
    const size_t esz = p->io_dtype == SS_BF16 ? 2 : 4;
    WsLayout w{};
    w.plan = plan;
    const size_t ns = (size_t)w.plan.nseg, split = ns > 1 ? 1 : 0;
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t at = off; off += round_up(bytes, 256); return at; };
    const size_t groups = ((size_t)slots(p) + 15) / 16;   // states are handled 16 at a time
    w.ckpt_group = nck * rows * 16 * sizeof(float);
    w.ckpt_off = take(for_bwd ? groups * w.ckpt_group : 0);
    // the pre-gate y: for the backward pass, and as the accumulator across state groups
    w.y_off = take((for_bwd || groups > 1) && (p->flags & SS_HAS_Z) ? rows * (size_t)pitch * esz : 0);
    w.segh_off = take(split * ns * rows * 16 * sizeof(float));
    w.segdt_off = take(split * ns * rows * sizeof(float));
    w.segg_off = take(for_bwd ? split * ns * rows * 16 * sizeof(float) : 0);
    w.dA_off = take(for_bwd ? ns * rows * 16 * sizeof(float) : 0);
    w.dD_off = take(for_bwd ? ns * rows * sizeof(float) : 0);
    w.db_off = take(for_bwd ? ns * rows * sizeof(float) : 0);
    // partial sums of the gradient of a time-invariant B / C, per batch entry and segment
    w.dBf_off = take(for_bwd && (p->flags & SS_B_FIXED) ? ns * rows * 16 * sizeof(float) : 0);
    w.dCf_off = take(for_bwd && (p->flags & SS_C_FIXED) ? ns * rows * 16 * sizeof(float) : 0);
    w.Lp = (p->seqlen + 31) / 32 * 32;
    w.bcs_off = take(stageable(p) ? (size_t)p->batch * (((size_t)slots(p) + 15) / 16 * 16) * w.Lp * 2 * esz : 0);
    w.total = off;
    return w;
}
WsLayout ws_layout(const ss_fwd_params* p, bool for_bwd, int pitch) { return ws_layout(p, for_bwd, pitch, plan_of(p, for_bwd)); }

int check_fwd(const ss_fwd_params* p, bool for_bwd, int pitch, bool bc_dense = true)
{
    if (!p) return SS_ERR_NULL;
    if (p->batch < 1 || p->dim < 1 || p->dstate < 1 || p->seqlen < 0) return SS_ERR_SHAPE;
    if (p->dstate > SS_MAX_DSTATE || slots(p) > SS_MAX_DSTATE) return SS_ERR_UNSUPPORTED;
    if ((p->flags & SS_COMPLEX_STATE) && (p->flags & SS_EXACT_ZOH_B)) return SS_ERR_UNSUPPORTED;
    if (p->io_dtype != SS_F32 && p->io_dtype != SS_BF16) return SS_ERR_UNSUPPORTED;
    if (p->flags & ~kFwdFlags) return SS_ERR_UNSUPPORTED;
    const bool empty = p->seqlen == 0;  // tensors with a zero-length axis may be NULL
    if (!p->A) return SS_ERR_NULL;
    if (!empty && (!p->u || !p->delta || !p->Bmat || !p->Cmat)) return SS_ERR_NULL;
    if (!empty && !for_bwd && !p->out) return SS_ERR_NULL;
    if (!empty && (p->flags & SS_HAS_Z) && !p->z) return SS_ERR_NULL;
    if ((p->flags & SS_HAS_D) && !p->Dskip) return SS_ERR_NULL;
    if ((p->flags & SS_HAS_DELTA_BIAS) && !p->delta_bias) return SS_ERR_NULL;
    if ((p->flags & SS_HAS_H0) && !p->h0) return SS_ERR_NULL;
    if (!for_bwd && (p->flags & SS_WRITE_H_LAST) && !p->h_last) return SS_ERR_NULL;
    const void* io[] = {p->u, p->delta, p->z, for_bwd ? nullptr : p->out};
    for (const void* q : io)
        if (q && !aligned(q, 16)) return SS_ERR_ALIGN;
    // B and C are read 16 bytes at a time only when every row is a whole number of such pieces;
    // the layer passes rows of a larger matrix here, which then are merely element-aligned
    const size_t bc_align = (p->seqlen % 8 == 0 || bc_dense) ? 16 : (p->io_dtype == SS_BF16 ? 2 : 4);
    if (p->Bmat && !aligned(p->Bmat, (p->flags & SS_B_FIXED) ? 4 : bc_align)) return SS_ERR_ALIGN;
    if (p->Cmat && !aligned(p->Cmat, (p->flags & SS_C_FIXED) ? 4 : bc_align)) return SS_ERR_ALIGN;
    const void* f32[] = {p->A, p->Dskip, p->delta_bias, p->h0, for_bwd ? nullptr : p->h_last};
    for (const void* q : f32)
        if (q && !aligned(q, 4)) return SS_ERR_ALIGN;
    if (!for_bwd && !(p->flags & SS_SAVE_FOR_BWD) && slots(p) > 16 && (p->flags & SS_HAS_Z) && p->seqlen > 0) {
        // the pre-gate output is accumulated over the groups of 16 states in the workspace
        if (!p->workspace || p->workspace_bytes < ws_layout(p, false, pitch).total) return SS_ERR_WORKSPACE;
        if (!aligned(p->workspace, 256)) return SS_ERR_ALIGN;
    }
    if (for_bwd || (p->flags & SS_SAVE_FOR_BWD)) {
        const size_t need = ws_layout(p, true, pitch).total;
        if (!p->workspace || p->workspace_bytes < need) return SS_ERR_WORKSPACE;
        if (!aligned(p->workspace, 256)) return SS_ERR_ALIGN;
    }
    return SS_OK;
}

// Whether a pass over fewer than 16 states deals them out to the waves in turn (FwdArgs::il): the
// common path only.  Forward and backward call derive it from the same arguments.
inline bool deals_states(int dpp_ok, uint32_t flags)
{
    return dpp_ok && !(flags & (SS_EXACT_ZOH_B | SS_B_FIXED | SS_C_FIXED | SS_COMPLEX_STATE));
}

// Whether the float results of a chunk wait for those of its neighbour, so that what shares a line is written together
// (FwdArgs::wait_fwd, wait_bwd).  That pays once the tensors leave the caches; with less it only costs instructions and registers.
// A chunk of the forward pass is a line: its results wait where rows are not whole lines and a gate leaves time beside the stores, or where
// two results go to rows that are all on one channel.  A block of the backward pass is half a line.  Calls whose results
// wait relative to the same whose do not, us, 256 forms and sizes, tensors apart by whole MiB and by 65 KiB more.
// Forward, off whole lines, gate: below 16 MB a tensor 1.013, 16 to 32 MB 1.018, 32 to 64 MB 0.996, above 0.974 (8 x 4096 x 2047 0.89, with
// the backward pass 0.98; 3 x 8192 x 3000 alone 1.07), without a gate 1.016; whole lines 1.018 and 1.035; 256 x 2^20 0.985 with the
// backward pass.  Backward: below 16 MB 1.025 off eight steps, else 1.006, 16 to 32 MB 0.975, above 0.96; without a gate and 16 states 0.99
// to 1.01, exact hold 1.00.
void choose_waits(ss::FwdArgs& a, const ss_fwd_params* p)
{
    const size_t mb = (size_t)p->batch * p->dim * p->seqlen * sizeof(float) >> 20;
    const bool gate = p->flags & SS_HAS_Z, one_channel = p->seqlen % (1 << 20) == 0 && (p->flags & SS_SAVE_FOR_BWD);
    a.wait_fwd = gate && mb >= 32 && (p->seqlen % 32 != 0 || one_channel);
    a.wait_bwd = mb >= 16;
}

ss::FwdArgs make_fwd_args(const ss_fwd_params* p, long bc_bstride, int pitch)
{
    ss::FwdArgs a{};
    a.B = p->batch; a.D = p->dim; a.L = p->seqlen; a.N = slots(p); a.NS = slots(p);
    a.acc_y = 0;
    a.flags = p->flags;
    // 16-byte slices, addressed through per-workgroup buffer resources (64 rows, 31-bit offsets)
    a.dpp_ok = p->seqlen >= 8 && (size_t)p->seqlen * 64 * sizeof(float) < ((size_t)1 << 31);
    a.vec_ok = a.dpp_ok && p->seqlen % 8 == 0;
    a.Li = a.Lb = pitch;
    a.il = deals_states(a.dpp_ok, p->flags) && a.N < 16;
    a.u = p->u; a.delta = p->delta; a.z = (p->flags & SS_HAS_Z) ? p->z : nullptr;
    a.Bm = p->Bmat; a.Cm = p->Cmat; a.A = p->A;
    a.bc_bstride = bc_bstride;
    a.Dskip = p->Dskip; a.bias = p->delta_bias; a.h0 = p->h0;
    a.out = p->out;
    a.h_last = (p->flags & SS_WRITE_H_LAST) ? p->h_last : nullptr;
    a.ckpt = nullptr;
    a.ysave = nullptr;
    a.nseg = 1;
    a.seg_len = (p->seqlen + 31) / 32 * 32 + 32;
    a.seg_h = nullptr;
    a.seg_sumdt = nullptr;
    a.bcs = nullptr; a.Lp = 0;
    a.W_dt = nullptr; a.rT = nullptr; a.R = 0; a.Rp = 0;
    choose_waits(a, p);
    return a;
}

// Narrows the arguments of a whole call to the g-th group of 16 states: every (..., n) pointer
// moves to the group's first state (the stride stays NS), checkpoints get the group's block.
template <typename P> P* at(P* base, long elems) { return base ? base + elems : base; }
const void* at_bytes(const void* base, size_t bytes) { return base ? static_cast<const char*>(base) + bytes : base; }

void narrow_to_group(ss::FwdArgs& a, const ss_fwd_params* p, int g, size_t ckpt_group_bytes)
{
    const int n0 = g * 16;
    const size_t esz = p->io_dtype == SS_BF16 ? 2 : 4;
    a.N = slots(p) - n0 < 16 ? slots(p) - n0 : 16;
    a.il = deals_states(a.dpp_ok, p->flags) && a.N < 16;
    a.A = at(a.A, n0);
    a.h0 = at(a.h0, n0);
    a.h_last = at(a.h_last, n0);
    a.Bm = (p->flags & SS_B_FIXED) ? at_bytes(a.Bm, (size_t)n0 * 4) : at_bytes(a.Bm, (size_t)n0 * a.Lb * esz);
    a.Cm = (p->flags & SS_C_FIXED) ? at_bytes(a.Cm, (size_t)n0 * 4) : at_bytes(a.Cm, (size_t)n0 * a.Lb * esz);
    a.bcs = at_bytes(a.bcs, (size_t)(n0 / 4) * (a.Lp / 4) * 32 * esz);   // the group's first packed piece
    if (a.ckpt) a.ckpt = reinterpret_cast<float*>(reinterpret_cast<char*>(a.ckpt) + (size_t)g * ckpt_group_bytes);
    if (g > 0) {
        a.flags &= ~(uint32_t)SS_HAS_D;   // the skip term enters once
        a.acc_y = 1;
    }
}

// Device address of `scratch` on the current device, looked up once per device.
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];
int static_scratch(void** out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SS_ERR_LAUNCH;
    void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!ptr) {
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return SS_ERR_LAUNCH;
        g_scratch_ptr[dev].store(ptr, std::memory_order_release);   // the same value from every thread
    }
    *out = ptr;
    return SS_OK;
}

}  // namespace

namespace ss {

// The fused projection exists for the plain bf16 kernel on an unsplit sequence of at least 8 steps,
// with a workspace.  It is taken up to a rank of 128 on whole 8-step slices, and for the ranks that the matrix-core product does
// not reach (above 192).  Layer forward, us, fused / product and plain scan:
//   8 x 2048 tokens, D = 4096, R = 128     419 / 429       16 x 2048 tokens, D = 2048, R = 64   387 / 397
//   16 x 104 tokens, D = 3072, R = 96       87 / 92        8 x 2048 tokens, D = 3072, R = 96    383 / 377
// Above 128 the pieces of W_dt take the registers that a second workgroup per CU needs:
//   6 x 8192 tokens, D = 5120, R = 160    2474 / 1618      16 x 504 tokens    457 / 328      16 x 128 tokens    169 / 131
// and off whole slices:
//   16 x 2047 tokens, D = 4096, R = 128   1025 / 1000      4 x 101 tokens     57 / 55
//   16 x 2047 tokens, D = 5120, R = 160   1701 / 1342      4 x 101 tokens     79 / 68
//   16 x 701 tokens,  D = 6144, R = 192    856 / 698       4 x 127 tokens    101 / 91
//   16 x 1001 tokens, D = 6400, R = 200   1297 / 1308      8 x 117 tokens    161 / 489
bool scan_fwd_fusable(const ss_fwd_params* p, int pitch, int R)
{
    if (!p || p->seqlen < 1 || p->io_dtype != SS_BF16 || !stageable(p) || slots(p) > 16) return false;
    if (R < 8 || R % 8 != 0 || R > 256 || (p->flags & SS_EXACT_ZOH_B)) return false;
    if (p->seqlen < 8 || (size_t)p->seqlen * 64 * sizeof(float) >= ((size_t)1 << 31)) return false;
    if (R <= 192 && (R > 128 || p->seqlen % 8 != 0)) return false;
    // eight states or fewer are dealt out to kernels of one or two slots per lane, which are built without the projection
    if (slots(p) <= 8) return false;
    if (plan_of(p, true).nseg != 1) return false;   // stageable: B and C selective
    return p->workspace && aligned(p->workspace, 256) &&
           p->workspace_bytes >= ws_layout(p, (p->flags & SS_SAVE_FOR_BWD) != 0, pitch).total;
}

// Whether rows of the caller's own tensors may be that far apart: the kernels that own_rows() names take it.
static bool pitch_ok(const ss_fwd_params* p, int pitch)
{
    if (pitch == p->seqlen) return true;
    return pitch > p->seqlen && p->seqlen >= 8 && p->seqlen % 8 != 0 && p->io_dtype == SS_BF16 && !(p->flags & SS_EXACT_ZOH_B) && stageable(p) &&
           (size_t)pitch * 64 * sizeof(float) < ((size_t)1 << 31);
}

// Whether the forward pass goes over whole rows in workgroups of eight waves (launch_fwd_whole), whatever the plan of the backward
// pass: where every row group has a compute unit of its own and that is less than what the pass in nseg segments is modelled to
// take.  In steps of a workgroup of four waves alone, a whole row is `step` per step and `fixed` more, fitted for what differs
// between the kernels: the rule, the dtype and, in bf16, the slots per lane (with fewer the four waves are done sooner, the
// pointwise waves here are not).  Measured: 1 to 256 row groups x 32 to 16384 steps, on and off eight steps, N = 1, 4, 8, 16 and the
// exact hold, forward alone and with the backward pass; profiles/whole_rows_line.txt has both sides of every point.  Where the line
// sends a call whole that is faster in segments, that costs 3 % at most, float rows of up to four states 4 % (136 x 3072).
// us, in segments / whole, forward alone.  Sent whole: 192 x 2048 N = 16 bf16 181 / 133, float 186 / 130, exact hold 305 / 235, N = 4 bf16
// 110 / 93; 160 x 16384 bf16 1110 / 1006; float 160 x 8192 598 / 497.  Kept in segments: 128 x 2048 bf16 127 / 132, N = 4 160 x 16384
// 647 / 708, 136 x 3072 129 / 143, N = 8 155 / 158; exact hold, float 80 x 320 34.0 / 40.8, bf16 1 x 192 23.1 / 24.9.  With the backward pass:
// 192 x 2048 518 / 464, exact hold 821 / 749, 160 x 16384 3171 / 3044, N = 4 2182 / 2215, 128 x 2048 350 / 350, float 192 x 2048 560 / 490.
static bool runs_whole(const ss_fwd_params* p, const ss::FwdArgs& a)
{
    const long wgs = (long)p->batch * ((p->dim + 63) / 64), L = p->seqlen;
    if (!a.dpp_ok || !stageable(p) || slots(p) > 16 || wgs > 256) return false;
    const int spl = ss::slots_for(a.N, a.il);
    // not split: always (256 x 64 9.3 / 7.9 us), but for a single chunk, which has nothing to run beside, with one slot per lane
    // (192 x 32 float 5.04 / 5.24, bf16 4.69 / 4.76; two slots bf16 5.26 / 5.12)
    if (a.nseg == 1) return spl > 1 || L > 32;
    double step = 0.48, fixed = 32.0;   // float
    if (p->flags & SS_EXACT_ZOH_B) {
        step = 0.535;
        fixed = 48.0;
    } else if (p->io_dtype == SS_BF16) {
        step = spl == 1 ? 0.605 : (spl == 2 ? 0.59 : 0.55);
        fixed = spl == 2 ? -12.0 : 0.0;
    }
    return step * (double)L + fixed <= launch_cost(wgs * a.nseg, a.seg_len) + AGG_COST * launch_cost(wgs * (a.nseg - 1), a.seg_len);
}

static int scan_fwd_impl(const ss_fwd_params* p, long bc_bstride, int pitch, const void* W_dt, int R, const void* rT, void* stream)
{
    if (p && !pitch_ok(p, pitch)) return SS_ERR_UNSUPPORTED;
    const int rc = check_fwd(p, false, pitch, p && bc_bstride == (long)slots(p) * p->seqlen);
    if (rc != SS_OK) return rc;
    ss::FwdArgs a = make_fwd_args(p, bc_bstride, pitch);
    if (W_dt) {
        if (!scan_fwd_fusable(p, pitch, R) || !aligned(W_dt, 16) || !aligned(rT, 16)) return SS_ERR_UNSUPPORTED;
        a.W_dt = W_dt; a.rT = rT; a.R = R; a.Rp = (R + 31) / 32 * 32;
    }
    char* ws = static_cast<char*>(p->workspace);
    const int groups = p->seqlen == 0 ? 1 : (slots(p) + 15) / 16;
    size_t ckpt_group = 0;
    // the repacked copy serves the scalar path only: the other kernels stage B and C through LDS instead
    auto stage = [&](const WsLayout& w) {
        a.Lp = w.Lp;
        if (a.dpp_ok) return true;
        if (ss::launch_stage_bc(a, ws + w.bcs_off, p->io_dtype, static_cast<hipStream_t>(stream)) != 0) return false;
        a.bcs = ws + w.bcs_off;
        return true;
    };
    if (p->flags & SS_SAVE_FOR_BWD) {
        const WsLayout w = ws_layout(p, true, pitch);
        if (stageable(p) && !stage(w)) return SS_ERR_LAUNCH;
        ckpt_group = w.ckpt_group;
        a.ckpt = reinterpret_cast<float*>(ws + w.ckpt_off);
        a.ysave = (p->flags & SS_HAS_Z) ? ws + w.y_off : nullptr;
        if (w.plan.nseg > 1) {
            a.nseg = w.plan.nseg; a.seg_len = w.plan.seg_len;
            a.seg_h = reinterpret_cast<float*>(ws + w.segh_off);
            a.seg_sumdt = reinterpret_cast<float*>(ws + w.segdt_off);
        }
    } else {
        // a plain forward call splits the sequence only if the caller lent the scratch for it
        const WsLayout w = ws_layout(p, false, pitch);
        const bool lent = ws && p->workspace_bytes >= w.total && aligned(ws, 256);
        if (stageable(p) && lent && !stage(w)) return SS_ERR_LAUNCH;
        if (groups > 1 && (p->flags & SS_HAS_Z)) a.ysave = ws + w.y_off;   // checked to be there
        if (w.plan.nseg > 1 && lent) {
            a.nseg = w.plan.nseg; a.seg_len = w.plan.seg_len;
            a.seg_h = reinterpret_cast<float*>(ws + w.segh_off);
            a.seg_sumdt = reinterpret_cast<float*>(ws + w.segdt_off);
        }
    }
    if (!W_dt && runs_whole(p, a)) {
        if (!(p->flags & SS_SAVE_FOR_BWD)) a.seg_sumdt = nullptr;
        return ss::launch_fwd_whole(a, p->io_dtype, static_cast<hipStream_t>(stream)) == 0 ? SS_OK : SS_ERR_LAUNCH;
    }
    // one pass per group of 16 states; the passes run in stream order and share the segment
    // buffers, each adds its C*h to the y of the ones before it
    for (int g = 0; g < groups; ++g) {
        ss::FwdArgs ag = a;
        if (groups > 1) narrow_to_group(ag, p, g, ckpt_group);
        if (ss::launch_fwd(ag, p->io_dtype, static_cast<hipStream_t>(stream)) != 0) return SS_ERR_LAUNCH;
    }
    return SS_OK;
}


int scan_fwd_strided(const ss_fwd_params* p, long bc_bstride, int pitch, void* stream)
{
    return scan_fwd_impl(p, bc_bstride, pitch, nullptr, 0, nullptr, stream);
}

size_t scan_workspace_bytes(const ss_fwd_params* p, int for_backward, int pitch)
{
    if (!p || p->batch < 1 || p->dim < 1 || p->seqlen < 0) return 0;
    // of the split plan, whether or not it pays: that depends on what a query need not give (SS_EXACT_ZOH_B)
    return ws_layout(p, for_backward != 0, pitch, plan_segments(p->batch, p->dim, split_steps(p, for_backward != 0))).total;
}

int scan_fwd_fused(const ss_fwd_params* p, long bc_bstride, int pitch, const void* W_dt, int R, const void* rT, void* stream)
{
    if (!W_dt || !rT) return SS_ERR_NULL;
    return scan_fwd_impl(p, bc_bstride, pitch, W_dt, R, rT, stream);
}

int scan_bwd_strided(const ss_bwd_params* p, long bc_bstride, int pitch, const BwdSide* side, void* stream)
{
    if (!p) return SS_ERR_NULL;
    if (!pitch_ok(&p->fwd, pitch)) return SS_ERR_UNSUPPORTED;
    const int rc = check_fwd(&p->fwd, true, pitch, bc_bstride == (long)slots(&p->fwd) * p->fwd.seqlen);
    if (rc != SS_OK) return rc;
    const ss_fwd_params* f = &p->fwd;
    const bool empty = f->seqlen == 0;
    if (!p->dA) return SS_ERR_NULL;
    if (!empty && (!p->dout || !p->du || !p->ddelta || !p->dB || !p->dC)) return SS_ERR_NULL;
    if (((f->flags & SS_B_FIXED) && !p->dB) || ((f->flags & SS_C_FIXED) && !p->dC)) return SS_ERR_NULL;
    if (!empty && (f->flags & SS_HAS_Z) && !p->dz) return SS_ERR_NULL;
    if ((f->flags & SS_HAS_D) && !p->dD) return SS_ERR_NULL;
    if ((f->flags & SS_HAS_DELTA_BIAS) && !p->ddelta_bias) return SS_ERR_NULL;
    const void* io[] = {p->dout, p->du, p->ddelta, p->dz};
    for (const void* q : io)
        if (q && !aligned(q, 16)) return SS_ERR_ALIGN;
    const void* f32[] = {p->dh_last, p->dB, p->dC, p->dA, p->dD, p->ddelta_bias, p->dh0};
    for (const void* q : f32)
        if (q && !aligned(q, 4)) return SS_ERR_ALIGN;

    const WsLayout w = ws_layout(f, true, pitch);
    char* ws = static_cast<char*>(f->workspace);
    ss::BwdArgs a{};
    a.f = make_fwd_args(f, bc_bstride, pitch);
    a.f.out = nullptr;
    a.f.h_last = nullptr;
    a.f.ckpt = reinterpret_cast<float*>(ws + w.ckpt_off);
    a.f.ysave = (f->flags & SS_HAS_Z) ? ws + w.y_off : nullptr;
    if (w.plan.nseg > 1) {
        a.f.nseg = w.plan.nseg; a.f.seg_len = w.plan.seg_len;
        a.f.seg_h = reinterpret_cast<float*>(ws + w.segh_off);
        a.f.seg_sumdt = reinterpret_cast<float*>(ws + w.segdt_off);
        a.seg_g = reinterpret_cast<float*>(ws + w.segg_off);
    }
    a.dout = p->dout; a.dh_last = p->dh_last;
    a.du = p->du; a.ddelta = p->ddelta; a.dz = (f->flags & SS_HAS_Z) ? p->dz : nullptr;
    a.dB = p->dB; a.dC = p->dC;
    a.dA_part = reinterpret_cast<float*>(ws + w.dA_off);
    a.dBf_part = reinterpret_cast<float*>(ws + w.dBf_off);
    a.dCf_part = reinterpret_cast<float*>(ws + w.dCf_off);
    a.dD_part = reinterpret_cast<float*>(ws + w.dD_off);
    a.db_part = reinterpret_cast<float*>(ws + w.db_off);
    a.dh0 = p->dh0;
    a.dA = p->dA;
    a.dD = (f->flags & SS_HAS_D) ? p->dD : nullptr;
    a.dbias = (f->flags & SS_HAS_DELTA_BIAS) ? p->ddelta_bias : nullptr;
    a.acc = 0;
    a.dbc_bstride = (long)slots(f) * f->seqlen;
    if (side) a.bc_cleared = side->bc_cleared;
    // one pass per group of 16 states, in stream order: each adds its share of du, ddelta and
    // dbias to the earlier ones' and writes its own slices of dA, dB, dC and dh0
    const int groups = (slots(f) + 15) / 16;
    for (int g = 0; g < groups; ++g) {
        ss::BwdArgs ag = a;
        if (groups > 1) {
            const int n0 = g * 16;
            narrow_to_group(ag.f, f, g, w.ckpt_group);
            ag.f.acc_y = 0;
            ag.acc = g > 0;
            ag.dh_last = at(ag.dh_last, n0);
            ag.dh0 = at(ag.dh0, n0);
            ag.dA = at(ag.dA, n0);
            ag.dB = at(ag.dB, (f->flags & SS_B_FIXED) ? (long)n0 : (long)n0 * f->seqlen);
            ag.dC = at(ag.dC, (f->flags & SS_C_FIXED) ? (long)n0 : (long)n0 * f->seqlen);
            if (g > 0) { ag.dz = nullptr; ag.dD = nullptr; }
        }
        if (side && g == groups - 1) {   // all of dB and dC are there
            ag.pack = side->pack; ag.pack_ld = side->pack_ld; ag.pack_bstride = side->pack_bstride;
            ag.pack_dB = p->dB; ag.pack_dC = p->dC;
        }
        if (ss::launch_bwd(ag, f->io_dtype, static_cast<hipStream_t>(stream)) != 0) return SS_ERR_LAUNCH;
    }
    return SS_OK;
}


static int step_impl(const ss_step_params* p, long bc_stride, const float* P, const void* W_dt, int R, int ldp, void* conv_state,
                     const void* x_t, void* stream)
{
    if (!p) return SS_ERR_NULL;
    if (p->batch < 1 || p->dim < 1 || p->dstate < 1) return SS_ERR_SHAPE;
    if (p->dstate > SS_MAX_DSTATE || slots(p) > SS_MAX_DSTATE) return SS_ERR_UNSUPPORTED;
    if ((p->flags & SS_COMPLEX_STATE) && (p->flags & SS_EXACT_ZOH_B)) return SS_ERR_UNSUPPORTED;
    if (p->io_dtype != SS_F32 && p->io_dtype != SS_BF16) return SS_ERR_UNSUPPORTED;
    if (p->flags & ~kStepFlags) return SS_ERR_UNSUPPORTED;
    if (!p->h || !p->u_t || !p->A || !p->out_t) return SS_ERR_NULL;
    if (!P && (!p->delta_t || !p->B_t || !p->C_t)) return SS_ERR_NULL;
    if ((p->flags & SS_HAS_Z) && !p->z_t) return SS_ERR_NULL;
    if ((p->flags & SS_HAS_D) && !p->Dskip) return SS_ERR_NULL;
    if ((p->flags & SS_HAS_DELTA_BIAS) && !p->delta_bias) return SS_ERR_NULL;
    if (!aligned(p->h, 16)) return SS_ERR_ALIGN;
    const size_t esz = p->io_dtype == SS_BF16 ? 2 : 4;
    const void* io[] = {p->u_t, p->delta_t, p->z_t, p->out_t};
    for (const void* q : io)
        if (q && !aligned(q, esz)) return SS_ERR_ALIGN;
    if (!P && (!aligned(p->B_t, (p->flags & SS_B_FIXED) ? 4 : esz) || !aligned(p->C_t, (p->flags & SS_C_FIXED) ? 4 : esz)))
        return SS_ERR_ALIGN;
    if (P && (!aligned(P, 16) || !aligned(W_dt, 16) || !aligned(p->h, 16))) return SS_ERR_ALIGN;
    const void* f32[] = {p->A, p->Dskip, p->delta_bias};
    for (const void* q : f32)
        if (q && !aligned(q, 4)) return SS_ERR_ALIGN;
    ss::StepArgs a{};
    a.B = p->batch; a.D = p->dim; a.N = slots(p); a.flags = p->flags;
    a.h = p->h; a.u_t = p->u_t; a.delta_t = p->delta_t; a.z_t = p->z_t;
    a.B_t = P ? nullptr : p->B_t; a.C_t = P ? nullptr : p->C_t; a.bc_stride = bc_stride;
    a.P = P; a.W_dt = W_dt; a.R = R; a.ldp = ldp; a.conv_state = conv_state; a.x_t = x_t; a.A = p->A; a.Dskip = p->Dskip; a.bias = p->delta_bias;
    a.out_t = p->out_t;
    if (P) return ss::launch_step_projected(a, p->io_dtype, static_cast<hipStream_t>(stream)) == 0 ? SS_OK : SS_ERR_LAUNCH;
    return ss::launch_step(a, p->io_dtype, static_cast<hipStream_t>(stream)) == 0 ? SS_OK : SS_ERR_LAUNCH;
}

int step_strided(const ss_step_params* p, long bc_stride, void* stream)
{
    return step_impl(p, bc_stride, nullptr, nullptr, 0, 0, nullptr, nullptr, stream);
}

int step_projected(const ss_step_params* p, const float* P, const void* W_dt, int R, int ldp, void* conv_state, const void* x_t,
                   void* stream)
{
    if (!p || !P || !W_dt) return SS_ERR_NULL;
    if (R < 8 || R > 256 || p->dstate > 16 || ldp != R + 2 * p->dstate) return SS_ERR_UNSUPPORTED;
    return step_impl(p, 0, P, W_dt, R, ldp, conv_state, x_t, stream);
}

}  // namespace ss

extern "C" {

size_t ss_workspace_bytes(const ss_fwd_params* p, int for_backward)
{
    return p ? ss::scan_workspace_bytes(p, for_backward, p->seqlen) : 0;
}

int ss_scan_fwd(const ss_fwd_params* p, void* stream)
{
    if (!p) return SS_ERR_NULL;
    return ss::scan_fwd_strided(p, (long)slots(p) * p->seqlen, p->seqlen, stream);
}

int ss_scan_fwd_static(const ss_fwd_params* p, void* stream)
{
    if (!p) return SS_ERR_NULL;
    if (p->flags & SS_SAVE_FOR_BWD) return SS_ERR_UNSUPPORTED;
    ss_fwd_params q = *p;
    q.workspace = nullptr;
    q.workspace_bytes = 0;
    // everything else is checked first, so that an invalid call reports its own error
    const int rc = check_fwd(&q, false, q.seqlen);
    if (rc != SS_OK && rc != SS_ERR_WORKSPACE) return rc;
    if (ws_layout(&q, false, q.seqlen).total > (size_t)SS_STATIC_SCRATCH_BYTES) return SS_ERR_WORKSPACE;
    void* ptr = nullptr;
    const int rs = static_scratch(&ptr);
    if (rs != SS_OK) return rs;
    q.workspace = ptr;
    q.workspace_bytes = SS_STATIC_SCRATCH_BYTES;
    return ss::scan_fwd_strided(&q, (long)slots(&q) * q.seqlen, q.seqlen, stream);
}

int ss_scan_bwd(const ss_bwd_params* p, void* stream)
{
    if (!p) return SS_ERR_NULL;
    return ss::scan_bwd_strided(p, (long)slots(&p->fwd) * p->fwd.seqlen, p->fwd.seqlen, nullptr, stream);
}

int ss_step(const ss_step_params* p, void* stream)
{
    if (!p) return SS_ERR_NULL;
    return ss::step_strided(p, slots(p), stream);
}

const char* ss_strerror(int code)
{
    switch (code) {
    case SS_OK: return "success";
    case SS_ERR_NULL: return "a required pointer is NULL";
    case SS_ERR_SHAPE: return "batch, dim and dstate must be >= 1 and seqlen >= 0";
    case SS_ERR_UNSUPPORTED: return "unsupported dstate, io_dtype or flag";
    case SS_ERR_ALIGN: return "a pointer is not aligned as required";
    case SS_ERR_WORKSPACE: return "workspace missing or too small";
    case SS_ERR_LAUNCH: return "the HIP runtime refused a kernel launch";
    case SS_ERR_BACKEND: return "backend failure (reserved; not returned by any current entry point)";
    default: return "unknown error code";
    }
}

int ss_version(void) { return 100; }

}  // extern "C"
