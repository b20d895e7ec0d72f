// Forward selective scan (Algorithm 2 steps 5-6, fused as in Appendix D "Speed") and the
// single-token recurrent step (Section 2, Eq. 2a/2b applied once).
#include <type_traits>

#include "ss_kernels.h"
#include "ss_device.h"

namespace ss {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));   // MFMA operand and accumulator types

// One workgroup = 64 rows x 4 waves.  Per chunk of CHUNK_T steps:
//   A. (pointwise view) load 64 rows x 32 steps of u, delta, z with 16-byte accesses, form
//      dt = softplus(delta + bias) and dt*u, park them in LDS;
//   B. (state view) wave w runs Eq. 2a/2b sequentially over the 32 steps for states
//      4w..4w+3 of its 64 rows, B and C arriving as scalar operands, and writes its
//      partial sum over those states of C*h to LDS;
//   C. (pointwise view) add the 4 partial sums, the skip term and the gate, and store.
// The state never leaves registers between chunks (Appendix D: the scan continues from
// the previous chunk's state).  Steps past the end of the sequence use dt = 0, which is
// the identity of the recurrence (abar = 1, input term 0).
//
// When the sequence is split into segments (blockIdx.y), the kernel runs twice: first with
// AGG = true on every segment but the last, from the zero state (segment 0: from h0),
// producing only the segment's end state and the sum of its step sizes; then, after
// carry_fwd_kernel has turned those into each segment's incoming state (with few segments every workgroup of the
// second run does that for itself, chain_segments), with AGG = false.
// ZOH selects the exact zero-order-hold B-bar of Eq. 4: the LDS tile that otherwise carries
// dt*u then carries u, and each state multiplies it by phi(dt, A) = (abar - 1) / A.
// BCFIX: bit 0 / bit 1 set when B / C is the time-invariant (D,N) float32 parameter of
// Algorithm 1 instead of the selective (B,N,L) tensor: it then sits in registers like A.
// CPLX: the lane's four state slots are two complex states (re, im) each (Section 3.6); only
// the recurrence and the read-out differ, everything around them sees 2N real "states".
// STAGED (rows of fewer than 8 or at least 2^23 steps, with a workspace): B and C come from the
// wave-packed copy a.bcs that stage_bc_kernel made: one scalar
// load per group instead of eight, one address per wave instead of eight clamped ones, so the
// scalar registers suffice for a whole group of prefetch and the scalar unit does little but
// widen bf16.  (Read in place, the eight loads of the next group compete with the current
// group's operands for scalar registers, some are issued only right before their use, and the
// wait for those drains the whole prefetch: the loads' latency shows once per group.)
// FUSED_KS > 0 (bf16, PAT, main pass of an unsplit sequence): delta_raw = W_dt r is not
// read but formed here, per chunk, as a 64 x 32 product over R <= 32 * FUSED_KS on the matrix
// cores: wave w owns rows 16w..16w+15 (its pieces of W_dt stay in registers for the whole
// kernel) and both 16-step halves of the chunk; the result goes through the dt tile in LDS to
// the pointwise threads, rounded to bf16 as the stored delta would be.  Saves the projection
// kernel and the write and read of a (B,D,L) tensor.
// SPL: slots per lane the recurrence is built for (4, or ceil(N / 4) rounded up to 1 or 2 when the
// states are dealt out to the waves in turn, FwdArgs::il).
// PAT (VEC, real state, selective B and C): B and C take neither scalar path.  The chunk's B and C are
// requested with the chunk's u, delta and z by ordinary buffer loads (thread -> B or C, state, group
// of four steps), widened to float and put into an LDS tile [group][state][step]; lane l of wave w
// reads, per group, one float4 with the state of slot l % 4 at the group's four steps, and the
// recurrence takes a state's value from that register as a quad-broadcast DPP operand
// (input_step_dpp, readout_step_dpp).  No scalar loads or their waits (which also drain LDS reads and
// vice versa), no repacking pass, no touching of cache lines ahead, and no vector-memory wait that
// has to cover the previous chunk's stores.
// RAG (PAT): rows of any length >= 8.  Slices are read in one access at element alignment, the
// one that reaches past the end from inside the row (row_piece), and shifted into place in the last chunk
// only; a partial slice is stored element by element.  Everything else is the aligned kernel's.  Such rows
// used to take the scalar path with one access per element: 8 x 1536 x 2047 in bf16, main + aggregate pass
// 309 + 139 -> 158 + 90 us (2048 steps: 137 + 86), backward 1632 + 385 -> 445 + 93 us (320 + 84); float32,
// 4 x 1536 x 2047, all passes: 865 -> 512 us.
template <typename T, bool VEC, bool FULLN, bool AGG, bool ZOH, int BCFIX = 0, bool CPLX = false, bool STAGED = false,
          int FUSED_KS = 0, int SPL = STATES_PER_LANE, bool PAT = false, bool RAG = false, bool SHORT = false, bool WAIT = true>
__global__ void __launch_bounds__(THREADS, PAT && AGG ? 4 : ((PAT && FUSED_KS <= 4) ? 2 : 1)) scan_fwd_kernel(const FwdArgs a)
{
    static_assert(!PAT || (VEC && BCFIX == 0 && !CPLX && !STAGED), "PAT: vector path, real state, selective B and C");
    static_assert(!RAG || PAT, "RAG: a form of the PAT kernel");
    constexpr int NGC = CHUNK_T / GROUP_T;
    __shared__ __attribute__((aligned(16))) float s_bc[PAT ? 2 : 1][PAT ? NGC : 1][PAT ? NPAD : 1][GROUP_T];   // PAT: B (0) and C (1) of the chunk
    __shared__ __attribute__((aligned(16))) float s_dt[ROWS][TPAD];
    __shared__ __attribute__((aligned(16))) float s_du[ROWS][TPAD];
    __shared__ __attribute__((aligned(16))) float s_yp[NWAVES][ROWS][TPAD];
    __shared__ __attribute__((aligned(16))) float s_raw[FUSED_KS > 0 ? ROWS : 1][TPAD];   // FUSED: delta_raw of the next chunk
    constexpr int RT_PITCH = 32 * (FUSED_KS > 0 ? FUSED_KS : 1) + 8;                     // bf16 elements; rows 16 bytes off the banks
    __shared__ __attribute__((aligned(16))) bf16_t s_rT[FUSED_KS > 0 ? CHUNK_T : 1][RT_PITCH];   // FUSED: r of the next chunk's steps

    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, provably uniform
    const int lane = tid & (WAVE - 1);
    const int groups = (a.D + ROWS - 1) / ROWS;
    // Workgroups go to the eight XCDs in turn by index; with this renumbering each XCD gets a contiguous
    // run of row groups, i.e. one batch entry's rows, whose shared operands (B, C, r) then meet in its L2.
    const unsigned bx = xcd_contiguous(blockIdx.x, gridDim.x);
    const int b = bx / groups;
    const int d0 = (bx % groups) * ROWS;
    const int L = a.L, N = a.N, NS = a.NS;
    const bool has_z = !AGG && (a.flags & F_HAS_Z), has_D = !AGG && (a.flags & F_HAS_D);
    const bool softplus = a.flags & F_DELTA_SOFTPLUS;
    const int seg = blockIdx.y;
    const int c_begin = seg * (a.seg_len / CHUNK_T);
    const int c_end = min((L + CHUNK_T - 1) / CHUNK_T, (seg + 1) * (a.seg_len / CHUNK_T));

    // ---- pointwise view: thread -> (row pr, slice pq) -----------------------------------
    // A slice is PC pieces of PE consecutive steps, one 16-byte access each (float with PC = 1, rows of any length and off the quad-broadcast kernels: two)
    constexpr int PC = PAT ? slice_pieces<T, RAG>() : 1, PE = SLICE / PC, PSTEP = CHUNK_T / PC;
    constexpr int HALF4 = PC == 2 ? PSTEP / 4 : 1;   // float4s from a slice's first four steps to its last four
    typedef slice_io<T, PC> pio;
    static_assert(!RAG || PC == 1, "rows of any length: a slice is one piece");
    const int pr = PC == 2 ? pointwise_row_pitch5(tid) : pointwise_row_pitch9(tid), pq = tid & 3;   // TPAD = 36 floats
    const bool p_ok = d0 + pr < a.D;
    const int pd = p_ok ? d0 + pr : a.D - 1;  // out-of-range rows shadow the last row; stores masked
    const long prow = (long)b * a.D + pd;
    const T* __restrict__ gu = static_cast<const T*>(a.u) + prow * L;
    const T* __restrict__ gdl = static_cast<const T*>(a.delta) + prow * L;
    const T* __restrict__ gz = static_cast<const T*>(a.z) + prow * L;  // not dereferenced without z
    T* __restrict__ gout = static_cast<T*>(a.out) + prow * L;
    const float bias = (a.flags & F_HAS_DELTA_BIAS) ? a.bias[pd] : 0.0f;
    const float Dsk = has_D ? a.Dskip[pd] : 0.0f;
    // VEC: buffer resources over this workgroup's rows of each tensor (a size of zero switches
    // an optional tensor off), so that the accesses in the loop are issued unconditionally
    const int rows_here = min(ROWS, a.D - d0);
    const long wg_first = ((long)b * a.D + d0) * L;
    const uint32_t wg_bytes = (uint32_t)rows_here * (uint32_t)L * (uint32_t)sizeof(T);
    const uint32_t row_off = (uint32_t)pr * (uint32_t)L * (uint32_t)sizeof(T);   // past the resource for rows past D
    const bool keep_y = !AGG && has_z && a.ysave;
    const rsrc_t bu = make_rsrc(static_cast<const T*>(a.u) + wg_first, wg_bytes);
    const rsrc_t bd = make_rsrc(static_cast<const T*>(a.delta) + wg_first, wg_bytes);
    const rsrc_t bz = make_rsrc(static_cast<const T*>(has_z ? a.z : a.u) + wg_first, has_z ? wg_bytes : 0u);
    const rsrc_t bo = make_rsrc(static_cast<T*>(AGG ? const_cast<void*>(a.u) : a.out) + wg_first, AGG ? 0u : wg_bytes);
    const rsrc_t by = make_rsrc(static_cast<T*>(keep_y ? a.ysave : const_cast<void*>(a.u)) + wg_first, keep_y ? wg_bytes : 0u);
    // what the earlier state groups left (more than 16 states): prefetched like an input, so that no wait in the loop has to drain the memory pipeline
    const bool acc_on = !AGG && a.acc_y;
    const rsrc_t bp = make_rsrc(static_cast<const T*>(acc_on ? (has_z ? a.ysave : a.out) : a.u) + wg_first, acc_on ? wg_bytes : 0u);
    // PAT staging view: waves 0, 1 stage B, waves 2, 3 stage C (not needed for the aggregates);
    // thread -> (state s_n, group of four steps s_tq) of the chunk
    const int s_which = w >> 1, s_n = (tid >> 3) & (NPAD - 1), s_tq = tid & (NGC - 1);
    const bool s_on = PAT && !(AGG && s_which == 1);
    const rsrc_t bbc = make_rsrc(static_cast<const T*>(s_which ? a.Cm : a.Bm) + (long)b * a.bc_bstride,
                                 s_on ? (uint32_t)N * (uint32_t)L * (uint32_t)sizeof(T) : 0u);
    const uint32_t bc_row_off = s_n < N ? (uint32_t)s_n * (uint32_t)L * (uint32_t)sizeof(T) : BUF_OFF;
    // RAG: plain pointers to the workgroup's first row and offsets of this thread's row, clamped to a valid one
    const uint32_t esz = (uint32_t)sizeof(T);
    const int r_row = min(pr, rows_here - 1);
    const uint32_t r_off = (uint32_t)r_row * (uint32_t)L * esz;
    // ... u, delta, ysave and B, C have rows of their own (FwdArgs::Li)
    constexpr bool OWN = own_rows<T, RAG, ZOH>();
    const int Li = OWN ? a.Li : L;
    const uint32_t r_off_bc = (uint32_t)min(s_n, N - 1) * (uint32_t)(OWN ? a.Lb : L) * esz;
    const long wg_first_i = ((long)b * a.D + d0) * Li;
    const uint32_t r_off_i = (uint32_t)r_row * (uint32_t)Li * esz, r_off_p = has_z ? r_off_i : r_off;
    const T* const ru_p = static_cast<const T*>(a.u) + wg_first_i;
    const T* const rd_p = static_cast<const T*>(a.delta) + wg_first_i;
    const T* const rz_p = has_z ? static_cast<const T*>(a.z) + wg_first : ru_p;
    const T* const rp_p = !acc_on ? ru_p : (has_z ? static_cast<const T*>(a.ysave) + wg_first_i : static_cast<const T*>(a.out) + wg_first);
    const T* const rbc_p = static_cast<const T*>(s_which ? a.Cm : a.Bm) + (long)b * a.bc_bstride;

    // ---- state view: lane -> row, wave -> states 4w..4w+3 -------------------------------
    const bool s_ok = d0 + lane < a.D;
    const int sd = s_ok ? d0 + lane : a.D - 1;
    const long srow = (long)b * a.D + sd;
    constexpr bool BFIX = BCFIX & 1, CFIX = BCFIX & 2;
    float A2[STATES_PER_LANE], An[STATES_PER_LANE], invA[STATES_PER_LANE], h[STATES_PER_LANE];
    float Bf[STATES_PER_LANE], Cf[STATES_PER_LANE];
    const T* __restrict__ gB[STATES_PER_LANE];
    const T* __restrict__ gC[STATES_PER_LANE];
    bool n_ok[STATES_PER_LANE];
    // the incoming state is worked out here from the aggregates of the segments before (see chain_segments)
    const bool chained = PAT && !AGG && FUSED_KS == 0 && a.nseg <= CARRY_INLINE;
#pragma unroll
    for (int k = 0; k < STATES_PER_LANE; ++k) {
        const int n = slot_state(w, k, a.il);
        n_ok[k] = n < N && k < SPL;
        const int nc = n_ok[k] ? n : 0;
        An[k] = n_ok[k] ? a.A[(long)sd * NS + nc] : 0.0f;
        A2[k] = An[k] * LOG2E;
        invA[k] = An[k] != 0.0f ? 1.0f / An[k] : 0.0f;
        if (seg == 0) h[k] = (n_ok[k] && (a.flags & F_HAS_H0)) ? a.h0[srow * NS + nc] : 0.0f;
        else h[k] = AGG || chained ? 0.0f : a.seg_h[((long)seg * a.B * a.D + srow) * NPAD + w * STATES_PER_LANE + k];
        gB[k] = BFIX ? nullptr : static_cast<const T*>(a.Bm) + (long)b * a.bc_bstride + (long)nc * L;
        gC[k] = CFIX ? nullptr : static_cast<const T*>(a.Cm) + (long)b * a.bc_bstride + (long)nc * L;
        Bf[k] = (BFIX && n_ok[k]) ? static_cast<const float*>(a.Bm)[(long)sd * NS + nc] : 0.0f;
        Cf[k] = (CFIX && n_ok[k]) ? static_cast<const float*>(a.Cm)[(long)sd * NS + nc] : 0.0f;
    }
    if constexpr (PAT && !AGG && FUSED_KS == 0) {
        if (chained && seg > 0) {
            const long rows = (long)a.B * a.D;
            const f32x4_t c = chain_segments(
                seg, A2, [&](int s) { return *(reinterpret_cast<const f32x4_t*>(a.seg_h + (s * rows + srow) * NPAD) + w); },
                [&](int s) { return a.seg_sumdt[s * rows + srow]; });
#pragma unroll
            for (int k = 0; k < STATES_PER_LANE; ++k) h[k] = c[k];
        }
    }
    // staged B and C: this wave's pieces, one per group of steps, consecutive in memory
    const T* __restrict__ const sbc =
        STAGED ? static_cast<const T*>(a.bcs) + (((long)b * ((NS + NPAD - 1) / NPAD * NWAVES) + w) * (a.Lp / GROUP_T)) * STAGE_GROUP
               : nullptr;
    // the selective operands (if any) whose cache lines are touched one chunk ahead
    const void* const touchB = BFIX ? a.Cm : a.Bm;
    const void* const touchC = CFIX ? a.Bm : a.Cm;
    // staged: the wave's pieces of a chunk are contiguous; a lane touches every 16th element
    const rsrc_t bt = make_rsrc(sbc, STAGED ? (uint32_t)(a.Lp / GROUP_T) * STAGE_GROUP * (uint32_t)sizeof(T) : 0u);
    auto touch = [&](int t) -> uint32_t {
        if constexpr (STAGED) {   // an unconditional buffer load; lanes with nothing to touch are out of range
            constexpr int per_chunk = CHUNK_T / GROUP_T * STAGE_GROUP;
            const bool on = lane * 16 < per_chunk && t >= 0 && t < a.Lp;
            const uint32_t off = on ? (uint32_t)((t / GROUP_T) * STAGE_GROUP + lane * 16) * (uint32_t)sizeof(T) : BUF_OFF;
            return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(bt, (int)off, 0, 0);
        } else {
            return touch_bc<T>(touchB, touchC, b, a.bc_bstride, N, L, w, lane, t);
        }
    };
    float sum_dt = 0.0f;  // AGG: this thread's share of the segment's sum of step sizes

    // FUSED: operand fragments of the 16x16x32 bf16 MFMA.  Lane l holds row (column) l % 16 of
    // the first (second) operand at contraction indices 8 * (l / 16) ..+7 of each 32-wide step;
    // accumulator element i of lane l is row 4 * (l / 16) + i, column l % 16.
    constexpr int KS = FUSED_KS > 0 ? FUSED_KS : 1;
    union Frag { unsigned short s[8]; bf16x8_t v; };
    Frag wfr[KS];
    constexpr int RLD = (KS + 1) / 2;          // 16-byte pieces of the chunk's r per thread: 32 steps x Rp / 256 threads
    Frag rld[RLD];
    const int fsub = 8 * (lane >> 4);
    const int rt_t = tid >> 3, rt_col = (tid & 7) * 4 * KS;   // this thread's piece of the (32 steps, Rp) tile
    if constexpr (FUSED_KS > 0) {
        const bf16_t* wp = static_cast<const bf16_t*>(a.W_dt) + (long)min(d0 + 16 * w + (lane & 15), a.D - 1) * a.R;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int k = 32 * ks + fsub;
            wfr[ks].v = *reinterpret_cast<const bf16x8_t*>(wp + min(k, a.R - 8));   // R is a multiple of 8
            if (k >= a.R) {
#pragma unroll
                for (int e = 0; e < 8; ++e) wfr[ks].s[e] = 0;
            }
        }
    }
    // u, delta and z are requested PF chunks ahead (slot = chunk index mod PF): the scan is not long
    // enough to cover a memory round trip under load, and with one chunk in flight per workgroup
    // the kernel ran at the pace of that latency whatever the state size.
    constexpr int PF = VEC ? 2 : 1;
    typename pio::raw ru_[PF][PC], rd_[PF][PC], rz_[PF][PC];
    typename io4<T>::raw rbc_[PF];   // PAT: the thread's four steps of B or C
    typename pio::raw rp_[PF][PC];   // VEC: the pre-gate y of the earlier state groups (zeros if there are none)
    auto issue_loads = [&](int c, auto slot_tag) {   // chunk c into the slot given at compile time
        constexpr int s = decltype(slot_tag)::value;
        if constexpr (RAG) {   // past the segment's end: its last chunk again (never used)
            const int cc = min(c, c_end - 1) * CHUNK_T;
            const uint32_t t = (uint32_t)row_piece(cc + pq * SLICE, SLICE, L) * esz;
            ru_[s][0] = pio::load_elem(ru_p, r_off_i + t);
            if constexpr (FUSED_KS == 0) rd_[s][0] = pio::load_elem(rd_p, r_off_i + t);
            if constexpr (!AGG) {
                rz_[s][0] = pio::load_elem(rz_p, has_z ? r_off + t : 0u);
                rp_[s][0] = pio::load_elem(rp_p, acc_on ? r_off_p + t : 0u);
            }
            rbc_[s] = io4<T>::load_elem(rbc_p, r_off_bc + (uint32_t)row_piece(cc + s_tq * GROUP_T, GROUP_T, L) * esz);
        } else if constexpr (VEC) {   // pieces are whole or empty
#pragma unroll
            for (int p = 0; p < PC; ++p) {
                const int t = c * CHUNK_T + p * PSTEP + pq * PE;
                const uint32_t off = (t < L && c < c_end) ? row_off + (uint32_t)t * (uint32_t)sizeof(T) : BUF_OFF;
                ru_[s][p] = pio::load_buf(bu, off);
                if constexpr (FUSED_KS == 0) rd_[s][p] = pio::load_buf(bd, off);
                if constexpr (!AGG) {
                    rz_[s][p] = pio::load_buf(bz, off);
                    rp_[s][p] = pio::load_buf(bp, off);
                }
            }
            if constexpr (PAT) {   // L % 8 == 0: a group of four steps is whole or past the end
                const int ts = c * CHUNK_T + s_tq * GROUP_T;
                rbc_[s] = io4<T>::load_buf(bbc, (ts < L && c < c_end) ? bc_row_off + (uint32_t)ts * (uint32_t)sizeof(T) : BUF_OFF);
            }
        } else {
            const int t0 = c * CHUNK_T + pq * SLICE;
            ru_[s][0] = load_slice8<T, VEC, SHORT>(gu, t0, L, true);
            rd_[s][0] = load_slice8<T, VEC, SHORT>(gdl, t0, L, true);
            if (has_z) rz_[s][0] = load_slice8<T, VEC, SHORT>(gz, t0, L, true);
        }
    };
    // FUSED: delta_raw of a chunk from the fragments in registers: two 16 x 16 tiles per wave,
    // into rows 16w..16w+15 of s_raw -- the rows this wave's own pointwise threads read, so the
    // exchange needs no workgroup barrier (a wave's LDS instructions execute in order).  Called
    // for the next chunk after the recurrence, where the matrix-core latency hides behind the
    // pointwise post-processing.
    auto project = [&]() {
        if constexpr (FUSED_KS > 0) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // earlier reads of s_raw are done
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    if (32 * ks < a.Rp) {
                        const bf16x8_t rv = *reinterpret_cast<const bf16x8_t*>(&s_rT[16 * nt + (lane & 15)][32 * ks + fsub]);
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wfr[ks].v, rv, acc, 0, 0, 0);
                    }
#pragma unroll
                for (int i = 0; i < 4; ++i) s_raw[16 * w + 4 * (lane >> 4) + i][16 * nt + (lane & 15)] = acc[i];
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    };
    // FUSED: r of a chunk's 32 steps (transposed and padded, so always in range) is read once per
    // workgroup, two chunks ahead into registers, one chunk ahead into LDS
    auto issue_r = [&](int c) {
        if constexpr (FUSED_KS > 0) {
            const bf16_t* rp = static_cast<const bf16_t*>(a.rT) + ((long)b * a.Lp + min(max(c, 0) * CHUNK_T, a.Lp - CHUNK_T) + rt_t) * a.Rp;
#pragma unroll
            for (int j = 0; j < RLD; ++j)
                rld[j].v = *reinterpret_cast<const bf16x8_t*>(rp + min(rt_col + 8 * j, a.Rp - 8));
        }
    };
    auto stage_r = [&]() {   // this thread's piece of the chunk's r, from registers to LDS
        if constexpr (FUSED_KS > 0) {
#pragma unroll
            for (int j = 0; j < RLD; ++j)
                if (rt_col + 8 * j < a.Rp) *reinterpret_cast<bf16x8_t*>(&s_rT[rt_t][rt_col + 8 * j]) = rld[j].v;
        }
    };
    // The wait the compiler puts before a chunk's first use of its inputs allows as many memory
    // operations in flight as the shortest path into that point issues after them.  The way in from
    // here must not be that path, or every iteration would drain the stores it has just issued: the
    // first chunk's requests go out first and stay in that order.
    issue_loads(c_begin, std::integral_constant<int, 0>{});
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (PF > 1) issue_loads(c_begin + 1, std::integral_constant<int, 1>{});
    __builtin_amdgcn_sched_barrier(0);
    // PAIR (16-bit elements): a 32-step chunk is 64 bytes of a row, half a 128-byte line.  Writes of
    // half lines reach about half the throughput of whole lines (and reads somewhat less than whole
    // ones), so the traffic of an even chunk and the odd one after it (segments start at even
    // chunks) is issued together: both chunks' inputs are requested in the odd chunk's phase A, tensor
    // by tensor, and the even chunk's results wait in registers for the odd chunk's.  A float chunk is a whole
    // line: its inputs are better requested one by one (8 x 2048 x 4096 forward 293 us, in pairs 306), its results
    // wait where that pays (WAIT, see choose_waits).
    constexpr bool PAIR = PAT && sizeof(T) == 2;
    auto issue_pair = [&](int c0) {   // chunks c0 (slot 0) and c0 + 1 (slot 1)
      if constexpr (PAIR && RAG) {
        uint32_t t[2], tb[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int cc = min(c0 + s, c_end - 1) * CHUNK_T;
            t[s] = (uint32_t)row_piece(cc + pq * SLICE, SLICE, L) * esz;
            tb[s] = r_off_bc + (uint32_t)row_piece(cc + s_tq * GROUP_T, GROUP_T, L) * esz;
        }
        ru_[0][0] = io8<T>::load_elem(ru_p, r_off_i + t[0]); ru_[1][0] = io8<T>::load_elem(ru_p, r_off_i + t[1]);
        if constexpr (FUSED_KS == 0) { rd_[0][0] = io8<T>::load_elem(rd_p, r_off_i + t[0]); rd_[1][0] = io8<T>::load_elem(rd_p, r_off_i + t[1]); }
        if constexpr (!AGG) {
            rz_[0][0] = io8<T>::load_elem(rz_p, has_z ? r_off + t[0] : 0u); rz_[1][0] = io8<T>::load_elem(rz_p, has_z ? r_off + t[1] : 0u);
            rp_[0][0] = io8<T>::load_elem(rp_p, acc_on ? r_off_p + t[0] : 0u); rp_[1][0] = io8<T>::load_elem(rp_p, acc_on ? r_off_p + t[1] : 0u);
        }
        rbc_[0] = io4<T>::load_elem(rbc_p, tb[0]); rbc_[1] = io4<T>::load_elem(rbc_p, tb[1]);
      } else if constexpr (PAIR) {
        uint32_t off[2], boff[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int c = c0 + s;
            const int t0 = c * CHUNK_T + pq * SLICE;
            off[s] = (t0 + SLICE <= L && c < c_end) ? row_off + (uint32_t)t0 * (uint32_t)sizeof(T) : BUF_OFF;
            const int ts = c * CHUNK_T + s_tq * GROUP_T;
            boff[s] = (ts < L && c < c_end) ? bc_row_off + (uint32_t)ts * (uint32_t)sizeof(T) : BUF_OFF;
        }
        ru_[0][0] = io8<T>::load_buf(bu, off[0]); ru_[1][0] = io8<T>::load_buf(bu, off[1]);
        if constexpr (FUSED_KS == 0) { rd_[0][0] = io8<T>::load_buf(bd, off[0]); rd_[1][0] = io8<T>::load_buf(bd, off[1]); }
        if constexpr (!AGG) {
            rz_[0][0] = io8<T>::load_buf(bz, off[0]); rz_[1][0] = io8<T>::load_buf(bz, off[1]);
            rp_[0][0] = io8<T>::load_buf(bp, off[0]); rp_[1][0] = io8<T>::load_buf(bp, off[1]);
        }
        rbc_[0] = io4<T>::load_buf(bbc, boff[0]); rbc_[1] = io4<T>::load_buf(bbc, boff[1]);
      }
    };
    typename pio::packed held_y[PC]{}, held_o[PC]{};
    if constexpr (FUSED_KS > 0) {
        issue_r(c_begin);
        stage_r();
        __syncthreads();
        project();
        __syncthreads();   // s_rT is rewritten in the first chunk's phase A
        issue_r(c_begin + 1);
    }
    uint32_t touched = 0u;
    if (BCFIX != 3 && !PAT) touched = touch(c_begin * CHUNK_T);

    // One chunk; the slot of its prefetched inputs (chunk index from c_begin, mod PF) is a compile-time
    // constant, so the prefetch registers are addressed statically and the loads just issued are
    // not touched again before their chunk comes up.
    auto do_chunk = [&](const int c, auto slot_tag) {
        constexpr int SLOT = decltype(slot_tag)::value;
        float u8[SLICE], z8[SLICE], v8[SLICE];
        const int tc = c * CHUNK_T;
        const int t0 = tc + pq * PE;
        int nv[PC];   // steps of each piece inside the row
#pragma unroll
        for (int p = 0; p < PC; ++p) nv[p] = min(max(L - t0 - p * PSTEP, 0), PE);
        // ---- A: pointwise pre-processing --------------------------------------------
        typename pio::raw ru[PC], rd[PC], rz[PC];
#pragma unroll
        for (int p = 0; p < PC; ++p) { ru[p] = ru_[SLOT][p]; rd[p] = rd_[SLOT][p]; rz[p] = rz_[SLOT][p]; }
        typename io4<T>::raw rbc = rbc_[SLOT];
        if constexpr (RAG) {
            if (tc + CHUNK_T > L) {   // uniform: the last chunk of a row that does not fill it
                const int sh = t0 - row_piece(t0, SLICE, L), ts = tc + s_tq * GROUP_T;
                pio::drop(ru[0], sh);
                if constexpr (FUSED_KS == 0) pio::drop(rd[0], sh);
                if constexpr (!AGG) pio::drop(rz[0], sh);
                if (acc_on) pio::drop(rp_[SLOT][0], sh);
                io4<T>::drop(rbc, ts - row_piece(ts, GROUP_T, L));
            }
        }
        float p8[SLICE];
        if constexpr (VEC) {
            if (acc_on) unpack_slice<pio, PC>(rp_[SLOT], p8);   // uniform: only with more than 16 states
        }
        if constexpr (PAT) {
            float bc4[GROUP_T];
            io4<T>::unpack(rbc, bc4);
            if constexpr (RAG) {   // slots without a state
#pragma unroll
                for (int j = 0; j < GROUP_T; ++j) bc4[j] = s_n < N ? bc4[j] : 0.0f;
            }
            *reinterpret_cast<float4*>(&s_bc[s_which][s_tq][s_n][0]) = make_float4(bc4[0], bc4[1], bc4[2], bc4[3]);
        }
        unpack_slice<pio, PC>(ru, u8);
        if constexpr (FUSED_KS > 0) {   // delta_raw of this chunk: left in s_raw by this same wave (project)
            const float4 d0v = *reinterpret_cast<const float4*>(&s_raw[pr][pq * SLICE]);
            const float4 d1v = *reinterpret_cast<const float4*>(&s_raw[pr][pq * SLICE + 4]);
            const float raw[SLICE] = {d0v.x, d0v.y, d0v.z, d0v.w, d1v.x, d1v.y, d1v.z, d1v.w};
#pragma unroll
            for (int j = 0; j < SLICE; ++j) v8[j] = bf16_to_f32(bf16_t(f32_to_bf16_bits(raw[j])));   // as the stored delta would be
        } else {
            unpack_slice<pio, PC>(rd, v8);
        }
        if (has_z) unpack_slice<pio, PC>(rz, z8);
        {
            float dt8[SLICE], du8[SLICE];
            // PAT without the in-kernel projection: a piece is whole or empty, and an empty one was read as
            // zeros; a bias of -1e30 (0 without softplus) then makes its step sizes exactly 0, the identity of
            // the recurrence, without a select per element
            constexpr bool ZERO_BY_BIAS = PAT && FUSED_KS == 0 && !RAG;
            float bias_e[PC];   // selected here: inside the loop the select is made again in front of every softplus
#pragma unroll
            for (int p = 0; p < PC; ++p) bias_e[p] = !ZERO_BY_BIAS || nv[p] == PE ? bias : (softplus ? -1e30f : 0.0f);
#pragma unroll
            for (int j = 0; j < SLICE; ++j) {
                float sp = v8[j] + bias_e[j / PE];
                if (softplus) sp = ss::softplus(sp);
                if constexpr (!ZERO_BY_BIAS) sp = (j % PE < nv[j / PE]) ? sp : 0.0f;
                dt8[j] = sp;
                du8[j] = ZOH ? u8[j] : sp * u8[j];
                if (AGG) sum_dt += sp;
            }
            float4* const pd4 = reinterpret_cast<float4*>(&s_dt[pr][pq * PE]);   // four steps each
            float4* const pu4 = reinterpret_cast<float4*>(&s_du[pr][pq * PE]);
            pd4[0] = make_float4(dt8[0], dt8[1], dt8[2], dt8[3]);
            pd4[HALF4] = make_float4(dt8[4], dt8[5], dt8[6], dt8[7]);
            pu4[0] = make_float4(du8[0], du8[1], du8[2], du8[3]);
            pu4[HALF4] = make_float4(du8[4], du8[5], du8[6], du8[7]);
        }
        // The touch of the next chunk's B and C goes here, after the wait for this chunk's u,
        // delta and z: the value touched a chunk ago is older than those and costs no wait of
        // its own.
        if constexpr (!PAT) {
            consume_touch(touched);
            if (BCFIX != 3) touched = touch((c + 1) * CHUNK_T);
        }
        // checkpoint: the state entering every CKPT_T-step block (read back by the backward pass)
        auto save_ckpt = [&](int block) {
            if constexpr (AGG) return;
            if constexpr (VEC) {   // the block's 64 rows x 16 states; nothing is written if there is no block or no buffer
                const bool on = a.ckpt && block * CKPT_T < L;
                const rsrc_t bc = make_rsrc(a.ckpt + (((long)block * a.B + b) * a.D + d0) * NPAD,
                                            on ? (uint32_t)rows_here * NPAD * (uint32_t)sizeof(float) : 0u);
                buf_store16(bc, (uint32_t)(lane * NPAD + w * STATES_PER_LANE) * (uint32_t)sizeof(float),
                            make_uint4(__float_as_uint(h[0]), __float_as_uint(h[1]), __float_as_uint(h[2]), __float_as_uint(h[3])));
            } else if (a.ckpt && s_ok && block * CKPT_T < L) {
                float4* ck = reinterpret_cast<float4*>(a.ckpt + (((long)block * a.B + b) * a.D + sd) * NPAD) + w;
                *ck = make_float4(h[0], h[1], h[2], h[3]);
            }
        };
        save_ckpt(c * (CHUNK_T / CKPT_T));
        if constexpr (PAIR) {
            if constexpr (SLOT == 1) issue_pair(c + 1);
        } else {
            if (VEC || c + PF < c_end) issue_loads(c + PF, slot_tag);  // in flight during the scans below (VEC: switched off past the end, not branched around)
        }
        if constexpr (FUSED_KS > 0) {
            stage_r();          // r of chunk c + 1, requested a chunk ago; read by project() after the recurrence
            issue_r(c + 2);
        }
        __syncthreads();
        // ---- B: sequential recurrence over the chunk ---------------------------------
        __builtin_amdgcn_s_setprio(2);   // raised wave priority for the recurrence (see scan_bwd_kernel)
        constexpr int NG = CHUNK_T / GROUP_T;
        bc_group<T> Bg[2][STATES_PER_LANE], Cg[2][STATES_PER_LANE];
        constexpr int FB = 1;            // staged: groups fetched together (two gain nothing and spill scalar registers)
        bcs_group<T> Sg[2 * FB];
        const T* __restrict__ const sbc_chunk = STAGED ? sbc + (long)(tc / GROUP_T) * STAGE_GROUP : nullptr;
        auto fetch_bc = [&](int g, int slot) {
            if constexpr (PAT) {
                return;
            } else if constexpr (STAGED) {
                Sg[slot] = load_bcs<T>(sbc_chunk + g * STAGE_GROUP);
            } else {
#pragma unroll
                for (int k = 0; k < STATES_PER_LANE; ++k) {
                    if (!BFIX) Bg[slot][k] = load_bc<T, VEC, !FULLN, SHORT>(gB[k], tc + g * GROUP_T, L, n_ok[k]);
                    if (!CFIX && !AGG) Cg[slot][k] = load_bc<T, VEC, !FULLN, SHORT>(gC[k], tc + g * GROUP_T, L, n_ok[k]);
                }
            }
        };
        auto Bval = [&](int slot, int k, int j) -> float {
            if constexpr (STAGED) return Sg[slot].B(k, j); else return BFIX ? Bf[k] : Bg[slot][k].get(j);
        };
        auto Cval = [&](int slot, int k, int j) -> float {
            if constexpr (STAGED) return Sg[slot].C(k, j); else return CFIX ? Cf[k] : Cg[slot][k].get(j);
        };
        // Scalar loads return out of order and share their counter with LDS reads, so a wait
        // for either drains both: the step sizes of the whole chunk are read from LDS before
        // the loop, and inside it only the scalar loads of the next group are outstanding.
        float4 dtc[NG], duc[NG], Bpc[PAT ? NG : 1], Cpc[PAT ? NG : 1];
        const int pat = slot_state(w, lane & 3, a.il);   // PAT: the state of slot lane % 4
        auto read_group = [&](int g) {
            dtc[g] = *reinterpret_cast<const float4*>(&s_dt[lane][g * GROUP_T]);
            duc[g] = *reinterpret_cast<const float4*>(&s_du[lane][g * GROUP_T]);
            if constexpr (PAT) {
                Bpc[g] = *reinterpret_cast<const float4*>(&s_bc[0][g][pat][0]);
                if (!AGG) Cpc[g] = *reinterpret_cast<const float4*>(&s_bc[1][g][pat][0]);
            }
        };
        // The aggregate pass has little LDS and nothing but the recurrence, so it runs four waves per SIMD: a group
        // is read one ahead, and the barrier below keeps the scheduler from starting every later group early
        // (which took all 256 or 512 registers, spills included, and one or two waves per SIMD).  The float main
        // pass, whose inputs take twice the registers, spills up to 20 otherwise (4 x 1536 x 2047, forward +
        // backward: 448 -> 422 us); the bf16 one does not, and gains nothing.
        constexpr bool LEAN = PAT && (AGG || sizeof(T) == 4);
        // The read-outs of a group of steps together (readout_group_dpp) and B dt u from the matrix cores (input_step_mfma):
        // forward 357 -> 345 us at 8 x 4096 x 2048 bf16; layer prefill 4 x 4096 x 1531 281 -> 269.  The kernel that
        // forms delta itself has no registers for either (layer training 8 x 4096 x 2048: 1515 -> 1560 us).
        constexpr bool GROUP_OUT = PAT && !AGG && SPL == 4 && FUSED_KS == 0;
        if constexpr (LEAN) {
            read_group(0);
        } else {
#pragma unroll
            for (int g = 0; g < NG; ++g) read_group(g);
        }
        if constexpr (STAGED) {
#pragma unroll
            for (int i = 0; i < FB; ++i) fetch_bc(i, i);
        } else {
            fetch_bc(0, 0);
        }
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int cur = STAGED ? g % (2 * FB) : (g & 1);
            if constexpr (!STAGED) {
                if (g + 1 < NG) fetch_bc(g + 1, cur ^ 1);  // in flight while group g is consumed
            }
            const int tl = g * GROUP_T;  // step within the chunk
            if constexpr (LEAN) {
                __builtin_amdgcn_sched_barrier(0);
                if (g + 1 < NG) read_group(g + 1);
            }
            const float4 dt4 = dtc[g], du4 = duc[g];
            if (g > 0 && tl % CKPT_T == 0) save_ckpt((tc + tl) / CKPT_T);
            float yp[GROUP_T], hq[GROUP_T][STATES_PER_LANE];
#pragma unroll
            for (int j = 0; j < GROUP_T; ++j) {
                const float dt = f4_get(dt4, j), du = f4_get(du4, j);
                float y = 0.0f;
                if constexpr (CPLX) {
#pragma unroll
                    for (int k = 0; k < STATES_PER_LANE; k += 2) {
                        const cplx ab = complex_decay(dt, A2[k], An[k + 1]);         // Eq. 4 over C
                        const float br = du * Bval(cur, k, j);
                        const float bi = du * Bval(cur, k + 1, j);
                        const float hr = fmaf(ab.re, h[k], fmaf(-ab.im, h[k + 1], br));  // Eq. 2a over C
                        const float hi = fmaf(ab.im, h[k], fmaf(ab.re, h[k + 1], bi));
                        h[k] = hr;
                        h[k + 1] = hi;
                        if (!AGG) {                                                  // Re(C h)
                            y = fmaf(Cval(cur, k, j), hr, y);
                            y = fmaf(-Cval(cur, k + 1, j), hi, y);
                        }
                    }
                } else if constexpr (PAT) {
                    float bu[STATES_PER_LANE];
                    if constexpr (FUSED_KS == 0) input_step_mfma<SPL>(bu, f4_get(Bpc[g], j), du);
                    else input_step_dpp<SPL>(bu, f4_get(Bpc[g], j), du);
#pragma unroll
                    for (int k = 0; k < SPL; ++k) {
                        const float x2 = dt * A2[k];
                        const float abar = exp2_fast(x2);                            // Eq. 4
                        if (ZOH) bu[k] *= zoh_phi_fast(dt, x2, abar, invA[k]);
                        h[k] = fmaf(abar, h[k], bu[k]);                              // Eq. 2a
                    }
                    if constexpr (!AGG && !GROUP_OUT) readout_step_dpp<SPL>(y, f4_get(Cpc[g], j), h);        // Eq. 2b
                    if constexpr (GROUP_OUT) {
#pragma unroll
                        for (int k = 0; k < SPL; ++k) hq[j][k] = h[k];
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < SPL; ++k) {
                        const float abar = exp2_fast(dt * A2[k]);                    // Eq. 4
                        float bu = du * Bval(cur, k, j);
                        if (ZOH) bu *= zoh_phi(dt, An[k], invA[k], abar, false).phi;
                        h[k] = fmaf(abar, h[k], bu);                                 // Eq. 2a
                        if (!AGG) y = fmaf(Cval(cur, k, j), h[k], y);                         // Eq. 2b
                    }
                }
                yp[j] = y;
                if constexpr (STAGED) {
                    // The next group's load is issued after this group's first step, i.e. after
                    // the wait for this group's own operands, so that that wait does not drain
                    // it; the scheduling barriers keep the compiler from moving it either way.
                    if (j == 0 && g % FB == 0 && g + FB < NG) {
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int i = 0; i < FB; ++i) fetch_bc(g + FB + i, (g + FB + i) % (2 * FB));
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            if constexpr (GROUP_OUT) readout_group_dpp(yp, Cpc[g], hq);              // Eq. 2b
            if (!AGG)
                *reinterpret_cast<float4*>(&s_yp[w][lane][tl]) = make_float4(yp[0], yp[1], yp[2], yp[3]);
            if constexpr (PAT && AGG)   // the group ends here: left alone, half of the chunk's arithmetic sinks below the barriers
                asm volatile("" : "+v"(h[0]), "+v"(h[1]), "+v"(h[2]), "+v"(h[3]));
        }
        // delta_raw of the next chunk, before the barrier: the next phase A rewrites s_rT after it
        if (c + 1 < c_end) project();
        __syncthreads();
        // ---- C: pointwise post-processing --------------------------------------------
        __builtin_amdgcn_s_setprio(0);
        if (!AGG) {
            float y8[SLICE];
#pragma unroll
            for (int j = 0; j < SLICE; ++j) y8[j] = has_D ? Dsk * u8[j] : 0.0f;
#pragma unroll
            for (int ww = 0; ww < NWAVES; ++ww) {
                const float4* const p4 = reinterpret_cast<const float4*>(&s_yp[ww][pr][pq * PE]);
                const float4 p0 = p4[0], p1 = p4[HALF4];
                y8[0] += p0.x; y8[1] += p0.y; y8[2] += p0.z; y8[3] += p0.w;
                y8[4] += p1.x; y8[5] += p1.y; y8[6] += p1.z; y8[7] += p1.w;
            }
            if constexpr (VEC) {   // states beyond the first 16: add to what the earlier groups left
                if (acc_on) {
#pragma unroll
                    for (int j = 0; j < SLICE; ++j) y8[j] += p8[j];
                }
            } else if (a.acc_y) {
                const T* prev = (has_z ? static_cast<const T*>(a.ysave) : static_cast<const T*>(a.out)) + prow * L;
                io8<T>::unpack(load_slice8<T, VEC, SHORT>(prev, t0, L, p_ok), p8);
#pragma unroll
                for (int j = 0; j < SLICE; ++j) y8[j] += p8[j];
            }
            if constexpr (PAT) {
                uint32_t off[PC], off_e[PC];   // a piece, and the same piece of the even chunk (whole before an odd one; a lone even chunk has nothing waiting)
                typename pio::packed py[PC], po[PC];
#pragma unroll
                for (int p = 0; p < PC; ++p) {
                    const uint32_t at = row_off + (uint32_t)(t0 + p * PSTEP) * esz;
                    off[p] = nv[p] == PE ? at : BUF_OFF;
                    off_e[p] = SLOT == 1 ? at - CHUNK_T * esz : BUF_OFF;
                }
                pack_slice<pio, PC>(y8, py);   // y before the gate, for the backward pass's dz (if kept)
                if (has_z) {
#pragma unroll
                    for (int j = 0; j < SLICE; ++j) y8[j] *= z8[j] * sigmoid_fast(z8[j]);
                }
                pack_slice<pio, PC>(y8, po);
                if (WAIT && SLOT == 0 && c + 1 < c_end) {   // for the odd chunk
#pragma unroll
                    for (int p = 0; p < PC; ++p) { held_y[p] = py[p]; held_o[p] = po[p]; }
                } else if constexpr (RAG) {
                    if (p_ok) {
                        T* const yp = static_cast<T*>(a.ysave) + wg_first_i;
                        T* const op = static_cast<T*>(a.out) + wg_first;
                        const uint32_t yt = r_off_i + (uint32_t)t0 * esz, ot = r_off + (uint32_t)t0 * esz;
                        if (WAIT && SLOT == 1 && keep_y) pio::store_elem(yp, yt - CHUNK_T * esz, held_y[0], SLICE);
                        if (keep_y) pio::store_elem(yp, yt, py[0], nv[0]);
                        if (WAIT && SLOT == 1) pio::store_elem(op, ot - CHUNK_T * esz, held_o[0], SLICE);
                        pio::store_elem(op, ot, po[0], nv[0]);
                    }
                } else if constexpr (!WAIT) {
#pragma unroll
                    for (int p = 0; p < PC; ++p) pio::store_packed(by, off[p], py[p]);
#pragma unroll
                    for (int p = 0; p < PC; ++p) pio::store_packed(bo, off[p], po[p]);
                } else {
#pragma unroll
                    for (int p = 0; p < PC; ++p) pio::store_packed(by, off_e[p], held_y[p]);
#pragma unroll
                    for (int p = 0; p < PC; ++p) pio::store_packed(by, off[p], py[p]);
#pragma unroll
                    for (int p = 0; p < PC; ++p) pio::store_packed(bo, off_e[p], held_o[p]);
#pragma unroll
                    for (int p = 0; p < PC; ++p) pio::store_packed(bo, off[p], po[p]);
                }
            } else if constexpr (VEC) {
                const uint32_t off = nv[0] == SLICE ? row_off + (uint32_t)t0 * (uint32_t)sizeof(T) : BUF_OFF;
                io8<T>::store_buf(by, off, y8);   // y before the gate, for the backward pass's dz (if kept)
                if (has_z) {
#pragma unroll
                    for (int j = 0; j < SLICE; ++j) y8[j] *= z8[j] * sigmoid_fast(z8[j]);
                }
                io8<T>::store_buf(bo, off, y8);
            } else {
                const int nvs = p_ok ? nv[0] : 0;
                if (has_z) {
                    if (a.ysave)  // y before the gate, for the backward pass's dz
                        store_slice<T, VEC, SHORT, io8, SLICE>(static_cast<T*>(a.ysave) + prow * L + t0, y8, nvs);
#pragma unroll
                    for (int j = 0; j < SLICE; ++j) y8[j] *= z8[j] * sigmoid_fast(z8[j]);
                }
                store_slice<T, VEC, SHORT, io8, SLICE>(gout + t0, y8, nvs);
            }
        }
        // no barrier needed here: the next phase A writes s_dt/s_du, which every wave has
        // finished reading (barrier above), and s_yp is rewritten only after the next barrier
    };
    for (int c = c_begin; c < c_end; c += PF) {
        do_chunk(c, std::integral_constant<int, 0>{});
        if constexpr (PF > 1) {
            if (c + 1 < c_end) do_chunk(c + 1, std::integral_constant<int, 1>{});
        }
    }

    if (AGG) {
        if (s_ok) {
            float4* dst = reinterpret_cast<float4*>(a.seg_h + ((long)seg * a.B * a.D + srow) * NPAD) + w;
            *dst = make_float4(h[0], h[1], h[2], h[3]);
        }
        sum_dt += __shfl_xor(sum_dt, 1);
        sum_dt += __shfl_xor(sum_dt, 2);
        if (p_ok && pq == 0) a.seg_sumdt[(long)seg * a.B * a.D + prow] = sum_dt;
    } else if (a.h_last && s_ok && seg == a.nseg - 1) {
#pragma unroll
        for (int k = 0; k < STATES_PER_LANE; ++k)
            if (n_ok[k]) a.h_last[srow * NS + slot_state(w, k, a.il)] = h[k];
    }
}

// Turns the segments' local end states into incoming states, in place:
// in[1] = loc[0];  in[s+1] = exp(A * sum_dt[s]) * in[s] + loc[s]   (one thread per (b,d,n)).
__global__ void carry_fwd_kernel(const FwdArgs a)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long rows = (long)a.B * a.D;
    if (i >= rows * NPAD) return;
    const long row = i / NPAD;
    const int n = position_state((int)(i % NPAD), a.il), d = row % a.D;   // the state this slot of the record holds
    const float A2 = n < a.N ? a.A[(long)d * a.NS + n] * LOG2E : 0.0f;
    // complex state: slots (n, n^1) are (re, im) of one state; the thread carries both parts
    // and writes its own (slot n even: real part)
    const bool cplx_state = a.flags & F_COMPLEX;
    const long ip = i ^ 1;
    const float A2r = cplx_state && (n & ~1) < a.N ? a.A[(long)d * a.NS + (n & ~1)] * LOG2E : 0.0f;
    const float Aim = cplx_state && (n | 1) < a.N ? a.A[(long)d * a.NS + (n | 1)] : 0.0f;
    float carry = a.seg_h[i];  // loc[0]: already includes h0
    float other = cplx_state ? a.seg_h[ip] : 0.0f;
    // Segments are taken CARRY_BATCH at a time: their loads do not depend on the carry, so
    // they are issued together and only the multiply-adds form the serial chain.
    constexpr int CARRY_BATCH = 16;
    for (int s0 = 1; s0 < a.nseg; s0 += CARRY_BATCH) {
        float loc[CARRY_BATCH], locp[CARRY_BATCH], sdt[CARRY_BATCH];
#pragma unroll
        for (int j = 0; j < CARRY_BATCH; ++j) {
            const int s = s0 + j;
            loc[j] = s < a.nseg - 1 ? a.seg_h[(long)s * rows * NPAD + i] : 0.0f;   // the last segment has no aggregate
            locp[j] = (cplx_state && s < a.nseg - 1) ? a.seg_h[(long)s * rows * NPAD + ip] : 0.0f;
            sdt[j] = s < a.nseg - 1 ? a.seg_sumdt[(long)s * rows + row] : 0.0f;
        }
#pragma unroll
        for (int j = 0; j < CARRY_BATCH; ++j) {
            const int s = s0 + j;
            if (s < a.nseg) {
                a.seg_h[(long)s * rows * NPAD + i] = carry;  // incoming state of segment s
                if (cplx_state) {
                    const cplx ab = complex_decay(sdt[j], A2r, Aim);
                    const float re = (n & 1) ? other : carry, im = (n & 1) ? carry : other;
                    const float nre = fmaf(ab.re, re, -ab.im * im) + ((n & 1) ? locp[j] : loc[j]);
                    const float nim = fmaf(ab.im, re, ab.re * im) + ((n & 1) ? loc[j] : locp[j]);
                    carry = (n & 1) ? nim : nre;
                    other = (n & 1) ? nre : nim;
                } else {
                    carry = fmaf(exp2_fast(A2 * sdt[j]), carry, loc[j]);
                }
            }
        }
    }
}

// Single-token step: 4 lanes per row, 4 states each; the state is read and written once,
// in place.  With N == 16 every per-state operand (state, A, B_t, C_t) is one aligned
// 16- or 8-byte access per lane.
template <typename T, bool FULLN, bool ZOH>
__global__ void __launch_bounds__(256) step_kernel(const StepArgs a)
{
    const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long rowi = gid >> 2;
    const int q = gid & 3;
    const long rows = (long)a.B * a.D;
    const bool row_ok = rowi < rows;
    const long row = row_ok ? rowi : rows - 1;
    const int b = row / a.D, d = row % a.D;
    const int N = a.N;

    const T* u_t = static_cast<const T*>(a.u_t);
    const T* dl_t = static_cast<const T*>(a.delta_t);
    const T* z_t = static_cast<const T*>(a.z_t);
    const T* B_t = static_cast<const T*>(a.B_t);
    const T* C_t = static_cast<const T*>(a.C_t);
    // time-invariant B / C are (D,N) float32 parameters; the launcher sends them down the generic path
    const bool bfix = !FULLN && (a.flags & F_B_FIXED), cfix = !FULLN && (a.flags & F_C_FIXED);
    auto ld = [](const T* p, long i) -> float {
        if constexpr (sizeof(T) == 2) return bf16_to_f32(p[i]); else return p[i];
    };
    // Every global load of the thread is requested here (and, on the vector path, right below),
    // back to back: optional operands through a valid stand-in pointer, and no arithmetic on a
    // loaded value in between, either of which would make the compiler wait for one load before
    // issuing the next -- four memory round trips instead of one.
    const bool has_bias = a.flags & F_HAS_DELTA_BIAS, has_D = a.flags & F_HAS_D, has_z = a.flags & F_HAS_Z;
    const T u_raw = u_t[row], dl_raw = dl_t[row], z_raw = (has_z ? z_t : u_t)[row];
    const float bias_raw = (has_bias ? a.bias : a.A)[has_bias ? d : 0];
    const float D_raw = (has_D ? a.Dskip : a.A)[has_D ? d : 0];
    float4 h4_first = make_float4(0.f, 0.f, 0.f, 0.f), A4_first = h4_first;
    uint4 B_first = make_uint4(0u, 0u, 0u, 0u), C_first = B_first;   // bf16: two words each; float: four
    if constexpr (FULLN) {
        h4_first = *reinterpret_cast<const float4*>(a.h + row * N + q * STATES_PER_LANE);
        A4_first = *reinterpret_cast<const float4*>(a.A + (long)d * NPAD + q * STATES_PER_LANE);
        const long bo = (long)b * a.bc_stride + q * STATES_PER_LANE;
        if constexpr (sizeof(T) == 2) {
            const uint2 Bw = *reinterpret_cast<const uint2*>(B_t + bo), Cw = *reinterpret_cast<const uint2*>(C_t + bo);
            B_first.x = Bw.x; B_first.y = Bw.y; C_first.x = Cw.x; C_first.y = Cw.y;
        } else {
            B_first = *reinterpret_cast<const uint4*>(B_t + bo);
            C_first = *reinterpret_cast<const uint4*>(C_t + bo);
        }
    }
    auto cvt = [](T v) -> float {
        if constexpr (sizeof(T) == 2) return bf16_to_f32(v); else return v;
    };
    const float u = cvt(u_raw);
    float x = cvt(dl_raw) + (has_bias ? bias_raw : 0.0f);
    float dt = x, sg;
    if (a.flags & F_DELTA_SOFTPLUS) softplus_sigmoid(x, dt, sg);
    const float du = ZOH ? u : dt * u, dt2 = dt * LOG2E;

    float y = 0.0f;
    // 16 states per pass: one pass when N <= 16 (always so on the vector path)
    for (int n0 = 0; n0 < (FULLN ? NPAD : N); n0 += NPAD) {
        float hv[STATES_PER_LANE], Av[STATES_PER_LANE], Bv[STATES_PER_LANE], Cv[STATES_PER_LANE];
        float* hp = a.h + row * N + n0 + q * STATES_PER_LANE;
        if (FULLN) {   // one pass; loaded above
            const float4 h4 = h4_first, A4 = A4_first;
            hv[0] = h4.x; hv[1] = h4.y; hv[2] = h4.z; hv[3] = h4.w;
            Av[0] = A4.x; Av[1] = A4.y; Av[2] = A4.z; Av[3] = A4.w;
            if constexpr (sizeof(T) == 2) {
                Bv[0] = bf16_lo(B_first.x); Bv[1] = bf16_hi(B_first.x); Bv[2] = bf16_lo(B_first.y); Bv[3] = bf16_hi(B_first.y);
                Cv[0] = bf16_lo(C_first.x); Cv[1] = bf16_hi(C_first.x); Cv[2] = bf16_lo(C_first.y); Cv[3] = bf16_hi(C_first.y);
            } else {
                Bv[0] = __uint_as_float(B_first.x); Bv[1] = __uint_as_float(B_first.y);
                Bv[2] = __uint_as_float(B_first.z); Bv[3] = __uint_as_float(B_first.w);
                Cv[0] = __uint_as_float(C_first.x); Cv[1] = __uint_as_float(C_first.y);
                Cv[2] = __uint_as_float(C_first.z); Cv[3] = __uint_as_float(C_first.w);
            }
        } else {
#pragma unroll
            for (int k = 0; k < STATES_PER_LANE; ++k) {
                const int n = n0 + q * STATES_PER_LANE + k;
                const bool ok = n < N;
                hv[k] = ok ? hp[k] : 0.0f;
                Av[k] = ok ? a.A[(long)d * N + n] : 0.0f;
                Bv[k] = !ok ? 0.0f : bfix ? static_cast<const float*>(a.B_t)[(long)d * N + n] : ld(B_t, (long)b * a.bc_stride + n);
                Cv[k] = !ok ? 0.0f : cfix ? static_cast<const float*>(a.C_t)[(long)d * N + n] : ld(C_t, (long)b * a.bc_stride + n);
            }
        }
        if (a.flags & F_COMPLEX) {   // slots (0,1) and (2,3) are (re, im) of two complex states
#pragma unroll
            for (int k = 0; k < STATES_PER_LANE; k += 2) {
                const cplx ab = complex_decay(dt, Av[k] * LOG2E, Av[k + 1]);
                const float hr = fmaf(ab.re, hv[k], fmaf(-ab.im, hv[k + 1], du * Bv[k]));
                const float hi = fmaf(ab.im, hv[k], fmaf(ab.re, hv[k + 1], du * Bv[k + 1]));
                hv[k] = hr;
                hv[k + 1] = hi;
                y = fmaf(Cv[k], hr, fmaf(-Cv[k + 1], hi, y));
            }
        } else {
#pragma unroll
            for (int k = 0; k < STATES_PER_LANE; ++k) {
                const float abar = exp2_fast(dt2 * Av[k]);                  // Eq. 4
                float bu = du * Bv[k];
                if (ZOH) bu *= zoh_phi(dt, Av[k], Av[k] != 0.0f ? 1.0f / Av[k] : 0.0f, abar, false).phi;
                hv[k] = fmaf(abar, hv[k], bu);                              // Eq. 2a
                y = fmaf(Cv[k], hv[k], y);                                  // Eq. 2b
            }
        }
        if (row_ok) {
            if (FULLN) {
                *reinterpret_cast<float4*>(hp) = make_float4(hv[0], hv[1], hv[2], hv[3]);
            } else {
#pragma unroll
                for (int k = 0; k < STATES_PER_LANE; ++k)
                    if (n0 + q * STATES_PER_LANE + k < N) hp[k] = hv[k];
            }
        }
    }
    // sum over the 4 lanes of the row
    y += __shfl_xor(y, 1);
    y += __shfl_xor(y, 2);
    if (has_D) y = fmaf(D_raw, u, y);
    if (has_z) {
        const float z = cvt(z_raw);
        y *= z * sigmoid_fast(z);
    }
    if (row_ok && q == 0) {
        if constexpr (sizeof(T) == 2) static_cast<bf16_t*>(a.out_t)[row] = bf16_t(f32_to_bf16_bits(y));
        else static_cast<float*>(a.out_t)[row] = y;
    }
}

// Single-token step, the common case at scale (N == 16, real state, first-order B-bar, selective
// B / C, vector-aligned operands): as step_kernel, with RPT batch entries (b, b + B/RPT, ...) of the
// same channel per thread.  A, bias and D are fetched once for them, and RPT state vectors per lane
// are in flight at once, which a streaming kernel this short needs to fill the memory pipeline.
template <typename T, int RPT>
__global__ void __launch_bounds__(256) step_multi_kernel(const StepArgs a)
{
    const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long rowi = gid >> 2;
    const int q = gid & 3;
    const int bpart = a.B / RPT;                       // the launcher checks B % RPT == 0
    const long rows_part = (long)bpart * a.D;
    const bool row_ok = rowi < rows_part;
    const long row0 = row_ok ? rowi : rows_part - 1;
    const int b0 = row0 / a.D, d = row0 % a.D;
    const T* u_t = static_cast<const T*>(a.u_t);
    const T* dl_t = static_cast<const T*>(a.delta_t);
    const T* z_t = static_cast<const T*>(a.z_t);
    const T* B_t = static_cast<const T*>(a.B_t);
    const T* C_t = static_cast<const T*>(a.C_t);
    const bool has_bias = a.flags & F_HAS_DELTA_BIAS, has_D = a.flags & F_HAS_D, has_z = a.flags & F_HAS_Z;
    // all loads first, none behind a branch or behind arithmetic on a loaded value (see step_kernel)
    float4 h4[RPT];
    T u_raw[RPT], dl_raw[RPT], z_raw[RPT];
    uint4 Bw[RPT], Cw[RPT];
    long row[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int b = b0 + i * bpart;
        row[i] = (long)b * a.D + d;
        h4[i] = *reinterpret_cast<const float4*>(a.h + row[i] * NPAD + q * STATES_PER_LANE);
        u_raw[i] = u_t[row[i]];
        dl_raw[i] = dl_t[row[i]];
        z_raw[i] = (has_z ? z_t : u_t)[row[i]];
        const long bo = (long)b * a.bc_stride + q * STATES_PER_LANE;
        Bw[i] = make_uint4(0u, 0u, 0u, 0u);
        Cw[i] = Bw[i];
        if constexpr (sizeof(T) == 2) {
            const uint2 x = *reinterpret_cast<const uint2*>(B_t + bo), y = *reinterpret_cast<const uint2*>(C_t + bo);
            Bw[i].x = x.x; Bw[i].y = x.y; Cw[i].x = y.x; Cw[i].y = y.y;
        } else {
            Bw[i] = *reinterpret_cast<const uint4*>(B_t + bo);
            Cw[i] = *reinterpret_cast<const uint4*>(C_t + bo);
        }
    }
    const float4 A4 = *reinterpret_cast<const float4*>(a.A + (long)d * NPAD + q * STATES_PER_LANE);
    const float bias_raw = (has_bias ? a.bias : a.A)[has_bias ? d : 0];
    const float D_raw = (has_D ? a.Dskip : a.A)[has_D ? d : 0];
    auto cvt = [](T v) -> float {
        if constexpr (sizeof(T) == 2) return bf16_to_f32(v); else return v;
    };
    const float Av[STATES_PER_LANE] = {A4.x * LOG2E, A4.y * LOG2E, A4.z * LOG2E, A4.w * LOG2E};
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const float u = cvt(u_raw[i]);
        float x = cvt(dl_raw[i]) + (has_bias ? bias_raw : 0.0f);
        float dt = x, sg;
        if (a.flags & F_DELTA_SOFTPLUS) softplus_sigmoid(x, dt, sg);
        const float du = dt * u;
        float hv[STATES_PER_LANE] = {h4[i].x, h4[i].y, h4[i].z, h4[i].w}, Bv[STATES_PER_LANE], Cv[STATES_PER_LANE];
        if constexpr (sizeof(T) == 2) {
            Bv[0] = bf16_lo(Bw[i].x); Bv[1] = bf16_hi(Bw[i].x); Bv[2] = bf16_lo(Bw[i].y); Bv[3] = bf16_hi(Bw[i].y);
            Cv[0] = bf16_lo(Cw[i].x); Cv[1] = bf16_hi(Cw[i].x); Cv[2] = bf16_lo(Cw[i].y); Cv[3] = bf16_hi(Cw[i].y);
        } else {
            Bv[0] = __uint_as_float(Bw[i].x); Bv[1] = __uint_as_float(Bw[i].y); Bv[2] = __uint_as_float(Bw[i].z); Bv[3] = __uint_as_float(Bw[i].w);
            Cv[0] = __uint_as_float(Cw[i].x); Cv[1] = __uint_as_float(Cw[i].y); Cv[2] = __uint_as_float(Cw[i].z); Cv[3] = __uint_as_float(Cw[i].w);
        }
        float y = 0.0f;
#pragma unroll
        for (int k = 0; k < STATES_PER_LANE; ++k) {
            const float abar = exp2_fast(dt * Av[k]);                       // Eq. 4
            hv[k] = fmaf(abar, hv[k], du * Bv[k]);                          // Eq. 2a
            y = fmaf(Cv[k], hv[k], y);                                      // Eq. 2b
        }
        if (row_ok)
            *reinterpret_cast<float4*>(a.h + row[i] * NPAD + q * STATES_PER_LANE) = make_float4(hv[0], hv[1], hv[2], hv[3]);
        y += __shfl_xor(y, 1);
        y += __shfl_xor(y, 2);
        if (has_D) y = fmaf(D_raw, u, y);
        if (has_z) {
            const float z = cvt(z_raw[i]);
            y *= z * sigmoid_fast(z);
        }
        if (row_ok && q == 0) {
            if constexpr (sizeof(T) == 2) static_cast<bf16_t*>(a.out_t)[row[i]] = bf16_t(f32_to_bf16_bits(y));
            else static_cast<float*>(a.out_t)[row[i]] = y;
        }
    }
}

// Single-token step of the layer's decode : as step_kernel, but delta_t, B_t and C_t come
// from the float32 output P = [r; B; C] of the projection (the sum of STEP_NPARTS partial results,
// rounded to the io type as the layer stores it) and delta_t = W_dt r_t + bias is formed here.  A workgroup
// owns 64 channels and a tile of BT = 16 or 8 batch entries.  It stages the tile's rows of P in LDS;
// four of its eight waves (in float32 all eight, two to a tile, every other contraction step each) then form the 16 x 64 block of
// W_dt r_t on the matrix cores (16 x 16 tiles, rows past the tile shadowing its last one, W_dt rows straight from global memory)
// and leave softplus(. + bias) in LDS, once per (b, d) instead of once per quarter; after that a
// thread is (channel d, quarter q, half of the batch tile) as in step_kernel and walks its BT / 2
// batch entries.  The 8-entry tile needs fewer registers (two workgroups per CU instead of one) and
// gives twice the workgroups; the launcher picks the tile from the number of workgroups each gives.  The state, u and z of those entries are
// requested before anything else, so that their latency overlaps the projection.  Real, first-order,
// selective B / C only; 8 <= R <= 256, N <= 16.  Rows of W_dt are read at element alignment, their last piece cut.
constexpr int SP_MFMA_ROWS = 16;                  // rows of the MFMA tile: the largest batch tile
constexpr int SP_THREADS = 512;                   // 64 channels x 4 quarters x 2 halves of the batch tile
constexpr int SP_MAX_R = 256;
constexpr int STEP_MAX_LDP = SP_MAX_R + 2 * NPAD;   // R <= 256 and N <= 16 on this path
constexpr int SP_LDP = STEP_MAX_LDP + 4;          // row stride of the staged P in floats: 16-byte rows, off the banks

// WIN: the convolution's window slides here, the projection having formed u itself (see StepArgs).
template <typename T, bool FULLN, int SP_BT, bool WIN = false>
__global__ void __launch_bounds__(SP_THREADS, SP_BT == 8 ? 4 : 2) step_proj_kernel(const StepArgs a)
{
    static_assert(SP_BT == 8 || SP_BT == SP_MFMA_ROWS, "batch tile");
    constexpr int SP_PER = SP_BT / 2;                // batch entries per thread
    using mma = tile_mma<T>;
    // Contraction steps of the delta projection a wave takes.  In float, where they are twice as many and four dependent MFMAs each, all eight
    // waves share them, the second four every other step: half the registers for W_dt, so that two workgroups of the 8-entry tile fit a CU
    // (float32, D 5120, kernel: batch 64 28.4 -> 18.8 us, 256 86 -> 50; D 1536, batch 128, the 16-entry tile 10.8 -> 9.8).
    constexpr bool HALVES = sizeof(T) == 4;
    constexpr int SP_MAX_KSTEPS = SP_MAX_R / mma::K / (HALVES ? 2 : 1), KSTRIDE = HALVES ? 2 * mma::K : mma::K;
    __shared__ __attribute__((aligned(16))) float s_p[SP_BT][SP_LDP];   // r, and from SP_MAX_R on B and C
    __shared__ float s_dt[SP_MFMA_ROWS][64];
    __shared__ f32x4_t s_half[HALVES ? 4 : 1][HALVES ? 64 : 1];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = tid & 3, dl = (tid >> 2) & 63, half = tid >> 8;
    const int d0 = blockIdx.x * 64;
    const bool d_ok = d0 + dl < a.D;
    const int d = d_ok ? d0 + dl : a.D - 1;
    const int N = a.N, R = a.R;
    const int b0 = blockIdx.y * SP_BT;
    const int nbt = min(SP_BT, a.B - b0);            // batch entries of this tile
    const T* u_t = static_cast<const T*>(a.u_t);
    const T* z_t = static_cast<const T*>(a.z_t);
    auto cvt = [](T v) -> float {
        if constexpr (sizeof(T) == 2) return bf16_to_f32(v); else return v;
    };
    auto as_stored = [](float v) -> float {
        if constexpr (sizeof(T) == 2) return bf16_to_f32(bf16_t(f32_to_bf16_bits(v))); else return v;
    };

    // Everything the thread needs from global memory is requested here, in straight-line code
    // with no branch between the loads (optional operands are read through a valid stand-in
    // pointer and discarded) and no arithmetic on a loaded value: either would make the compiler
    // wait for that load before issuing the next, one memory latency after another.
    const int sq = q * STATES_PER_LANE;               // this quarter's first state
    const bool has_z = a.flags & F_HAS_Z, has_D = a.flags & F_HAS_D, has_bias = a.flags & F_HAS_DELTA_BIAS;
    const T* zp = has_z ? z_t : u_t;
    float hv[SP_PER][STATES_PER_LANE];
    T ub_raw[SP_PER], zb_raw[SP_PER];
    T slot_raw[SP_PER];   // WIN: quarter q < 3 moves slot q of its (b, d)
#pragma unroll
    for (int i = 0; i < SP_PER; ++i) {
        const int b = min(b0 + half * SP_PER + i, a.B - 1);
        const long row = (long)b * a.D + d;
        if constexpr (FULLN) {
            const float4 h4 = *reinterpret_cast<const float4*>(a.h + row * N + sq);
            hv[i][0] = h4.x; hv[i][1] = h4.y; hv[i][2] = h4.z; hv[i][3] = h4.w;
        } else {
#pragma unroll
            for (int k = 0; k < STATES_PER_LANE; ++k) hv[i][k] = a.h[row * N + min(sq + k, N - 1)];   // a valid element; masked below
        }
        ub_raw[i] = u_t[row];
        zb_raw[i] = zp[row];
        if constexpr (WIN) slot_raw[i] = *(q < 2 ? static_cast<const T*>(a.conv_state) + row * 3 + q + 1 : static_cast<const T*>(a.x_t) + row);
    }
    float A_raw[STATES_PER_LANE];
#pragma unroll
    for (int k = 0; k < STATES_PER_LANE; ++k) A_raw[k] = a.A[(long)d * N + min(sq + k, N - 1)];
    const float D_raw = (has_D ? a.Dskip : a.A)[has_D ? d : 0];

    // Waves 0-3 form the tile (batch entries) x (channels d0 + 16 * wave ..+15) of r W_dt^T after
    // the staging below (fragments as tile_mma describes).  Their pieces of W_dt are requested now, with everything
    // else (from a clamped, valid place; what lies past R meets zeros of r).
    const int dcol = 16 * (wave & 3) + (lane & 15);
    const int wrow = min(d0 + dcol, a.D - 1);
    const int ksub = mma::E * (lane >> 4);
    const int kfirst = HALVES ? mma::K * (wave >> 2) : 0;   // this wave's first step
    u32x4 wfrag[SP_MAX_KSTEPS];
    const float bias_raw = (has_bias ? a.bias : a.A)[has_bias ? wrow : 0];
    {
        const T* wp = static_cast<const T*>(a.W_dt) + (long)d0 * R;   // the workgroup's first row
        const int woff = (wrow - d0) * R;
#pragma unroll
        for (int i = 0; i < SP_MAX_KSTEPS; ++i)
            wfrag[i] = load_any<u32x4>(wp, (uint32_t)(woff + row_piece(kfirst + KSTRIDE * i + ksub, mma::E, R)) * (uint32_t)sizeof(T));
    }

    {
        // P of the tile: all loads first (STEP_NPARTS x STAGE_ITEMS per thread, independent), then
        // the parts added in a fixed order and rounded as stored
        constexpr int STAGE_ITEMS = (SP_BT * STEP_MAX_LDP + SP_THREADS - 1) / SP_THREADS;
        const long part = (long)a.B * a.ldp;   // floats between partial results
        const int count = nbt * a.ldp;
        float v[STAGE_ITEMS][STEP_NPARTS];
#pragma unroll
        for (int j = 0; j < STAGE_ITEMS; ++j) {
            const int i = tid + SP_THREADS * j;
            const long g = (long)b0 * a.ldp + min(i, count - 1);
#pragma unroll
            for (int k = 0; k < STEP_NPARTS; ++k) v[j][k] = a.P[k * part + g];
        }
#pragma unroll
        for (int j = 0; j < STAGE_ITEMS; ++j) {
            const int i = tid + SP_THREADS * j;
            float s = v[j][0];
#pragma unroll
            for (int k = 1; k < STEP_NPARTS; ++k) s += v[j][k];
            const int col = i % a.ldp;
            if (i < count) s_p[i / a.ldp][col < R ? col : SP_MAX_R + col - R] = as_stored(s);
        }
        // r up to a whole step of the product
        const int zcol = R + (tid & 31);
        if ((tid >> 5) < SP_BT && zcol < (R + mma::K - 1) / mma::K * mma::K) s_p[tid >> 5][zcol] = 0.0f;
    }
    __syncthreads();

    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    if (HALVES || wave < 4) {
        const int arow = min(lane & 15, nbt - 1);             // rows past the end shadow the last one
        const float* pp = &s_p[arow][ksub];
#pragma unroll
        for (int i = 0; i < SP_MAX_KSTEPS; ++i) {
            const int k = kfirst + KSTRIDE * i;
            if (k < R) {                                      // uniform
                float pv[mma::E];
#pragma unroll
                for (int e = 0; e < mma::E; e += 4) {
                    const float4 p4 = *reinterpret_cast<const float4*>(pp + k + e);
                    pv[e] = p4.x; pv[e + 1] = p4.y; pv[e + 2] = p4.z; pv[e + 3] = p4.w;
                }
                u32x4 av, wv = wfrag[i];
                if (R % mma::E != 0 && k + mma::K > R) wv = mma::cut(wv, k + ksub, R);   // uniform
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (sizeof(T) == 2) av[e] = pack_bf16x2(pv[2 * e], pv[2 * e + 1]);   // exact: rounded above
                    else av[e] = __float_as_uint(pv[e]);
                }
                acc = mma::step(av, wv, acc);
            }
        }
    }
    if constexpr (HALVES) {
        if (wave >= 4) s_half[wave & 3][lane] = acc;
        __syncthreads();
        if (wave < 4) acc += s_half[wave][lane];
    }
    if (wave < 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float x = as_stored(acc[i]) + (has_bias ? bias_raw : 0.0f), dt = x, sg;
            if (a.flags & F_DELTA_SOFTPLUS) softplus_sigmoid(x, dt, sg);
            s_dt[4 * (lane >> 4) + i][dcol] = dt;
        }
    }
    __syncthreads();

    float Av[STATES_PER_LANE];
#pragma unroll
    for (int k = 0; k < STATES_PER_LANE; ++k) Av[k] = (sq + k < N) ? A_raw[k] * LOG2E : 0.0f;
    const float Dsk = has_D ? D_raw : 0.0f;
#pragma unroll
    for (int i = 0; i < SP_PER; ++i) {
        const int bl = half * SP_PER + i;
        if (bl >= nbt) break;
        if constexpr (!FULLN) {
#pragma unroll
            for (int k = 0; k < STATES_PER_LANE; ++k) hv[i][k] = (sq + k < N) ? hv[i][k] : 0.0f;
        }
        const long row = (long)(b0 + bl) * a.D + d;
        const float* pb = s_p[bl];
        const float dt = s_dt[bl][dl];
        const float u = cvt(ub_raw[i]);
        const float du = dt * u;
        float Bq[STATES_PER_LANE], Cq[STATES_PER_LANE];
        if constexpr (FULLN) {
            const float4 b4 = *reinterpret_cast<const float4*>(pb + SP_MAX_R + sq);
            const float4 c4 = *reinterpret_cast<const float4*>(pb + SP_MAX_R + NPAD + sq);
            Bq[0] = b4.x; Bq[1] = b4.y; Bq[2] = b4.z; Bq[3] = b4.w;
            Cq[0] = c4.x; Cq[1] = c4.y; Cq[2] = c4.z; Cq[3] = c4.w;
        } else {
#pragma unroll
            for (int k = 0; k < STATES_PER_LANE; ++k) {
                const bool ok = sq + k < N;
                Bq[k] = ok ? pb[SP_MAX_R + sq + k] : 0.0f;
                Cq[k] = ok ? pb[SP_MAX_R + N + sq + k] : 0.0f;
            }
        }
        float y = 0.0f;
#pragma unroll
        for (int k = 0; k < STATES_PER_LANE; ++k) {
            const float abar = exp2_fast(dt * Av[k]);          // Eq. 4
            hv[i][k] = fmaf(abar, hv[i][k], du * Bq[k]);       // Eq. 2a
            y = fmaf(Cq[k], hv[i][k], y);                      // Eq. 2b
        }
        if (d_ok) {
            float* hp = a.h + row * N + sq;
            if constexpr (FULLN) {
                *reinterpret_cast<float4*>(hp) = make_float4(hv[i][0], hv[i][1], hv[i][2], hv[i][3]);
            } else {
#pragma unroll
                for (int k = 0; k < STATES_PER_LANE; ++k)
                    if (sq + k < N) hp[k] = hv[i][k];
            }
        }
        y += __shfl_xor(y, 1);
        y += __shfl_xor(y, 2);
        y = fmaf(Dsk, u, y);
        if (has_z) {
            const float z = cvt(zb_raw[i]);
            y *= z * sigmoid_fast(z);
        }
        if (d_ok && q == 0) {
            if constexpr (sizeof(T) == 2) static_cast<bf16_t*>(a.out_t)[row] = bf16_t(f32_to_bf16_bits(y));
            else static_cast<float*>(a.out_t)[row] = y;
        }
        if constexpr (WIN) {
            if (d_ok && q < 3) static_cast<T*>(a.conv_state)[row * 3 + q] = slot_raw[i];
        }
    }
}

// h_last for an empty sequence: h0 or zero
__global__ void copy_state_kernel(const float* __restrict__ src, float* __restrict__ dst, long n)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src ? src[i] : 0.0f;
}

// Wave-packed copy of the selective B and C for the forward kernels (layout: FwdArgs::bcs).
// A thread writes the four steps of one (batch entry, state, group of steps, B or C).
// The scalar path does not deal its states out (FwdArgs::il is 0 there).
template <typename T>
__global__ void stage_bc_kernel(const T* __restrict__ Bm, const T* __restrict__ Cm, long bstride, T* __restrict__ dst,
                                int B, int NS, int L, int Lp)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const int tgroups = Lp / GROUP_T, sgroups = (NS + NPAD - 1) / NPAD * NWAVES;   // every wave of every pass has a piece
    if (i >= (long)B * sgroups * tgroups * 2 * STATES_PER_LANE) return;
    const int r = (int)(i % (2 * STATES_PER_LANE));            // which * 4 + k
    const long piece = i / (2 * STATES_PER_LANE);
    const int tg = (int)(piece % tgroups);
    const int sg = (int)((piece / tgroups) % sgroups);
    const int b = (int)(piece / ((long)tgroups * sgroups));
    const int grp = sg / NWAVES;
    const int n = grp * NPAD + slot_state(sg % NWAVES, r % STATES_PER_LANE, 0), t = tg * GROUP_T;
    const T* src = (r >= STATES_PER_LANE ? Cm : Bm) + (long)b * bstride + (long)n * L + t;
    T v[GROUP_T];
#pragma unroll
    for (int j = 0; j < GROUP_T; ++j) v[j] = (n < NS && t + j < L) ? src[j] : T(0);
    T* out = dst + i * GROUP_T;
    if constexpr (sizeof(T) == 2) {
        *reinterpret_cast<uint2*>(out) = make_uint2(uint32_t(v[0]) | (uint32_t(v[1]) << 16), uint32_t(v[2]) | (uint32_t(v[3]) << 16));
    } else {
        *reinterpret_cast<float4*>(out) = make_float4(v[0], v[1], v[2], v[3]);
    }
}

int launch_stage_bc(const FwdArgs& a, void* bcs, int io_dtype, hipStream_t stream)
{
    const long n = (long)a.B * ((a.NS + NPAD - 1) / NPAD * NWAVES) * (a.Lp / GROUP_T) * 2 * STATES_PER_LANE;
    const dim3 grid((unsigned)((n + 255) / 256));
    if (io_dtype == 0)
        stage_bc_kernel<float><<<grid, dim3(256), 0, stream>>>(static_cast<const float*>(a.Bm), static_cast<const float*>(a.Cm),
                                                               a.bc_bstride, static_cast<float*>(bcs), a.B, a.NS, a.L, a.Lp);
    else
        stage_bc_kernel<bf16_t><<<grid, dim3(256), 0, stream>>>(static_cast<const bf16_t*>(a.Bm), static_cast<const bf16_t*>(a.Cm),
                                                                a.bc_bstride, static_cast<bf16_t*>(bcs), a.B, a.NS, a.L, a.Lp);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// The main pass off the quad-broadcast kernels; rows that are not whole slices by elements if they are short (never split).
template <typename T, bool VEC, bool FULLN, bool ZOH, int BCFIX, bool CPLX = false, bool STAGED = false>
static void launch_fwd_rows(const FwdArgs& a, dim3 grid, hipStream_t stream)
{
    if constexpr (!VEC) {
        if (short_rows<T>(a.L, SLICE)) {
            scan_fwd_kernel<T, false, FULLN, false, ZOH, BCFIX, CPLX, STAGED, 0, STATES_PER_LANE, false, false, true><<<grid, dim3(THREADS), 0, stream>>>(a);
            return;
        }
    }
    scan_fwd_kernel<T, VEC, FULLN, false, ZOH, BCFIX, CPLX, STAGED><<<grid, dim3(THREADS), 0, stream>>>(a);
}

// The aggregate pass of a real state with time-invariant B and / or C.  It has no use for C: with a selective B it is the
// common path's (or the scalar path's) and with a time-invariant one the kernel that reads neither along the sequence, each
// given B in the place of C.
template <typename T, bool VEC, bool FULLN, bool ZOH, int BCFIX>
static void launch_agg_fixed(const FwdArgs& a, hipStream_t stream)
{
    const int groups = (a.D + ROWS - 1) / ROWS;
    const dim3 grid((unsigned)(a.B * groups), (unsigned)(a.nseg - 1)), block(THREADS);
    FwdArgs b = a;
    b.Cm = a.Bm;
    if constexpr (BCFIX & 1) {
        scan_fwd_kernel<T, VEC, FULLN, true, ZOH, 3><<<grid, block, 0, stream>>>(b);
    } else {
        if (a.vec_ok) scan_fwd_kernel<T, true, false, true, ZOH, 0, false, false, 0, STATES_PER_LANE, true, false><<<grid, block, 0, stream>>>(b);
        else if (a.dpp_ok) scan_fwd_kernel<T, true, false, true, ZOH, 0, false, false, 0, STATES_PER_LANE, true, true><<<grid, block, 0, stream>>>(b);
        else scan_fwd_kernel<T, false, false, true, ZOH><<<grid, block, 0, stream>>>(b);
    }
    const long n = (long)a.B * a.D * NPAD;
    carry_fwd_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream>>>(a);
}

template <typename T, bool VEC, bool FULLN, bool ZOH, int BCFIX>
static void launch_fwd_fixed(const FwdArgs& a, hipStream_t stream)
{
    const int groups = (a.D + ROWS - 1) / ROWS;
    if (a.nseg > 1) launch_agg_fixed<T, VEC, FULLN, ZOH, BCFIX>(a, stream);
    launch_fwd_rows<T, VEC, FULLN, ZOH, BCFIX>(a, dim3((unsigned)(a.B * groups), (unsigned)a.nseg), stream);
}

// complex state: first-order B-bar only; selective or time-invariant B / C
template <typename T, bool VEC, bool FULLN, int BCFIX>
static void launch_fwd_complex(const FwdArgs& a, hipStream_t stream)
{
    const int groups = (a.D + ROWS - 1) / ROWS;
    const dim3 block(THREADS);
    if (a.nseg > 1) {
        scan_fwd_kernel<T, VEC, FULLN, true, false, BCFIX, true><<<dim3((unsigned)(a.B * groups), (unsigned)(a.nseg - 1)), block, 0, stream>>>(a);
        const long n = (long)a.B * a.D * NPAD;
        carry_fwd_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream>>>(a);
    }
    launch_fwd_rows<T, VEC, FULLN, false, BCFIX, true>(a, dim3((unsigned)(a.B * groups), (unsigned)a.nseg), stream);
}

// Real state, selective B and C, rows of at least 8 steps: B and C as quad-broadcast operands.
template <typename T, bool ZOH, int SPL, bool RAG>
static void launch_fwd_dpp_t(const FwdArgs& a, hipStream_t stream)
{
    const int groups = (a.D + ROWS - 1) / ROWS;
    const dim3 block(THREADS);
    if (a.nseg > 1) {
        scan_fwd_kernel<T, true, false, true, ZOH, 0, false, false, 0, SPL, true, RAG><<<dim3((unsigned)(a.B * groups), (unsigned)(a.nseg - 1)), block, 0, stream>>>(a);
        const long n = (long)a.B * a.D * NPAD;
        if (a.nseg > CARRY_INLINE) carry_fwd_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream>>>(a);
    }
    if constexpr (sizeof(T) == 2 && !ZOH && SPL == STATES_PER_LANE) {
        if (a.W_dt) {   // the caller has checked: unsplit, R <= 256
            if (!RAG && a.Rp <= 128)   // rows off whole slices come here for more than 192 ranks only
                scan_fwd_kernel<T, true, false, false, ZOH, 0, false, false, 4, SPL, true, false><<<dim3((unsigned)(a.B * groups), 1u), block, 0, stream>>>(a);
            else
                scan_fwd_kernel<T, true, false, false, ZOH, 0, false, false, 8, SPL, true, RAG><<<dim3((unsigned)(a.B * groups), 1u), block, 0, stream>>>(a);
            return;
        }
    }
    if (sizeof(T) == 2 || a.wait_fwd)
        scan_fwd_kernel<T, true, false, false, ZOH, 0, false, false, 0, SPL, true, RAG><<<dim3((unsigned)(a.B * groups), (unsigned)a.nseg), block, 0, stream>>>(a);
    else
        scan_fwd_kernel<T, true, false, false, ZOH, 0, false, false, 0, SPL, true, RAG, false, sizeof(T) == 2><<<dim3((unsigned)(a.B * groups), (unsigned)a.nseg), block, 0, stream>>>(a);
}
// Rows of whole 16-byte pieces take the kernel with buffer-addressed accesses, all others the one for any row length.
// Fewer than 16 states dealt out to the waves: kernels built for 1 or 2 slots per lane.
template <typename T, bool RAG>
static void launch_fwd_dpp(const FwdArgs& a, hipStream_t stream)
{
    if (a.flags & F_EXACT_ZOH_B) return launch_fwd_dpp_t<T, true, STATES_PER_LANE, RAG>(a, stream);
    const int spl = slots_for(a.N, a.il);
    if (spl == 1) return launch_fwd_dpp_t<T, false, 1, RAG>(a, stream);
    if (spl == 2) return launch_fwd_dpp_t<T, false, 2, RAG>(a, stream);
    launch_fwd_dpp_t<T, false, STATES_PER_LANE, RAG>(a, stream);
}

// Real state, selective B and C, fewer than 8 steps or rows beyond the kernels above: the scalar path (from the
// repacked copy of B and C if there is one).
template <typename T, bool ZOH>
static void launch_fwd_scalar(const FwdArgs& a, hipStream_t stream)
{
    const int groups = (a.D + ROWS - 1) / ROWS;
    const dim3 block(THREADS), main_grid((unsigned)(a.B * groups), (unsigned)a.nseg);
    if (a.nseg > 1) {
        const dim3 agg_grid((unsigned)(a.B * groups), (unsigned)(a.nseg - 1));
        if (a.bcs) scan_fwd_kernel<T, false, false, true, ZOH, 0, false, true><<<agg_grid, block, 0, stream>>>(a);
        else scan_fwd_kernel<T, false, false, true, ZOH><<<agg_grid, block, 0, stream>>>(a);
        const long n = (long)a.B * a.D * NPAD;
        carry_fwd_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream>>>(a);
    }
    if (a.bcs) launch_fwd_rows<T, false, false, ZOH, 0, false, true>(a, main_grid, stream);
    else launch_fwd_rows<T, false, false, ZOH, 0>(a, main_grid, stream);
}

// complex state and time-invariant B and / or C
template <typename T, bool VEC, bool FULLN, bool ZOH>
static void launch_fwd_variant(const FwdArgs& a, hipStream_t stream)
{
    const int bcfix = ((a.flags & F_B_FIXED) ? 1 : 0) | ((a.flags & F_C_FIXED) ? 2 : 0);
    if constexpr (!ZOH) {
        if (a.flags & F_COMPLEX) {
            if (bcfix == 0) return launch_fwd_complex<T, VEC, FULLN, 0>(a, stream);
            if (bcfix == 1) return launch_fwd_complex<T, VEC, FULLN, 1>(a, stream);
            if (bcfix == 2) return launch_fwd_complex<T, VEC, FULLN, 2>(a, stream);
            return launch_fwd_complex<T, VEC, FULLN, 3>(a, stream);
        }
    }
    if (bcfix == 1) return launch_fwd_fixed<T, VEC, FULLN, ZOH, 1>(a, stream);
    if (bcfix == 2) return launch_fwd_fixed<T, VEC, FULLN, ZOH, 2>(a, stream);
    launch_fwd_fixed<T, VEC, FULLN, ZOH, 3>(a, stream);
}

template <typename T>
static void launch_fwd_io(const FwdArgs& a, hipStream_t stream)
{
    const bool zoh = a.flags & F_EXACT_ZOH_B, fulln = a.N == NPAD;
    if (!(a.flags & (F_B_FIXED | F_C_FIXED | F_COMPLEX))) {
        if (a.vec_ok) return launch_fwd_dpp<T, false>(a, stream);
        if (a.dpp_ok) return launch_fwd_dpp<T, true>(a, stream);
        if (zoh) return launch_fwd_scalar<T, true>(a, stream);
        return launch_fwd_scalar<T, false>(a, stream);
    }
    if (zoh) {   // built for the fastest and the most general shape only
        if (a.vec_ok && fulln) return launch_fwd_variant<T, true, true, true>(a, stream);
        return launch_fwd_variant<T, false, false, true>(a, stream);
    }
    if (a.vec_ok && fulln) return launch_fwd_variant<T, true, true, false>(a, stream);
    if (a.vec_ok) return launch_fwd_variant<T, true, false, false>(a, stream);
    launch_fwd_variant<T, false, false, false>(a, stream);
}

int launch_fwd(const FwdArgs& a, int io_dtype, hipStream_t stream)
{
    if (a.L == 0) {
        if (a.h_last) {
            const long n = (long)a.B * a.D * a.NS;
            copy_state_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream>>>(
                (a.flags & F_HAS_H0) ? a.h0 : nullptr, a.h_last, n);
        }
        return hipGetLastError() == hipSuccess ? 0 : -1;
    }
    if (io_dtype == 0) launch_fwd_io<float>(a, stream);
    else launch_fwd_io<bf16_t>(a, stream);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_step(const StepArgs& a, int io_dtype, hipStream_t stream)
{
    const long lanes = (long)a.B * a.D * 4;
    const dim3 grid((unsigned)((lanes + 255) / 256)), block(256);
    // the vector path also needs B_t / C_t rows aligned to 8 (bf16) or 16 (float) bytes,
    // which N == 16 and the element-aligned base pointers checked by the caller give only
    // when the bases themselves are that aligned
    const size_t va = io_dtype == 0 ? 16 : 8;
    const bool vec = a.N == NPAD && !(a.flags & (F_B_FIXED | F_C_FIXED)) && (a.bc_stride * (io_dtype == 0 ? 4 : 2)) % va == 0 &&
                     reinterpret_cast<uintptr_t>(a.B_t) % va == 0 &&
                     reinterpret_cast<uintptr_t>(a.C_t) % va == 0 && reinterpret_cast<uintptr_t>(a.A) % 16 == 0;
    const bool zoh = a.flags & F_EXACT_ZOH_B;
    // Several batch entries per thread once that still leaves every CU its 2048 threads
    if (vec && !zoh && !(a.flags & F_COMPLEX)) {
        const long full = 256L * 2048;
        const int rpt = (a.B % 4 == 0 && lanes / 4 >= full) ? 4 : (a.B % 2 == 0 && lanes / 2 >= full) ? 2 : 1;
        if (rpt > 1) {
            const dim3 g((unsigned)((lanes / rpt + 255) / 256));
            if (io_dtype == 0) {
                if (rpt == 4) step_multi_kernel<float, 4><<<g, block, 0, stream>>>(a);
                else step_multi_kernel<float, 2><<<g, block, 0, stream>>>(a);
            } else {
                if (rpt == 4) step_multi_kernel<bf16_t, 4><<<g, block, 0, stream>>>(a);
                else step_multi_kernel<bf16_t, 2><<<g, block, 0, stream>>>(a);
            }
            return hipGetLastError() == hipSuccess ? 0 : -1;
        }
    }
#define SS_LAUNCH_STEP(T, V, Z) step_kernel<T, V, Z><<<grid, block, 0, stream>>>(a)
    if (io_dtype == 0) {
        if (vec) { if (zoh) SS_LAUNCH_STEP(float, true, true); else SS_LAUNCH_STEP(float, true, false); }
        else { if (zoh) SS_LAUNCH_STEP(float, false, true); else SS_LAUNCH_STEP(float, false, false); }
    } else {
        if (vec) { if (zoh) SS_LAUNCH_STEP(bf16_t, true, true); else SS_LAUNCH_STEP(bf16_t, true, false); }
        else { if (zoh) SS_LAUNCH_STEP(bf16_t, false, true); else SS_LAUNCH_STEP(bf16_t, false, false); }
    }
#undef SS_LAUNCH_STEP
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <typename T>
static void launch_step_projected_t(const StepArgs& a, hipStream_t stream)
{
    // One workgroup per CU is the fastest arrangement (the state streams while the projection's
    // dependent steps run), so: 8-entry batch tiles while they fit the chip's 256 CUs once, 16-entry
    // tiles while those still do, and 8-entry tiles again beyond that, where two of them share a CU.  A token, us, 16 / 8 entries in between:
    // 64 x 4096 bf16 17.5 / 18.4, float32 20.6 / 21.7, 48 x 5120 17.4 / 17.5, 22.3 / 23.4, 128 x 2048 16.1 / 17.2, 18.0 / 19.2, but
    // 128 x 1536 13.9 / 13.7 (float32 15.6 / 16.0), 256 x 768 13.5 / 13.3.
    const long groups = (a.D + 63) / 64;
    const long n16 = groups * ((a.B + SP_MFMA_ROWS - 1) / SP_MFMA_ROWS), n8 = groups * ((a.B + 7) / 8);
    const bool wide = n8 > 256 && n16 <= 256;
    const dim3 grid((unsigned)groups, (unsigned)(wide ? (a.B + SP_MFMA_ROWS - 1) / SP_MFMA_ROWS : (a.B + 7) / 8));
    const dim3 block(SP_THREADS);
    if (a.conv_state) {   // a few entries only: never wide
        const dim3 g((unsigned)groups, (unsigned)((a.B + 7) / 8));
        if (a.N == NPAD) step_proj_kernel<T, true, 8, true><<<g, block, 0, stream>>>(a);
        else step_proj_kernel<T, false, 8, true><<<g, block, 0, stream>>>(a);
    } else if (a.N == NPAD) {
        if (wide) step_proj_kernel<T, true, SP_MFMA_ROWS><<<grid, block, 0, stream>>>(a);
        else step_proj_kernel<T, true, 8><<<grid, block, 0, stream>>>(a);
    } else {
        if (wide) step_proj_kernel<T, false, SP_MFMA_ROWS><<<grid, block, 0, stream>>>(a);
        else step_proj_kernel<T, false, 8><<<grid, block, 0, stream>>>(a);
    }
}

int launch_step_projected(const StepArgs& a, int io_dtype, hipStream_t stream)
{
    if (io_dtype == 0) launch_step_projected_t<float>(a, stream);
    else launch_step_projected_t<bf16_t>(a, stream);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace ss
