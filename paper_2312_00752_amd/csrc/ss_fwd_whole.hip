// Forward selective scan of grids that leave a compute unit one row group: whole rows, eight waves.
#include <type_traits>

#include "ss_kernels.h"
#include "ss_device.h"

namespace ss {

// The common path of scan_fwd_kernel (real state, selective B and C, rows of at least 8 steps) where there are at most as many row groups as
// compute units.  There a workgroup of four waves has a unit to itself and nothing to run while it waits at its barriers or for its
// own chains, and the split of the sequence that fills the unit with a second one costs an aggregate pass, about half of a main
// pass.  Here the two kinds of work run beside each other instead: waves 0..3 (state) carry the recurrence over chunk
// i while waves 4..7 (pointwise), one on the SIMD of each, finish chunk i - 1 and prepare chunk i + 1.  One barrier a
// chunk; every LDS tile exists twice (119 KB), and a chunk's inputs are requested three to four chunks ahead, which these
// waves have the registers for.  Same values and the same order of every sum as scan_fwd_kernel.
constexpr int WHOLE_THREADS = 2 * THREADS;

// the values exist from here on: their arithmetic does not sink to its uses
template <int SPL>
__device__ __forceinline__ void pin_slots(float (&v)[STATES_PER_LANE])
{
    if constexpr (SPL == 4) asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
    else if constexpr (SPL == 2) asm volatile("" : "+v"(v[0]), "+v"(v[1]));
    else asm volatile("" : "+v"(v[0]));
}

template <typename T, int SPL, bool ZOH, bool RAG>
__global__ void __launch_bounds__(WHOLE_THREADS, 2) scan_fwd_whole_kernel(const FwdArgs a)
{
    constexpr int NG = CHUNK_T / GROUP_T;
    __shared__ __attribute__((aligned(16))) float s_bc[2][2][NG][NPAD][GROUP_T];   // [chunk % 2][B, C]
    __shared__ __attribute__((aligned(16))) float s_dt[2][ROWS][TPAD];
    __shared__ __attribute__((aligned(16))) float s_du[2][ROWS][TPAD];
    __shared__ __attribute__((aligned(16))) float s_yp[2][NWAVES][ROWS][TPAD];

    const int tid = threadIdx.x & (THREADS - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool pointwise = __builtin_amdgcn_readfirstlane((int)threadIdx.x) >= THREADS;
    const int lane = tid & (WAVE - 1);
    const int groups = (a.D + ROWS - 1) / ROWS;
    const unsigned bx = xcd_contiguous(blockIdx.x, gridDim.x);
    const int b = bx / groups;
    const int d0 = (bx % groups) * ROWS;
    const int L = a.L, N = a.N, NS = a.NS;
    const int chunks = (L + CHUNK_T - 1) / CHUNK_T;
    const int rows_here = min(ROWS, a.D - d0);

    if (pointwise) {
        const bool has_z = a.flags & F_HAS_Z, has_D = a.flags & F_HAS_D, softplus = a.flags & F_DELTA_SOFTPLUS;
        const bool keep_y = has_z && a.ysave;
        // by fours in rows of any length as well: 8 x 1536 x 2047 forward + backward 742 us, by eights 795 (spills)
        constexpr int PC = slice_pieces<T, false>(), PE = SLICE / PC, PSTEP = CHUNK_T / PC, HALF4 = PC == 2 ? PSTEP / 4 : 1;
        typedef slice_io<T, PC> pio;
        const uint32_t esz = (uint32_t)sizeof(T);
        const int pr = PC == 2 ? pointwise_row_pitch5(tid) : pointwise_row_pitch9(tid), pq = tid & 3;
        const bool p_ok = d0 + pr < a.D;
        const int pd = p_ok ? d0 + pr : a.D - 1;
        const float bias = (a.flags & F_HAS_DELTA_BIAS) ? a.bias[pd] : 0.0f;
        const float Dsk = has_D ? a.Dskip[pd] : 0.0f;
        // whole slices: buffer resources over the workgroup's rows; rows past D lie beyond them
        const long wg_first = ((long)b * a.D + d0) * L;
        const uint32_t wg_bytes = (uint32_t)rows_here * (uint32_t)L * esz;
        const uint32_t row_off = (uint32_t)pr * (uint32_t)L * esz;
        const rsrc_t bu = make_rsrc(static_cast<const T*>(a.u) + wg_first, wg_bytes);
        const rsrc_t bd = make_rsrc(static_cast<const T*>(a.delta) + wg_first, wg_bytes);
        const rsrc_t bz = make_rsrc(static_cast<const T*>(has_z ? a.z : a.u) + wg_first, has_z ? wg_bytes : 0u);
        const rsrc_t bo = make_rsrc(static_cast<T*>(a.out) + wg_first, wg_bytes);
        const rsrc_t by = make_rsrc(static_cast<T*>(keep_y ? a.ysave : const_cast<void*>(a.u)) + wg_first, keep_y ? wg_bytes : 0u);
        // staging view: waves 0, 1 of these B, 2, 3 C; thread -> (state s_n, group of four steps s_tq) of the chunk
        const int s_which = w >> 1, s_n = (tid >> 3) & (NPAD - 1), s_tq = tid & (NG - 1);
        const rsrc_t bbc = make_rsrc(static_cast<const T*>(s_which ? a.Cm : a.Bm) + (long)b * a.bc_bstride, (uint32_t)N * (uint32_t)L * esz);
        const uint32_t bc_row_off = s_n < N ? (uint32_t)s_n * (uint32_t)L * esz : BUF_OFF;
        // rows of any length: plain pointers and offsets of this thread's row, clamped to a valid one
        constexpr bool OWN = own_rows<T, RAG, ZOH>();
        const int Li = OWN ? a.Li : L;
        const int r_row = min(pr, rows_here - 1);
        const uint32_t r_off = (uint32_t)r_row * (uint32_t)L * esz, r_off_i = (uint32_t)r_row * (uint32_t)Li * esz;
        const uint32_t r_off_bc = (uint32_t)min(s_n, N - 1) * (uint32_t)(OWN ? a.Lb : L) * esz;
        const long wg_first_i = ((long)b * a.D + d0) * Li;
        const T* const ru_p = static_cast<const T*>(a.u) + wg_first_i;
        const T* const rd_p = static_cast<const T*>(a.delta) + wg_first_i;
        const T* const rz_p = has_z ? static_cast<const T*>(a.z) + wg_first : ru_p;
        const T* const rbc_p = static_cast<const T*>(s_which ? a.Cm : a.Bm) + (long)b * a.bc_bstride;

        // inputs of chunk c in slot c % 4; what the second half of a chunk's work takes two chunks later in slot c % 2: u and z as they
        // came, or, in the kernel that would spill then (float rows of any length, 4 x 3072 x 2047 749 -> 717 us), the skip term and the gate
        constexpr bool RAW = !(RAG && sizeof(T) == 4);
        constexpr int RING = 4;
        typename pio::raw ru_[RING][PC], rd_[RING][PC], rz_[RING][PC], hu_[2][PC], hz_[2][PC];
        float skip_[2][SLICE], gate_[2][SLICE];
        typename io4<T>::raw rbc_[RING];
        // chunks c (into slot S) to c + COUNT - 1, tensor by tensor: bf16 by twos, the 128 bytes of a line; past the end the last
        // chunk again (rows of any length) or nothing
        auto issue = [&](int c, auto slot_tag, auto count_tag) {
            constexpr int S = decltype(slot_tag)::value, COUNT = decltype(count_tag)::value;
            uint32_t off[COUNT][PC], boff[COUNT];
#pragma unroll
            for (int k = 0; k < COUNT; ++k) {
                const int cc = RAG ? min(c + k, chunks - 1) : c + k, ts = cc * CHUNK_T + s_tq * GROUP_T;
#pragma unroll
                for (int p = 0; p < PC; ++p) {
                    const int t = cc * CHUNK_T + p * PSTEP + pq * PE;
                    if constexpr (RAG) off[k][p] = (uint32_t)row_piece(t, PE, L) * esz;
                    else off[k][p] = t < L ? row_off + (uint32_t)t * esz : BUF_OFF;
                }
                if constexpr (RAG) boff[k] = r_off_bc + (uint32_t)row_piece(ts, GROUP_T, L) * esz;
                else boff[k] = ts < L ? bc_row_off + (uint32_t)ts * esz : BUF_OFF;
            }
#pragma unroll
            for (int k = 0; k < COUNT; ++k)
#pragma unroll
                for (int p = 0; p < PC; ++p) {
                    if constexpr (RAG) ru_[S + k][p] = pio::load_elem(ru_p, r_off_i + off[k][p]);
                    else ru_[S + k][p] = pio::load_buf(bu, off[k][p]);
                }
#pragma unroll
            for (int k = 0; k < COUNT; ++k)
#pragma unroll
                for (int p = 0; p < PC; ++p) {
                    if constexpr (RAG) rd_[S + k][p] = pio::load_elem(rd_p, r_off_i + off[k][p]);
                    else rd_[S + k][p] = pio::load_buf(bd, off[k][p]);
                }
#pragma unroll
            for (int k = 0; k < COUNT; ++k)
#pragma unroll
                for (int p = 0; p < PC; ++p) {
                    if constexpr (RAG) rz_[S + k][p] = pio::load_elem(rz_p, has_z ? r_off + off[k][p] : 0u);
                    else rz_[S + k][p] = pio::load_buf(bz, off[k][p]);
                }
#pragma unroll
            for (int k = 0; k < COUNT; ++k) {
                if constexpr (RAG) rbc_[S + k] = io4<T>::load_elem(rbc_p, boff[k]);
                else rbc_[S + k] = io4<T>::load_buf(bbc, boff[k]);
            }
        };
        // this thread's share of the step sizes of a segment: what a backward pass in segments chains them by
        float sum_dt = 0.0f;
        float* sum_to = a.seg_sumdt + (long)b * a.D + pd;
        int sum_end = a.seg_sumdt ? min(a.seg_len, L) : 0x7fffffff;
        auto leave_sum = [&](int end) {   // the chunk that ends here is prepared
            if (end < sum_end) return;    // uniform
            sum_dt += __shfl_xor(sum_dt, 1);
            sum_dt += __shfl_xor(sum_dt, 2);
            if (p_ok && pq == 0) *sum_to = sum_dt;
            sum_dt = 0.0f;
            sum_to += (long)a.B * a.D;
            sum_end = sum_end >= L ? 0x7fffffff : min(sum_end + a.seg_len, L);
        };
        // what the recurrence over chunk c takes, into the tiles of parity S % 2
        auto prepare = [&](const int c, auto slot_tag) {
            constexpr int S = decltype(slot_tag)::value, H = S % 2;
            const int tc = c * CHUNK_T, t0 = tc + pq * PE;
            if constexpr (RAG) {
                if (tc + CHUNK_T > L) {   // uniform: the last chunk of a row that does not fill it
                    const int ts = tc + s_tq * GROUP_T;
#pragma unroll
                    for (int p = 0; p < PC; ++p) {
                        const int t = t0 + p * PSTEP, sh = t - row_piece(t, PE, L);
                        pio::drop(ru_[S][p], sh);
                        pio::drop(rd_[S][p], sh);
                        pio::drop(rz_[S][p], sh);
                    }
                    io4<T>::drop(rbc_[S], ts - row_piece(ts, GROUP_T, L));
                }
            }
            float bc4[GROUP_T], u8[SLICE], v8[SLICE], z8[SLICE];
            io4<T>::unpack(rbc_[S], bc4);
            if constexpr (RAG) {   // slots without a state
#pragma unroll
                for (int j = 0; j < GROUP_T; ++j) bc4[j] = s_n < N ? bc4[j] : 0.0f;
            }
            *reinterpret_cast<float4*>(&s_bc[H][s_which][s_tq][s_n][0]) = make_float4(bc4[0], bc4[1], bc4[2], bc4[3]);
            unpack_slice<pio, PC>(ru_[S], u8);
            unpack_slice<pio, PC>(rd_[S], v8);
            if constexpr (RAW) {
#pragma unroll
                for (int p = 0; p < PC; ++p) { hu_[H][p] = ru_[S][p]; hz_[H][p] = rz_[S][p]; }
            } else {
                if (has_z) unpack_slice<pio, PC>(rz_[S], z8);
#pragma unroll
                for (int j = 0; j < SLICE; ++j) {
                    skip_[H][j] = has_D ? Dsk * u8[j] : 0.0f;
                    gate_[H][j] = has_z ? z8[j] * sigmoid_fast(z8[j]) : 1.0f;
                }
            }
            float dt8[SLICE], du8[SLICE], bias_e[PC];   // an empty piece runs with dt = 0
#pragma unroll
            for (int p = 0; p < PC; ++p) bias_e[p] = RAG || t0 + p * PSTEP < L ? bias : (softplus ? -1e30f : 0.0f);
#pragma unroll
            for (int j = 0; j < SLICE; ++j) {
                float sp = v8[j] + bias_e[j / PE];
                if (softplus) sp = ss::softplus(sp);
                if constexpr (RAG) sp = t0 + j / PE * PSTEP + j % PE < L ? sp : 0.0f;
                dt8[j] = sp;
                du8[j] = ZOH ? u8[j] : sp * u8[j];
                sum_dt += sp;
            }
            float4* const pd4 = reinterpret_cast<float4*>(&s_dt[H][pr][pq * PE]);   // four steps each
            float4* const pu4 = reinterpret_cast<float4*>(&s_du[H][pr][pq * PE]);
            pd4[0] = make_float4(dt8[0], dt8[1], dt8[2], dt8[3]);
            pd4[HALF4] = make_float4(dt8[4], dt8[5], dt8[6], dt8[7]);
            pu4[0] = make_float4(du8[0], du8[1], du8[2], du8[3]);
            pu4[HALF4] = make_float4(du8[4], du8[5], du8[6], du8[7]);
        };
        typename pio::packed held_y[PC]{}, held_o[PC]{};
        // the waves' shares of chunk c (parity H) added up, the skip term, the gate; an even chunk's results wait for the odd one's
        auto finish = [&](const int c, auto parity_tag) {
            constexpr int H = decltype(parity_tag)::value;
            const int t0 = c * CHUNK_T + pq * PE;
            float u8[SLICE], z8[SLICE], y8[SLICE];
            if constexpr (RAW) {
                unpack_slice<pio, PC>(hu_[H], u8);
                if (has_z) unpack_slice<pio, PC>(hz_[H], z8);
            }
#pragma unroll
            for (int j = 0; j < SLICE; ++j) y8[j] = RAW ? (has_D ? Dsk * u8[j] : 0.0f) : skip_[H][j];
#pragma unroll
            for (int ww = 0; ww < NWAVES; ++ww) {
                const float4* const p4 = reinterpret_cast<const float4*>(&s_yp[H][ww][pr][pq * PE]);
                const float4 p0 = p4[0], p1 = p4[HALF4];
                y8[0] += p0.x; y8[1] += p0.y; y8[2] += p0.z; y8[3] += p0.w;
                y8[4] += p1.x; y8[5] += p1.y; y8[6] += p1.z; y8[7] += p1.w;
            }
            int nv[PC];
            uint32_t off[PC], off_e[PC];
            typename pio::packed py[PC], po[PC];
#pragma unroll
            for (int p = 0; p < PC; ++p) {
                nv[p] = min(max(L - t0 - p * PSTEP, 0), PE);
                const uint32_t at = row_off + (uint32_t)(t0 + p * PSTEP) * esz;
                off[p] = nv[p] == PE ? at : BUF_OFF;
                off_e[p] = H == 1 ? at - CHUNK_T * esz : BUF_OFF;
            }
            pack_slice<pio, PC>(y8, py);   // y before the gate, for the backward pass's dz (if kept)
            if (has_z) {
#pragma unroll
                for (int j = 0; j < SLICE; ++j) y8[j] *= RAW ? z8[j] * sigmoid_fast(z8[j]) : gate_[H][j];
            }
            pack_slice<pio, PC>(y8, po);
            if (H == 0 && c + 1 < chunks) {
#pragma unroll
                for (int p = 0; p < PC; ++p) { held_y[p] = py[p]; held_o[p] = po[p]; }
            } else if constexpr (RAG) {
                if (p_ok) {
                    T* const yp = static_cast<T*>(a.ysave) + wg_first_i;
                    T* const op = static_cast<T*>(a.out) + wg_first;
                    const uint32_t yt = r_off_i + (uint32_t)t0 * esz, ot = r_off + (uint32_t)t0 * esz;
#pragma unroll
                    for (int p = 0; p < PC; ++p) {
                        if (H == 1 && keep_y) pio::store_elem(yp, yt + (uint32_t)(p * PSTEP - CHUNK_T) * esz, held_y[p], PE);
                        if (H == 1) pio::store_elem(op, ot + (uint32_t)(p * PSTEP - CHUNK_T) * esz, held_o[p], PE);
                    }
#pragma unroll
                    for (int p = 0; p < PC; ++p) {
                        if (keep_y) pio::store_elem(yp, yt + (uint32_t)(p * PSTEP) * esz, py[p], nv[p]);
                        pio::store_elem(op, ot + (uint32_t)(p * PSTEP) * esz, po[p], nv[p]);
                    }
                }
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
        };
        constexpr int LOADS = sizeof(T) == 2 ? 2 : 1;   // chunks requested together
        issue(0, std::integral_constant<int, 0>{}, std::integral_constant<int, 2>{});
        __builtin_amdgcn_sched_barrier(0);
        issue(2, std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{});
        __builtin_amdgcn_sched_barrier(0);
        prepare(0, std::integral_constant<int, 0>{});
        if constexpr (LOADS == 1) issue(4, std::integral_constant<int, 0>{}, std::integral_constant<int, 1>{});
        leave_sum(CHUNK_T);
        __syncthreads();
        // Beside the recurrence over chunk i (i % 4 = K).  Nothing of it is conditional, also where chunk i + 1 is past the end (its tiles
        // are not read): where requests stand behind a branch, their registers are copied at its end, and waited for there.
        auto next = [&](const int i, auto k_tag) {
            constexpr int S = (decltype(k_tag)::value + 1) % RING;
            prepare(i + 1, std::integral_constant<int, S>{});
            if constexpr (LOADS == 1) issue(i + 1 + RING, std::integral_constant<int, S>{}, std::integral_constant<int, 1>{});
            else if constexpr (S % 2 == 1) issue(i + RING, std::integral_constant<int, S - 1>{}, std::integral_constant<int, 2>{});
            leave_sum((i + 2) * CHUNK_T);
            __syncthreads();
        };
        auto beside = [&](const int i, auto k_tag) {
            finish(i - 1, std::integral_constant<int, (decltype(k_tag)::value + 1) % 2>{});
            next(i, k_tag);
        };
        next(0, std::integral_constant<int, 0>{});
        for (int i = 1; i < chunks; i += RING) {
            beside(i, std::integral_constant<int, 1>{});
            if (i + 1 >= chunks) break;
            beside(i + 1, std::integral_constant<int, 2>{});
            if (i + 2 >= chunks) break;
            beside(i + 2, std::integral_constant<int, 3>{});
            if (i + 3 >= chunks) break;
            beside(i + 3, std::integral_constant<int, 0>{});
        }
        if (chunks & 1) finish(chunks - 1, std::integral_constant<int, 0>{});
        else finish(chunks - 1, std::integral_constant<int, 1>{});
        return;
    }

    // ---- state waves: lane -> row, wave -> states 4w..4w+3 (see scan_fwd_kernel) -------------------------------
    __builtin_amdgcn_s_setprio(2);
    const bool s_ok = d0 + lane < a.D;
    const int sd = s_ok ? d0 + lane : a.D - 1;
    const long srow = (long)b * a.D + sd;
    float A2[STATES_PER_LANE], invA[STATES_PER_LANE], h[STATES_PER_LANE];
    bool n_ok[STATES_PER_LANE];
#pragma unroll
    for (int k = 0; k < STATES_PER_LANE; ++k) {
        const int n = slot_state(w, k, a.il);
        n_ok[k] = n < N && k < SPL;
        const int nc = n_ok[k] ? n : 0;
        const float An = n_ok[k] ? a.A[(long)sd * NS + nc] : 0.0f;
        A2[k] = An * LOG2E;
        invA[k] = An != 0.0f ? 1.0f / An : 0.0f;
        h[k] = (n_ok[k] && (a.flags & F_HAS_H0)) ? a.h0[srow * NS + nc] : 0.0f;
    }
    const int pat = slot_state(w, lane & 3, a.il);   // the state of slot lane % 4
    // the state entering every CKPT_T-step block; nothing is written if there is no block or no buffer
    auto save_ckpt = [&](int block) {
        const bool on = a.ckpt && block * CKPT_T < L;
        const rsrc_t bc = make_rsrc(a.ckpt + (((long)block * a.B + b) * a.D + d0) * NPAD, on ? (uint32_t)rows_here * NPAD * (uint32_t)sizeof(float) : 0u);
        buf_store16(bc, (uint32_t)(lane * NPAD + w * STATES_PER_LANE) * (uint32_t)sizeof(float),
                    make_uint4(__float_as_uint(h[0]), __float_as_uint(h[1]), __float_as_uint(h[2]), __float_as_uint(h[3])));
    };
    __syncthreads();
    for (int i = 0; i < chunks; ++i) {
        const int H = i & 1;
        constexpr int AHEAD = ZOH ? 2 : 3;   // groups read before their turn: all of them take the registers that the lines below need
        float4 dtc[NG], duc[NG], Bpc[NG], Cpc[NG];
        auto read_group = [&](int g) {
            dtc[g] = *reinterpret_cast<const float4*>(&s_dt[H][lane][g * GROUP_T]);
            duc[g] = *reinterpret_cast<const float4*>(&s_du[H][lane][g * GROUP_T]);
            Bpc[g] = *reinterpret_cast<const float4*>(&s_bc[H][0][g][pat][0]);
            Cpc[g] = *reinterpret_cast<const float4*>(&s_bc[H][1][g][pat][0]);
        };
#pragma unroll
        for (int g = 0; g < AHEAD; ++g) read_group(g);
        save_ckpt(i * (CHUNK_T / CKPT_T));
        // The decays and inputs of a group are formed beside the chain and the read-outs of the group before it: left to itself the
        // compiler forms each right before its use, and the only state wave of a SIMD waits for every one.
        float ab[2][GROUP_T][STATES_PER_LANE], bu[2][GROUP_T][STATES_PER_LANE];
        auto form = [&](auto g_tag) {
            constexpr int g = decltype(g_tag)::value, P = g & 1;
#pragma unroll
            for (int j = 0; j < GROUP_T; ++j) {
                const float dt = f4_get(dtc[g], j), du = f4_get(duc[g], j);
                input_step_mfma<SPL>(bu[P][j], f4_get(Bpc[g], j), du);
#pragma unroll
                for (int k = 0; k < SPL; ++k) {
                    const float x2 = dt * A2[k];
                    ab[P][j][k] = exp2_fast(x2);                                 // Eq. 4
                    if (ZOH) bu[P][j][k] *= zoh_phi_fast(dt, x2, ab[P][j][k], invA[k]);
                }
            }
        };
        auto formed = [&](auto p_tag) {   // all of them by here
#pragma unroll
            for (int j = 0; j < GROUP_T; ++j) pin_slots<SPL>(ab[decltype(p_tag)::value][j]);
        };
        auto group = [&](auto g_tag) {
            constexpr int g = decltype(g_tag)::value, P = g & 1, tl = g * GROUP_T;
            if constexpr (g > 0 && tl % CKPT_T == 0) save_ckpt((i * CHUNK_T + tl) / CKPT_T);
            float yp[GROUP_T], hq[GROUP_T][STATES_PER_LANE];
            if constexpr (ZOH) __builtin_amdgcn_sched_barrier(0);
            if constexpr (g + AHEAD < NG) read_group(g + AHEAD);
            if constexpr (g + 1 < NG) form(std::integral_constant<int, g + 1>{});
#pragma unroll
            for (int j = 0; j < GROUP_T; ++j) {
#pragma unroll
                for (int k = 0; k < SPL; ++k) {
                    h[k] = fmaf(ab[P][j][k], h[k], bu[P][j][k]);                 // Eq. 2a
                    hq[j][k] = h[k];
                }
                if constexpr (SPL < 4) readout_step_dpp<SPL>(yp[j], f4_get(Cpc[g], j), h);   // Eq. 2b
            }
            if constexpr (SPL == 4) readout_group_dpp(yp, Cpc[g], hq);           // Eq. 2b
            *reinterpret_cast<float4*>(&s_yp[H][w][lane][tl]) = make_float4(yp[0], yp[1], yp[2], yp[3]);
            if constexpr (g + 1 < NG) formed(std::integral_constant<int, P ^ 1>{});
        };
        form(std::integral_constant<int, 0>{});
        formed(std::integral_constant<int, 0>{});
        group(std::integral_constant<int, 0>{});
        group(std::integral_constant<int, 1>{});
        group(std::integral_constant<int, 2>{});
        group(std::integral_constant<int, 3>{});
        group(std::integral_constant<int, 4>{});
        group(std::integral_constant<int, 5>{});
        group(std::integral_constant<int, 6>{});
        group(std::integral_constant<int, 7>{});
        __syncthreads();
    }
    if (a.h_last && s_ok) {
#pragma unroll
        for (int k = 0; k < STATES_PER_LANE; ++k)
            if (n_ok[k]) a.h_last[srow * NS + slot_state(w, k, a.il)] = h[k];
    }
}

template <typename T, bool RAG>
static void launch_whole(const FwdArgs& a, hipStream_t stream)
{
    const dim3 grid((unsigned)(a.B * ((a.D + ROWS - 1) / ROWS))), block(WHOLE_THREADS);
    const int spl = slots_for(a.N, a.il);
    if (a.flags & F_EXACT_ZOH_B) scan_fwd_whole_kernel<T, STATES_PER_LANE, true, RAG><<<grid, block, 0, stream>>>(a);
    else if (spl == 1) scan_fwd_whole_kernel<T, 1, false, RAG><<<grid, block, 0, stream>>>(a);
    else if (spl == 2) scan_fwd_whole_kernel<T, 2, false, RAG><<<grid, block, 0, stream>>>(a);
    else scan_fwd_whole_kernel<T, STATES_PER_LANE, false, RAG><<<grid, block, 0, stream>>>(a);
}

int launch_fwd_whole(const FwdArgs& a, int io_dtype, hipStream_t stream)
{
    if (a.L <= 0 || !a.dpp_ok || a.acc_y) return -1;
    if (io_dtype == 0) a.vec_ok ? launch_whole<float, false>(a, stream) : launch_whole<float, true>(a, stream);
    else a.vec_ok ? launch_whole<bf16_t, false>(a, stream) : launch_whole<bf16_t, true>(a, stream);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace ss
