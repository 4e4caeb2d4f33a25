// Forward pass of the GLA recurrence in one launch, two waves per 64-token chunk (bf16 hi/lo MFMA operands)
// (DiG paper, Sec. 3.5: chunks of M = 64 tokens computed on-chip; recurrence of Sec. 3.1 Eq. (attn_gla) rows 1-3 with
// beta = 1; heads of 17 .. 36 key channels and 33 .. 72 value columns, see onepass_covers).
//
// A work-group holds a span of NC chunks from the first load to the last store: every input is read once.  With the mid-chunk
// anchor m (after the chunk's 32nd token) and, per key channel, b_j the inclusive prefix sum of log2 alpha inside the chunk,
//     q~_j = q_j 2^(b_j - b_m),   k~_i = k_i 2^(b_m - b_i),   A = tril(Q~ K~^T)
//     U_c = 2^(b_C - b_m) K~^T V                      (the chunk's own state)
//     o_j = sum_{i<=j} A_ji v_i + q~_j P_c ,  P_c = 2^(b_m) S_c ,   S_{c+1} = 2^(b_C) S_c + U_c .
// The waves of a chunk own its 16-token tiles 0 and 3, and 1 and 2 (as many causal score tiles either way).  Lane (lm, g) =
// (lane % 16, lane / 16) holds of the tokens 16 t + lm the channels 16 u + 4 g .. + 3 and 32 + g, the layout of the MFMA
// operands, so q~ stays in registers; k~ goes to LDS for the partner and, with v (loaded straight to LDS), for the
// transposing reads of U_c.  The two waves wait for each other only (meet), so that a chunk whose rows have come is worked on
// while those of the next are on their way.  Then the group's threads add the U_c up to the span's state and publish it, the
// waves multiply the scores with v, the group looks back over the states that the spans before it have published until the
// decay leaves nothing of the earlier ones, turns every U_c into P_c, and each wave adds q~ P_c and stores.
//
// Looking back: a wave publishes its part of the span's state with device-scope stores, waits for them to arrive, and stores
// the call's nonce behind them; the same wave of a later span polls for that nonce.  A span waits for nothing before it publishes, and then
// only for earlier spans of its sequence.  These have smaller work-group numbers, are earlier ones of the same XCD, or are at the end of the range of
// spans of the XCD before (onepass_block), whose own waits go the same way, so the earliest span that has not published can always go on.  That holds while the GPU starts groups
// in the order of their numbers and has room for them; where something else is in the way, a poll can run out (`polls`), and the wave forms its part of
// the entering state from the inputs, token by token: every wait ends, and the result then differs in the order of the sum only.
// Operands are pairs of bf16 (hi + remainder; v as given), so products carry 16 bits; states, decays and sums are fp32.
//
// What bounds it on MI355X (36 / 72 channels, 1024 chunks in 256 groups of 4, 20 us): the rows of all groups come at the
// memory's rate until 7 us, then 9 us of dependent stages (scores and U_c 3, publishing and looking back 4, outputs 2), then the
// stores; at 4096 chunks two rounds of 28 us.  Against a state pass and an output pass, which read k, v and the gates twice (calls): 1024
// chunks 29.1 -> 21.7 us, 2048 with gate prologue and epilogue 43.4 -> 30.0, 4096 70.7 -> 65.4, and of those in a column scan whose gates
// hardly decay 89.8 -> 77.4 (a column's neighbours are loaded at the same time, so the lines that they share are fetched once); 1024 with the
// two-sided gate 45.4 -> 26.2.
// Why this shape: 128 registers and 20 KB of LDS a chunk, so 16 waves and 8 chunks on a compute unit (a wave per chunk with 256
// registers: 72 us at 4096 chunks where this took 64, and 31 at 1024 where this took 25).  Straight-line code for waves whose
// chunk is not there, arguments and lane numbers loaded afresh in each stage: with branches around the stages the registers
// spilled (150 us).  Tried: publishing in the XCD's L2 first (an L1 may hold a neighbouring span's line: wrong), group barriers for
// the two waves of a chunk (up to 4 us of waiting for the slowest rows).
#include <type_traits>

#include "gla_common.h"
#include "gla_onepass_plan.h"
#include "gla_onepass_util.h"

namespace gla {
namespace {

typedef unsigned long long flag_t;

template <typename HD, int NC, bool FUSE, bool BETA>
struct WLayout {
    static constexpr int kRow = 72;                                  // bf16 per row of k~ (32 hi, 32 lo, 4 x (hi, lo))
    static constexpr int kState = 36;                                // floats per value column of a state
    static constexpr int kUBytes = HD::NV * kState * 4;
    static constexpr int kKBytes = kChunk * kRow * 2 > kUBytes ? kChunk * kRow * 2 : kUBytes;   // k~, then U_c, then P_c
    static constexpr int kVRows = kChunk * HD::NV * 2;               // v, as it comes in: 16-byte pieces row by row
    static constexpr int kVBytes = (BETA ? 2 : 1) * kVRows;          // (v~ of the two-sided gate: hi rows, then lo rows)
    static constexpr int kOne = kKBytes + kVBytes;
    static constexpr int oDecay = NC * kOne;                         // float[NC][4][36]: totals of the tiles, then kDecay ..
    static constexpr int kCols = 16 * HD::NX;
    static constexpr int oCols = oDecay + NC * 4 * kState * 4;       // float[NC][4][kCols]: the same of the value columns (BETA)
    static constexpr int oPair = oCols + (BETA ? NC * 4 * kCols * 4 : 0);    // int[2 NC]: how often a wave has met its partner
    static constexpr int oLn = oPair + 2 * NC * 4;                   // float[2][16 NX]: LayerNorm weight, bias (FUSE)
    static constexpr int kBytes = oLn + (FUSE ? 2 * 16 * HD::NX * 4 : 0);
    static_assert(kBytes <= 160 * 1024 / (BETA ? 4 / NC : 8 / NC), "16 waves on a compute unit, 8 with the two-sided gate");
};
// Accesses at device scope (sc1): past the L1s and past the L2s, of which every XCD has one of its own
constexpr int kDeviceScope = 16;
__device__ inline void publish(Rsrc r, uint32_t at, uint32_t from, float x) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), r, (int)at, (int)from, kDeviceScope);
}
__device__ inline float published(Rsrc r, uint32_t at, uint32_t from) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)at, (int)from, kDeviceScope));
}
__device__ inline f32x4 published4(Rsrc r, uint32_t at, uint32_t from) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)at, (int)from, kDeviceScope));
}

typedef const __attribute__((address_space(4))) OnePassParams *Args;

// FUSE = the gate prologue and the optional output epilogue; ACC = rows are added to the fp32 rows already in `out`; BETA = the
// two-sided gate (log_beta): with c_j the prefix sums of log2 beta per value column, v~_i = v_i 2^(c_m - c_i) takes the place of v as
// a hi/lo pair, the state decays by 2^(c_C) as well, and output rows are scaled by 2^(c_j - c_m).
template <typename HD, int NC, bool FUSE, bool ACC, typename TOut, bool BETA>
__global__ __launch_bounds__(128 * NC, BETA ? 2 : 4) void chunk_pair_kernel(OnePassParams) {
    const Args args = (Args)__builtin_amdgcn_kernarg_segment_ptr();
    using L = WLayout<HD, NC, FUSE, BETA>;
    static_assert(!BETA || (!FUSE && !ACC), "two-sided gate: from log gates, no sums");
    constexpr int DT = HD::DT, NX = HD::NX, NG = 8 + DT, NT = 128 * NC, NW = 2 * NC;
    constexpr int RS = L::kRow, US = L::kState;
    constexpr int VP = HD::NV / 8;                    // 16-byte pieces of a v row; a chunk's go to LDS 64 at a time
    constexpr int kQuads = HD::NV * (8 + DT);         // (value column, four channels) pieces of a state
    constexpr int KQ = (kQuads + NT - 1) / NT;        // ... of a thread

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int W = w & 1;                              // tiles W and 3 - W of chunk w / 2
    unsigned char *mine = smem + (w >> 1) * L::kOne;
    uint16_t *s_k = reinterpret_cast<uint16_t *>(mine);
    float *s_u = reinterpret_cast<float *>(mine);
    uint16_t *s_v = reinterpret_cast<uint16_t *>(mine + L::kKBytes);
    float *s_decay = reinterpret_cast<float *>(smem + L::oDecay);
    float *my_decay = s_decay + (w >> 1) * 4 * US;
    float *s_cols = reinterpret_cast<float *>(smem + L::oCols), *my_cols = s_cols + (w >> 1) * 4 * L::kCols;
    float *s_lnw = reinterpret_cast<float *>(smem + L::oLn), *s_lnb = s_lnw + 16 * NX;

    // The two waves of a chunk wait for each other without the group's others (a chunk whose rows have come is not held up by
    // those of the next).  LDS accesses of a wave are done in order.
    int *s_pair = reinterpret_cast<int *>(smem + L::oPair);
    int met = 0;
    auto meet = [&]() {
        ++met;
        asm volatile("" ::: "memory");
        __hip_atomic_store(s_pair + w, met, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(s_pair + (w ^ 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) < met) {
        }
        asm volatile("" ::: "memory");
    };
    if (tid < NW) s_pair[tid] = 0;

    // what the first loads need, all at once: a group's first access to a line of its arguments takes as long as one to memory (with a load at each use, in five
    // dependent rounds, a launch took 0.9 us longer: 1024 chunks in a reversed column scan 22.7 us, now 21.7)
    int B = args->B, H = args->H, T = args->T, dk = args->dk, dv = args->dv, grid_h = args->grid_h, grid_w = args->grid_w,
        scan_dir = args->scan_dir, nspans = args->nspans, span_len = args->span_len, st_k = args->st_k, st_v = args->st_v;
    long long sb_k = args->sb_k, sh_k = args->sh_k, sb_v = args->sb_v, sh_v = args->sh_v;
    const float *initial = args->initial_state;
    const void *from_v = args->v, *from_k = args->k, *from_q = args->q, *from_gate = FUSE ? args->z_gate : (const void *)args->log_alpha;
    asm volatile("" : "+s"(B), "+s"(H), "+s"(T), "+s"(dk), "+s"(dv), "+s"(grid_h), "+s"(grid_w), "+s"(scan_dir), "+s"(nspans), "+s"(span_len),
                 "+s"(st_k), "+s"(st_v), "+s"(sb_k), "+s"(sh_k), "+s"(sb_v), "+s"(sh_v), "+s"(initial), "+s"(from_v), "+s"(from_k), "+s"(from_q), "+s"(from_gate));
    __syncthreads();           // (the counters of meet are there)
    const int blk = onepass_block((int)blockIdx.x, B * H * nspans, onepass_in_ranges(B * H, nspans, onepass_resident(NC, BETA)));
    const int bh = blk / nspans, sp = blk - bh * nspans;
    const int s_begin = sp * span_len, s_end = min(T, s_begin + span_len);

    const int batch = bh / H, head = bh - batch * H;
    const size_t base_k = (size_t)batch * (size_t)sb_k + (size_t)head * (size_t)sh_k,
                 base_v = (size_t)batch * (size_t)sb_v + (size_t)head * (size_t)sh_v;
    const uint32_t dk2 = 2u * (uint32_t)st_k, dv2 = 2u * (uint32_t)st_v;   // bytes from one bf16 row to the next
    const uint32_t bytes_k = (uint32_t)(T - 1) * dk2 + 2u * (uint32_t)dk, bytes_v = (uint32_t)(T - 1) * dv2 + 2u * (uint32_t)dv;
    constexpr uint32_t OE = sizeof(TOut) / 2;         // bytes of `out` per byte of a bf16 row
    auto view_k = [&](const void *x, uint32_t bytes) { return view(static_cast<const char *>(x) + afresh(base_k) * bytes, bytes_k / 2 * bytes); };
    auto view_v = [&](const void *x, uint32_t bytes) { return view(static_cast<const char *>(x) + afresh(base_v) * bytes, bytes_v / 2 * bytes); };
    const bool epilogue = FUSE && args->r_pre != nullptr;   // uniform
    if constexpr (FUSE) {
        if (epilogue) {
            const int h = bh % ARG->H;
            for (int n = tid; n < dv; n += NT) {
                s_lnw[n] = ARG->ln_weight != nullptr ? ARG->ln_weight[h * dv + n] : 1.f;
                s_lnb[n] = ARG->ln_bias != nullptr ? ARG->ln_bias[h * dv + n] : 0.f;
            }
        }
    }
    auto gate1 = [&](float z) {     // log2(sigmoid(z)) / tau = (min(t, 0) - log2(1 + 2^-|t|)) / tau with t = z log2(e)
        const float t = z * kLog2e;
        return (fminf(t, 0.f) - __builtin_amdgcn_logf(1.f + exp2_fast(-fabsf(t)))) * ARG->inv_tau;
    };

    // this thread's pieces of a state: column qn, channels 4 qc .. + 3 (value columns on neighbouring lanes)
    struct Pieces {
        int n[KQ], c[KQ];
        uint32_t at[KQ], at_dk[KQ];      // byte offsets of the first channel in a [dk][dv] state, of the channels in [dk] (or nowhere)
    };
    auto pieces = [&](int thread) {
        Pieces q;
#pragma unroll
        for (int i = 0; i < KQ; ++i) {
            const int idx = min(thread + NT * i, kQuads - 1);      // threads past the end repeat the last piece
            q.c[i] = idx / HD::NV;
            q.n[i] = idx - q.c[i] * HD::NV;
            const bool real = 4 * q.c[i] < dk && q.n[i] < dv;      // (dk is a multiple of 4)
            q.at[i] = real ? 4u * (uint32_t)(4 * q.c[i] * dv + q.n[i]) : kNowhere;
            q.at_dk[i] = real ? 16u * (uint32_t)q.c[i] : kNowhere;
        }
        return q;
    };
    f32x4 S[KQ];
#pragma unroll
    for (int i = 0; i < KQ; ++i) S[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto owns = [&](int i) { return tid + NT * i < kQuads; };
    const uint32_t ne4 = 4u * (uint32_t)(dk * dv), dv4 = 4u * (uint32_t)dv;
    auto view_init = [&]() { return view(ARG->initial_state + (size_t)afresh(bh) * dk * dv, ne4); };
    if (sp == 0 && initial != nullptr) {
        const Pieces q = pieces(tid);
        const Rsrc b_init = view_init();
#pragma unroll
        for (int i = 0; i < KQ; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) S[i][r] = fetch<float>(b_init, q.at[i] + r * dv4);
    }

    {
        const int c_begin = s_begin + (w >> 1) * kChunk;
        // (Waves whose chunk is not there go along with rows of zeros: straight-line code keeps the registers.)
        using GatePiece = std::conditional_t<FUSE, u32x2, f32x4>;
        using GateTail = std::conditional_t<FUSE, uint16_t, float>;
        // each lane finds one row's token (a row past the span's end repeats the last)
        int tok;
        {
            const int col_len = scan_dir >= 2 ? grid_h : 1;       // (uniform)
            const int s0 = min(c_begin + (recompute_per_chunk(tid) & 63), s_end - 1), s = (scan_dir & 1) ? T - 1 - s0 : s0;
            const int tc = s / col_len;
            tok = (s - tc * col_len) * grid_w + tc;
        }
        auto token_of = [&](int j) { return (uint32_t)__builtin_amdgcn_ds_bpermute(4 * j, tok); };
        // rows of v's shape straight to LDS, half of the pieces from either wave of the chunk
        auto v_to_lds = [&](Rsrc from) {
            const int lane = recompute_per_chunk(tid) & 63;
#pragma unroll
            for (int i = 0; i < (VP + 1) / 2; ++i) {
                if (2 * i + W < VP) {
                    const int at = lane + 64 * (2 * i + W), vr = at / VP, vp = at - vr * VP;
                    const int piece = DT ? vp : vp ^ (2 * ((vr >> 1) & 3));
                    load_to_lds(from, mine + L::kKBytes + 1024 * (2 * i + W), token_of(vr) * dv2 + 16u * (uint32_t)min(piece, dv / 8 - 1));
                }
            }
        };
        u32x4 qh[2], ql[2];
        uint32_t qt[2];
        uint32_t rowv[2];
        const int tile[2] = {W, 3 - W};
        float b[2][NG];
        u32x2 rk[2][2], rq[2][2];
        uint32_t rkt[2], rqt[2];
        u32x2 rv[2][BETA ? NX : 1];                    // BETA: v and the sums of log2 beta, columns 16 x + 4 g .. + 3
        f32x4 cx[2][BETA ? NX : 1];
        {
            LANE;
            uint32_t chb[2];                     // byte offset of the lane's units in a bf16 row
#pragma unroll
            for (int u = 0; u < 2; ++u) chb[u] = 16 * u + 4 * g < dk ? 2u * (uint32_t)(16 * u + 4 * g) : kNowhere / 2;
            const uint32_t tcb = 32 + g < dk ? 2u * (uint32_t)(32 + g) : kNowhere / 2;    // the same for the tail channel
            uint32_t row[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const bool there = c_begin + 16 * tile[t] + lm < s_end;
                const uint32_t tk = token_of(16 * tile[t] + lm);
                row[t] = there ? tk * dk2 : kNowhere / 2;
                rowv[t] = there ? tk * dv2 : kNowhere / 2;
            }
            if constexpr (!BETA) v_to_lds(view_v(from_v, 2));       // (a row that is not there meets k~ = 0; columns past dv are not read)
            const Rsrc bg = view_k(from_gate, FUSE ? 2 : 4), bk = view_k(from_k, 2), bq = view_k(from_q, 2);
            GatePiece la[2][2];
            GateTail lat[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int u = 0; u < 2; ++u) la[t][u] = fetch<GatePiece>(bg, FUSE ? row[t] + chb[u] : f32_at(row[t], chb[u]));
                if constexpr (DT) lat[t] = fetch<GateTail>(bg, FUSE ? row[t] + tcb : f32_at(row[t], tcb));
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int u = 0; u < 2; ++u) rk[t][u] = fetch<u32x2>(bk, row[t] + chb[u]);
                if constexpr (DT) rkt[t] = fetch<uint16_t>(bk, row[t] + tcb);
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) {
#pragma unroll
                for (int u = 0; u < 2; ++u) rq[t][u] = fetch<u32x2>(bq, row[t] + chb[u]);
                if constexpr (DT) rqt[t] = fetch<uint16_t>(bq, row[t] + tcb);
            }

            if constexpr (BETA) {
                const Rsrc bv = view_v(ARG->v, 2), bb = view_v(ARG->log_beta, 4);
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int x = 0; x < NX; ++x) {
                        const uint32_t col = 4 * g + 16 * x < dv ? 8u * (uint32_t)g + 32u * (uint32_t)x : kNowhere / 2;
                        cx[t][x] = fetch<f32x4>(bb, f32_at(rowv[t], col));
                        rv[t][x] = fetch<u32x2>(bv, rowv[t] + col);
                    }
            }

            // ---- gates: prefix sums inside the 16-token tiles, totals of the tiles ----
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if constexpr (FUSE) {
                    const float least = c_begin + 16 * tile[t] + lm < s_end ? kLeastGate2 : 0.f;   // (a row that is not there decays by nothing)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            b[t][4 * u + 2 * h] = fmaxf(gate1(bf16_lo_as_float(la[t][u][h])), least);
                            b[t][4 * u + 2 * h + 1] = fmaxf(gate1(bf16_hi_as_float(la[t][u][h])), least);
                        }
                    if constexpr (DT) b[t][8] = fmaxf(gate1(bf16_bits_to_float(lat[t])), least);
                    row_scan16x4(b[t][0], b[t][1], b[t][2], b[t][3]);
                    row_scan16x4(b[t][4], b[t][5], b[t][6], b[t][7]);
                } else {
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int e = 0; e < 4; ++e) b[t][4 * u + e] = la[t][u][e] * kLog2e;
                    if constexpr (DT) b[t][8] = fmaxf(lat[t] * kLog2e, kLeastGate2);
                    row_scan16x4_least(b[t][0], b[t][1], b[t][2], b[t][3], kLeastGate2);
                    row_scan16x4_least(b[t][4], b[t][5], b[t][6], b[t][7], kLeastGate2);
                }
                if constexpr (DT) b[t][8] = row_scan16(b[t][8]);
                if constexpr (BETA) {
#pragma unroll
                    for (int x = 0; x < NX; ++x) {
                        float c0 = cx[t][x][0] * kLog2e, c1 = cx[t][x][1] * kLog2e, c2 = cx[t][x][2] * kLog2e, c3 = cx[t][x][3] * kLog2e;
                        row_scan16x4_least(c0, c1, c2, c3, kLeastGate2);
                        cx[t][x] = f32x4{c0, c1, c2, c3};
                        if (lm == 15) *reinterpret_cast<f32x4 *>(my_cols + tile[t] * L::kCols + 16 * x + 4 * g) = cx[t][x];
                    }
                }
                if (lm == 15) {
                    float *d = my_decay + tile[t] * US;
                    *reinterpret_cast<f32x4 *>(d + 4 * g) = f32x4{b[t][0], b[t][1], b[t][2], b[t][3]};
                    *reinterpret_cast<f32x4 *>(d + 16 + 4 * g) = f32x4{b[t][4], b[t][5], b[t][6], b[t][7]};
                    if constexpr (DT) d[32 + g] = b[t][8];
                }
            }
        }
        meet();
        {
            LANE;
            // ---- relative to the anchor: tiles 0, 1 lie before it (-(t0 + t1), -t1), tile 2 starts at it, tile 3 follows tile
            // 2 (+t2).  Gated operands: k~ to LDS, q~ in registers ----
            const float first = W == 0 ? 1.f : 0.f;
            float off[2][NG];
#pragma unroll
            for (int i = 0; i < NG; i += 4) {
                if (i < 8) {
                    const float *d = my_decay + 4 * i + 4 * g;
                    const f32x4 t0 = *reinterpret_cast<const f32x4 *>(d), t1 = *reinterpret_cast<const f32x4 *>(d + US),
                                t2 = *reinterpret_cast<const f32x4 *>(d + 2 * US);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        off[0][i + e] = -fmaf(first, t0[e], t1[e]);
                        off[1][i + e] = first * t2[e];
                    }
                } else {
                    const float *d = my_decay + 32 + g;
                    off[0][i] = -fmaf(first, d[0], d[US]);
                    off[1][i] = first * d[2 * US];
                }
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                float eq[NG], ek[NG];
#pragma unroll
                for (int i = 0; i < NG; ++i) {
                    const float ex = b[t][i] + off[t][i];
                    // (clamped so that gates beyond the range leave nothing infinite; q~ can only exceed 1 before the
                    // anchor, k~ only behind it)
                    eq[i] = exp2_fast(t == 0 ? fminf(ex, kMaxExp2) : ex);
                    ek[i] = exp2_fast(t == 0 ? -ex : fminf(-ex, kMaxExp2));
                }
                u32x4 kh, kl;
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        SPLIT_PAIR(bf16_lo_as_float(rk[t][u][h]) * ek[4 * u + 2 * h], bf16_hi_as_float(rk[t][u][h]) * ek[4 * u + 2 * h + 1],
                                   kh[2 * u + h], kl[2 * u + h]);
                        SPLIT_PAIR(bf16_lo_as_float(rq[t][u][h]) * eq[4 * u + 2 * h], bf16_hi_as_float(rq[t][u][h]) * eq[4 * u + 2 * h + 1],
                                   qh[t][2 * u + h], ql[t][2 * u + h]);
                    }
                uint16_t *krow = s_k + (16 * tile[t] + lm) * RS;
                *reinterpret_cast<u32x4 *>(krow + 8 * g) = kh;
                *reinterpret_cast<u32x4 *>(krow + 32 + 8 * g) = kl;
                if constexpr (DT) {
                    const float kx = bf16_lo_as_float(rkt[t]) * ek[NG - 1];
                    const uint32_t hh = pack_bf16(kx, kx);
                    const float rem = kx - bf16_lo_as_float(hh);
                    *reinterpret_cast<uint32_t *>(krow + 64 + 2 * g) = (hh & 0xffffu) | (pack_bf16(rem, rem) << 16);
                    const float qx = bf16_lo_as_float(rqt[t]) * eq[NG - 1];
                    const uint32_t qhh = pack_bf16(qx, qx);
                    const float qrem = qx - bf16_lo_as_float(qhh);
                    qt[t] = (qhh & 0xffffu) | (pack_bf16(qrem, qrem) << 16);           // slots hi, lo, hi, lo
                }
            }
            if constexpr (BETA) {
#pragma unroll
                for (int x = 0; x < NX; ++x) {
                    const float *d = my_cols + 16 * x + 4 * g;
                    const f32x4 t0 = *reinterpret_cast<const f32x4 *>(d), t1 = *reinterpret_cast<const f32x4 *>(d + L::kCols),
                                t2 = *reinterpret_cast<const f32x4 *>(d + 2 * L::kCols);
                    cx[0][x] -= first * t0 + t1;
                    cx[1][x] += first * t2;
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        f32x4 y;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const float vv = r & 1 ? bf16_hi_as_float(rv[t][x][r >> 1]) : bf16_lo_as_float(rv[t][x][r >> 1]);
                            y[r] = vv * exp2_fast(fminf(-cx[t][x][r], kMaxExp2));
                        }
                        u32x2 h, l;
                        SPLIT_PAIR(y[0], y[1], h[0], l[0]);
                        SPLIT_PAIR(y[2], y[3], h[1], l[1]);
                        uint16_t *vrow = s_v + (16 * tile[t] + lm) * HD::NV + ((16 * x) ^ (DT ? 0 : 16 * ((lm >> 1) & 3))) + 4 * g;
                        if (16 * x + 4 * g < HD::NV) {
                            *reinterpret_cast<u32x2 *>(vrow) = h;
                            *reinterpret_cast<u32x2 *>(vrow + kChunk * HD::NV) = l;
                        }
                    }
                }
            } else {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // (v is in LDS)
            }
        }
        meet();
        // This lane, and its operand of the products with v: transposing reads of columns 16 x + lm, slot (g, e) of step q32 = token
        // 32 q32 + 16 (e / 4) + 4 g + e % 4; part 1: the lo rows.  (Rows of 128 bytes: tiles change places, see load_to_lds.)
#define TR_LANE \
        LANE; \
        const int tr_row = lm >> 2, tr_col = 4 * (lm & 3);     /* token-in-4 and column quad of this lane */ \
        const uint16_t *vtr = s_v + (4 * g + tr_row) * HD::NV + tr_col; \
        const int v_swz = DT ? 0 : 16 * ((2 * g + (tr_row >> 1)) & 3); \
        auto v_frag = [&](int q32, int x, int part = 0) { \
            const u32x2 lo = lds_read_tr(vtr + (32 * q32 + kChunk * part) * HD::NV + ((16 * x) ^ v_swz)); \
            const u32x2 hi = lds_read_tr(vtr + (32 * q32 + 16 + kChunk * part) * HD::NV + ((16 * x) ^ v_swz)); \
            return u32x4{lo[0], lo[1], hi[0], hi[1]}; \
        }
        // slots hi, hi, lo, lo of a tail channel's pair
        auto tail_operand = [](uint32_t pair) {
            return u32x4{__builtin_amdgcn_perm(pair, pair, 0x01000100u), __builtin_amdgcn_perm(pair, pair, 0x03020302u), 0, 0};
        };
        u32x4 pah[3], pal[3];                          // scores of tile W; of tile 3 - W, tokens 0 .. 31 and 32 .. 63
        f32x4 acc[2][2 + DT], acc4[1 + DT];            // column tiles W and W + 2; of tile 4 the channels of tile W, and the tail's
        {
            TR_LANE;
            // (the totals of the tiles have been read)
            if (W == 0 && lane < US) {
                float *d = my_decay + lane;
                const float m = d[0] + d[US], e = d[2 * US] + d[3 * US];
                d[kDecay * US] = exp2_fast(m + e);
                d[kToAnchor * US] = exp2_fast(m);
                d[kFromAnchor * US] = exp2_fast(e);
                d[kLogDecay * US] = m + e;
            }
            if constexpr (BETA) {
                if (W == 1) {
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        if (lane + 64 * i < L::kCols) {
                            float *d = my_cols + lane + 64 * i;
                            const float m = d[0] + d[L::kCols], e = d[2 * L::kCols] + d[3 * L::kCols];
                            d[kDecay * L::kCols] = exp2_fast(m + e);
                            d[kToAnchor * L::kCols] = exp2_fast(m);
                            d[kFromAnchor * L::kCols] = exp2_fast(e);
                            d[kLogDecay * L::kCols] = m + e;
                        }
                    }
                }
            }
            // ---- scores, transposed: lane (lm, g) gets A[i = 16 t + lm][j = 16 jt + 4 g + r]: of tile W with token tile 0, of tile
            // 3 - W with 0, 1, 2, and the last one of its two diagonals: tile 3 with 3 (W = 0), 1 with 1 (W = 1) ----
            f32x4 d[5];
            const u32x4 dqh = W ? qh[0] : qh[1], dql = W ? ql[0] : ql[1];
            const uint32_t dqt = W ? qt[0] : qt[1];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint16_t *krow = s_k + (16 * (j < 3 ? j : (W ? 1 : 3)) + lm) * RS;
                const u32x4 kh = *reinterpret_cast<const u32x4 *>(krow + 8 * g), kl = *reinterpret_cast<const u32x4 *>(krow + 32 + 8 * g);
                u32x4 kt = u32x4{0, 0, 0, 0};
                if constexpr (DT) kt = tail_operand(*reinterpret_cast<const uint32_t *>(krow + 64 + 2 * g));
                auto product = [&](u32x4 h, u32x4 l, uint32_t t) {
                    f32x4 x = mfma(kh, h, f32x4{0.f, 0.f, 0.f, 0.f});
                    x = mfma(kh, l, x);
                    x = mfma(kl, h, x);
                    x = mfma(kl, l, x);
                    if constexpr (DT) x = mfma(kt, u32x4{t, t, 0, 0}, x);
                    return x;
                };
                if (j == 0) d[0] = product(qh[0], ql[0], qt[0]);
                d[j + 1] = j < 3 ? product(qh[1], ql[1], qt[1]) : product(dqh, dql, dqt);
            }
            // causal masks: d[4] always, d[0] for W = 0 (tile 0), d[3] for W = 1 (tile 2)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool past = 4 * g + r > lm;
                d[4][r] = past ? 0.f : d[4][r];
                d[0][r] = past && W == 0 ? 0.f : d[0][r];
                d[3][r] = past && W == 1 ? 0.f : d[3][r];
            }
            auto split = [&](f32x4 x, u32x2 &h, u32x2 &l) {
                const HiLo a = split_pair_val(x[0], x[1]), c = split_pair_val(x[2], x[3]);
                h = u32x2{a.hi, c.hi};
                l = u32x2{a.lo, c.lo};
            };
            u32x2 h, l, h2, l2, eh, el;
            const u32x2 none = u32x2{0, 0};
            split(d[4], eh, el);
            split(d[0], h, l);
            pah[0] = u32x4{h[0], h[1], W ? eh[0] : 0, W ? eh[1] : 0};
            pal[0] = u32x4{l[0], l[1], W ? el[0] : 0, W ? el[1] : 0};
            split(d[1], h, l);
            split(d[2], h2, l2);
            pah[1] = u32x4{h[0], h[1], h2[0], h2[1]};
            pal[1] = u32x4{l[0], l[1], l2[0], l2[1]};
            split(d[3], h, l);
            h2 = W ? none : eh;
            l2 = W ? none : el;
            pah[2] = u32x4{h[0], h[1], h2[0], h2[1]};
            pal[2] = u32x4{l[0], l[1], l2[0], l2[1]};
            // ---- U_c = 2^(b_C - b_m) K~^T V: main tile ct, column tile x: channel 16 (g & 1) + 4 (2 ct + g / 2) + r, column
            // 16 x + lm; tail tile: rows hi, lo of the channels 32 + 2 g and 33 + 2 g (g < 2) ----
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int ct = 0; ct < 2 + DT; ++ct) acc[i][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < 1 + DT; ++i) acc4[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            const uint16_t *ktr = s_k + (4 * g + tr_row) * RS + tr_col;
            auto k_frag = [&](int q32, int col) {
                const u32x2 lo = lds_read_tr(ktr + 32 * q32 * RS + col);
                const u32x2 hi = lds_read_tr(ktr + (32 * q32 + 16) * RS + col);
                return u32x4{lo[0], lo[1], hi[0], hi[1]};
            };
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                u32x4 kf[4 + DT];
#pragma unroll
                for (int i = 0; i < 4 + DT; ++i) kf[i] = k_frag(q, 16 * i);      // hi of ct 0, 1; lo of ct 0, 1; tail
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const u32x4 vf = v_frag(q, 2 * i + W);
                    acc[i][0] = mfma(kf[0], vf, acc[i][0]);
                    acc[i][1] = mfma(kf[1], vf, acc[i][1]);
                    if constexpr (DT) acc[i][2] = mfma(kf[4], vf, acc[i][2]);
                    acc[i][0] = mfma(kf[2], vf, acc[i][0]);
                    acc[i][1] = mfma(kf[3], vf, acc[i][1]);
                    if constexpr (BETA) {
                        const u32x4 vl = v_frag(q, 2 * i + W, 1);
                        acc[i][0] = mfma(kf[0], vl, acc[i][0]);
                        acc[i][1] = mfma(kf[1], vl, acc[i][1]);
                        if constexpr (DT) acc[i][2] = mfma(kf[4], vl, acc[i][2]);
                        acc[i][0] = mfma(kf[2], vl, acc[i][0]);
                        acc[i][1] = mfma(kf[3], vl, acc[i][1]);
                    }
                }
                if constexpr (NX == 5) {
                    const u32x4 vf = v_frag(q, 4), kh = k_frag(q, 16 * W), kl = k_frag(q, 32 + 16 * W);
                    acc4[0] = mfma(kh, vf, acc4[0]);
                    if constexpr (DT) acc4[DT] = mfma(kf[4], vf, acc4[DT]);
                    acc4[0] = mfma(kl, vf, acc4[0]);
                    if constexpr (BETA) {
                        const u32x4 vl = v_frag(q, 4, 1);
                        acc4[0] = mfma(kh, vl, acc4[0]);
                        if constexpr (DT) acc4[DT] = mfma(kf[4], vl, acc4[DT]);
                        acc4[0] = mfma(kl, vl, acc4[0]);
                    }
                }
            }
        }
        meet();      // (k~ has been read)
        {
            LANE;
            const float *fa = my_decay + kFromAnchor * US;
            f32x4 fac[2];
            f32x2 fact = f32x2{0.f, 0.f};
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) fac[ct] = *reinterpret_cast<const f32x4 *>(fa + 16 * (g & 1) + 4 * (2 * ct + (g >> 1)));
            if constexpr (DT) fact = *reinterpret_cast<const f32x2 *>(fa + 32 + 2 * (g & 1));
            auto leave = [&](float *u, int ct, f32x4 a, f32x4 f) {
                *reinterpret_cast<f32x4 *>(u + 16 * (g & 1) + 4 * (2 * ct + (g >> 1))) = a * f;
            };
            auto leave_tail = [&](float *u, f32x4 a) {
                if (g < 2) *reinterpret_cast<f32x2 *>(u + 32 + 2 * g) = f32x2{(a[0] + a[1]) * fact[0], (a[2] + a[3]) * fact[1]};
            };
            if constexpr (BETA) {
                const float *ca = my_cols + kFromAnchor * L::kCols + lm;
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int ct = 0; ct < 2 + DT; ++ct) acc[i][ct] *= ca[16 * (2 * i + W)];
#pragma unroll
                for (int i = 0; i < 1 + DT; ++i) acc4[i] *= ca[NX == 5 ? 64 : 0];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                float *u = s_u + (16 * (2 * i + W) + lm) * US;
                leave(u, 0, acc[i][0], fac[0]);
                leave(u, 1, acc[i][1], fac[1]);
                if constexpr (DT) leave_tail(u, acc[i][2]);
            }
            if constexpr (NX == 5) {
                if (64 + lm < HD::NV) {
                    float *u = s_u + (64 + lm) * US;
                    leave(u, W, acc4[0], W ? fac[1] : fac[0]);
                    if constexpr (DT) {
                        if (W == 0) leave_tail(u, acc4[DT]);
                    }
                }
            }
        }
        __syncthreads();
        const Pieces qp = pieces(recompute_per_chunk(tid));
        const float *u_of = reinterpret_cast<const float *>(smem);       // of chunk c: + c * kWave / 4
        auto state_at = [&](int c, int i) { return u_of + c * (L::kOne / 4) + qp.n[i] * US + 4 * qp.c[i]; };
        auto decay_at = [&](int c, int i, int what) {
            f32x4 d = *reinterpret_cast<const f32x4 *>(s_decay + (4 * c + what) * US + 4 * qp.c[i]);
            if constexpr (BETA) d *= s_cols[(4 * c + what) * L::kCols + qp.n[i]];
            return d;
        };
        // ---- the span's own state for the spans behind it ----
        auto flags_of = [&]() { return ARG->flags + (size_t)afresh(bh) * ARG->nspans * NW; };
        auto view_state = [&]() { return view(ARG->ws_state + (size_t)afresh(bh) * ARG->nspans * dk * dv, (uint32_t)ARG->nspans * ne4); };
        auto view_lgam = [&]() { return view(ARG->ws_lgam + (size_t)afresh(bh) * ARG->nspans * dk, 4u * (uint32_t)(ARG->nspans * dk)); };
        auto view_lgam_b = [&]() { return view(ARG->ws_lgam_b + (size_t)afresh(bh) * ARG->nspans * dv, (uint32_t)ARG->nspans * dv4); };
        const bool gives = sp + 1 < ARG->nspans;
        if (gives) {
            const Rsrc b_state = view_state(), b_lgam = view_lgam();
#pragma unroll
            for (int i = 0; i < KQ; ++i) {
                f32x4 u = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = 0; c < NC; ++c) u = decay_at(c, i, kDecay) * u + *reinterpret_cast<const f32x4 *>(state_at(c, i));
#pragma unroll
                for (int r = 0; r < 4; ++r) publish(b_state, owns(i) ? qp.at[i] : kNowhere, (uint32_t)sp * ne4 + r * dv4, u[r]);
            }
            if (tid < dk) {     // (the workspace keeps natural logarithms)
                float sum = 0.f;
#pragma unroll
                for (int c = 0; c < NC; ++c) sum += s_decay[(4 * c + kLogDecay) * US + tid];
                publish(b_lgam, 4u * (uint32_t)tid, 4u * (uint32_t)(sp * dk), sum * kLn2);
            }
            if constexpr (BETA) {
                if (w == 0) {       // (the wave whose flag stands for the decays)
                    const Rsrc b_lgam_b = view_lgam_b();
                    for (int n = tid; n < dv; n += 64) {
                        float sum = 0.f;
#pragma unroll
                        for (int c = 0; c < NC; ++c) sum += s_cols[(4 * c + kLogDecay) * L::kCols + n];
                        publish(b_lgam_b, 4u * (uint32_t)n, (uint32_t)sp * dv4, sum * kLn2);
                    }
                }
            }
        }
        // ---- O^T = V^T A^T: lane (lm, g) accumulates O[i = 16 t + lm][n = 16 x + 4 g + r] ----
        f32x4 o[2][NX];
        auto view_out = [&]() { return view_v(ARG->out, sizeof(TOut)); };
        {
            TR_LANE;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int x = 0; x < NX; ++x) o[t][x] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int x = 0; x < NX; ++x) {
                    const u32x4 vf = v_frag(q, x);
                    if (q == 0) o[0][x] = mfma(vf, pah[0], o[0][x]);
                    o[1][x] = mfma(vf, pah[1 + q], o[1][x]);
                    if (q == 0) o[0][x] = mfma(vf, pal[0], o[0][x]);
                    o[1][x] = mfma(vf, pal[1 + q], o[1][x]);
                    if constexpr (BETA) {
                        const u32x4 vl = v_frag(q, x, 1);
                        if (q == 0) o[0][x] = mfma(vl, pah[0], o[0][x]);
                        o[1][x] = mfma(vl, pah[1 + q], o[1][x]);
                        if (q == 0) o[0][x] = mfma(vl, pal[0], o[0][x]);
                        o[1][x] = mfma(vl, pal[1 + q], o[1][x]);
                    }
                }
        }
        if (gives) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // (the wave's stores have arrived)
            if ((tid & 63) == 0) __hip_atomic_store(flags_of() + sp * NW + w, ARG->nonce, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if constexpr (FUSE) {      // output-gate pre-activations of the chunk, in the place of v
            if (epilogue) {
                meet();
                v_to_lds(view_v(ARG->r_pre, 2));
            }
        }
        // ---- the state entering the span ----
        if (sp > 0 && 64 * w < kQuads) {
            const Rsrc b_state = view_state(), b_lgam = view_lgam();
            float wb[BETA ? KQ : 1];   // the value column's part of the weight
#pragma unroll
            for (int i = 0; i < (BETA ? KQ : 1); ++i) wb[i] = 0.f;
            f32x4 wl[KQ], ref[KQ];     // log2 of the weight of the next span; the same behind the nearest spans that were all zero
#pragma unroll
            for (int i = 0; i < KQ; ++i) wl[i] = ref[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            int have = sp;        // the spans from this one on are there, as far as is known
            auto wait_for = [&](int lowest) {      // false: the poll ran out
                const int lane = tid & 63;
                for (int i = 0; have > lowest; ++i) {
                    if (i >= ARG->polls) return false;
                    if (i > 0) __builtin_amdgcn_s_sleep(1);
                    const int s = have - 1 - (lane >> 1);       // two flags each: this wave's part, and that with the decays
                    const flag_t f = __hip_atomic_load(flags_of() + max(s, 0) * NW + ((lane & 1) ? w : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const unsigned long long there = __ballot(f == ARG->nonce || s < 0);
                    const unsigned long long missing = ~there;
                    have -= missing ? __builtin_ctzll(missing) >> 1 : 32;
                }
                return true;
            };
            auto alive = [&]() {
                bool a = false;
#pragma unroll
                for (int i = 0; i < KQ; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) a = a || (qp.at[i] != kNowhere && wl[i][r] > ref[i][r] - 40.f);
                return (bool)__any(a);
            };
            constexpr int N = KQ == 1 ? 4 : 2;
            bool ok = true;
            int r0 = sp - 1;
            for (; r0 >= 0 && alive(); r0 -= N) {
                ok = wait_for(max(r0 - N + 1, 0));
                if (!ok) break;
                asm volatile("" ::: "memory");
                f32x4 u[N][KQ], d[N][KQ];
                float db[N][BETA ? KQ : 1];
#pragma unroll
                for (int n = 0; n < N; ++n) {
                    const uint32_t at = (uint32_t)max(r0 - n, 0);
#pragma unroll
                    for (int i = 0; i < KQ; ++i) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) u[n][i][r] = published(b_state, qp.at[i], at * ne4 + r * dv4);
                        d[n][i] = published4(b_lgam, qp.at_dk[i], at * 4u * (uint32_t)dk);
                        if constexpr (BETA) db[n][i] = published(view_lgam_b(), 4u * (uint32_t)min(qp.n[i], dv - 1), at * dv4);
                    }
                }
#pragma unroll
                for (int n = 0; n < N; ++n) {
                    if (r0 - n < 0) break;
#pragma unroll
                    for (int i = 0; i < KQ; ++i) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            S[i][r] = fmaf(exp2_fast(BETA ? wl[i][r] + wb[BETA ? i : 0] : wl[i][r]), u[n][i][r], S[i][r]);
                            wl[i][r] += d[n][i][r] * kLog2e;
                        }
                        if constexpr (BETA) wb[i] += db[n][i] * kLog2e;
                        const bool zero = S[i][0] == 0.f && S[i][1] == 0.f && S[i][2] == 0.f && S[i][3] == 0.f;
#pragma unroll
                        for (int r = 0; r < 4; ++r) ref[i][r] = zero ? wl[i][r] : ref[i][r];
                    }
                }
            }
            if (!ok) {       // the poll ran out: from the inputs
                const Rsrc bg = FUSE ? view_k(ARG->z_gate, 2) : view_k(ARG->log_alpha, 4), bk = view_k(ARG->k, 2), bv = view_v(ARG->v, 2), b_init = view_init();
#pragma unroll
                for (int i = 0; i < KQ; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) S[i][r] = ARG->initial_state != nullptr ? fetch<float>(b_init, qp.at[i] + r * dv4) : 0.f;
                for (int s = 0; s < s_begin; ++s) {
                    const uint32_t tok = (uint32_t)scan_token(ARG->scan_dir, s, T, ARG->grid_h, ARG->grid_w);
#pragma unroll
                    for (int i = 0; i < KQ; ++i) {
                        const uint32_t at_v = tok * dv2 + 2u * (uint32_t)min(qp.n[i], dv - 1);
                        const float x = bf16_bits_to_float(fetch<uint16_t>(bv, at_v));
                        float beta = 0.f;
                        if constexpr (BETA) beta = fetch<float>(view_v(ARG->log_beta, 4), 2u * at_v) * kLog2e;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const uint32_t at = tok * dk2 + 2u * (uint32_t)min(4 * qp.c[i] + r, dk - 1);
                            const float a = FUSE ? gate1(bf16_bits_to_float(fetch<uint16_t>(bg, at))) : fetch<float>(bg, 2u * at) * kLog2e;
                            S[i][r] = fmaf(exp2_fast(BETA ? a + beta : a), S[i][r], bf16_bits_to_float(fetch<uint16_t>(bk, at)) * x);
                        }
                    }
                }
            } else if (r0 < 0 && ARG->initial_state != nullptr) {
                const Rsrc b_init = view_init();
#pragma unroll
                for (int i = 0; i < KQ; ++i)
#pragma unroll
                    for (int r = 0; r < 4; ++r) S[i][r] = fmaf(exp2_fast(BETA ? wl[i][r] + wb[BETA ? i : 0] : wl[i][r]), fetch<float>(b_init, qp.at[i] + r * dv4), S[i][r]);
            }
        }
        constexpr int NB = KQ == 1 ? 2 : 4;       // chunks whose reads go together (registers)
        // ---- P_c = 2^(b_m) S_c in the place of U_c: of a piece's four channels the hi parts, then the lo parts (in the tail, pairs) ----
#pragma unroll
        for (int i = 0; i < KQ; ++i) {
            if (!owns(i)) continue;
#pragma unroll
            for (int c0 = 0; c0 < NC; c0 += NB) {
                f32x4 u[NB], m[NB], e[NB];
#pragma unroll
                for (int c = 0; c < NB; ++c) {
                    u[c] = *reinterpret_cast<const f32x4 *>(state_at(c0 + c, i));
                    m[c] = decay_at(c0 + c, i, kToAnchor);
                    e[c] = decay_at(c0 + c, i, kDecay);
                }
#pragma unroll
                for (int c = 0; c < NB; ++c) {
                    const f32x4 x = S[i] * m[c];
                    u32x4 y;
                    SPLIT_PAIR(x[0], x[1], y[0], y[2]);
                    SPLIT_PAIR(x[2], x[3], y[1], y[3]);
                    if (DT && qp.c[i] == 8)
                        y = u32x4{__builtin_amdgcn_perm(y[2], y[0], 0x05040100u), __builtin_amdgcn_perm(y[2], y[0], 0x07060302u),
                                  __builtin_amdgcn_perm(y[3], y[1], 0x05040100u), __builtin_amdgcn_perm(y[3], y[1], 0x07060302u)};
                    *reinterpret_cast<u32x4 *>(const_cast<float *>(state_at(c0 + c, i))) = y;
                    S[i] = e[c] * S[i] + u[c];
                }
            }
        }
        f32x4 prev[2][ACC ? NX : 1];
        auto fetch_prev = [&](int t) {      // rows to add to
            const Rsrc bo = view_out();
            const int g = recompute_per_chunk(threadIdx.x) >> 4 & 3;
#pragma unroll
            for (int x = 0; x < NX; ++x)
                prev[t][x] = fetch<f32x4>(bo, OE * (4 * g + 16 * x < dv ? rowv[t] + 8u * (uint32_t)g + 32u * (uint32_t)x : kNowhere / 2));
        };
        if constexpr (ACC) fetch_prev(0);
        __syncthreads();
        {
            LANE;
            // offset (bf16 row) of the four columns this lane holds of column tile x of its token in tile t
            auto ocol = [&](int t, int x) { return 4 * g + 16 * x < dv ? rowv[t] + 8u * (uint32_t)g + 32u * (uint32_t)x : kNowhere / 2; };
            // ---- O^T += P^T Q~^T ----
#pragma unroll
            for (int x = 0; x < NX; ++x) {
                const float *s = s_u + min(16 * x + lm, HD::NV - 1) * US;
                const u32x4 y0 = *reinterpret_cast<const u32x4 *>(s + 4 * g), y1 = *reinterpret_cast<const u32x4 *>(s + 16 + 4 * g);
                const u32x4 ph = u32x4{y0[0], y0[1], y1[0], y1[1]}, pl = u32x4{y0[2], y0[3], y1[2], y1[3]};
                u32x4 pt = u32x4{0, 0, 0, 0};
                if constexpr (DT) pt = tail_operand(*reinterpret_cast<const uint32_t *>(s + 32 + g));
#pragma unroll
                for (int t = 0; t < 2; ++t) o[t][x] = mfma(ph, qh[t], o[t][x]);
#pragma unroll
                for (int t = 0; t < 2; ++t) o[t][x] = mfma(ph, ql[t], o[t][x]);
#pragma unroll
                for (int t = 0; t < 2; ++t) o[t][x] = mfma(pl, qh[t], o[t][x]);
#pragma unroll
                for (int t = 0; t < 2; ++t) o[t][x] = mfma(pl, ql[t], o[t][x]);
                if constexpr (DT) {
#pragma unroll
                    for (int t = 0; t < 2; ++t) o[t][x] = mfma(pt, u32x4{qt[t], qt[t], 0, 0}, o[t][x]);
                }
            }
            if constexpr (ACC) fetch_prev(1);
            if constexpr (FUSE) {
                if (epilogue) {
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    meet();
                }
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                if constexpr (FUSE) {
                    if (epilogue) {
                        // Swish(r) * LN(o): a token's row is spread over the four lanes lm, lm+16, lm+32, lm+48
                        // (columns past dv are left out)
                        const uint16_t *rrow = s_v + (16 * tile[t] + lm) * HD::NV + 4 * g;
                        const int r_swz = DT ? 0 : 16 * ((lm >> 1) & 3);
                        const float inv_n = 1.f / (float)dv;
                        float sum = 0.f;
#pragma unroll
                        for (int x = 0; x < NX; ++x)
                            if (4 * g + 16 * x < dv) sum += (o[t][x][0] + o[t][x][1]) + (o[t][x][2] + o[t][x][3]);
                        sum += __shfl_xor(sum, 16);
                        sum += __shfl_xor(sum, 32);
                        const float mean = sum * inv_n;
                        float sq = 0.f;
#pragma unroll
                        for (int x = 0; x < NX; ++x) {
                            if (4 * g + 16 * x < dv) {
#pragma unroll
                                for (int r = 0; r < 4; ++r) {
                                    const float d = o[t][x][r] - mean;
                                    sq = fmaf(d, d, sq);
                                }
                            }
                        }
                        sq += __shfl_xor(sq, 16);
                        sq += __shfl_xor(sq, 32);
                        const float rstd = __builtin_amdgcn_rsqf(sq * inv_n + ARG->ln_eps);
#pragma unroll
                        for (int x = 0; x < NX; ++x) {
                            if (4 * g + 16 * x < dv) {
                                const f32x4 lw = *reinterpret_cast<const f32x4 *>(s_lnw + 16 * x + 4 * g);
                                const f32x4 lb = *reinterpret_cast<const f32x4 *>(s_lnb + 16 * x + 4 * g);
                                const u32x2 rg = *reinterpret_cast<const u32x2 *>(rrow + ((16 * x) ^ r_swz));
                                const float rv[4] = {bf16_lo_as_float(rg[0]), bf16_hi_as_float(rg[0]),
                                                     bf16_lo_as_float(rg[1]), bf16_hi_as_float(rg[1])};
#pragma unroll
                                for (int r = 0; r < 4; ++r) {
                                    const float sw = rv[r] * __builtin_amdgcn_rcpf(1.f + exp2_fast(-rv[r] * kLog2e));
                                    o[t][x][r] = fmaf((o[t][x][r] - mean) * rstd, lw[r], lb[r]) * sw;
                                }
                            }
                        }
                    }
                }
                const Rsrc bo = view_out();
                if constexpr (BETA) {
#pragma unroll
                    for (int x = 0; x < NX; ++x)
#pragma unroll
                        for (int r = 0; r < 4; ++r) o[t][x][r] *= exp2_fast(fminf(cx[t][x][r], kMaxExp2));
                }
                if constexpr (ACC) {
#pragma unroll
                    for (int x = 0; x < NX; ++x) o[t][x] += prev[t][x];
                }
#pragma unroll
                for (int x = 0; x < NX; ++x) {        // dv is a multiple of 8: all four columns or none
                    if constexpr (sizeof(TOut) == 4) put(bo, OE * ocol(t, x), o[t][x]);
                    else put(bo, OE * ocol(t, x), u32x2{pack_bf16(o[t][x][0], o[t][x][1]), pack_bf16(o[t][x][2], o[t][x][3])});
                }
            }
        }
    }
    if (sp == ARG->nspans - 1 && ARG->final_state != nullptr) {      // the last span ends in the final state
        const Pieces q = pieces(tid);
        const Rsrc b_fin = view(ARG->final_state + (size_t)bh * dk * dv, ne4);
#pragma unroll
        for (int i = 0; i < KQ; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float x = S[i][r];
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), b_fin, (int)(owns(i) ? q.at[i] + r * dv4 : kNowhere), 0, 0);
            }
    }
}

// Flags of a call that is recorded into a graph: its nonce is the same in every replay, so they are cleared ahead of it.
__global__ __launch_bounds__(256) void clear_flags_kernel(flag_t *flags, long long n) {
    for (long long i = blockIdx.x * 256ll + threadIdx.x; i < n; i += gridDim.x * 256ll) flags[i] = 0;
}

template <typename HD, int NC, bool FUSE, bool ACC, typename TOut, bool BETA = false>
hipError_t launch_one(const OnePassParams &p, hipStream_t stream) {
    using L = WLayout<HD, NC, FUSE, BETA>;
    auto kernel = chunk_pair_kernel<HD, NC, FUSE, ACC, TOut, BETA>;
    static std::atomic<bool> configured[kMaxDevices] = {};  // per instantiation and device
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), L::kBytes, configured);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(p.B * p.H * p.nspans)), dim3(128 * NC), L::kBytes, stream, p);
    return hipGetLastError();
}

template <typename HD, int NC>
hipError_t launch_heads(const OnePassParams &p, hipStream_t stream) {
    const bool bf16 = p.out_dtype == GLA_DT_BF16;
    if constexpr (NC == 4) {
        if (p.log_beta != nullptr)
            return bf16 ? launch_one<HD, 4, false, false, uint16_t, true>(p, stream) : launch_one<HD, 4, false, false, float, true>(p, stream);
    }
    if (p.z_gate != nullptr)
        return bf16 ? launch_one<HD, NC, true, false, uint16_t>(p, stream) : launch_one<HD, NC, true, false, float>(p, stream);
    if (p.accumulate) return launch_one<HD, NC, false, true, float>(p, stream);   // host checks fp32 out
    return bf16 ? launch_one<HD, NC, false, false, uint16_t>(p, stream) : launch_one<HD, NC, false, false, float>(p, stream);
}

}  // namespace

// (Smaller heads would leave most of the tiles empty, and stay with the kernels that have classes for them.)
bool onepass_covers(const Params &p) {
    return (!two_sided(p) || (p.z_gate == nullptr && p.z_beta == nullptr)) && p.dk > 16 && p.dk <= 36 && p.dv > 32 && p.dv <= 72;
}

hipError_t launch_onepass(const OnePassParams &p, int chunks, hipStream_t stream) {
    if (p.nspans > 1) {
        hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(stream, &status) != hipSuccess) {
            (void)hipGetLastError();
            status = hipStreamCaptureStatusNone;
        }
        if (status != hipStreamCaptureStatusNone) {
            const long long n = (long long)p.B * p.H * p.nspans * 2 * chunks;
            hipLaunchKernelGGL(clear_flags_kernel, dim3((unsigned)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024)), dim3(256), 0, stream, p.flags, n);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    if (p.dk <= 32 && p.dv <= 64) return chunks == 8 ? launch_heads<HeadsS, 8>(p, stream) : launch_heads<HeadsS, 4>(p, stream);
    return chunks == 8 ? launch_heads<HeadsXL, 8>(p, stream) : launch_heads<HeadsXL, 4>(p, stream);
}

}  // namespace gla
