// bf16 hi/lo MFMA engine for one span of the GLA recurrence in its chunk form, rows held in registers
// (DiG paper, Sec. 3.5: chunks of M = 64 tokens computed on-chip; recurrence of Sec. 3.1 Eq. (attn_gla) rows 1-3 with
// beta = 1; up to 36 key channels and 80 value columns, see hilo_kernels_cover).
//
// Chunk form around a mid-chunk anchor.  With b_j = sum_{i<=j} log2 alpha_i inside a chunk (inclusive, per key channel),
// b_m its value after the chunk's 32nd token and b_C after its last, and S_0 the state entering the chunk,
//     q~_j = q_j 2^(b_j - b_m),   k~_i = k_i 2^(b_m - b_i),   P = diag(2^b_m) S_0
//     o_j = sum_{i<=j} (q~_j . k~_i) v_i + q~_j P ,           S_C = diag(2^(b_C - b_m)) (P + K~^T V).
// Every gated operand (q~, k~, the scores, P) is a bf16 "hi" part and a bf16 "lo" remainder, so that the products carry
// about 16 mantissa bits; v is used as given.  The state lives in fp32 accumulators for the whole span.
//
// Wave w of the four owns tokens 16 w .. 16 w + 15 of every chunk, and fetches their rows straight into the layout of the
// MFMA operands: lane (lm, g) = (lane % 16, lane / 16) holds, for token 16 w + lm, channels 16 u + 4 g .. + 3 of the units
// u = 0, 1 (one 32-channel step: slot (g, e) is channel 16 (e / 4) + 4 g + e % 4) and the "tail" channel 32 + g.  q~
// therefore never leaves the wave's registers, the gates' prefix sums are 4-step scans over the 16 lanes of a DPP row plus
// the totals of the other waves' tiles, and only k~, v and P go through LDS, each written once.
// A tail channel fills the four contraction slots of its lane group with its four hi/lo products: (hi, hi, lo, lo) on the
// side of k~ and P, (hi, lo, hi, lo) on that of q~; one MFMA takes them all.  The same 16 columns read over the tokens
// give the state update of the four tail channels (rows hi, hi, lo, lo of each: the sum of the first and the third).
//
// LDS rows of k~ (per token) and P (per value column): 32 hi, 32 lo (position 8 g + 4 u + r for channel 16 u + 4 g + r),
// then 16 for the tail channels, and the operands of two chunks: while the waves contract chunk c from one set, they gate
// chunk c + 1 and scale the state into the other and scan the gates of chunk c + 2, with one barrier a chunk, so that the
// vector instructions of the gating stand between the matrix instructions of the contraction (both are chains of dependent
// instructions, and a SIMD holds two waves: 69 KB a group, two groups a compute unit).
//
// LDS rows are 160 bytes (40 banks) long, and the 16-byte units of rows 8 .. 15 of every 16 change places in pairs: the
// reads of 16 rows (8- and 16-byte pieces, transposing or not) then fall into different banks.  (With rows an odd number of
// 16-byte units long the transposing reads of 8 rows overlapped in twos.)
//
// What bounds it on MI355X: up to 1024 px the instruction streams (one group alone on a compute unit: 5300 clocks a chunk at
// 36 / 72 channels, 6500 when two share it), at 2048 px the memory (output pass 195 MB in 30 us once the pipeline is filled).
// Before, with the rows staged through LDS, three barriers a chunk and single sets (output pass / state pass of 2048 chunks
// in gla_fwd_fused: 36.7 / 16.6 us, here 30 / 13.9): a chunk of a lone group took 6800 clocks and two groups gained little
// on each other.  Tried: three groups of 168 registers with single sets (two barriers; 45.3 against 42.6 us a fused call),
// a chunk loop per wave with the scan inside (45.5), the state's chain with the decays read a run ahead (42.6 -> 43.3).
#include <type_traits>

#include "gla_common.h"
#include "gla_mfma_util.h"

namespace gla {
namespace {

template <int N>
using int_c = std::integral_constant<int, N>;

// What the heads come to: DT groups of four tail channels (33 .. 36), NDV16 tiles of 16 value columns.  (Smaller heads leave the
// rest of them empty, see hilo_kernels_cover.)
constexpr int DT = 1, NDV16 = 5;

template <bool OUT, bool FUSE>
struct HLayout {
    static_assert(64 + 16 * DT <= 80 && 16 * NDV16 <= 80, "rows of 160 bytes");
    static constexpr int NV = 8 + DT;                         // gate values per lane and chunk
    static constexpr int kTotStride = 12;                     // floats per (tile, g) of the tile totals
    static constexpr int kRow = 80, kVRow = 80;               // bf16 per row of k~ and P, of v (see swz)
    static constexpr int kTotBuf = 4 * 4 * kTotStride;        // floats per chunk: [tile][g][NV]
    static constexpr int oTot = 0;                            // three chunks
    static constexpr int oLn = oTot + 3 * kTotBuf * 4;        // float[2][16 NDV16]: LayerNorm weight, bias (FUSE)
    // two sets of operands (k~, v, P of one chunk each); chunk x uses set x % 2
    static constexpr int oK = oLn + (FUSE ? 2 * 16 * NDV16 * 4 : 0);
    static constexpr int oV = oK + kChunk * kRow * 2;
    static constexpr int oP = oV + kChunk * kVRow * 2;
    static constexpr int kSet = (OUT ? oP + 16 * NDV16 * kRow * 2 : oP) - oK;
    static constexpr int kBytes = oK + 2 * kSet;
    static constexpr int oChain = oK + kSet;                  // float[dk * dv] before the first chunk is gated into set 0
    static_assert(!OUT || kSet >= (32 + 4 * DT) * 16 * NDV16 * 4, "the chained start state must fit");
    static_assert(oK % 16 == 0 && oV % 16 == 0 && oP % 16 == 0 && kSet % 16 == 0, "16-byte LDS accesses");
};

// Which state tiles (tile t = row tile t % NCT of column tile t / NCT) a wave owns.  A wave's outputs cost more the later
// its tokens are (causal tiles), so the early waves own most of the state; in the state pass they share it evenly.
template <bool OUT>
struct Owned {
    static constexpr int NCT = 2 + DT, kTiles = NCT * NDV16;
    __host__ __device__ static constexpr int start(int w) {
        if (!OUT) return kTiles * w / 4;
        return w == 0 ? 0 : (w == 1 ? kTiles * 2 / 5 : (w == 2 ? kTiles * 3 / 4 : (w == 3 ? kTiles - 1 : kTiles)));   // (15: 6, 5, 3, 1)
    }
    __host__ __device__ static constexpr int count(int w) { return start(w + 1) - start(w); }
    static constexpr int kMost = OUT ? count(0) : (kTiles + 3) / 4;
};

// Last statement of code that exists once per wave: keeps the compiler from merging the copies' tails, which would
// address the accumulators through a wave-dependent pointer (they would leave the registers).
#define HILO_WAVE_END(W) asm volatile("; end of the code of wave %0" ::"n"(W))

// OUT: the output pass (or the single pass); otherwise the span-state pass (U and log Gamma of the span, from zero).
// FUSE = the gate prologue (gates from bf16 pre-activations) and, in the output pass, the optional epilogue.
// ACC = the output pass adds its rows to the fp32 rows already in `out`.
// SHIFT = p.gate_shift: a step uses the gate of the token visited a step earlier.
template <bool OUT, int MINW, bool FUSE, bool ACC, bool SHIFT, typename TOut>
__global__ __launch_bounds__(256, MINW) void hilo_span_kernel(Params p) {
    using L = HLayout<OUT, FUSE && OUT>;
    using OW = Owned<OUT>;
    constexpr int NV = L::NV, NCT = 2 + DT, RS = L::kRow, VS = L::kVRow, TS = L::kTotStride;
    constexpr int NVP = (2 * NDV16 + 3) / 4;          // 16-byte pieces of a v row per lane
    constexpr int NX = NDV16;
    static_assert(!ACC || (OUT && !FUSE && sizeof(TOut) == 4), "accumulation: plain output pass, fp32 rows");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    float *s_tot = reinterpret_cast<float *>(smem + L::oTot);
    uint16_t *s_k = reinterpret_cast<uint16_t *>(smem + L::oK);
    uint16_t *s_v = reinterpret_cast<uint16_t *>(smem + L::oV);
    uint16_t *s_p = reinterpret_cast<uint16_t *>(smem + L::oP);
    float *s_lnw = reinterpret_cast<float *>(smem + L::oLn), *s_lnb = s_lnw + 16 * NDV16;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15;
    const int g = lane >> 4;
    const int swz = 8 * (lm >> 3);            // of the rows 16 i + lm

    // contiguous ranges of spans per XCD; odd heads walk their spans backwards where the span states are chained here
    // (a long and a short chain then share a compute unit)
    int blk = blockIdx.x;
    {
        const int nb = gridDim.x;
        if ((nb & 7) == 0) blk = (blk & 7) * (nb >> 3) + (blk >> 3);
    }
    const int spans_here = (!OUT && p.chain_in_output) ? p.nspans - 1 : p.nspans;   // (nobody reads the last span's U)
    const int bh = blk / spans_here;
    int sp_ = blk - bh * spans_here;
    if (OUT && p.chain_in_output && (bh & 1)) sp_ = spans_here - 1 - sp_;
    const int sp = sp_;
    if constexpr (OUT) {
        // second opinion for the fp16 engine: a (batch, head) is recomputed if one of its spans raised its flag
        if (p.only_flagged) {
            int any = 0;
            for (int i = tid; i < p.fail_spans; i += 256) any |= p.ws_fail[(size_t)bh * p.fail_spans + i];
            if (!__syncthreads_or(any)) return;   // (uniform over the group)
        }
    }
    const int dk = p.dk, dv = p.dv, T = p.T;
    const int s_begin = sp * p.span_len;
    const int s_end = min(T, s_begin + p.span_len);
    const int nch = (s_end - s_begin + kChunk - 1) / kChunk;

    const size_t base_k = slab_k(p, bh), base_v = slab_v(p, bh);
    const uint32_t dk2 = 2u * (uint32_t)p.st_k, dv2 = 2u * (uint32_t)p.st_v;   // bytes from one bf16 row to the next
    const uint32_t bytes_k = (uint32_t)(T - 1) * dk2 + 2u * (uint32_t)dk, bytes_v = (uint32_t)(T - 1) * dv2 + 2u * (uint32_t)dv;
    const Rsrc bq = view(static_cast<const char *>(p.q) + base_k * 2, bytes_k);
    const Rsrc bk = view(static_cast<const char *>(p.k) + base_k * 2, bytes_k);
    const Rsrc bv = view(static_cast<const char *>(p.v) + base_v * 2, bytes_v);
    const Rsrc bg = FUSE ? view(static_cast<const char *>(p.z_gate) + base_k * 2, bytes_k)
                         : view(p.log_alpha + base_k, 2u * bytes_k);
    const Rsrc br = view(static_cast<const char *>(p.r_pre) + base_v * 2, bytes_v);
    constexpr uint32_t OE = sizeof(TOut) / 2;         // bytes of `out` per byte of a bf16 row
    const Rsrc bo = view(static_cast<char *>(p.out) + base_v * sizeof(TOut), OE * bytes_v);
    const bool epilogue = FUSE && OUT && p.r_pre != nullptr;   // uniform

    // ---- token of this lane's row (16 w + lm) as the wave moves from chunk to chunk: 64 scan steps further are 64 / R
    // columns and 64 % R rows of the scan (R tokens a column; a row scan: R = 1), with one wrap.  (Past the span's end it
    // is not looked at: such rows are nowhere.) ----
    const int row_s0 = s_begin + 16 * w + lm;
    auto row_is_token = [&](int x) { return row_s0 + x * kChunk < s_end; };
    const int col_len = p.scan_dir >= 2 ? p.grid_h : 1, dir = (p.scan_dir & 1) ? -1 : 1;   // (uniform)
    const int col_dq = dir * (kChunk / col_len), col_dr = dir * (kChunk % col_len);
    int tok, tok_c, tok_r, walk_s = row_s0;
    {
        const int s = (p.scan_dir & 1) ? T - 1 - min(row_s0, T - 1) : min(row_s0, T - 1);
        tok_c = s / col_len;
        tok_r = s - tok_c * col_len;
        tok = tok_r * p.grid_w + tok_c;
    }
    auto next_row_token = [&]() {
        walk_s += kChunk;
        tok_c += col_dq;
        tok_r += col_dr;
        const bool over = tok_r >= col_len, under = tok_r < 0;
        tok_r += under ? col_len : (over ? -col_len : 0);
        tok_c += under ? -1 : (over ? 1 : 0);
        tok = tok_r * p.grid_w + tok_c;
    };

    // ---- rows in registers ----
    uint32_t chb[2];                     // byte offset of the lane's units in a bf16 row
#pragma unroll
    for (int u = 0; u < 2; ++u) chb[u] = 16 * u + 4 * g < dk ? 2u * (uint32_t)(16 * u + 4 * g) : kNowhere / 2;
    uint32_t tcb[DT];                   // the same for the tail channels
#pragma unroll
    for (int e = 0; e < DT; ++e) tcb[e] = 32 + 4 * e + g < dk ? 2u * (uint32_t)(32 + 4 * e + g) : kNowhere / 2;
    using GatePiece = std::conditional_t<FUSE, u32x2, f32x4>;
    using GateTail = std::conditional_t<FUSE, uint16_t, float>;
    struct GateRow {
        GatePiece u[2];
        GateTail t[DT];
    };
    struct ActRow {
        u32x2 u[2];
        uint32_t t[DT];
    };
    GateRow r_la;
    ActRow r_q, r_k;
    u32x4 r_v[NVP];
    float r_b[8 + DT];                  // scanned gates (log2, prefix inside the 16-token tile)

    auto issue_la = [&](GateRow &dst, int step, int tk) {
        if constexpr (SHIFT) tk = scan_token(p.scan_dir, max(min(step, s_end - 1) - 1, 0), T, p.grid_h, p.grid_w);
        const uint32_t row = step < s_end ? (uint32_t)tk * dk2 : kNowhere / 2;
#pragma unroll
        for (int u = 0; u < 2; ++u) dst.u[u] = fetch<GatePiece>(bg, FUSE ? row + chb[u] : f32_at(row, chb[u]));
#pragma unroll
        for (int e = 0; e < DT; ++e) dst.t[e] = fetch<GateTail>(bg, FUSE ? row + tcb[e] : f32_at(row, tcb[e]));
    };
    auto issue_qkv = [&](int step, int tk) {
        const uint32_t row = step < s_end ? (uint32_t)tk * dk2 : kNowhere / 2;
        const uint32_t rowv = step < s_end ? (uint32_t)tk * dv2 : kNowhere / 2;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            r_k.u[u] = fetch<u32x2>(bk, row + chb[u]);
            if constexpr (OUT) r_q.u[u] = fetch<u32x2>(bq, row + chb[u]);
        }
#pragma unroll
        for (int e = 0; e < DT; ++e) {
            r_k.t[e] = fetch<uint16_t>(bk, row + tcb[e]);
            if constexpr (OUT) r_q.t[e] = fetch<uint16_t>(bq, row + tcb[e]);
        }
#pragma unroll
        for (int i = 0; i < NVP; ++i) {
            const int col = min(8 * (g + 4 * i), 16 * NDV16 - 8);     // (lanes past the last piece repeat it)
            r_v[i] = fetch<u32x4>(bv, rowv + (col < dv ? 2u * (uint32_t)col : kNowhere / 2));
        }
    };

    auto ring = [](int x) { return x % 3; };
    // prefix sums of log2(alpha) of chunk x inside this wave's tile; tile totals to LDS
    auto scan = [&](int x, const GateRow &la) {
        if constexpr (FUSE) {
            // log2(alpha) = log2(sigmoid(z)) / tau = (min(t, 0) - log2(1 + 2^-|t|)) / tau with t = z log2(e)
            auto gate1 = [&](float z) {
                const float t = z * kLog2e;
                return (fminf(t, 0.f) - __builtin_amdgcn_logf(1.f + exp2_fast(-fabsf(t)))) * p.inv_tau;
            };
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    r_b[4 * u + 2 * h] = gate1(bf16_lo_as_float(la.u[u][h]));
                    r_b[4 * u + 2 * h + 1] = gate1(bf16_hi_as_float(la.u[u][h]));
                }
#pragma unroll
            for (int e = 0; e < DT; ++e) r_b[8 + e] = gate1(bf16_bits_to_float(la.t[e]));
        } else {
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) r_b[4 * u + e] = la.u[u][e] * kLog2e;
#pragma unroll
            for (int e = 0; e < DT; ++e) r_b[8 + e] = fmaxf(la.t[e] * kLog2e, kLeastGate2);
        }
        if constexpr (FUSE) {     // (a row that is not there decays by nothing; the gate of z = 0 is not 1)
            const float least = row_is_token(x) ? kLeastGate2 : 0.f;      // (gates are at most 0)
#pragma unroll
            for (int i = 0; i < NV; ++i) r_b[i] = fmaxf(r_b[i], least);
            row_scan16x4(r_b[0], r_b[1], r_b[2], r_b[3]);
            row_scan16x4(r_b[4], r_b[5], r_b[6], r_b[7]);
        } else {
            row_scan16x4_least(r_b[0], r_b[1], r_b[2], r_b[3], kLeastGate2);
            row_scan16x4_least(r_b[4], r_b[5], r_b[6], r_b[7], kLeastGate2);
        }
#pragma unroll
        for (int e = 0; e < DT; ++e) r_b[8 + e] = row_scan16(r_b[8 + e]);
        if (lm == 15) {
            float *tot = s_tot + ring(x) * L::kTotBuf + (4 * w + g) * TS;
            *reinterpret_cast<f32x4 *>(tot) = f32x4{r_b[0], r_b[1], r_b[2], r_b[3]};
            *reinterpret_cast<f32x4 *>(tot + 4) = f32x4{r_b[4], r_b[5], r_b[6], r_b[7]};
#pragma unroll
            for (int e = 0; e < DT; ++e) tot[8 + e] = r_b[8 + e];
        }
    };

    constexpr int SET = L::kSet / 2;      // 16-bit elements from an operand to its twin in the other set
    struct QFrag {                        // q~ of the wave's tokens, B operand: 32-channel step hi, lo; tail
        u32x4 h, l, t;
    };
    QFrag qf;
    // gate chunk x: q~ to registers, k~ and v to LDS.  The prefix sums of this wave's tile are offset by totals of other
    // tiles: tiles 0, 1 lie before the anchor (-(t0 + t1), -t1), tile 2 starts at it, tile 3 follows tile 2 (+t2).
    auto gate = [&](auto wave_c, int x, QFrag &qn) {
        constexpr int W = decltype(wave_c)::value;
        const float *tot = s_tot + ring(x) * L::kTotBuf + g * TS;        // + tile * 4 * TS
        float off[8 + DT];
        if constexpr (W != 2) {
            const float *t1 = tot + (W == 3 ? 2 : 1) * 4 * TS;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                f32x4 o4 = *reinterpret_cast<const f32x4 *>(t1 + 4 * u);
                if constexpr (W == 0) o4 += *reinterpret_cast<const f32x4 *>(tot + 4 * u);
#pragma unroll
                for (int e = 0; e < 4; ++e) off[4 * u + e] = o4[e];
            }
#pragma unroll
            for (int e = 0; e < DT; ++e) {
                off[8 + e] = t1[8 + e];
                if constexpr (W == 0) off[8 + e] += tot[8 + e];
            }
        }
        uint16_t *krow = s_k + (x & 1) * SET + (16 * W + lm) * RS;
        qn.t = u32x4{0, 0, 0, 0};
        float eq[8 + DT], ek[8 + DT];
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const float ex = W == 2 ? r_b[i] : (W == 3 ? r_b[i] + off[i] : r_b[i] - off[i]);
            // (clamped so that gates beyond the range leave nothing infinite; q~ can only exceed 1 before the anchor, k~
            // only behind it)
            if constexpr (OUT) eq[i] = exp2_fast(W < 2 ? fminf(ex, kMaxExp2) : ex);
            ek[i] = exp2_fast(W < 2 ? -ex : fminf(-ex, kMaxExp2));
        }
        u32x4 kh, kl;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t kr = r_k.u[u][h];
                SPLIT_PAIR(bf16_lo_as_float(kr) * ek[4 * u + 2 * h], bf16_hi_as_float(kr) * ek[4 * u + 2 * h + 1],
                           kh[2 * u + h], kl[2 * u + h]);
                if constexpr (OUT) {
                    const uint32_t qr = r_q.u[u][h];
                    SPLIT_PAIR(bf16_lo_as_float(qr) * eq[4 * u + 2 * h], bf16_hi_as_float(qr) * eq[4 * u + 2 * h + 1],
                               qn.h[2 * u + h], qn.l[2 * u + h]);
                }
            }
        }
        *reinterpret_cast<u32x4 *>(krow + (8 * g ^ swz)) = kh;
        *reinterpret_cast<u32x4 *>(krow + 32 + (8 * g ^ swz)) = kl;
#pragma unroll
        for (int e = 0; e < DT; ++e) {
            const float kx = bf16_lo_as_float(r_k.t[e]) * ek[8 + e];
            const uint32_t hh = pack_bf16(kx, kx);
            const float rem = kx - bf16_lo_as_float(hh);
            *reinterpret_cast<u32x2 *>(krow + 64 + 16 * e + (4 * g ^ swz)) = u32x2{hh, pack_bf16(rem, rem)};
            if constexpr (OUT) {
                const float qx = bf16_lo_as_float(r_q.t[e]) * eq[8 + e];
                const uint32_t qh = pack_bf16(qx, qx);
                const float qrem = qx - bf16_lo_as_float(qh);
                const uint32_t hl = (qh & 0xffffu) | (pack_bf16(qrem, qrem) << 16);
                qn.t[2 * e] = hl;
                qn.t[2 * e + 1] = hl;
            }
        }
        uint16_t *vrow = s_v + (x & 1) * SET + (16 * W + lm) * VS;
#pragma unroll
        for (int i = 0; i < NVP; ++i) *reinterpret_cast<u32x4 *>(vrow + (min(8 * (g + 4 * i), 16 * NDV16 - 8) ^ swz)) = r_v[i];
    };

    // ---- state tiles owned by this wave: acc[i][r] of a main tile ct = 0, 1 is S[channel 16 (g & 1) + 4 (2 ct + g / 2) + r]
    // [column 16 nt + lm] (times 2^(b_m - ..) inside a chunk); of a tail tile it is the hi and lo share of channel 32 + 4 e + g
    // in r = 0 and 2 (r = 1, 3: copies) ----
    f32x4 acc[OW::kMost];
#pragma unroll
    for (int i = 0; i < OW::kMost; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto main_channel = [&](int ct) { return 16 * (g & 1) + 4 * (2 * ct + (g >> 1)); };    // of r = 0

    // scale the tiles from the anchor of chunk c to that of chunk c + 1 (c = -1: the span's start; c = nch - 1: to the
    // span's end) and leave P of chunk c + 1 in LDS
    auto publish = [&](auto wave_c, int c) {
        constexpr int W = decltype(wave_c)::value;
        constexpr int t_lo = OW::start(W), t_hi = OW::start(W + 1);
        const float *t_c = s_tot + ring(c + 3) * L::kTotBuf;           // totals of chunk c
        const float *t_n = s_tot + ring(c + 1) * L::kTotBuf;           // totals of chunk c + 1
        f32x4 fac[2];
        float fact[DT];
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
            bool used = false;
            for (int t = t_lo; t < t_hi; ++t) used = used || (t % NCT == ct);
            if (!used) continue;
            if (ct < 2) {
                const int at = (2 * ct + (g >> 1)) * TS + 4 * (g & 1);
                f32x4 h = f32x4{0.f, 0.f, 0.f, 0.f};
                if (c >= 0)
                    h += *reinterpret_cast<const f32x4 *>(t_c + 2 * 4 * TS + at) + *reinterpret_cast<const f32x4 *>(t_c + 3 * 4 * TS + at);
                h += *reinterpret_cast<const f32x4 *>(t_n + at) + *reinterpret_cast<const f32x4 *>(t_n + 4 * TS + at);
                fac[ct < 2 ? ct : 0] = f32x4{exp2_fast(h[0]), exp2_fast(h[1]), exp2_fast(h[2]), exp2_fast(h[3])};
            } else {
                const int at = g * TS + 8 + (ct - 2);
                float h = 0.f;
                if (c >= 0) h += t_c[2 * 4 * TS + at] + t_c[3 * 4 * TS + at];
                h += t_n[at] + t_n[4 * TS + at];
                fact[ct >= 2 ? ct - 2 : 0] = exp2_fast(h);
            }
        }
#pragma unroll
        for (int i = 0; i < t_hi - t_lo; ++i) {
            const int ct = (t_lo + i) % NCT, nt = (t_lo + i) / NCT;
            uint16_t *prow = s_p + ((c + 1) & 1) * SET + (16 * nt + lm) * RS;
            if (ct < 2) {
                acc[i] = acc[i] * fac[ct < 2 ? ct : 0];
                if constexpr (OUT) {
                    u32x2 hi, lo;
                    SPLIT_PAIR(acc[i][0], acc[i][1], hi[0], lo[0]);
                    SPLIT_PAIR(acc[i][2], acc[i][3], hi[1], lo[1]);
                    *reinterpret_cast<u32x2 *>(prow + 16 * ct + (4 * g ^ swz)) = hi;
                    *reinterpret_cast<u32x2 *>(prow + 32 + 16 * ct + (4 * g ^ swz)) = lo;
                }
            } else {
                const int e = ct >= 2 ? ct - 2 : 0;
                const float s = (acc[i][0] + acc[i][2]) * fact[e];
                acc[i] = f32x4{s, 0.f, 0.f, 0.f};
                if constexpr (OUT) {
                    const uint32_t hh = pack_bf16(s, s);
                    const float rem = s - bf16_lo_as_float(hh);
                    *reinterpret_cast<u32x2 *>(prow + 64 + 16 * e + (4 * g ^ swz)) = u32x2{hh, pack_bf16(rem, rem)};
                }
            }
        }
    };
    auto per_wave = [&](auto fn, int c) {
        switch (w) {
        case 0: fn(int_c<0>{}, c); break;
        case 1: fn(int_c<1>{}, c); break;
        case 2: fn(int_c<2>{}, c); break;
        default: fn(int_c<3>{}, c); break;
        }
    };
    // Copies the state of this wave's tiles to or from a [dk][dv] array.
    auto each_state = [&](auto wave_c, auto fn) {
        constexpr int W = decltype(wave_c)::value;
#pragma unroll
        for (int i = 0; i < OW::count(W); ++i) {
            const int ct = (OW::start(W) + i) % NCT, n = 16 * ((OW::start(W) + i) / NCT) + lm;
            if (ct < 2) {
#pragma unroll
                for (int r = 0; r < 4; ++r) fn(i, r, main_channel(ct) + r, n);
            } else {
                fn(i, 0, 32 + 4 * (ct - 2) + g, n);
            }
        }
    };

    // ---- prologue: request everything the first stages need, then chain the state entering the span ----
    int tok0 = tok, tok1;               // tokens of the chunk contracted next, and of the one after it
    {
        GateRow la1;
        issue_la(r_la, row_s0, tok);
        issue_qkv(row_s0, tok);
        next_row_token();
        tok1 = tok;
        issue_la(la1, row_s0 + kChunk, tok);
        next_row_token();
        const float *s0 = nullptr;
        const bool chained = OUT && p.chain_in_output && (sp > 0 || p.initial_state != nullptr);   // uniform
        if constexpr (OUT) {
            if (chained) {
                constexpr int kV4 = ((32 + 4 * DT) * 16 * NDV16 / 4 + 255) / 256;
                chain_span_states<256, kV4, 16 / kV4, false, true>(p, bh, sp, tid, reinterpret_cast<float *>(smem + L::oChain));
            } else if (p.nspans > 1 && !p.chain_in_output) {
                s0 = p.ws_state + ((size_t)bh * p.nspans + sp) * dk * dv;      // as the carry kernel left it
            } else if (p.nspans == 1 && p.initial_state != nullptr) {
                s0 = p.initial_state + (size_t)bh * dk * dv;
            }
        }
        if constexpr (FUSE && OUT) {
            if (epilogue) {
                const int h = bh % p.H;
                for (int n = tid; n < dv; n += 256) {
                    s_lnw[n] = p.ln_weight != nullptr ? p.ln_weight[h * dv + n] : 1.f;
                    s_lnb[n] = p.ln_bias != nullptr ? p.ln_bias[h * dv + n] : 0.f;
                }
            }
        }
        scan(0, r_la);
        r_la = la1;
        __syncthreads();
        auto take_state = [&](auto load) {
            per_wave([&](auto wave_c, int) {
                f32x4 x[OW::kMost];
                each_state(wave_c, [&](int i, int r, int c, int n) { x[i][r] = load(c, n); });
                each_state(wave_c, [&](int i, int r, int c, int n) { acc[i][r] = c < dk && n < dv ? x[i][r] : 0.f; });
                HILO_WAVE_END(decltype(wave_c)::value);
            }, 0);
        };
        if (chained) {
            const float *s_chain = reinterpret_cast<const float *>(smem + L::oChain);
            take_state([&](int c, int n) { return s_chain[min(c, dk - 1) * dv + min(n, dv - 1)]; });
        } else if (s0 != nullptr) {
            const Rsrc bs = view(s0, 4u * (uint32_t)(dk * dv));
            take_state([&](int c, int n) { return fetch<float>(bs, 4u * (uint32_t)(min(c, dk - 1) * dv + min(n, dv - 1))); });
        }
    }
    float lg_sum = 0.f;       // state pass, wave 0: log2 of the span's total decay on channel `tid`
    const int lg_at = tid < 32 ? ((tid & 15) >> 2) * TS + 4 * (tid >> 4) + (tid & 3) : ((tid & 3) * TS + 8 + ((tid - 32) >> 2));

    per_wave([&](auto wave_c, int) {
        gate(wave_c, 0, qf);
        publish(wave_c, -1);
        HILO_WAVE_END(decltype(wave_c)::value);
    }, 0);
    issue_qkv(row_s0 + kChunk, tok1);        // (in the order in which the loop leaves its loads)
    scan(1, r_la);
    issue_la(r_la, walk_s, tok);             // chunk 2
    __syncthreads();

    // Iteration c: contraction of chunk c from one set, gating of chunk c + 1 into the other, scan of chunk c + 2.  (Past the
    // span's end rows are nothing: what is gated and scanned there is not read.)
    const int tr_row = lm >> 2, tr_col = (4 * (lm & 3)) ^ (8 * (g >> 1));   // transposing reads: token-in-4 and column quad of this lane
    for (int c = 0; c < nch; ++c) {
        auto step = [&](auto wave_c, int) {
            constexpr int W = decltype(wave_c)::value;
            constexpr int NQ = W / 2 + 1;                     // 32-token steps that hold causal tokens for this wave
            constexpr int t_lo = OW::start(W), t_hi = OW::start(W + 1);
            const uint16_t *vtr = s_v + (c & 1) * SET + (4 * g + tr_row) * VS + tr_col;
            const uint16_t *ktr = s_k + (c & 1) * SET + (4 * g + tr_row) * RS + tr_col;
            auto v_frag = [&](int q32, int x) {   // slot (g, e) of step q32 = token 32 q32 + 16 (e / 4) + 4 g + e % 4
                const u32x2 lo = lds_read_tr(vtr + 32 * q32 * VS + 16 * x);
                const u32x2 hi = lds_read_tr(vtr + (32 * q32 + 16) * VS + 16 * x);
                return u32x4{lo[0], lo[1], hi[0], hi[1]};
            };
            auto tail_frag = [&](const uint16_t *at) {
                u32x4 t = u32x4{0, 0, 0, 0};
#pragma unroll
                for (int e = 0; e < DT; ++e) {
                    const u32x2 y = *reinterpret_cast<const u32x2 *>(at + 16 * e);
                    t[2 * e] = y[0];
                    t[2 * e + 1] = y[1];
                }
                return t;
            };
            auto k_frag = [&](int q32, int col) {
                const u32x2 lo = lds_read_tr(ktr + 32 * q32 * RS + col);
                const u32x2 hi = lds_read_tr(ktr + (32 * q32 + 16) * RS + col);
                return u32x4{lo[0], lo[1], hi[0], hi[1]};
            };
            // ---- state tiles of this wave: P + K~^T V ----
            if constexpr (t_lo < t_hi) {
                constexpr int NT_LO = t_lo / NCT, NT_HI = (t_hi - 1) / NCT;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    u32x4 kf[2 + 2 + DT];        // hi of ct 0, 1; lo of ct 0, 1; tails
#pragma unroll
                    for (int ct = 0; ct < NCT; ++ct) {
                        bool used = false;
                        for (int t = t_lo; t < t_hi; ++t) used = used || (t % NCT == ct);
                        if (!used) continue;
                        if (ct < 2) {
                            kf[ct] = k_frag(q, 16 * ct);
                            kf[2 + ct] = k_frag(q, 32 + 16 * ct);
                        } else {
                            kf[2 + ct] = k_frag(q, 64 + 16 * (ct - 2));
                        }
                    }
#pragma unroll
                    for (int nt = NT_LO; nt <= NT_HI; ++nt) {
                        const u32x4 vf = v_frag(q, nt);
#pragma unroll
                        for (int ct = 0; ct < NCT; ++ct) {
                            const int t = nt * NCT + ct;
                            if (t < t_lo || t >= t_hi) continue;
                            f32x4 a = acc[t - t_lo];
                            if (ct < 2) a = mfma(kf[ct], vf, a);
                            a = mfma(kf[2 + ct], vf, a);
                            acc[t - t_lo] = a;
                        }
                    }
                }
            }
            if constexpr (OUT) {
                // offset (bf16 row) of the four columns this lane holds of column tile x of its token's row
                const uint32_t orow = row_is_token(c) ? (uint32_t)tok0 * dv2 + 8u * (uint32_t)g : kNowhere / 2;
                auto ocol = [&](int x) { return 4 * g + 16 * x < dv ? orow + 32u * (uint32_t)x : kNowhere / 2; };
                f32x4 o[NX];
                u32x2 rg[FUSE ? NX : 1];
                f32x4 prev[ACC ? NX : 1];
                if constexpr (FUSE) {
                    // output-gate pre-activations of the wave's tokens, fetched now so that they have arrived at the end
                    if (epilogue) {
#pragma unroll
                        for (int x = 0; x < NX; ++x) rg[x] = fetch<u32x2>(br, ocol(x));
                    }
                }
                if constexpr (ACC) {   // rows to add to
#pragma unroll
                    for (int x = 0; x < NX; ++x)
                        prev[x] = fetch<f32x4>(bo, OE * ocol(x));
                }
                // (The products of several tiles go round: each tile's are a chain of dependent instructions.)
                // ---- score tiles, transposed: lane (lm, g) gets A[i = 16 W + lm][j = 16 jt + 4 g + r] ----
                u32x4 pah[NQ], pal[NQ];                       // A^T hi, lo: B operand of O^T += V^T A^T
                {
                    u32x4 kh[W + 1], kl[W + 1], kt[W + 1];
                    f32x4 d[W + 1];
#pragma unroll
                    for (int jt = 0; jt <= W; ++jt) {
                        const uint16_t *krow = s_k + (c & 1) * SET + (16 * jt + lm) * RS;
                        kh[jt] = *reinterpret_cast<const u32x4 *>(krow + (8 * g ^ swz));
                        kl[jt] = *reinterpret_cast<const u32x4 *>(krow + 32 + (8 * g ^ swz));
                        kt[jt] = tail_frag(krow + 64 + (4 * g ^ swz));
                        d[jt] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
#pragma unroll
                    for (int m = 0; m < 5; ++m)
#pragma unroll
                        for (int jt = 0; jt <= W; ++jt)
                            d[jt] = mfma(m == 4 ? kt[jt] : (m < 2 ? kh[jt] : kl[jt]), m == 4 ? qf.t : ((m & 1) ? qf.l : qf.h), d[jt]);
                    // causal mask of the diagonal tile
                    d[W] = f32x4{4 * g + 0 > lm ? 0.f : d[W][0], 4 * g + 1 > lm ? 0.f : d[W][1], 4 * g + 2 > lm ? 0.f : d[W][2],
                                 4 * g + 3 > lm ? 0.f : d[W][3]};
#pragma unroll
                    for (int q = 0; q < NQ; ++q) pah[q] = pal[q] = u32x4{0, 0, 0, 0};
#pragma unroll
                    for (int jt = 0; jt <= W; ++jt) {
                        const int h = 2 * (jt & 1);
                        SPLIT_PAIR(d[jt][0], d[jt][1], pah[jt / 2][h], pal[jt / 2][h]);
                        SPLIT_PAIR(d[jt][2], d[jt][3], pah[jt / 2][h + 1], pal[jt / 2][h + 1]);
                    }
                }
                // ---- O^T = P^T Q~^T + V^T A^T: lane (lm, g) accumulates O[i = 16 W + lm][n = 16 x + 4 g + r] ----
                constexpr int GX = (NX + 1) / 2;
#pragma unroll
                for (int x0 = 0; x0 < NX; x0 += GX) {
                    u32x4 ph[GX], pl[GX], pt[GX];
#pragma unroll
                    for (int i = 0; i < GX; ++i) {
                        const uint16_t *prow = s_p + (c & 1) * SET + (16 * min(x0 + i, NX - 1) + lm) * RS;
                        ph[i] = *reinterpret_cast<const u32x4 *>(prow + (8 * g ^ swz));
                        pl[i] = *reinterpret_cast<const u32x4 *>(prow + 32 + (8 * g ^ swz));
                        pt[i] = tail_frag(prow + 64 + (4 * g ^ swz));
                    }
#pragma unroll
                    for (int m = 0; m < 5; ++m)
#pragma unroll
                        for (int i = 0; i < GX; ++i)
                            if (x0 + i < NX)
                                o[x0 + i] = mfma(m == 4 ? pt[i] : (m < 2 ? ph[i] : pl[i]), m == 4 ? qf.t : ((m & 1) ? qf.l : qf.h),
                                                 m == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : o[x0 + i]);
                }
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    u32x4 vf[NX];
#pragma unroll
                    for (int x = 0; x < NX; ++x) vf[x] = v_frag(q, x);
#pragma unroll
                    for (int x = 0; x < NX; ++x) o[x] = mfma(vf[x], pah[q], o[x]);
#pragma unroll
                    for (int x = 0; x < NX; ++x) o[x] = mfma(vf[x], pal[q], o[x]);
                }
                if constexpr (FUSE) {
                    if (epilogue) {
                        // Swish(r) * LN(o): a token's row is spread over the four lanes lm, lm+16, lm+32, lm+48
                        // (columns past dv are exact zeros: they add nothing to the sum and are left out of the squares)
                        const float inv_n = 1.f / (float)dv;
                        float sum = 0.f;
#pragma unroll
                        for (int x = 0; x < NX; ++x) sum += (o[x][0] + o[x][1]) + (o[x][2] + o[x][3]);
                        sum += __shfl_xor(sum, 16);
                        sum += __shfl_xor(sum, 32);
                        const float mean = sum * inv_n;
                        float sq = 0.f;
#pragma unroll
                        for (int x = 0; x < NX; ++x) {
                            if (4 * g + 16 * x < dv) {
#pragma unroll
                                for (int r = 0; r < 4; ++r) {
                                    const float d = o[x][r] - mean;
                                    sq = fmaf(d, d, sq);
                                }
                            }
                        }
                        sq += __shfl_xor(sq, 16);
                        sq += __shfl_xor(sq, 32);
                        const float rstd = __builtin_amdgcn_rsqf(sq * inv_n + p.ln_eps);
#pragma unroll
                        for (int x = 0; x < NX; ++x) {
                            if (4 * g + 16 * x < dv) {
                                const f32x4 lw = *reinterpret_cast<const f32x4 *>(s_lnw + 16 * x + 4 * g);
                                const f32x4 lb = *reinterpret_cast<const f32x4 *>(s_lnb + 16 * x + 4 * g);
                                const float rv[4] = {bf16_lo_as_float(rg[x][0]), bf16_hi_as_float(rg[x][0]),
                                                     bf16_lo_as_float(rg[x][1]), bf16_hi_as_float(rg[x][1])};
#pragma unroll
                                for (int r = 0; r < 4; ++r) {
                                    const float sw = rv[r] * __builtin_amdgcn_rcpf(1.f + exp2_fast(-rv[r] * kLog2e));
                                    o[x][r] = fmaf((o[x][r] - mean) * rstd, lw[r], lb[r]) * sw;
                                }
                            }
                        }
                    }
                }
                if constexpr (ACC) {
#pragma unroll
                    for (int x = 0; x < NX; ++x) o[x] += prev[x];
                }
#pragma unroll
                for (int x = 0; x < NX; ++x) {        // dv is a multiple of 8: all four columns or none
                    if constexpr (sizeof(TOut) == 4) put(bo, OE * ocol(x), o[x]);
                    else put(bo, OE * ocol(x), u32x2{pack_bf16(o[x][0], o[x][1]), pack_bf16(o[x][2], o[x][3])});
                }
            }
            QFrag qn;
            gate(wave_c, c + 1, qn);
            publish(wave_c, c);
            qf = qn;
            HILO_WAVE_END(W);
        };
        per_wave(step, c);
        if constexpr (!OUT) {
            if (tid < dk) {
                const float *t_c = s_tot + ring(c) * L::kTotBuf + lg_at;
                lg_sum += (t_c[0] + t_c[4 * TS]) + (t_c[8 * TS] + t_c[12 * TS]);
            }
        }
        tok0 = tok1;
        tok1 = tok;
        issue_qkv(walk_s, tok1);         // chunk c + 2
        scan(c + 2, r_la);
        next_row_token();
        issue_la(r_la, walk_s, tok);     // chunk c + 3
        __syncthreads();
    }

    // ---- the span's state ----
    float *dst = nullptr;
    if (!OUT)
        dst = p.ws_state + ((size_t)bh * p.nspans + sp) * dk * dv;
    else if ((p.nspans == 1 || p.chain_in_output) && sp == p.nspans - 1 && p.final_state != nullptr)
        dst = p.final_state + (size_t)bh * dk * dv;  // the last span ends in the final state
    if (dst != nullptr) {
        per_wave([&](auto wave_c, int) {
            each_state(wave_c, [&](int i, int r, int ch, int n) {
                if (ch < dk && n < dv) dst[ch * dv + n] = acc[i][r];
            });
            HILO_WAVE_END(decltype(wave_c)::value);
        }, 0);
    }
    // the workspace keeps natural logarithms
    if (!OUT && tid < dk) p.ws_lgam[((size_t)bh * p.nspans + sp) * dk + tid] = lg_sum * kLn2;
}

template <bool OUT, bool FUSE, bool ACC, bool SHIFT, typename TOut>
hipError_t launch_one(const Params &p, hipStream_t stream) {
    using L = HLayout<OUT, FUSE && OUT>;
    constexpr int MINW = OUT ? 2 : 3;
    auto kernel = hilo_span_kernel<OUT, MINW, FUSE, ACC, SHIFT, TOut>;
    const int spans = (!OUT && p.chain_in_output) ? p.nspans - 1 : p.nspans;
    static std::atomic<bool> configured[kMaxDevices] = {};  // per instantiation and device
    {
        hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), L::kBytes, configured);
        if (e != hipSuccess) return e;
    }
    return launch_in_parts(p, spans, 256, [&](const Params &part, int, int) {
        dim3 grid((unsigned)(part.B * part.H * spans)), block(256);
        hipLaunchKernelGGL(kernel, grid, block, L::kBytes, stream, part);
        return hipGetLastError();
    });
}

}  // namespace

// One-sided gates, the DiG-XL/2 heads (36 / 72) and what their registers hold (launch_mfma_span and launch_mfma_row_read leave
// the shortest spans of these to the kernels that stage rows through LDS).  Heads of up to 32 / 64 channels stay with the
// kernels in gla_mfma.hip: a chunk has less to overlap there, and those have an 8-wave form for few groups (6 sequences of 432
// tokens 14.6 us, here 17.0; backward of 42 sequences of 256 steps 27.8 and 30.0; only calls of more than 256 groups would
// gain, 24 sequences of 6292 tokens with the epilogue 49.8 and 46.6).
bool hilo_kernels_cover(const Params &p) {
    return !two_sided(p) && p.dk <= 36 && p.dv <= 80 && (p.dk > 32 || p.dv > 64);
}

hipError_t launch_hilo_span(const Params &p, SpanMode mode, hipStream_t stream) {
    const bool fuse = p.z_gate != nullptr, bf16 = p.out_dtype == GLA_DT_BF16;
    if (mode == kModeState) {
        if (fuse) return launch_one<false, true, false, false, float>(p, stream);
        return p.gate_shift ? launch_one<false, false, false, true, float>(p, stream)
                            : launch_one<false, false, false, false, float>(p, stream);
    }
    if (fuse)
        return bf16 ? launch_one<true, true, false, false, uint16_t>(p, stream)
                    : launch_one<true, true, false, false, float>(p, stream);
    if (p.accumulate) return launch_one<true, false, true, false, float>(p, stream);   // host checks fp32 out
    if (p.gate_shift) return launch_one<true, false, false, true, float>(p, stream);   // (backward: fp32 rows)
    return bf16 ? launch_one<true, false, false, false, uint16_t>(p, stream)
                : launch_one<true, false, false, false, float>(p, stream);
}

}  // namespace gla
