// bf16 MFMA kernel for the state reads of the backward pass of the GLA recurrence
// (DiG paper, Sec. 3.1 Eq. (attn_gla) rows 1-3 with beta = 1, differentiated; chunks of M = 64
// tokens computed on-chip as in Sec. 3.5).
//
// It computes r_s[c] = sum_n S_s[c,n] w_s[n] for every scan step s of a span, where S follows
// S_s = diag(alpha_s) S_{s-1} + k_s^T v_s: with w = dO this is dq, and on the reversed recurrence
// of G = dL/dS (k, v := q, dO, gates shifted by one step) with w = v it is dk.
//
// Chunk form.  With b_j the inclusive sum of log_alpha inside the chunk (per key channel),
// k~_j = k_j exp(-b_j), E_j = exp(b_j) and S_0 the state entering the chunk,
//     S_j = diag(E_j) (S_0 + sum_{i<=j} k~_i^T v_i)
//     r_j = E_j * ( sum_{i<=j} (w_j . v_i) k~_i  +  S_0 w_j )          ("*" elementwise over channels)
//     S_C = diag(E_C) (S_0 + K~^T V)
// i.e. per chunk  P = tril(W V^T)  (plain bf16 operands, contraction over the value columns),
// R = E * (P K~ + W S_0^T),  S += K~^T V then scaled.  P, K~ and S_0 are split into a bf16 "hi" part
// and a bf16 "lo" remainder (three products where two split operands meet, two otherwise).
//
// One work-group walks the chunks of its span.  With 4 waves, wave i owns the 16 tokens 16i..16i+15 of a
// chunk (all channels of R) and the state tiles of the value-column tiles i, i+4; with 8, waves i and i+4
// share those tokens and the state tiles go round over all of them (see the kernel).  The state is kept
// transposed, S^T[n][c], in fp32 accumulators: a lane then holds four consecutive value columns of one
// channel, which is (a) a 16-byte load from the [dk][dv] state the carry kernel left in the workspace,
// (b) an 8-byte LDS write of the bf16 parts as the channel-major rows that the S_0 term reads as its A
// operand, and (c) scaled by one exp(b_C) per lane.
// P is computed transposed (as in the forward kernel) so that its accumulator registers are the B
// operand of the next contraction: slot (g, e) of a 32-token step is token 32q + 16(e/4) + 4g + e%4,
// and K~ (contracted over tokens) is fetched in the same order by the transposing LDS read.
#include <type_traits>

#include "gla_common.h"
#include "gla_mfma_util.h"

namespace gla {
namespace {

template <int NDK8, int NDV16, bool DV, bool BETA, bool GS>
struct RLayout {
    static constexpr int kDkp = NDK8 * 8;
    static constexpr int kDvp = NDV16 * 16;
    static constexpr int kNct = (NDK8 + 1) / 2;                           // 16-channel tiles
    // bf16 per row of K~: whole 16-channel tiles, an odd number of 16-byte units
    static constexpr int kChStride = (NDK8 % 4 == 0) ? kDkp + 8 : ((kDkp + 8 + 15) / 16) * 16 + 8;
    // bf16 per row of V, W and S_0: the columns, then an all-zero group of 8 (lanes whose column group lies
    // beyond the last one read that group); again an odd number of 16-byte units
    static constexpr int kVStride = kDvp + 8;
    static constexpr int kZeroCol = kDvp;
    static constexpr int kLaStride = kDkp + 4;                            // fp32 per row of log_alpha, then E
    static constexpr int kRowK = kChunk * kChStride * 2;
    static constexpr int kRowV = kChunk * kVStride * 2;
    static constexpr int kSt = 16 * kNct * kVStride * 2;

    static constexpr int oTok = 0;                                        // int[4][64]
    static constexpr int oGam = oTok + 4 * kChunk * 4;                    // float[64] exp(b_C)
    static constexpr int oLa = oGam + 64 * 4;
    static constexpr int oKHi = oLa + kChunk * kLaStride * 4;
    static constexpr int oKLo = oKHi + kRowK;
    static constexpr int oV = oKLo + kRowK;
    static constexpr int oW = oV + kRowV;
    static constexpr int oStHi = oW + kRowV;
    static constexpr int oStLo = oStHi + kSt;
    static constexpr int oQHi = oStLo + kSt;                              // with DV or GS: raw q rows, then q~ hi / lo
    static constexpr int oQLo = oQHi + kRowK;
    static constexpr int oEndAlpha = DV || GS ? oQLo + kRowK : oStLo + kSt;
    // two-sided gate: raw log_beta rows, the bf16 remainders of the gated v and w rows, exp(c_C) per value column
    static constexpr int kLbStride = kDvp + 4;
    static constexpr int oLb = oEndAlpha;
    static constexpr int oVLo = oLb + kChunk * kLbStride * 4;
    static constexpr int oWLo = oVLo + kRowV;
    static constexpr int oGamB = oWLo + kRowV;                            // float[kDvp]
    // with DV, the gate gradients: sums of the waves' 16 tokens [4], and the sum over all later scan steps [2]
    static constexpr int oTot = BETA ? oGamB + kDvp * 4 : oEndAlpha;      // float[4 + 2][kDkp]
    static constexpr int oTotB = oTot + (DV ? 6 * kDkp * 4 : 0);          // float[4 + 2][kDvp]
    // with GS, the chunk's b_C and c_C (base 2)
    static constexpr int oLg = oTotB + (DV && BETA ? 6 * kDvp * 4 : 0);   // float[64]
    static constexpr int oLgB = oLg + (GS ? 64 * 4 : 0);                  // float[kDvp]
    static constexpr int kBytes = oLgB + (GS && BETA ? kDvp * 4 : 0);
    static_assert(kBytes % 16 == 0, "cleared in 16-byte pieces");
    // (the span plan and the choice of waves count on it; 81,600 bytes of 81,920 for 5 x 5 with DV)
    static_assert(BETA || NDK8 > 5 || kBytes <= 80 * 1024, "two groups per compute unit up to 40 / 80 channels");
};

template <int N>
using int_c = std::integral_constant<int, N>;

// DV = also compute the outputs o_j = q_j S_j of the same recurrence (fp32 rows to p.out; p.q holds q):
//     o_j = sum_{i<=j} (q~_j . k~_i) v_i + q~_j S_0 ,   q~_j = q_j E_j
// as the forward kernel does, on the operands that are already in LDS.  In the backward pass the reversed
// recurrence of G needs both: dk as the row read against v, and dv = k G as the output with q := k.
// BETA = two-sided gate (p.log_beta): with c_j the inclusive sum of log_beta inside the chunk (per value column),
// F_j = exp(c_j), v~_i = v_i / F_i and w~_j = w_j * F_j,
//     r_j = E_j * ( sum_{i<=j} (w~_j . v~_i) k~_i + S_0 w~_j ),   S_C = diag(E_C) (S_0 + K~^T V~) diag(F_C):
// the same contractions with v~ and w~ (bf16 hi/lo pairs, all four products) in the places of v and w; with DV the
// outputs are o_j = F_j * (sum_{i<=j} (q~_j . k~_i) v~_i + q~_j S_0) (F_j is left in place of the raw log_beta row).
// Gate gradients (DV, p.dlog_alpha): dlog_alpha_s = sum_{s' >= s} (q dq - k dk) runs along this very walk (it visits the
// last scan step first), so the kernel forms it from the dk rows it holds and the dq rows of the walk before, instead of
// two more kernels over q, k, dq, dk and the result (29.6 + 17 us at the size below; this kernel takes 21 us more, and
// the call 205 -> 182 us on MI355X: 16 sequences of 16384 steps, 36 / 72 channels).  The part of the sum that lies
// before the span is a product of two states (see the prologue), not a chain over spans; its error is five times
// smaller than that of a sum over all steps (2.7e-5 against 1.5e-4).  With the two-sided gate both gradients (4
// images of 1024 tokens): 244 -> 192 us for a training step, which includes that the chain of the span states keeps
// 4 instead of 16 spans in flight there and no longer spills.
//
// NW = 4: the waves own 16 tokens each.  NW = 8, where a group has its compute unit to itself anyway (the LDS of the
// large classes, or no more groups than compute units): two waves per 16 tokens, one for the row read (with DV; without,
// the channel tiles are shared), one for the outputs, so that a SIMD has a second wave to issue from.  MI355X: 256
// sequences of 256 steps at 36 / 72 channels, dk and dv 34.4 -> 28.2 us; two-sided gate, 64 sequences of 1024 steps,
// dk and dv 65.9 -> 50.7 us, dq 33.7 -> 31.8 us; 8 sequences of 2304 steps at 64 / 128, whole backward 105 -> 62 us.
//
// GS (the walk for dq): the local states of the reversed recurrence come along, so that it needs no state pass of its
// own (which would read q, dO and the gates once more; of these only q is new here).  From a zero state its span over
// the steps a .. b - 1 ends in
//     U[c,n] = sum_s prod_{a < u <= s} alpha_u[c] beta_u[n] q_s[c] dO_s[n],
// which a forward walk can sum chunk by chunk: the decay from a to the chunk times (q~^T dO~ of the chunk).  MI355X: the
// walk for dq takes 59 instead of 45 us (16 sequences of 16384 steps, 36 / 72 channels) and the state pass of 31 us
// goes, 182 -> 167 us for the call; two-sided gate, 64 sequences of 1024 steps: 32 -> 36 us, without a state pass of 21.
// FOUR: lo times lo as well where two split operands meet, for calls whose longer spans gla_hilo_bwd.hip walks that way (errors
// of dq and dk 4.3e-6 -> 3.5e-6, of dlog_alpha 1.4e-5 -> 1.0e-5 at two chunks a span; 0.3 % of a call).
template <int NDK8, int NDV16, int NW, int MINW, bool DV, bool BETA, bool GS, bool FOUR>
__global__ __launch_bounds__(NW * 64, MINW) void mfma_row_read_kernel(WalkParams p, const void *w_in, float *r_out) {
    using L = RLayout<NDK8, NDV16, DV, BETA, GS>;
    static_assert(!(DV && GS), "either walk");
    constexpr bool Q = DV || GS;     // q~ rows are needed
    constexpr int LBS = L::kLbStride;
    constexpr int NTHR = NW * 64;
    static_assert(NW == 4 || NW == 8, "one or two waves per 16 tokens");
    constexpr int CHS = L::kChStride, VS = L::kVStride, LAS = L::kLaStride;
    constexpr int NCT = L::kNct;
    constexpr int KSV = (NDV16 * 2 + 3) / 4;        // 32-column steps of the contractions over value columns
    constexpr int TPW = (NDV16 + NW - 1) / NW;      // value-column tiles of the state per wave
    constexpr int NTB = 4;       // token maps: the chunk before (its last token may be row 0's gate), this one, the next two
    static_assert(16 * NCT <= CHS, "channel tiles must fit the operand row");
    static_assert(NW * L::kDkp <= kChunk * LAS, "scratch of the prologue");
    auto gstate_tile = [](int w, int i) { return (w + NW - 1) % NW + NW * i; };     // GS: the same for U
    // value-column tile of the state that is the i-th of wave w (8 waves without DV: the second waves of the tokens,
    // which have fewer channel tiles of the row read, take the first four)
    auto state_tile = [](int w, int i) { return (NW == 8 && !DV ? (w + 4) % 8 : w) + NW * i; };

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    int *s_tok = reinterpret_cast<int *>(smem + L::oTok);
    float *s_gam = reinterpret_cast<float *>(smem + L::oGam);
    float *s_la = reinterpret_cast<float *>(smem + L::oLa);
    uint16_t *s_khi = reinterpret_cast<uint16_t *>(smem + L::oKHi);
    uint16_t *s_klo = reinterpret_cast<uint16_t *>(smem + L::oKLo);
    uint16_t *s_v = reinterpret_cast<uint16_t *>(smem + L::oV);
    uint16_t *s_w = reinterpret_cast<uint16_t *>(smem + L::oW);
    uint16_t *s_sthi = reinterpret_cast<uint16_t *>(smem + L::oStHi);
    uint16_t *s_stlo = reinterpret_cast<uint16_t *>(smem + L::oStLo);
    uint16_t *s_qhi = reinterpret_cast<uint16_t *>(smem + L::oQHi);
    uint16_t *s_qlo = reinterpret_cast<uint16_t *>(smem + L::oQLo);
    float *s_lb = reinterpret_cast<float *>(smem + L::oLb);            // BETA only, like the three below
    uint16_t *s_vlo = reinterpret_cast<uint16_t *>(smem + L::oVLo);
    uint16_t *s_wlo = reinterpret_cast<uint16_t *>(smem + L::oWLo);
    float *s_gamb = reinterpret_cast<float *>(smem + L::oGamB);
    float *s_tot = reinterpret_cast<float *>(smem + L::oTot), *s_later = s_tot + 4 * L::kDkp;         // DV
    float *s_lg = reinterpret_cast<float *>(smem + L::oLg), *s_lgb = reinterpret_cast<float *>(smem + L::oLgB);   // GS
    float *s_totb = reinterpret_cast<float *>(smem + L::oTotB), *s_laterb = s_totb + 4 * L::kDvp;     // DV, BETA

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lm = lane & 15;
    const int g = lane >> 4;

    // contiguous ranges of spans per XCD (work-groups are dealt round-robin to the 8 XCDs)
    int blk = blockIdx.x;
    {
        const int nb = gridDim.x;
        if ((nb & 7) == 0) blk = (blk & 7) * (nb >> 3) + (blk >> 3);
    }
    const int bh = blk / p.nspans;
    int sp_ = blk - bh * p.nspans;
    // when the work-groups chain the span states themselves the cost grows with the span index: odd heads walk
    // their spans backwards, so that the two groups sharing a compute unit pair a long chain with a short one
    if (p.chain_in_output && (bh & 1)) sp_ = p.nspans - 1 - sp_;
    const int sp = sp_;
    const int dk = p.dk, dv = p.dv, T = p.T;
    const int s_begin = span_begin(p, sp);
    const int s_end = span_end(p, sp);
    const int nch = (s_end - s_begin + kChunk - 1) / kChunk;

    const size_t base_k = slab_k(p, bh), base_v = slab_v(p, bh);
    const char *gk = static_cast<const char *>(p.k) + base_k * 2;
    const char *gv = static_cast<const char *>(p.v) + base_v * 2;
    const char *gw = static_cast<const char *>(w_in) + base_v * 2;
    const char *gla_ = reinterpret_cast<const char *>(p.log_alpha) + base_k * 4;
    char *gr = reinterpret_cast<char *>(r_out) + base_k * 4;
    const char *gq = static_cast<const char *>(p.q) + base_k * 2;
    const char *glb = reinterpret_cast<const char *>(p.log_beta) + base_v * 4;
    char *gout = static_cast<char *>(p.out) + base_v * 4;
    const char *gdq = reinterpret_cast<const char *>(p.fwd_dq) + base_k * 4;          // DV: the gate gradients
    const char *gof = reinterpret_cast<const char *>(p.fwd_out) + base_v * 4;
    char *gdla = reinterpret_cast<char *>(p.dlog_alpha) + base_k * 4;
    char *gdlb = reinterpret_cast<char *>(p.dlog_beta) + base_v * 4;

    // ---- state tiles of this wave, transposed: acc[i][ct][r] = S[c = 16 ct + lm][n = 16 state_tile(w, i) + 4 g + r] ----
    f32x4 acc[TPW][NCT];
#pragma unroll
    for (int i = 0; i < TPW; ++i)
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) acc[i][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    // GS: the tiles of U this wave sums, the log2 of the decay from the span's first step to the current chunk
    f32x4 accg[GS ? TPW : 1][NCT];
    float decay[NCT];
    f32x4 decay_b[GS && BETA ? TPW : 1];
    if constexpr (GS) {
#pragma unroll
        for (int i = 0; i < TPW; ++i)
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) accg[i][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // The state entering the span: what the carry kernel left in the workspace, or (chain_in_output) chained here
    // from the local states of the spans before it (chain_span_states: nearest span first, until the accumulated
    // decay makes the rest vanish in fp32); the result goes through LDS into the accumulator layout.
    {
        const bool chain = p.chain_in_output && sp > 0;   // uniform over the group
        if (chain) {
            constexpr int kV4 = (L::kDkp * L::kDvp / 4 + NTHR - 1) / NTHR;  // float4 per thread
            constexpr int kBudget = BETA ? 16 : 32;                         // float4 in flight (BETA: as many of log_beta)
            constexpr int kRun = kBudget / kV4 > 0 ? kBudget / kV4 : 1;     // spans in flight
            chain_span_states<NTHR, kV4, kRun, BETA>(p, bh, sp, tid, reinterpret_cast<float *>(smem));
        }
        __syncthreads();
        if (chain) {
            const float *s_chain = reinterpret_cast<const float *>(smem);
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                const int n = 16 * state_tile(w, i) + 4 * g;
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct) {
                    const int c = 16 * ct + lm;
                    if (c < dk && n < dv) acc[i][ct] = *reinterpret_cast<const f32x4 *>(s_chain + c * dv + n);
                }
            }
        }
        __syncthreads();
        if (!p.chain_in_output && p.nspans > 1) {
            const float *s0 = p.ws_state + ((size_t)bh * p.nspans + sp) * dk * dv;
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                const int n = 16 * state_tile(w, i) + 4 * g;
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct) {
                    const int c = 16 * ct + lm;
                    if (c < dk && n < dv) acc[i][ct] = *reinterpret_cast<const f32x4 *>(s0 + c * dv + n);
                }
            }
        }
    }

    // ---- prologue: clear LDS (pads must read as zero), token maps of the first two chunks ----
    for (int i = tid; i < L::kBytes / 16; i += NTHR)
        reinterpret_cast<u32x4 *>(smem)[i] = u32x4{0, 0, 0, 0};
    __syncthreads();
    if (tid < 2 * kChunk) {
        const int s = s_begin + tid;
        const int sc = (s < s_end) ? s : s_begin;
        s_tok[tid] = scan_token(p.scan_dir, sc, T, p.grid_h, p.grid_w);
    }
    const int tok_before = scan_token(p.scan_dir, max(s_begin - 1, 0), T, p.grid_h, p.grid_w);   // the step before the span
    if (tid == 0) s_tok[NTB * kChunk - 1] = tok_before;
    if constexpr (GS) {
        // (the first step's own gate does not act on its q^T dO, but is part of the chunk's prefix sums)
        const int tok_first = scan_token(p.scan_dir, s_begin, T, p.grid_h, p.grid_w);
        const float *la_a = reinterpret_cast<const float *>(gla_) + (size_t)tok_first * p.st_k;
        const float *lb_a = reinterpret_cast<const float *>(glb) + (size_t)tok_first * p.st_v;
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) decay[ct] = fminf(-la_a[min(16 * ct + lm, dk - 1)] * kLog2e, kMaxExp2);
        if constexpr (BETA) {
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                const f32x4 x = *reinterpret_cast<const f32x4 *>(lb_a + min(16 * gstate_tile(w, i) + 4 * g, dv - 4));
#pragma unroll
                for (int r = 0; r < 4; ++r) decay_b[i][r] = fminf(-x[r] * kLog2e, kMaxExp2);
            }
        }
    }
    if constexpr (DV) {
        // The gate gradients are sums over all later scan steps, i.e. over the steps this walk has made before:
        // those before the span add up to the gradient of the gate between it and them,
        //     sum_{s' >= b} (q dq - k dk)[c] = sum_n alpha_b[c] beta_b[n] G_b[c,n] S_{b-1}[c,n]
        // (and the sum over c for beta_b[n]), G_b being the state that enters this walk (acc) and S_{b-1} the one that
        // the forward walk left at the same place.
        if (p.dlog_alpha != nullptr && sp > 0) {       // (uniform)
            const float *sb = p.ws_bound + ((size_t)bh * p.bounds + (T - s_begin) / p.bound_len - 1) * (size_t)(dk * dv);
            const float *la_b = reinterpret_cast<const float *>(gla_) + (size_t)tok_before * p.st_k;
            const float *lb_b = reinterpret_cast<const float *>(glb) + (size_t)tok_before * p.st_v;
            float row_sum[NCT];
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) row_sum[ct] = 0.f;
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                const int n = 16 * state_tile(w, i) + 4 * g;
                f32x4 col_sum = f32x4{0.f, 0.f, 0.f, 0.f}, fb = f32x4{1.f, 1.f, 1.f, 1.f};
                if constexpr (BETA) {
                    if (n < dv) {
                        const f32x4 lb4 = *reinterpret_cast<const f32x4 *>(lb_b + n);
#pragma unroll
                        for (int r = 0; r < 4; ++r) fb[r] = exp2_fast(lb4[r] * kLog2e);
                    }
                }
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct) {
                    const int c = 16 * ct + lm;
                    if (c < dk && n < dv) {
                        const f32x4 s4 = *reinterpret_cast<const f32x4 *>(sb + c * dv + n);
                        const float a = exp2_fast(la_b[c] * kLog2e);
                        const f32x4 x = acc[i][ct] * s4 * fb * a;
                        row_sum[ct] += (x[0] + x[1]) + (x[2] + x[3]);
                        if constexpr (BETA) col_sum += x;
                    }
                }
                if constexpr (BETA) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float x = col_sum[r];
                        for (int m = 1; m < 16; m *= 2) x += __shfl_xor(x, m);
                        col_sum[r] = x;
                    }
                    if (lm == 0 && n < dv) *reinterpret_cast<f32x4 *>(s_laterb + n) = col_sum;
                }
            }
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) {
                float x = row_sum[ct];
                x += __shfl_xor(x, 16);
                x += __shfl_xor(x, 32);
                if (g == 0 && 16 * ct + lm < dk) s_la[w * L::kDkp + 16 * ct + lm] = x;
            }
            __syncthreads();
            if (tid < dk) {
                float x = 0.f;
#pragma unroll
                for (int u = 0; u < NW; ++u) x += s_la[u * L::kDkp + tid];
                s_later[tid] = x;
            }
        }
    }
    __syncthreads();

    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): keeps later reads of acc from waiting on the row prefetch

    // ---- HBM pieces staged by this thread: the 16-byte pieces of log_alpha (8-byte pieces of k) of a chunk and the
    // 16-byte pieces of v and w are numbered row by row; slot m of a thread is piece tid + NTHR m, so that a wave's
    // request covers neighbouring pieces of neighbouring rows.  Slots past the last piece repeat it (the load stays
    // in bounds; nothing is written to LDS for them) ----
    constexpr int kF = (kChunk * NDK8 * 2 + NTHR - 1) / NTHR;
    constexpr int kVF = (kChunk * NDV16 * 2 + NTHR - 1) / NTHR;
    const int pcs = dk >> 2, vpcs = dv >> 3;
    int frp[kF], fvrp[kVF];     // row << 8 | piece
#pragma unroll
    for (int m = 0; m < kF; ++m) {
        const int f = min(tid + NTHR * m, kChunk * pcs - 1);
        const int row = f / pcs;
        frp[m] = (row << 8) | (f - row * pcs);
    }
#pragma unroll
    for (int m = 0; m < kVF; ++m) {
        const int f = min(tid + NTHR * m, kChunk * vpcs - 1);
        const int row = f / vpcs;
        fvrp[m] = (row << 8) | (f - row * vpcs);
    }
    const uint32_t dk2 = 2u * (uint32_t)p.st_k, dv2 = 2u * (uint32_t)p.st_v;

    f32x4 r_la[kF];
    u32x2 r_k[kF];
    u32x2 r_q[Q ? kF : 1];
    u32x4 r_v[kVF], r_w[kVF];
    f32x4 r_lb[BETA ? kVF : 1][2];   // log_beta of the same 8 columns as the v piece
    auto load_chunk = [&](int chunk) {
        const int first = (chunk % NTB) * kChunk;
        const int *tok = s_tok + first;
        // token whose gate row `row` uses: with gate_shift the one visited a step earlier
        auto tokg = [&](int row) { return s_tok[(first + row - p.gate_shift) & (NTB * kChunk - 1)]; };
#pragma unroll
        for (int m = 0; m < kF; ++m) {
            const int row = frp[m] >> 8;
            const uint32_t pc = 8u * (uint32_t)(frp[m] & 255);
            r_la[m] = *reinterpret_cast<const f32x4 *>(gla_ + 2u * ((uint32_t)tokg(row) * dk2 + pc));
            r_k[m] = *reinterpret_cast<const u32x2 *>(gk + (uint32_t)tok[row] * dk2 + pc);
            if constexpr (Q) r_q[m] = *reinterpret_cast<const u32x2 *>(gq + (uint32_t)tok[row] * dk2 + pc);
        }
#pragma unroll
        for (int m = 0; m < kVF; ++m) {
            const uint32_t e2 = (uint32_t)tok[fvrp[m] >> 8] * dv2 + 16u * (uint32_t)(fvrp[m] & 255);
            r_v[m] = *reinterpret_cast<const u32x4 *>(gv + e2);
            r_w[m] = *reinterpret_cast<const u32x4 *>(gw + e2);
            if constexpr (BETA) {
                const char *lbp = glb + 2u * ((uint32_t)tokg(fvrp[m] >> 8) * dv2 + 16u * (uint32_t)(fvrp[m] & 255));
                r_lb[m][0] = *reinterpret_cast<const f32x4 *>(lbp);
                r_lb[m][1] = *reinterpret_cast<const f32x4 *>(lbp + 16);
            }
        }
    };
    load_chunk(0);

    for (int chunk = 0; chunk < nch; ++chunk) {
        const int *tok = s_tok + (chunk % NTB) * kChunk;
        // ================= (a) registers -> LDS =================
        const int nvalid = min(kChunk, s_end - s_begin - chunk * kChunk);
        if (nvalid < kChunk) {   // rows past the span: no decay, no contribution
#pragma unroll
            for (int m = 0; m < kF; ++m) {
                if ((frp[m] >> 8) >= nvalid) {
                    r_la[m] = f32x4{0.f, 0.f, 0.f, 0.f};
                    r_k[m] = u32x2{0, 0};
                    if constexpr (Q) r_q[m] = u32x2{0, 0};
                }
            }
#pragma unroll
            for (int m = 0; m < kVF; ++m) {
                if ((fvrp[m] >> 8) >= nvalid) {
                    r_v[m] = u32x4{0, 0, 0, 0};
                    r_w[m] = u32x4{0, 0, 0, 0};
                    if constexpr (BETA) r_lb[m][0] = r_lb[m][1] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
        }
#pragma unroll
        for (int m = 0; m < kF; ++m) {
            if (tid + NTHR * m < kChunk * pcs) {
                const int row = frp[m] >> 8, ch = 4 * (frp[m] & 255);
                *reinterpret_cast<f32x4 *>(s_la + row * LAS + ch) = r_la[m];
                *reinterpret_cast<u32x2 *>(s_khi + row * CHS + ch) = r_k[m];
                if constexpr (Q) *reinterpret_cast<u32x2 *>(s_qhi + row * CHS + ch) = r_q[m];
            }
        }
#pragma unroll
        for (int m = 0; m < kVF; ++m) {
            if (tid + NTHR * m < kChunk * vpcs) {
                const int row = fvrp[m] >> 8, col = 8 * (fvrp[m] & 255);
                *reinterpret_cast<u32x4 *>(s_v + row * VS + col) = r_v[m];
                *reinterpret_cast<u32x4 *>(s_w + row * VS + col) = r_w[m];
                if constexpr (BETA) {
                    *reinterpret_cast<f32x4 *>(s_lb + row * LBS + col) = r_lb[m][0];
                    *reinterpret_cast<f32x4 *>(s_lb + row * LBS + col + 4) = r_lb[m][1];
                }
            }
        }
        load_chunk(chunk + 1);   // past the span the clamped token map keeps the loads in bounds
        {
            // S_0 as bf16 hi/lo, channel-major
            const int ln = recompute_per_chunk(lane), lm2 = ln & 15, g2 = ln >> 4;
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                if (state_tile(w, i) < NDV16) {
#pragma unroll
                    for (int ct = 0; ct < NCT; ++ct) {
                        u32x2 hi, lo;
                        SPLIT_PAIR(acc[i][ct][0], acc[i][ct][1], hi[0], lo[0]);
                        SPLIT_PAIR(acc[i][ct][2], acc[i][ct][3], hi[1], lo[1]);
                        const int off = (16 * ct + lm2) * VS + 16 * state_tile(w, i) + 4 * g2;
                        *reinterpret_cast<u32x2 *>(s_sthi + off) = hi;
                        *reinterpret_cast<u32x2 *>(s_stlo + off) = lo;
                    }
                }
            }
        }
        if (w == NW - 1) {   // token map of the chunk loaded next time
            const int s = s_begin + (chunk + 2) * kChunk + lane;
            const int sc = (s < s_end) ? s : s_begin;
            s_tok[((chunk + 2) % NTB) * kChunk + lane] = scan_token(p.scan_dir, sc, T, p.grid_h, p.grid_w);
        }
        __syncthreads();

        // ================= (b) gates: lane = token, units of 4 channels dealt to the waves =================
        {
            const int j = lane;
            // (8 waves: a last round of at most half as many units as waves is dealt channel by channel below, 19.4 -> 18.1
            // and 28.2 -> 26.7 us for dq and dk, dv of 256 sequences of 256 steps at dk = 36; with 4 waves it costs registers
            // that spill, and with the two-sided gate the units of the value side, dealt from the last wave, even it out)
            const int rest = NW == 8 && !BETA && pcs % NW <= NW / 2 ? pcs % NW : 0, units = pcs - rest;
            for (int u = w; u < units; u += NW) {
                const int c0 = 4 * u;
                const f32x4 x = *reinterpret_cast<const f32x4 *>(s_la + j * LAS + c0);
                const u32x2 kr = *reinterpret_cast<const u32x2 *>(s_khi + j * CHS + c0);
                float bb[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) bb[i] = x[i] * kLog2e;
                wave_inclusive_scan4(bb[0], bb[1], bb[2], bb[3]);
                f32x4 e;
#pragma unroll
                for (int i = 0; i < 4; ++i) e[i] = exp2_fast(bb[i]);
                u32x2 khi, klo;
                SPLIT_PAIR(bf16_lo_as_float(kr[0]) * exp2_fast(fminf(-bb[0], kMaxExp2)),
                           bf16_hi_as_float(kr[0]) * exp2_fast(fminf(-bb[1], kMaxExp2)), khi[0], klo[0]);
                SPLIT_PAIR(bf16_lo_as_float(kr[1]) * exp2_fast(fminf(-bb[2], kMaxExp2)),
                           bf16_hi_as_float(kr[1]) * exp2_fast(fminf(-bb[3], kMaxExp2)), khi[1], klo[1]);
                *reinterpret_cast<u32x2 *>(s_khi + j * CHS + c0) = khi;
                *reinterpret_cast<u32x2 *>(s_klo + j * CHS + c0) = klo;
                if constexpr (Q) {
                    const u32x2 qr = *reinterpret_cast<const u32x2 *>(s_qhi + j * CHS + c0);
                    u32x2 qhi, qlo;
                    SPLIT_PAIR(bf16_lo_as_float(qr[0]) * e[0], bf16_hi_as_float(qr[0]) * e[1], qhi[0], qlo[0]);
                    SPLIT_PAIR(bf16_lo_as_float(qr[1]) * e[2], bf16_hi_as_float(qr[1]) * e[3], qhi[1], qlo[1]);
                    *reinterpret_cast<u32x2 *>(s_qhi + j * CHS + c0) = qhi;
                    *reinterpret_cast<u32x2 *>(s_qlo + j * CHS + c0) = qlo;
                }
                *reinterpret_cast<f32x4 *>(s_la + j * LAS + c0) = e;      // E_j in place of the raw gates
                if (lane == 63) {
                    *reinterpret_cast<f32x4 *>(s_gam + c0) = e;
                    if constexpr (GS) *reinterpret_cast<f32x4 *>(s_lg + c0) = f32x4{bb[0], bb[1], bb[2], bb[3]};
                }
            }
            if constexpr (NW == 8 && !BETA) for (int c = 4 * units + w; c < dk; c += NW) {
                const float b = wave_inclusive_scan(s_la[j * LAS + c] * kLog2e);
                const float e = exp2_fast(b);
                const float kx = bf16_bits_to_float(s_khi[j * CHS + c]) * exp2_fast(fminf(-b, kMaxExp2));
                const float qx = Q ? bf16_bits_to_float(s_qhi[j * CHS + c]) * e : 0.f;
                uint32_t h2, l2;
                SPLIT_PAIR(kx, qx, h2, l2);
                s_khi[j * CHS + c] = (uint16_t)(h2 & 0xffffu);
                s_klo[j * CHS + c] = (uint16_t)(l2 & 0xffffu);
                if constexpr (Q) {
                    s_qhi[j * CHS + c] = (uint16_t)(h2 >> 16);
                    s_qlo[j * CHS + c] = (uint16_t)(l2 >> 16);
                }
                s_la[j * LAS + c] = e;
                if (lane == 63) {
                    s_gam[c] = e;
                    if constexpr (GS) s_lg[c] = b;
                }
            }
            if constexpr (BETA) {
                // value side, 8-column units dealt from the last wave: v~ = v / F and w~ = w F as bf16 hi/lo
                for (int c0 = 8 * (NW - 1 - w); c0 < dv; c0 += 8 * NW) {
                    float cc[8];
#pragma unroll
                    for (int v4 = 0; v4 < 2; ++v4) {
                        const f32x4 x = *reinterpret_cast<const f32x4 *>(s_lb + j * LBS + c0 + 4 * v4);
#pragma unroll
                        for (int i = 0; i < 4; ++i) cc[4 * v4 + i] = x[i] * kLog2e;
                        wave_inclusive_scan4(cc[4 * v4], cc[4 * v4 + 1], cc[4 * v4 + 2], cc[4 * v4 + 3]);
                    }
                    const u32x4 vr = *reinterpret_cast<const u32x4 *>(s_v + j * VS + c0);
                    const u32x4 wr = *reinterpret_cast<const u32x4 *>(s_w + j * VS + c0);
                    u32x4 vh, vl, wh, wl;
                    float f[8];
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        f[2 * h] = exp2_fast(cc[2 * h]);
                        f[2 * h + 1] = exp2_fast(cc[2 * h + 1]);
                        SPLIT_PAIR(bf16_lo_as_float(vr[h]) * exp2_fast(fminf(-cc[2 * h], kMaxExp2)),
                                   bf16_hi_as_float(vr[h]) * exp2_fast(fminf(-cc[2 * h + 1], kMaxExp2)), vh[h], vl[h]);
                        SPLIT_PAIR(bf16_lo_as_float(wr[h]) * f[2 * h], bf16_hi_as_float(wr[h]) * f[2 * h + 1], wh[h], wl[h]);
                    }
                    *reinterpret_cast<u32x4 *>(s_v + j * VS + c0) = vh;
                    *reinterpret_cast<u32x4 *>(s_vlo + j * VS + c0) = vl;
                    *reinterpret_cast<u32x4 *>(s_w + j * VS + c0) = wh;
                    *reinterpret_cast<u32x4 *>(s_wlo + j * VS + c0) = wl;
                    if constexpr (DV) {
                        *reinterpret_cast<f32x4 *>(s_lb + j * LBS + c0) = f32x4{f[0], f[1], f[2], f[3]};
                        *reinterpret_cast<f32x4 *>(s_lb + j * LBS + c0 + 4) = f32x4{f[4], f[5], f[6], f[7]};
                    }
                    if (lane == 63) {
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            s_gamb[c0 + i] = f[i];
                            if constexpr (GS) s_lgb[c0 + i] = cc[i];
                        }
                    }
                }
            }
        }
        __syncthreads();

        // ================= (c) contractions =================
        const int ln = recompute_per_chunk(lane), lm3 = ln & 15, g3 = ln >> 4;
        int coln[KSV];   // column group of this lane in 32-column step ks; groups past the data alias the zero group
#pragma unroll
        for (int ks = 0; ks < KSV; ++ks) coln[ks] = (4 * ks + g3 < 2 * NDV16) ? 8 * (4 * ks + g3) : L::kZeroCol;
        const int tr_row = lm3 >> 2, tr_col = 4 * (lm3 & 3);
        auto contract = [&](auto wave_c) {
            constexpr int W = decltype(wave_c)::value;
            constexpr int IT = W & 3;                     // 16-token tile of this wave
            // what the wave does of the tile's work: the row read on channel tiles [CT0, CT1), the outputs
            constexpr bool READ = !(NW == 8 && DV) || W < 4, OUTPUTS = DV && (NW == 4 || W >= 4);
            constexpr int CT0 = NW == 8 && !DV && W >= 4 ? (NCT + 1) / 2 : 0;
            constexpr int CT1 = !READ ? 0 : (NW == 8 && !DV && W < 4 ? (NCT + 1) / 2 : NCT);
            constexpr int NQ = IT / 2 + 1;                // 32-token steps that hold tokens <= the tile's
            const int lm = lm3, g = g3;
            const uint16_t *krow_h = s_khi + (4 * g + tr_row) * CHS + tr_col;
            const uint16_t *krow_l = s_klo + (4 * g + tr_row) * CHS + tr_col;
            const uint16_t *vrow = s_v + (4 * g + tr_row) * VS + tr_col;
            const uint16_t *vrow_l = s_vlo + (4 * g + tr_row) * VS + tr_col;   // BETA
            u32x4 wf[KSV], wfl[BETA ? KSV : 1];
#pragma unroll
            for (int ks = 0; ks < (CT0 < CT1 ? KSV : 0); ++ks) {
                wf[ks] = *reinterpret_cast<const u32x4 *>(s_w + (16 * IT + lm) * VS + coln[ks]);
                if constexpr (BETA) wfl[ks] = *reinterpret_cast<const u32x4 *>(s_wlo + (16 * IT + lm) * VS + coln[ks]);
            }
            u32x4 kth[2][NCT], ktl[2][NCT];   // K~ over tokens: [32-token step][channel tile]
            auto load_k = [&](int q) {
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct) {
                    const u32x2 h0 = lds_read_tr(krow_h + 32 * q * CHS + 16 * ct);
                    const u32x2 h1 = lds_read_tr(krow_h + (32 * q + 16) * CHS + 16 * ct);
                    const u32x2 l0 = lds_read_tr(krow_l + 32 * q * CHS + 16 * ct);
                    const u32x2 l1 = lds_read_tr(krow_l + (32 * q + 16) * CHS + 16 * ct);
                    kth[q][ct] = u32x4{h0[0], h0[1], h1[0], h1[1]};
                    ktl[q][ct] = u32x4{l0[0], l0[1], l1[0], l1[1]};
                }
            };
            // rows of the gate gradient (key side), fetched now so that they have arrived when dk is there
            const int row = 16 * IT + lm;
            u32x2 raw_k[DV ? NCT : 1], raw_q[DV ? NCT : 1];
            f32x4 row_dq[DV ? NCT : 1];
            if constexpr (DV && READ) {
                if (p.dlog_alpha != nullptr) {
                    const uint32_t first = (uint32_t)tok[row] * (uint32_t)p.st_k;    // (rows past the span: a valid token's)
#pragma unroll
                    for (int ct = 0; ct < NCT; ++ct) {
                        const uint32_t e = first + (uint32_t)min(16 * ct + 4 * g, dk - 4);
                        raw_k[ct] = *reinterpret_cast<const u32x2 *>(gk + 2u * e);
                        raw_q[ct] = *reinterpret_cast<const u32x2 *>(gq + 2u * e);
                        row_dq[ct] = *reinterpret_cast<const f32x4 *>(gdq + 4u * e);
                    }
                }
            }
            f32x4 rr[NCT];
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) rr[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
            constexpr bool OWNS = (NW == 8 && !DV ? (W + 4) % 8 : W) < NDV16;   // state tiles of this wave
#pragma unroll
            for (int q = 0; q < (CT0 < CT1 ? NQ : 0); ++q) {
                u32x2 ph[2] = {u32x2{0, 0}, u32x2{0, 0}}, pl[2] = {u32x2{0, 0}, u32x2{0, 0}};
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int jt = 2 * q + u;
                    if (jt <= IT) {
                        // P^T tile: lane (lm, g) gets P[i = 16 IT + lm][j = 16 jt + 4 g + r]
                        f32x4 d = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int ks = 0; ks < KSV; ++ks) {
                            const u32x4 vf = *reinterpret_cast<const u32x4 *>(s_v + (16 * jt + lm) * VS + coln[ks]);
                            d = mfma(vf, wf[ks], d);
                            if constexpr (BETA) {
                                const u32x4 vfl = *reinterpret_cast<const u32x4 *>(s_vlo + (16 * jt + lm) * VS + coln[ks]);
                                d = mfma(vf, wfl[ks], d);
                                d = mfma(vfl, wf[ks], d);
                                d = mfma(vfl, wfl[ks], d);
                            }
                        }
                        if (jt == IT) {
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                if (4 * g + r > lm) d[r] = 0.f;
                        }
                        SPLIT_PAIR(d[0], d[1], ph[u][0], pl[u][0]);
                        SPLIT_PAIR(d[2], d[3], ph[u][1], pl[u][1]);
                    }
                }
                load_k(q);
                const u32x4 bh_ = u32x4{ph[0][0], ph[0][1], ph[1][0], ph[1][1]};
                const u32x4 bl_ = u32x4{pl[0][0], pl[0][1], pl[1][0], pl[1][1]};
#pragma unroll
                for (int ct = CT0; ct < CT1; ++ct) {
                    rr[ct] = mfma(kth[q][ct], bh_, rr[ct]);
                    rr[ct] = mfma(kth[q][ct], bl_, rr[ct]);
                    rr[ct] = mfma(ktl[q][ct], bh_, rr[ct]);
                    if constexpr (FOUR) rr[ct] = mfma(ktl[q][ct], bl_, rr[ct]);
                }
            }
            // + W S_0^T
#pragma unroll
            for (int ks = 0; ks < KSV; ++ks) {
#pragma unroll
                for (int ct = CT0; ct < CT1; ++ct) {
                    const int srow = (16 * ct + lm) * VS + coln[ks];
                    const u32x4 sh = *reinterpret_cast<const u32x4 *>(s_sthi + srow);
                    const u32x4 sl = *reinterpret_cast<const u32x4 *>(s_stlo + srow);
                    rr[ct] = mfma(sh, wf[ks], rr[ct]);
                    rr[ct] = mfma(sl, wf[ks], rr[ct]);
                    if constexpr (BETA) {
                        rr[ct] = mfma(sh, wfl[ks], rr[ct]);
                        rr[ct] = mfma(sl, wfl[ks], rr[ct]);
                    }
                }
            }
            // scale by E and store: lane (lm, g) holds channels 16 ct + 4 g .. + 3 of token 16 IT + lm
            if (row < nvalid) {
                char *orow = gr + ((uint32_t)tok[row] * (uint32_t)p.st_k + 4u * (uint32_t)g) * 4u;
#pragma unroll
                for (int ct = CT0; ct < CT1; ++ct) {
                    if (16 * ct + 4 * g < dk) {   // dk is a multiple of 4: all four channels or none
                        const f32x4 e = *reinterpret_cast<const f32x4 *>(s_la + row * LAS + 16 * ct + 4 * g);
                        f32x4 o = rr[ct];
#pragma unroll
                        for (int r = 0; r < 4; ++r) o[r] *= e[r];
                        *reinterpret_cast<f32x4 *>(orow + 64 * ct) = o;
                        if constexpr (DV) rr[ct] = o;
                    }
                }
            }
            // Gate gradient, key side: x_s = q_s * dq_s - k_s * dk_s summed over the steps walked so far (in this walk
            // the rows called k are q, those called q are k).  The sums inside the wave's 16 tokens take the place of
            // E in its rows; what the other waves' tokens and the earlier chunks add follows after the next barrier.
            if constexpr (DV && READ) {
                if (p.dlog_alpha != nullptr) {
#pragma unroll
                    for (int ct = 0; ct < NCT; ++ct) {
                        float x[4] = {0.f, 0.f, 0.f, 0.f};
                        if (row < nvalid && 16 * ct + 4 * g < dk) {
                            x[0] = fmaf(bf16_lo_as_float(raw_k[ct][0]), row_dq[ct][0], -bf16_lo_as_float(raw_q[ct][0]) * rr[ct][0]);
                            x[1] = fmaf(bf16_hi_as_float(raw_k[ct][0]), row_dq[ct][1], -bf16_hi_as_float(raw_q[ct][0]) * rr[ct][1]);
                            x[2] = fmaf(bf16_lo_as_float(raw_k[ct][1]), row_dq[ct][2], -bf16_lo_as_float(raw_q[ct][1]) * rr[ct][2]);
                            x[3] = fmaf(bf16_hi_as_float(raw_k[ct][1]), row_dq[ct][3], -bf16_hi_as_float(raw_q[ct][1]) * rr[ct][3]);
                        }
                        row_scan16x4(x[0], x[1], x[2], x[3]);
                        if (16 * ct + 4 * g < dk) {
                            const f32x4 x4 = f32x4{x[0], x[1], x[2], x[3]};
                            *reinterpret_cast<f32x4 *>(s_la + row * LAS + 16 * ct + 4 * g) = x4;
                            if (lm == 15) *reinterpret_cast<f32x4 *>(s_tot + IT * L::kDkp + 16 * ct + 4 * g) = x4;
                        }
                    }
                }
            }
            if constexpr (OUTPUTS) {
                // ---- outputs of the wave's 16 tokens: O^T[n][i], lane (lm, g) holds o[x][r] = O[i = 16 IT + lm][n = 16 x + 4 g + r]
                constexpr int NX = NDV16;
                constexpr int KS = (NDK8 + 3) / 4;            // 32-channel steps
                f32x4 o[NX];
#pragma unroll
                for (int x = 0; x < NX; ++x) o[x] = f32x4{0.f, 0.f, 0.f, 0.f};
                int colk[KS];   // channel group of this lane in step ks; groups past the data alias the all-zero group
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) colk[ks] = (4 * ks + g < NDK8) ? 8 * (4 * ks + g) : L::kDkp;
                u32x4 qfh[KS], qfl[KS];
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    qfh[ks] = *reinterpret_cast<const u32x4 *>(s_qhi + (16 * IT + lm) * CHS + colk[ks]);
                    qfl[ks] = *reinterpret_cast<const u32x4 *>(s_qlo + (16 * IT + lm) * CHS + colk[ks]);
                }
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    u32x2 ah[2] = {u32x2{0, 0}, u32x2{0, 0}}, al[2] = {u32x2{0, 0}, u32x2{0, 0}};
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int jt = 2 * q + u;
                        if (jt <= IT) {
                            // score tile, transposed: lane (lm, g) gets A[i = 16 IT + lm][j = 16 jt + 4 g + r]
                            f32x4 d = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                            for (int ks = 0; ks < KS; ++ks) {
                                const u32x4 kh = *reinterpret_cast<const u32x4 *>(s_khi + (16 * jt + lm) * CHS + colk[ks]);
                                const u32x4 kl = *reinterpret_cast<const u32x4 *>(s_klo + (16 * jt + lm) * CHS + colk[ks]);
                                d = mfma(kh, qfh[ks], d);
                                d = mfma(kh, qfl[ks], d);
                                d = mfma(kl, qfh[ks], d);
                                if constexpr (FOUR) d = mfma(kl, qfl[ks], d);
                            }
                            if (jt == IT) {
#pragma unroll
                                for (int r = 0; r < 4; ++r)
                                    if (4 * g + r > lm) d[r] = 0.f;
                            }
                            SPLIT_PAIR(d[0], d[1], ah[u][0], al[u][0]);
                            SPLIT_PAIR(d[2], d[3], ah[u][1], al[u][1]);
                        }
                    }
                    const u32x4 bh2 = u32x4{ah[0][0], ah[0][1], ah[1][0], ah[1][1]};
                    const u32x4 bl2 = u32x4{al[0][0], al[0][1], al[1][0], al[1][1]};
#pragma unroll
                    for (int x = 0; x < NX; ++x) {
                        const u32x2 v0 = lds_read_tr(vrow + 32 * q * VS + 16 * x);
                        const u32x2 v1 = lds_read_tr(vrow + (32 * q + 16) * VS + 16 * x);
                        const u32x4 vf = u32x4{v0[0], v0[1], v1[0], v1[1]};
                        o[x] = mfma(vf, bh2, o[x]);
                        o[x] = mfma(vf, bl2, o[x]);
                        if constexpr (BETA) {
                            const u32x2 l0 = lds_read_tr(vrow_l + 32 * q * VS + 16 * x);
                            const u32x2 l1 = lds_read_tr(vrow_l + (32 * q + 16) * VS + 16 * x);
                            const u32x4 vfl = u32x4{l0[0], l0[1], l1[0], l1[1]};
                            o[x] = mfma(vfl, bh2, o[x]);
                            o[x] = mfma(vfl, bl2, o[x]);
                        }
                    }
                }
                // + Q~ S_0: the state rows (channel-major in LDS) are read transposed, so the channels of a 32-channel
                // step come in the slot order 16 (e/4) + 4 g + e%4; the q~ operand is read in that order too
                const uint16_t *strow_h = s_sthi + (4 * g + tr_row) * VS + tr_col;
                const uint16_t *strow_l = s_stlo + (4 * g + tr_row) * VS + tr_col;
#pragma unroll
                for (int q = 0; q < KS; ++q) {
                    const bool second = 32 * q + 16 < 16 * NCT;    // the step's upper 16 channels exist in the state rows
                    const uint16_t *qh = s_qhi + (16 * IT + lm) * CHS + 32 * q + 4 * g;
                    const uint16_t *ql = s_qlo + (16 * IT + lm) * CHS + 32 * q + 4 * g;
                    const u32x2 qh0 = *reinterpret_cast<const u32x2 *>(qh), ql0 = *reinterpret_cast<const u32x2 *>(ql);
                    u32x2 qh1 = u32x2{0, 0}, ql1 = u32x2{0, 0};
                    if (second) {
                        qh1 = *reinterpret_cast<const u32x2 *>(qh + 16);
                        ql1 = *reinterpret_cast<const u32x2 *>(ql + 16);
                    }
                    const u32x4 qsh = u32x4{qh0[0], qh0[1], qh1[0], qh1[1]}, qsl = u32x4{ql0[0], ql0[1], ql1[0], ql1[1]};
#pragma unroll
                    for (int x = 0; x < NX; ++x) {
                        const u32x2 h0 = lds_read_tr(strow_h + 32 * q * VS + 16 * x);
                        const u32x2 l0 = lds_read_tr(strow_l + 32 * q * VS + 16 * x);
                        u32x2 h1 = u32x2{0, 0}, l1 = u32x2{0, 0};
                        if (second) {
                            h1 = lds_read_tr(strow_h + (32 * q + 16) * VS + 16 * x);
                            l1 = lds_read_tr(strow_l + (32 * q + 16) * VS + 16 * x);
                        }
                        const u32x4 sh = u32x4{h0[0], h0[1], h1[0], h1[1]}, sl = u32x4{l0[0], l0[1], l1[0], l1[1]};
                        o[x] = mfma(sh, qsh, o[x]);
                        o[x] = mfma(sh, qsl, o[x]);
                        o[x] = mfma(sl, qsh, o[x]);
                        if constexpr (FOUR) o[x] = mfma(sl, qsl, o[x]);
                    }
                }
                if (row < nvalid) {
                    char *orow2 = gout + ((uint32_t)tok[row] * (uint32_t)p.st_v + 4u * (uint32_t)g) * 4u;
#pragma unroll
                    for (int x = 0; x < NX; ++x) {
                        if (4 * g + 16 * x < dv) {
                            if constexpr (BETA) {   // row j of the outputs carries F_j per value column
                                const f32x4 f4 = *reinterpret_cast<const f32x4 *>(s_lb + row * LBS + 16 * x + 4 * g);
#pragma unroll
                                for (int r = 0; r < 4; ++r) o[x][r] *= f4[r];
                            }
                            *reinterpret_cast<f32x4 *>(orow2 + 64 * x) = o[x];
                        }
                    }
                }
                if (p.dlog_alpha != nullptr) {
                    if constexpr (BETA) {
                        // value side: y_s = o_s * dO_s - v_s * dv_s (dO are the rows called v, v those called w), the
                        // sums in the place of F
                        const uint32_t first = (uint32_t)tok[row] * (uint32_t)p.st_v;
#pragma unroll
                        for (int x = 0; x < NX; ++x) {
                            const uint32_t e = first + (uint32_t)min(16 * x + 4 * g, dv - 4);
                            const u32x2 rv = *reinterpret_cast<const u32x2 *>(gv + 2u * e);
                            const u32x2 rw = *reinterpret_cast<const u32x2 *>(gw + 2u * e);
                            const f32x4 of = *reinterpret_cast<const f32x4 *>(gof + 4u * e);
                            const bool there = row < nvalid && 16 * x + 4 * g < dv;
                            float y[4];
                            y[0] = fmaf(bf16_lo_as_float(rv[0]), of[0], -bf16_lo_as_float(rw[0]) * o[x][0]);
                            y[1] = fmaf(bf16_hi_as_float(rv[0]), of[1], -bf16_hi_as_float(rw[0]) * o[x][1]);
                            y[2] = fmaf(bf16_lo_as_float(rv[1]), of[2], -bf16_lo_as_float(rw[1]) * o[x][2]);
                            y[3] = fmaf(bf16_hi_as_float(rv[1]), of[3], -bf16_hi_as_float(rw[1]) * o[x][3]);
#pragma unroll
                            for (int r = 0; r < 4; ++r) y[r] = there ? y[r] : 0.f;
                            row_scan16x4(y[0], y[1], y[2], y[3]);
                            const f32x4 y4 = f32x4{y[0], y[1], y[2], y[3]};
                            *reinterpret_cast<f32x4 *>(s_lb + row * LBS + 16 * x + 4 * g) = y4;
                            if (lm == 15) *reinterpret_cast<f32x4 *>(s_totb + IT * L::kDvp + 16 * x + 4 * g) = y4;
                        }
                    }
                }
            }
            // state update on this wave's tiles: S^T += V^T K~, then the chunk's decay per channel
#pragma unroll
            for (int q = CT0 < CT1 ? NQ : 0; q < (OWNS ? 2 : 0); ++q) load_k(q);
            float gm[NCT];
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) gm[ct] = s_gam[16 * ct + lm];
#pragma unroll
            for (int i = 0; i < TPW; ++i) {
                const int nt = (NW == 8 && !DV ? (W + 4) % 8 : W) + NW * i;
                if (nt < NDV16) {
                    u32x4 vt[2], vtl[BETA ? 2 : 1];
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const u32x2 v0 = lds_read_tr(vrow + 32 * q * VS + 16 * nt);
                        const u32x2 v1 = lds_read_tr(vrow + (32 * q + 16) * VS + 16 * nt);
                        vt[q] = u32x4{v0[0], v0[1], v1[0], v1[1]};
                        if constexpr (BETA) {
                            const u32x2 l0 = lds_read_tr(vrow_l + 32 * q * VS + 16 * nt);
                            const u32x2 l1 = lds_read_tr(vrow_l + (32 * q + 16) * VS + 16 * nt);
                            vtl[q] = u32x4{l0[0], l0[1], l1[0], l1[1]};
                        }
                    }
                    f32x4 gb = f32x4{1.f, 1.f, 1.f, 1.f};     // BETA: decay of this lane's four value columns
                    if constexpr (BETA) gb = *reinterpret_cast<const f32x4 *>(s_gamb + 16 * nt + 4 * g);
#pragma unroll
                    for (int ct = 0; ct < NCT; ++ct) {
                        f32x4 a = acc[i][ct];
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            a = mfma(vt[q], kth[q][ct], a);
                            a = mfma(vt[q], ktl[q][ct], a);
                            if constexpr (BETA) {
                                a = mfma(vtl[q], kth[q][ct], a);
                                a = mfma(vtl[q], ktl[q][ct], a);
                            }
                        }
#pragma unroll
                        for (int r = 0; r < 4; ++r) a[r] *= BETA ? gm[ct] * gb[r] : gm[ct];
                        acc[i][ct] = a;
                    }
                }
            }
            if constexpr (GS) {
                // U += (decay from the span's first step) * Q~^T dO, transposed like the state
                constexpr int G0 = (W + NW - 1) % NW;
                if constexpr (G0 < NDV16) {
                    const uint16_t *qrow_h = s_qhi + (4 * g + tr_row) * CHS + tr_col;
                    const uint16_t *qrow_l = s_qlo + (4 * g + tr_row) * CHS + tr_col;
                    const uint16_t *wrow = s_w + (4 * g + tr_row) * VS + tr_col;
                    const uint16_t *wrow_l = s_wlo + (4 * g + tr_row) * VS + tr_col;   // BETA
                    u32x4 qth[2][NCT], qtl[2][NCT];
#pragma unroll
                    for (int q = 0; q < 2; ++q)
#pragma unroll
                        for (int ct = 0; ct < NCT; ++ct) {
                            const u32x2 h0 = lds_read_tr(qrow_h + 32 * q * CHS + 16 * ct);
                            const u32x2 h1 = lds_read_tr(qrow_h + (32 * q + 16) * CHS + 16 * ct);
                            const u32x2 l0 = lds_read_tr(qrow_l + 32 * q * CHS + 16 * ct);
                            const u32x2 l1 = lds_read_tr(qrow_l + (32 * q + 16) * CHS + 16 * ct);
                            qth[q][ct] = u32x4{h0[0], h0[1], h1[0], h1[1]};
                            qtl[q][ct] = u32x4{l0[0], l0[1], l1[0], l1[1]};
                        }
                    float fac[NCT];
#pragma unroll
                    for (int ct = 0; ct < NCT; ++ct) {
                        fac[ct] = exp2_fast(decay[ct]);
                        decay[ct] += s_lg[16 * ct + lm];
                    }
#pragma unroll
                    for (int i = 0; i < TPW; ++i) {
                        const int nt = G0 + NW * i;
                        if (nt < NDV16) {
                            u32x4 wt[2], wtl[BETA ? 2 : 1];
#pragma unroll
                            for (int q = 0; q < 2; ++q) {
                                const u32x2 v0 = lds_read_tr(wrow + 32 * q * VS + 16 * nt);
                                const u32x2 v1 = lds_read_tr(wrow + (32 * q + 16) * VS + 16 * nt);
                                wt[q] = u32x4{v0[0], v0[1], v1[0], v1[1]};
                                if constexpr (BETA) {
                                    const u32x2 l0 = lds_read_tr(wrow_l + 32 * q * VS + 16 * nt);
                                    const u32x2 l1 = lds_read_tr(wrow_l + (32 * q + 16) * VS + 16 * nt);
                                    wtl[q] = u32x4{l0[0], l0[1], l1[0], l1[1]};
                                }
                            }
                            f32x4 fb = f32x4{1.f, 1.f, 1.f, 1.f};
                            if constexpr (BETA) {
                                const f32x4 lb4 = *reinterpret_cast<const f32x4 *>(s_lgb + 16 * nt + 4 * g);
#pragma unroll
                                for (int r = 0; r < 4; ++r) fb[r] = exp2_fast(decay_b[i][r]);
                                decay_b[i] += lb4;
                            }
#pragma unroll
                            for (int ct = 0; ct < NCT; ++ct) {
                                f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                                for (int q = 0; q < 2; ++q) {
                                    a = mfma(wt[q], qth[q][ct], a);
                                    a = mfma(wt[q], qtl[q][ct], a);
                                    if constexpr (BETA) {
                                        a = mfma(wtl[q], qth[q][ct], a);
                                        a = mfma(wtl[q], qtl[q][ct], a);
                                    }
                                }
                                f32x4 u = accg[i][ct];
#pragma unroll
                                for (int r = 0; r < 4; ++r) u[r] = fmaf(BETA ? fac[ct] * fb[r] : fac[ct], a[r], u[r]);
                                accg[i][ct] = u;
                            }
                        }
                    }
                } else {
#pragma unroll
                    for (int ct = 0; ct < NCT; ++ct) decay[ct] += s_lg[16 * ct + lm];
                }
            }
            if constexpr (DV) {
                if (p.dlog_alpha != nullptr) {
                    // Sums over all later scan steps: the wave's own rows + the waves before it + everything before
                    // this chunk; the last wave leaves the total for the next chunk.  The barrier stands behind the state
                    // update, so that the waves with fewer causal tiles, which own the odd state tiles, have no less to
                    // do before it; and since only registers and the sums are read after it, it is also the one that
                    // lets the next chunk's rows into LDS.
                    constexpr int NA = READ ? NCT : 0, NB = BETA && OUTPUTS ? NDV16 : 0;
                    f32x4 xs[NA > 0 ? NA : 1], ys[NB > 0 ? NB : 1];
#pragma unroll
                    for (int x = 0; x < NA; ++x) xs[x] = *reinterpret_cast<const f32x4 *>(s_la + row * LAS + min(16 * x + 4 * g, L::kDkp - 4));
#pragma unroll
                    for (int x = 0; x < NB; ++x) ys[x] = *reinterpret_cast<const f32x4 *>(s_lb + row * LBS + 16 * x + 4 * g);
                    const uint32_t my_tok = (uint32_t)tok[row];
                    __syncthreads();
                    auto finish = [&](auto pitch_c, const f32x4 &sum, int x, const float *tot, float *later, char *dst, int stride, int width) {
                        constexpr int P = decltype(pitch_c)::value;
                        const int c = 16 * x + 4 * g;
                        if (c < width) {
                            f32x4 add = *reinterpret_cast<const f32x4 *>(later + (chunk & 1) * P + c);
#pragma unroll
                            for (int u = 0; u < IT; ++u) add += *reinterpret_cast<const f32x4 *>(tot + u * P + c);
                            if (row < nvalid)
                                *reinterpret_cast<f32x4 *>(dst + (my_tok * (uint32_t)stride + (uint32_t)c) * 4u) = sum + add;
                            if (IT == 3 && lm == 0)
                                *reinterpret_cast<f32x4 *>(later + ((chunk + 1) & 1) * P + c) =
                                    add + *reinterpret_cast<const f32x4 *>(tot + IT * P + c);
                        }
                    };
#pragma unroll
                    for (int x = 0; x < NA; ++x) finish(int_c<L::kDkp>{}, xs[x], x, s_tot, s_later, gdla, p.st_k, dk);
#pragma unroll
                    for (int x = 0; x < NB; ++x) finish(int_c<L::kDvp>{}, ys[x], x, s_totb, s_laterb, gdlb, p.st_v, dv);
                }
            }
        };
        switch (w) {
        case 0: contract(int_c<0>{}); break;
        case 1: contract(int_c<1>{}); break;
        case 2: contract(int_c<2>{}); break;
        case 3: contract(int_c<3>{}); break;
        case 4: if constexpr (NW > 4) contract(int_c<4>{}); break;
        case 5: if constexpr (NW > 4) contract(int_c<5>{}); break;
        case 6: if constexpr (NW > 4) contract(int_c<6>{}); break;
        default: if constexpr (NW > 4) contract(int_c<7>{}); break;
        }
        if constexpr (!DV) {
            const int done = s_begin + (chunk + 1) * kChunk;       // scan steps walked: a bound of the reversed walk's spans?
            if (p.ws_bound != nullptr && done < T && done % p.bound_len == 0) {
                float *dst = p.ws_bound + ((size_t)bh * p.bounds + done / p.bound_len - 1) * (size_t)(dk * dv);
#pragma unroll
                for (int i = 0; i < TPW; ++i) {
                    const int n = 16 * state_tile(w, i) + 4 * g;
#pragma unroll
                    for (int ct = 0; ct < NCT; ++ct) {
                        const int c = 16 * ct + lm;
                        if (c < dk && n < dv) *reinterpret_cast<f32x4 *>(dst + c * dv + n) = acc[i][ct];
                    }
                }
            }
        }
        if (!(DV && p.dlog_alpha != nullptr)) __syncthreads();
    }

    if constexpr (GS) {
        // U of the reversed walk's span, and the log of its decay: the gates of the steps a + 1 .. b (with gate_shift the
        // walk's first step decays by the gate of step b, the first one after this span)
        const size_t span = (size_t)bh * p.nspans + (p.nspans - 1 - sp);
        const int tok_after = scan_token(p.scan_dir, min(s_end, T - 1), T, p.grid_h, p.grid_w);
        float *u = p.ws_gstate + span * (size_t)(dk * dv);
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            const int n = 16 * gstate_tile(w, i) + 4 * g;
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) {
                const int c = 16 * ct + lm;
                if (c < dk && n < dv) *reinterpret_cast<f32x4 *>(u + c * dv + n) = accg[i][ct];
            }
            if constexpr (BETA) {
                if (lm == 0 && n < dv) {
                    const f32x4 x = *reinterpret_cast<const f32x4 *>(reinterpret_cast<const float *>(glb) + (size_t)tok_after * p.st_v + n);
                    *reinterpret_cast<f32x4 *>(p.ws_glgam_b + span * dv + n) = decay_b[i] * kLn2 + x;
                }
            }
        }
        if (w == 0 && g == 0) {
            const float *la = reinterpret_cast<const float *>(gla_) + (size_t)tok_after * p.st_k;
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct)
                if (16 * ct + lm < dk) p.ws_glgam[span * dk + 16 * ct + lm] = decay[ct] * kLn2 + la[16 * ct + lm];
        }
    }
}

template <int NDK8, int NDV16, int NW, int MINW, bool DV, bool BETA, bool GS, bool FOUR = false>
hipError_t launch_waves(const WalkParams &p, const void *w, float *r, hipStream_t stream) {
    using L = RLayout<NDK8, NDV16, DV, BETA, GS>;
    auto kernel = mfma_row_read_kernel<NDK8, NDV16, NW, MINW, DV, BETA, GS, FOUR>;
    static std::atomic<bool> configured[kMaxDevices] = {};  // per instantiation and device
    {
        hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), L::kBytes, configured);
        if (e != hipSuccess) return e;
    }
    return launch_in_parts(p, p.nspans, NW * 64, [&](const WalkParams &part, int b, int h) {
        dim3 grid((unsigned)(part.B * part.H * p.nspans)), block(NW * 64);
        const void *wp = static_cast<const char *>(w) + 2 * ((size_t)b * p.sb_v + (size_t)h * p.sh_v);
        hipLaunchKernelGGL(kernel, grid, block, L::kBytes, stream, part, wp, r + (size_t)b * p.sb_k + (size_t)h * p.sh_k);
        return hipGetLastError();
    });
}

template <int NDK8, int NDV16, bool DV, bool BETA, bool GS>
hipError_t launch_one(const WalkParams &p, const void *w, float *r, hipStream_t stream) {
    // 8 waves where a compute unit holds one group anyway: by its LDS, or because there are no more groups than units
    constexpr int kGroupsPerCu = (160 * 1024) / RLayout<NDK8, NDV16, DV, BETA, GS>::kBytes;
    if constexpr (kGroupsPerCu >= 2) {
        if ((long long)p.B * p.H * p.nspans > 256) return launch_waves<NDK8, NDV16, 4, 2, DV, BETA, GS>(p, w, r, stream);
    }
    return launch_waves<NDK8, NDV16, 8, 2, DV, BETA, GS>(p, w, r, stream);
}

template <bool DV, bool GS>
hipError_t launch_sizes(const WalkParams &p, const void *w, float *r, hipStream_t stream) {
    const int ndk8 = (p.dk + 7) / 8, ndv16 = (p.dv + 15) / 16;
    if (p.log_beta != nullptr) {   // two-sided gate: the head sizes whose extra rows fit the LDS (dk <= 40, dv <= 80)
        if (ndk8 <= 4 && ndv16 <= 4) return launch_one<4, 4, DV, true, GS>(p, w, r, stream);
        if (ndk8 <= 5 && ndv16 <= 5) return launch_one<5, 5, DV, true, GS>(p, w, r, stream);
        return hipErrorInvalidConfiguration;
    }
    if (ndk8 <= 4 && ndv16 <= 4) return launch_one<4, 4, DV, false, GS>(p, w, r, stream);
    if (ndk8 <= 5 && ndv16 <= 5) return launch_one<5, 5, DV, false, GS>(p, w, r, stream);
    return launch_one<8, 8, DV, false, GS>(p, w, r, stream);
}

}  // namespace

static hipError_t launch_four(const WalkParams &p, const void *w, float *r, hipStream_t stream, bool with_outputs);

// Same conditions as the forward MFMA engine (bf16 rows, dk % 4 == 0, dv % 8 == 0, 32-bit offsets).
// with_outputs: also write o_j = q_j S_j (p.q, fp32 rows to p.out).
hipError_t launch_mfma_row_read(const WalkParams &p, const void *w, float *r, hipStream_t stream, bool with_outputs) {
    // The kernels with the rows in registers take a compute unit per group: where there are more groups (a forward call's plan
    // adopted by gla_bwd_reuse, more than 256 sequences) those above, two groups a unit, are as fast or faster (16 x 256 chunks
    // at 36 / 72 channels in 512 spans 162 and 167 us a call, in 256 spans 178 and 155).  They also pay for a longer prologue
    // (both kinds of waves read the gates of three chunks) and for loads that touch 16 rows each, which tells where these are
    // those of [B,T,H,d].  Short spans therefore stay with those above.  Difference of a backward call over 64 to 256 groups,
    // the means of eleven numbers of sequences and spans (+: faster with the rows in registers), by chunks a span:
    //     walk for dq      [B,H,T,d] row scans 1: +0.9 %, 2: +3.1, 3: +4.0; column scans +0.6, +2.0, +2.4
    //                      [B,T,H,d] 2: -0.3 %, 3: 0.0, 4: +0.7, 6: +1.9, 12: +4.3
    //     walk for dk, dv  [B,H,T,d] row scans 1: -0.7 %, 2: +0.2, 3: +1.9; column scans 2: -0.8, 3: +0.3, 4: +2.0 (grids 64
    //                      tokens wide 3: -1.0, 4: -0.2, 12: +1.1)
    //                      [B,T,H,d] 1: -4.3 %, 2: -3.9, 4: -1.8, 8: -0.2, 10: +0.2, 16: +1.2
    // and of [B,H,T,d] by spans: one chunk in the walk for dq +0.2 to +5 % with 4 to 9 spans (grids 64 tokens wide, column scans
    // -0.8 to +0.2), -0.7 to -2.4 with two, -2.5 to -4 with 15 that hardly decay; row scans of two chunks in the walk for dk, dv
    // +1.3 to +2.8 % from four spans on, -0.4 to -3.8 with one or two.
    const bool heads_inside = p.st_k != p.dk;
    const int chunks = p.span_len / kChunk;
    int least;
    if (heads_inside) least = with_outputs ? 10 : 4;
    else if (!with_outputs) least = p.nspans > 2 && p.nspans <= 10 ? 1 : 2;
    else least = p.scan_dir >= GLA_SCAN_COL_FWD ? 4 : (p.nspans > 2 ? 2 : 3);
    if (hilo_kernels_cover(p) && (long long)p.B * p.H * p.nspans <= 256)
        return chunks >= least ? launch_hilo_walk(p, w, r, stream, with_outputs) : launch_four(p, w, r, stream, with_outputs);
    if (with_outputs) return launch_sizes<true, false>(p, w, r, stream);
    return p.ws_gstate != nullptr ? launch_sizes<false, true>(p, w, r, stream) : launch_sizes<false, false>(p, w, r, stream);
}

// Short spans of the heads of 33 to 36 channels.  (Last in this file, so that the other kernels stay where they are in the code
// object: a two-sided training step of 64 sequences of 16 chunks takes 143.2 us then, 143.6 with these in between.)
static hipError_t launch_four(const WalkParams &p, const void *w, float *r, hipStream_t stream, bool with_outputs) {
    if (with_outputs) return launch_waves<5, 5, 8, 2, true, false, false, true>(p, w, r, stream);
    return p.ws_gstate != nullptr ? launch_waves<5, 5, 8, 2, false, false, true, true>(p, w, r, stream)
                                  : launch_waves<5, 5, 8, 2, false, false, false, true>(p, w, r, stream);
}

}  // namespace gla
