// bf16 hi/lo MFMA kernel for the walks of the backward pass of the GLA recurrence, rows held in registers
// (DiG paper, Sec. 3.1 Eq. (attn_gla) rows 1-3, differentiated; chunks of M = 64 tokens computed on-chip as in Sec. 3.5;
// up to 36 key channels and 80 value columns).
//
// It computes r_s[c] = sum_n S_s[c,n] w_s[n] for every scan step s of a span, where S follows
// S_s = diag(alpha_s) S_{s-1} + k_s^T v_s: with w = dO this is dq, and on the reversed recurrence of G = dL/dS
// (k, v := q, dO, gates shifted by one step) with w = v it is dk.
//
// Chunk form around a mid-chunk anchor (gla_hilo.hip).  With b the inclusive sums of log2 alpha inside the chunk (per
// channel), m its 32nd token, E_j = 2^(b_j - b_m) and S_0 the state entering the chunk,
//     k~_i = k_i / E_i,  q~_j = q_j E_j,  P = diag(2^b_m) S_0
//     r_j = E_j * ( sum_{i<=j} (w_j . v_i) k~_i + P w_j ),     S_C = diag(2^(b_C - b_m)) (P + K~^T V)
// DV: also o_j = q_j S_j = sum_{i<=j} (q~_j . k~_i) v_i + q~_j P (fp32 rows to p.out): the reversed walk needs both, dk as
// the row read against v and dv = k G as the output with q := k; and the gate gradient (see gla_mfma_bwd.hip).
// GS: also the local states of the reversed recurrence over the span, U = sum_s (decay from the span's first step to s) *
// q_s^T dO_s, chunk by chunk (decay to the chunk's anchor times Q~^T dO), so that G needs no state pass of its own.
// q~, k~, P and the scores are bf16 hi/lo pairs, of whose products all four are taken.
//
// Two waves share tokens 16 w .. 16 w + 15 of every chunk: w of the four readers (k~, the row read, the gate gradient) and w
// of the four others (v, q~, the outputs or U, most of the state tiles), so that each has the registers for its rows and a
// SIMD has two chains of dependent instructions to issue from; one group a compute unit, one barrier a chunk (operands of
// two chunks in LDS).  Lane (lm, g) of either holds, for token 16 w + lm, channels 16 u + 4 g .. + 3 of the units u = 0, 1,
// the tail channel 32 + g (dk > 32), and columns 16 x + 4 g .. + 3 of the column tiles x: this is at once the layout of the
// MFMA operands (slot (g, e) of a 32-wide step is 16 (e / 4) + 4 g + e % 4; LDS rows are in plain order and read in two
// 8-byte pieces) and that of the result rows, so that E, the rows of the gate gradient, q~ and w never leave the wave's
// registers.  A tail channel's four hi/lo products share an MFMA as in gla_hilo.hip.  The state is kept transposed,
// S^T[n][c]: a lane holds four columns of one channel, which is a 16-byte piece of the [dk][dv] states in memory and an
// 8-byte piece of the channel-major rows of P in LDS; the contraction over columns reads these rows plainly, that over
// channels with the transposing read.
//
// MI355X, 16 sequences of 16384 steps at 36 / 72 channels, against the walks with rows staged through LDS (two 4-wave groups
// a compute unit): dk, dv and gate gradient 85 -> 76 us (340 MB, 63 us at the copy rate; 8500 clocks a chunk, of which
// the vector unit is busy 57 % and the LDS 35 %), dq 58 -> 59 us, whole call (with the state pass of gla_hilo.hip) 166.5 ->
// 154.9 us; errors of dq, dk, dv against 64 bits 4.3e-6 -> 3.5e-6 (all four products), of dlog_alpha 2.7e-5 at twice the
// steps a span.  Tried: 4 waves that do everything, two groups a compute unit (256 registers spill: 84 us, dq 55.5).
#include <type_traits>

#include "gla_common.h"
#include "gla_mfma_util.h"

namespace gla {
namespace {

template <int N>
using int_c = std::integral_constant<int, N>;

#define HILO_WAVE_END(W) asm volatile("; end of the code of wave %0" ::"n"(W))

// groups of four tail channels, tiles of 16 value columns (gla_hilo.hip)
constexpr int DT = 1, NDV16 = 5;

template <bool DV, bool GS>
struct WLayout {
    static constexpr int NV = 8 + DT, NX = NDV16;
    static constexpr int kTS = 12;                            // floats per (tile, g) of the key-side totals
    static constexpr int kRow = 80;       // bf16 per row of k~, q~: 32 hi, 32 lo, 16 of the tail (swz: see gla_hilo.hip)
    static constexpr int kVRow = 80;      // ... of v, w, P
    static constexpr int kK = kChunk * kRow * 2, kV = kChunk * kVRow * 2;
    static constexpr int kP = (64 + 16 * DT) * kVRow * 2;     // rows of P: 32 channels hi, lo, 16 of the tail
    static constexpr int oTot = 0;                                        // float[3][tile][g][kTS]: gates
    static constexpr int oX = oTot + 3 * 16 * kTS * 4;             // float[2][tile][g][kTS]: gate gradient
    static constexpr int oDump = oX + (DV ? 2 * 16 * kTS * 4 : 0);   // where the lanes without a total write theirs
    static constexpr int oSet = oDump + 4 * kTS * 4;
    // operands of a chunk
    static constexpr int oK = oSet, oV = oK + kK, oP = oV + kV;
    static constexpr int oQ = oP + kP, oW = oQ + (GS ? kK : 0);
    static constexpr int kSet = oW + (GS ? kV : 0) - oSet;
    static constexpr int kBytes = oSet + 2 * kSet;      // operands of two chunks: one barrier a chunk
    static_assert(kSet >= (32 + 4 * DT) * 16 * NDV16 * 4 + 8 * 40 * 4, "start state and the sums of the prologue fit");
    static_assert(oSet % 16 == 0 && kSet % 16 == 0 && kBytes <= 160 * 1024, "16-byte accesses, one compute unit");
};

// State tiles (tile t = channel tile t % NCT of column tile t / NCT) of a wave: the readers own the few that even the two
// kinds of waves out.
template <bool DV, bool GS>
struct WOwned {
    static constexpr int NCT = 2 + DT, kTiles = NCT * NDV16;
    static constexpr int kCount[8] = {DV ? 2 : 1, 1, 1, DV || GS ? 1 : 0, 3, 3, DV ? 2 : 3, DV || GS ? 2 : 3};
    __host__ __device__ static constexpr int count(int w) { return kCount[w]; }
    __host__ __device__ static constexpr int start(int w) {
        int n = 0;
        for (int i = 0; i < w; ++i) n += kCount[i];
        return n;
    }
    static_assert(start(8) == kTiles, "every tile has an owner");
    static constexpr int kMost = 3;
};

// A copy that stays one: where it were merged with its source, a register that is being loaded, the next load would go
// elsewhere and be copied into place at the loop's end, i.e. waited for.
__device__ inline uint32_t kept(uint32_t x) {
    uint32_t y;
    asm volatile("v_mov_b32 %0, %1" : "=v"(y) : "v"(x));
    return y;
}
__device__ inline u32x2 kept(u32x2 x) { return u32x2{kept(x[0]), kept(x[1])}; }

__device__ inline f32x4 exp2_4(f32x4 x) { return f32x4{exp2_fast(x[0]), exp2_fast(x[1]), exp2_fast(x[2]), exp2_fast(x[3])}; }
__device__ inline f32x4 scan16_4(f32x4 x) {      // prefix sums over the 16 lanes of a DPP row
    float a = x[0], b = x[1], c = x[2], d = x[3];
    row_scan16x4(a, b, c, d);
    return f32x4{a, b, c, d};
}
// x + the value two lanes further in the quad (hi and lo share of a tail channel)
__device__ inline float quad_add2(float x) { return x + dpp_move<0x4E, 0xF, true>(x); }

template <bool DV, bool GS>
__global__ __launch_bounds__(512, 2) void hilo_walk_kernel(WalkParams p, const void *w_in, float *r_out) {
    using L = WLayout<DV, GS>;
    using OW = WOwned<DV, GS>;
    static_assert(!(DV && GS), "either walk");
    constexpr int NCT = 2 + DT, RS = L::kRow, VS = L::kVRow, TS = L::kTS, NX = NDV16;
    constexpr int KSV = (NX + 1) / 2;                 // 32-column steps
    constexpr int SET = L::kSet / 2;                  // 16-bit elements from an operand to its twin in the other set

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    float *s_tot = reinterpret_cast<float *>(smem + L::oTot), *s_x = reinterpret_cast<float *>(smem + L::oX);
    uint16_t *s_k = reinterpret_cast<uint16_t *>(smem + L::oK), *s_v = reinterpret_cast<uint16_t *>(smem + L::oV);
    uint16_t *s_p = reinterpret_cast<uint16_t *>(smem + L::oP);
    uint16_t *s_q = reinterpret_cast<uint16_t *>(smem + L::oQ), *s_w = reinterpret_cast<uint16_t *>(smem + L::oW);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w8 = __builtin_amdgcn_readfirstlane(tid >> 6), w = w8 & 3;     // 0..3 readers, 4..7 the others; 16-token tile
    int lm = lane & 15, g = lane >> 4;
    int swz = 8 * (lm >> 3);                  // of the rows 16 i + lm

    int blk = blockIdx.x;    // contiguous ranges of spans per XCD
    {
        const int nb = gridDim.x;
        if ((nb & 7) == 0) blk = (blk & 7) * (nb >> 3) + (blk >> 3);
    }
    const int bh = blk / p.nspans;
    int sp_ = blk - bh * p.nspans;
    if (p.chain_in_output && (bh & 1)) sp_ = p.nspans - 1 - sp_;   // (long and short chains share a compute unit)
    const int sp = sp_;
    const int dk = p.dk, dv = p.dv, T = p.T;
    const int s_begin = span_begin(p, sp), s_end = span_end(p, sp);
    const int nch = (s_end - s_begin + kChunk - 1) / kChunk;
    const bool with_gates = DV && p.dlog_alpha != nullptr;          // uniform

    const size_t base_k = slab_k(p, bh), base_v = slab_v(p, bh);
    const uint32_t dk2 = 2u * (uint32_t)p.st_k, dv2 = 2u * (uint32_t)p.st_v;   // bytes from one bf16 row to the next
    const uint32_t bytes_k = (uint32_t)(T - 1) * dk2 + 2u * (uint32_t)dk, bytes_v = (uint32_t)(T - 1) * dv2 + 2u * (uint32_t)dv;
    const Rsrc bk = view(static_cast<const char *>(p.k) + base_k * 2, bytes_k), bq = view(static_cast<const char *>(p.q) + base_k * 2, bytes_k);
    const Rsrc bv = view(static_cast<const char *>(p.v) + base_v * 2, bytes_v), bw = view(static_cast<const char *>(w_in) + base_v * 2, bytes_v);
    const Rsrc bg = view(p.log_alpha + base_k, 2u * bytes_k), br = view(r_out + base_k, 2u * bytes_k);
    const Rsrc bo = view(static_cast<float *>(p.out) + base_v, 2u * bytes_v);
    const Rsrc bdq = view(p.fwd_dq + base_k, 2u * bytes_k), bda = view(p.dlog_alpha + base_k, 2u * bytes_k);

    // ---- token of this lane's row as the wave moves from chunk to chunk (see gla_hilo.hip), and of the step before it,
    // whose gate the row uses with gate_shift ----
    const int row_s0 = s_begin + 16 * w + lm;
    const int col_len = p.scan_dir >= 2 ? p.grid_h : 1, dir = (p.scan_dir & 1) ? -1 : 1;   // (uniform)
    const int col_dq = dir * (kChunk / col_len), col_dr = dir * (kChunk % col_len);
    struct Walker {
        int tok, c, r;
    };
    auto walker_at = [&](int step) {
        const int s = (p.scan_dir & 1) ? T - 1 - min(step, T - 1) : min(step, T - 1);
        Walker x;
        x.c = s / col_len;
        x.r = s - x.c * col_len;
        x.tok = x.r * p.grid_w + x.c;
        return x;
    };
    auto advance = [&](Walker &x) {
        x.c += col_dq;
        x.r += col_dr;
        const bool over = x.r >= col_len, under = x.r < 0;
        x.r += under ? col_len : (over ? -col_len : 0);
        x.c += under ? -1 : (over ? 1 : 0);
        x.tok = x.r * p.grid_w + x.c;
    };
    int walk_s = row_s0;
    Walker row = walker_at(row_s0), grow = walker_at(row_s0);
    auto next_row = [&]() {
        walk_s += kChunk;
        advance(row);
        if constexpr (DV || !GS) advance(grow);
    };
    // (the very first step has no step before it: its own gate, which multiplies a zero state.  Its walker starts one step
    // back, i.e. at the walker of the first step of the chunk, only where there is one.)
    bool first_row = false;
    if constexpr (DV || !GS) {
        if (p.gate_shift) {
            first_row = row_s0 == 0;
            // one step back along the scan
            grow = row;
            const bool fwd = dir > 0;
            if (fwd) {
                const bool wrap = grow.r == 0;
                grow.c -= (col_len == 1 || wrap) ? 1 : 0;
                grow.r = wrap ? col_len - 1 : grow.r - 1;
            } else {
                const bool wrap = grow.r == col_len - 1;
                grow.c += wrap ? 1 : 0;
                grow.r = wrap ? 0 : grow.r + 1;
            }
            grow.tok = grow.r * p.grid_w + grow.c;
        }
    }

    // Everything from here on exists once per kind of wave.
    auto walk = [&](auto reads) {
        constexpr bool READ = decltype(reads)::value;
        constexpr bool Q = READ ? DV : DV || GS;              // rows of q: raw for the gate gradient; gated
        // ---- rows in registers ----
        uint32_t chb[2], tcb[DT], vcb[NX];       // byte offsets of the lane's units in a bf16 row, or nowhere
#pragma unroll
        for (int u = 0; u < 2; ++u) chb[u] = 16 * u + 4 * g < dk ? 2u * (uint32_t)(16 * u + 4 * g) : kNowhere / 2;
#pragma unroll
        for (int e = 0; e < DT; ++e) tcb[e] = 32 + 4 * e + g < dk ? 2u * (uint32_t)(32 + 4 * e + g) : kNowhere / 2;
#pragma unroll
        for (int x = 0; x < NX; ++x) vcb[x] = 16 * x + 4 * g < dv ? 2u * (uint32_t)(16 * x + 4 * g) : kNowhere / 2;
        struct FRow {           // a row of the key side in fp32
            f32x4 u[2];
            float t[DT];
        };
        struct HRow {           // ... in bf16
            u32x2 u[2];
            uint32_t t[DT];
        };
        auto fetch_f = [&](Rsrc b, uint32_t at) {
            FRow x;
#pragma unroll
            for (int u = 0; u < 2; ++u) x.u[u] = fetch<f32x4>(b, f32_at(at, chb[u]));
#pragma unroll
            for (int e = 0; e < DT; ++e) x.t[e] = fetch<float>(b, f32_at(at, tcb[e]));
            return x;
        };
        auto fetch_h = [&](Rsrc b, uint32_t at) {
            HRow x;
#pragma unroll
            for (int u = 0; u < 2; ++u) x.u[u] = fetch<u32x2>(b, at + chb[u]);
#pragma unroll
            for (int e = 0; e < DT; ++e) x.t[e] = fetch<uint16_t>(b, at + tcb[e]);
            return x;
        };
        auto put_f = [&](Rsrc b, uint32_t at, const FRow &x) {
#pragma unroll
            for (int u = 0; u < 2; ++u) put(b, f32_at(at, chb[u]), x.u[u]);
#pragma unroll
            for (int e = 0; e < DT; ++e)
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x.t[e]), b, (int)f32_at(at, tcb[e]), 0, 0);
        };
        auto at_k = [&](int step, int tk) { return step < s_end ? (uint32_t)tk * dk2 : kNowhere / 2; };
        auto at_v = [&](int step, int tk) { return step < s_end ? (uint32_t)tk * dv2 : kNowhere / 2; };
        FRow r_la, r_dq;
        HRow r_q, r_k;
        u32x2 r_v[NX], r_w[NX];
        FRow r_b;                            // scanned gates (log2, prefix inside the 16-token tile) of the chunk gated next

        auto issue_gates = [&]() {           // the rows at the walkers
            const int tk = p.gate_shift && !(first_row && walk_s == 0) ? grow.tok : row.tok;
            r_la = fetch_f(bg, at_k(walk_s, tk));
        };
        auto issue_rows = [&](int step, int tk) {
            const uint32_t at = at_k(step, tk), atv = at_v(step, tk);
            if constexpr (READ) r_k = fetch_h(bk, at);
            if constexpr (Q) r_q = fetch_h(bq, at);
#pragma unroll
            for (int x = 0; x < NX; ++x) {
                if constexpr (!READ) r_v[x] = fetch<u32x2>(bv, atv + vcb[x]);
                if constexpr (READ) r_w[x] = fetch<u32x2>(bw, atv + vcb[x]);
            }
        };
        auto issue_grad = [&](int step, int tk) {     // rows of the gate gradients
            if constexpr (DV) {
                if constexpr (READ) r_dq = fetch_f(bdq, with_gates ? at_k(step, tk) : kNowhere / 2);
            }
        };

        auto ring = [](int x) { return x % 3; };
        auto scan_rows = [&](FRow &b) {
            b.u[0] = scan16_4(b.u[0]);
            b.u[1] = scan16_4(b.u[1]);
#pragma unroll
            for (int e = 0; e < DT; ++e) b.t[e] = row_scan16(b.t[e]);
        };
        // the last lane of every row of 16 holds the tile's total (written without a branch: the others write elsewhere)
        float *s_dump = reinterpret_cast<float *>(smem + L::oDump);
        auto put_tot = [&](float *tot, const FRow &b) {    // [g][kTS]
            tot = lm == 15 ? tot : s_dump;
            *reinterpret_cast<f32x4 *>(tot + g * TS) = b.u[0];
            *reinterpret_cast<f32x4 *>(tot + g * TS + 4) = b.u[1];
#pragma unroll
            for (int e = 0; e < DT; ++e) tot[g * TS + 8 + e] = b.t[e];
        };
        auto get_tot = [&](const float *tot) {
            FRow b;
            b.u[0] = *reinterpret_cast<const f32x4 *>(tot + g * TS);
            b.u[1] = *reinterpret_cast<const f32x4 *>(tot + g * TS + 4);
#pragma unroll
            for (int e = 0; e < DT; ++e) b.t[e] = tot[g * TS + 8 + e];
            return b;
        };
        auto add_row = [](const FRow &a, const FRow &b) {
            FRow c;
            c.u[0] = a.u[0] + b.u[0];
            c.u[1] = a.u[1] + b.u[1];
#pragma unroll
            for (int e = 0; e < DT; ++e) c.t[e] = a.t[e] + b.t[e];
            return c;
        };
        // prefix sums of the gates of chunk x inside this wave's tile; tile totals to LDS
        auto scan = [&](int x, FRow &b) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                float l[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) l[i] = r_la.u[u][i] * kLog2e;
                row_scan16x4_least(l[0], l[1], l[2], l[3], kLeastGate2);
                b.u[u] = f32x4{l[0], l[1], l[2], l[3]};
            }
#pragma unroll
            for (int e = 0; e < DT; ++e) b.t[e] = row_scan16(fmaxf(r_la.t[e] * kLog2e, kLeastGate2));
            if constexpr (READ) put_tot(s_tot + (ring(x) * 4 + w) * 4 * TS, b);
        };

        // operands of the wave's own tokens: E (and F), q~ (DV) and w~
        struct Own {
            FRow e;
            u32x4 qh, ql, qt;
            u32x4 wh[KSV];
            HRow raw_q, raw_k;
        };
        Own own;
        // gate chunk x: what its own tokens need to registers; k~, v~ (GS: q~, w~) to LDS
        auto gate = [&](auto wave_c, int x, Own &n) {
            constexpr int W = decltype(wave_c)::value & 3;
            // exponents relative to the anchor: tiles 0, 1 lie before it (-(t0 + t1), -t1), tile 2 starts at it, tile 3 follows (+t2)
            auto offset = [&](f32x4 b, const float *tot, int stride) {
                if constexpr (W == 0) b -= *reinterpret_cast<const f32x4 *>(tot) + *reinterpret_cast<const f32x4 *>(tot + stride);
                if constexpr (W == 1) b -= *reinterpret_cast<const f32x4 *>(tot + stride);
                if constexpr (W == 3) b += *reinterpret_cast<const f32x4 *>(tot + 2 * stride);
                return b;
            };
            auto offset1 = [&](float b, const float *tot, int stride) {
                if constexpr (W == 0) b -= tot[0] + tot[stride];
                if constexpr (W == 1) b -= tot[stride];
                if constexpr (W == 3) b += tot[2 * stride];
                return b;
            };
            // (clamped so that gates beyond the range leave nothing infinite)
            auto up = [](float ex) { return exp2_fast(W < 2 ? fminf(ex, kMaxExp2) : ex); };          // towards the row
            auto down = [](float ex) { return exp2_fast(W < 2 ? -ex : fminf(-ex, kMaxExp2)); };      // away from it
            const float *tot = s_tot + ring(x) * 16 * TS + g * TS;
            uint16_t *krow = s_k + (x & 1) * SET + (16 * W + lm) * RS, *qrow = s_q + (x & 1) * SET + (16 * W + lm) * RS;
            const int vat = (x & 1) * SET + (16 * W + lm) * VS + (4 * g ^ swz);
            if constexpr (READ || DV || GS) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const f32x4 ex = offset(r_b.u[u], tot + 4 * u, 4 * TS);
#pragma unroll
                    for (int i = 0; i < 4; ++i) n.e.u[u][i] = up(ex[i]);
                    if constexpr (READ) {
                        u32x2 kh, kl;
#pragma unroll
                        for (int h = 0; h < 2; ++h)
                            SPLIT_PAIR(bf16_lo_as_float(r_k.u[u][h]) * down(ex[2 * h]), bf16_hi_as_float(r_k.u[u][h]) * down(ex[2 * h + 1]),
                                       kh[h], kl[h]);
                        *reinterpret_cast<u32x2 *>(krow + 16 * u + (4 * g ^ swz)) = kh;
                        *reinterpret_cast<u32x2 *>(krow + 32 + 16 * u + (4 * g ^ swz)) = kl;
                    } else {
#pragma unroll
                        for (int h = 0; h < 2; ++h)
                            SPLIT_PAIR(bf16_lo_as_float(r_q.u[u][h]) * n.e.u[u][2 * h], bf16_hi_as_float(r_q.u[u][h]) * n.e.u[u][2 * h + 1],
                                       n.qh[2 * u + h], n.ql[2 * u + h]);
                        if constexpr (GS) {
                            *reinterpret_cast<u32x2 *>(qrow + 16 * u + (4 * g ^ swz)) = u32x2{n.qh[2 * u], n.qh[2 * u + 1]};
                            *reinterpret_cast<u32x2 *>(qrow + 32 + 16 * u + (4 * g ^ swz)) = u32x2{n.ql[2 * u], n.ql[2 * u + 1]};
                        }
                    }
                }
                n.qt = u32x4{0, 0, 0, 0};
#pragma unroll
                for (int e = 0; e < DT; ++e) {
                    const float ex = offset1(r_b.t[e], tot + 8 + e, 4 * TS);
                    n.e.t[e] = up(ex);
                    const float y = READ ? bf16_lo_as_float(r_k.t[e]) * down(ex) : bf16_lo_as_float(r_q.t[e]) * n.e.t[e];
                    const uint32_t hi = pack_bf16(y, y);
                    const float rem = y - bf16_lo_as_float(hi);
                    const uint32_t lo = pack_bf16(rem, rem);
                    if constexpr (READ || GS) *reinterpret_cast<u32x2 *>((READ ? krow : qrow) + 64 + 16 * e + (4 * g ^ swz)) = u32x2{hi, lo};
                    else n.qt[2 * e] = n.qt[2 * e + 1] = (hi & 0xffffu) | (lo << 16);
                }
            }
            if constexpr (READ) {
                if constexpr (NX % 2) n.wh[KSV - 1] = u32x4{0, 0, 0, 0};
#pragma unroll
                for (int i = 0; i < NX; ++i) {
                    if constexpr (GS) *reinterpret_cast<u32x2 *>(s_w + vat + 16 * i) = r_w[i];
                    n.wh[i / 2][2 * (i & 1)] = kept(r_w[i][0]);
                    n.wh[i / 2][2 * (i & 1) + 1] = kept(r_w[i][1]);
                }
            } else {
#pragma unroll
                for (int i = 0; i < NX; ++i) *reinterpret_cast<u32x2 *>(s_v + vat + 16 * i) = r_v[i];
            }
            if constexpr (READ && DV) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    n.raw_k.u[u] = kept(r_k.u[u]);
                    n.raw_q.u[u] = kept(r_q.u[u]);
                }
#pragma unroll
                for (int e = 0; e < DT; ++e) {
                    n.raw_k.t[e] = kept(r_k.t[e]);
                    n.raw_q.t[e] = kept(r_q.t[e]);
                }
            }
        };

        // ---- state tiles of this wave, transposed: acc[i][r] = S[channel][column 16 nt + 4 g + r], the channel 16 ct + lm of a
        // main tile, 32 + 4 e + lm / 4 of a tail tile: there lanes lm % 4 = 0, 1 hold the hi share (twice), 2, 3 the lo share ----
        f32x4 acc[OW::kMost], accg[GS ? OW::kMost : 1];
#pragma unroll
        for (int i = 0; i < OW::kMost; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (GS) {
#pragma unroll
            for (int i = 0; i < OW::kMost; ++i) accg[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        const bool tail_hi = (lm & 3) < 2;
        auto channel = [&](int ct) { return ct < 2 ? 16 * ct + lm : 32 + 4 * (ct - 2) + (lm >> 2); };
        // where a lane finds its channel's entry of a [g][kTS] row of totals
        auto tot_at = [&](int ct) { return (lm >> 2) * TS + (ct < 2 ? 4 * ct + (lm & 3) : 8 + (ct - 2)); };
        auto whole = [&](int ct, f32x4 x) {      // a tile's values; a tail tile's in all four lanes of a channel
            return ct < 2 ? x : f32x4{quad_add2(x[0]), quad_add2(x[1]), quad_add2(x[2]), quad_add2(x[3])};
        };
        auto zero4 = f32x4{0.f, 0.f, 0.f, 0.f};
        // scale the tiles from the anchor of chunk c to that of chunk c + 1 (or from the span's start, or to its end: what lies
        // past it decays by nothing) and leave P of chunk c + 1 in LDS
        auto publish = [&](auto wave_c, int c) {
            constexpr int W = decltype(wave_c)::value;
            const float *t_c = s_tot + ring(c + 3) * 16 * TS, *t_n = s_tot + ring(c + 1) * 16 * TS;
            uint16_t *prow = s_p + ((c + 1) & 1) * SET + (4 * g ^ swz);
            float fac[NCT];
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) {
                bool used = false;
                for (int t = OW::start(W); t < OW::start(W + 1); ++t) used = used || (t % NCT == ct);
                if (!used) continue;
                const int at = tot_at(ct);
                float h = t_n[at] + t_n[4 * TS + at];
                if (c >= 0) h += t_c[8 * TS + at] + t_c[12 * TS + at];
                fac[ct] = exp2_fast(h);
            }
#pragma unroll
            for (int i = 0; i < OW::count(W); ++i) {
                const int ct = (OW::start(W) + i) % NCT, nt = (OW::start(W) + i) / NCT;
                f32x4 s = whole(ct, acc[i]) * fac[ct];
                u32x2 hi, lo;
                SPLIT_PAIR(s[0], s[1], hi[0], lo[0]);
                SPLIT_PAIR(s[2], s[3], hi[1], lo[1]);
                if (ct < 2) {
                    *reinterpret_cast<u32x2 *>(prow + (16 * ct + lm) * VS + 16 * nt) = hi;
                    *reinterpret_cast<u32x2 *>(prow + (32 + 16 * ct + lm) * VS + 16 * nt) = lo;
                    acc[i] = s;
                } else {
                    *reinterpret_cast<u32x2 *>(prow + (64 + 16 * (ct - 2) + lm) * VS + 16 * nt) =
                        u32x2{tail_hi ? hi[0] : lo[0], tail_hi ? hi[1] : lo[1]};
                    acc[i] = f32x4{tail_hi ? s[0] : 0.f, tail_hi ? s[1] : 0.f, tail_hi ? s[2] : 0.f, tail_hi ? s[3] : 0.f};
                }
            }
        };
        auto per_wave = [&](auto fn, int c) {
            constexpr int W0 = READ ? 0 : 4;
            switch (w) {
            case 0: fn(int_c<W0>{}, c); break;
            case 1: fn(int_c<W0 + 1>{}, c); break;
            case 2: fn(int_c<W0 + 2>{}, c); break;
            default: fn(int_c<W0 + 3>{}, c); break;
            }
        };
        auto store_state = [&](auto wave_c, float *dst, const f32x4 *a) {
            constexpr int W = decltype(wave_c)::value;
#pragma unroll
            for (int i = 0; i < OW::count(W); ++i) {
                const int ct = (OW::start(W) + i) % NCT, c = channel(ct), n = 16 * ((OW::start(W) + i) / NCT) + 4 * g;
                const f32x4 s = whole(ct, a[i]);
                if (c < dk && n < dv && (ct < 2 || (lm & 3) == 0)) *reinterpret_cast<f32x4 *>(dst + c * dv + n) = s;
            }
        };

        // GS: log2 of the decay from the span's first step to the chunk, per channel tile and column tile of this wave's tiles
        float decay[NCT];
        // ---- prologue: request everything the first stages need, then chain the state entering the span ----
        int tok0 = row.tok, tok1;            // tokens of the chunk contracted next, and of the one after it
        FRow later;                          // gate gradients: sums over the scan steps walked before the chunk
        later.u[0] = later.u[1] = zero4;
#pragma unroll
        for (int e = 0; e < DT; ++e) later.t[e] = 0.f;
        {
            issue_gates();
            issue_rows(row_s0, row.tok);
            issue_grad(row_s0, row.tok);
            next_row();
            tok1 = row.tok;
            if constexpr (GS) {
                // (the first step's own gate does not act on its q^T dO, but is part of the chunk's prefix sums)
                const int tf = scan_token(p.scan_dir, s_begin, T, p.grid_h, p.grid_w);
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct)
                    decay[ct] = fminf(-fetch<float>(bg, channel(ct) < dk ? 2u * ((uint32_t)tf * dk2 + 2u * (uint32_t)channel(ct)) : kNowhere) * kLog2e, kMaxExp2);
            }
            const bool chained = p.chain_in_output && sp > 0;   // uniform
            float *s_chain = reinterpret_cast<float *>(smem + L::oSet);
            float *s_sum = s_chain + (32 + 4 * DT) * 16 * NX;            // [8][40]: sums of the waves
            if (chained) {
                constexpr int kV4 = ((32 + 4 * DT) * 16 * NDV16 / 4 + 511) / 512;
                constexpr int kRun = 16 / kV4;
                chain_span_states<512, kV4, kRun, false, true>(p, bh, sp, tid, s_chain);
            }
            if constexpr (DV)     // (totals of the chunk before the first)
                for (int i = tid; i < (L::oSet - L::oX) / 4; i += 512) s_x[i] = 0.f;
            scan(0, r_b);
            issue_gates();                   // chunk 1
            __syncthreads();
            if (chained || (!p.chain_in_output && p.nspans > 1)) {
                const Rsrc bs = view(p.ws_state + ((size_t)bh * p.nspans + sp) * dk * dv, 4u * (uint32_t)(dk * dv));
                per_wave([&](auto wave_c, int) {
                    constexpr int W = decltype(wave_c)::value;
#pragma unroll
                    for (int i = 0; i < OW::count(W); ++i) {
                        const int ct = (OW::start(W) + i) % NCT, c = channel(ct), n = 16 * ((OW::start(W) + i) / NCT) + 4 * g;
                        const int at = min(c, dk - 1) * dv + min(n, dv - 4);
                        const f32x4 s = chained ? *reinterpret_cast<const f32x4 *>(s_chain + at) : fetch<f32x4>(bs, 4u * (uint32_t)at);
                        const bool there = c < dk && n < dv && (ct < 2 || tail_hi);
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[i][r] = there ? s[r] : 0.f;
                    }
                    HILO_WAVE_END(W);
                }, 0);
            }
            if constexpr (DV) {
                // The gate gradients are sums over all later scan steps, i.e. over the steps this walk has made before: those
                // before the span add up to the gradient of the gate between it and them,
                //     sum_{s' >= b} (q dq - k dk)[c] = sum_n alpha_b[c] G_b[c,n] S_{b-1}[c,n],
                // G_b being the state that enters this walk (acc) and S_{b-1} the one that
                // the forward walk left at the same place.
                if (with_gates && sp > 0) {       // (uniform)
                    const Rsrc bs = view(p.ws_bound + ((size_t)bh * p.bounds + (T - s_begin) / p.bound_len - 1) * (size_t)(dk * dv), 4u * (uint32_t)(dk * dv));
                    const uint32_t tb = (uint32_t)scan_token(p.scan_dir, s_begin - 1, T, p.grid_h, p.grid_w);
                    for (int i = tid; i < 8 * 40; i += 512) s_sum[i] = 0.f;
                    __syncthreads();
                    per_wave([&](auto wave_c, int) {
                        constexpr int W = decltype(wave_c)::value;
                        float row_sum[NCT];
#pragma unroll
                        for (int ct = 0; ct < NCT; ++ct) row_sum[ct] = 0.f;
#pragma unroll
                        for (int i = 0; i < OW::count(W); ++i) {
                            const int ct = (OW::start(W) + i) % NCT, nt = (OW::start(W) + i) / NCT, c = channel(ct), n = 16 * nt + 4 * g;
                            const bool there = c < dk && n < dv && (ct < 2 || (lm & 3) == 0);
                            const f32x4 s = fetch<f32x4>(bs, there ? 4u * (uint32_t)(c * dv + n) : kNowhere);
                            const float a = exp2_fast(fetch<float>(bg, c < dk ? 2u * (tb * dk2 + 2u * (uint32_t)c) : kNowhere) * kLog2e);
                            f32x4 x = acc[i] * s * a;
                            row_sum[ct] += (x[0] + x[1]) + (x[2] + x[3]);
                        }
#pragma unroll
                        for (int ct = 0; ct < NCT; ++ct) {
                            float x = row_sum[ct];
                            x += __shfl_xor(x, 16);
                            x += __shfl_xor(x, 32);
                            if (g == 0 && (ct < 2 || (lm & 3) == 0)) s_sum[40 * W + channel(ct)] = x;
                        }
                        HILO_WAVE_END(W);
                    }, 0);
                    __syncthreads();
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
#pragma unroll
                        for (int h = 0; h < 2; ++h) later.u[h] += *reinterpret_cast<const f32x4 *>(s_sum + 40 * u + 16 * h + 4 * g);
#pragma unroll
                        for (int e = 0; e < DT; ++e) later.t[e] += s_sum[40 * u + 32 + 4 * e + g];
                    }
                }
            }
            __syncthreads();      // the start state and the sums have been read
        }
        per_wave([&](auto wave_c, int) {
            gate(wave_c, 0, own);
            HILO_WAVE_END(decltype(wave_c)::value);
        }, 0);
        scan(1, r_b);
        next_row();
        issue_gates();                           // chunk 2 (in the order in which the loop leaves its loads)
        issue_rows(row_s0 + kChunk, tok1);
        per_wave([&](auto wave_c, int) {
            publish(wave_c, -1);
            HILO_WAVE_END(decltype(wave_c)::value);
        }, 0);
        __syncthreads();

        FRow xs;                             // gate gradients of the chunk before: sums inside the wave's tile
        uint32_t xs_at = kNowhere / 2;       // their row
        // the gate gradients of chunk c - 1: the wave's own rows + the tiles before it + everything before the chunk
        auto finish = [&](auto wave_c, int c) {
            constexpr int W = decltype(wave_c)::value & 3;
            if constexpr (DV && READ) {
                const float *t = s_x + ((c + 1) & 1) * 16 * TS;
                FRow add = later;
#pragma unroll
                for (int u = 0; u < W; ++u) add = add_row(add, get_tot(t + u * 4 * TS));
                put_f(bda, xs_at, add_row(xs, add));
                later = add;
#pragma unroll
                for (int u = W; u < 4; ++u) later = add_row(later, get_tot(t + u * 4 * TS));
            }
        };
        for (int c = 0; c < nch; ++c) {
            {   // (LDS offsets are derived afresh in every chunk: kept across the loop they would take too many registers)
                const int ln = recompute_per_chunk(lane);
                lm = ln & 15;
                g = ln >> 4;
                swz = 8 * (lm >> 3);
            }
            const int tr_row = lm >> 2, tr_col = (4 * (lm & 3)) ^ (8 * (g >> 1));   // transposing reads: row-in-4 and column quad of this lane
            // Gates of chunk c + 2, requested an iteration ago.  (Here and not behind the contraction: a wait for them there would
            // wait for the rows stored in it as well.)
            FRow b_next;
            scan(c + 2, b_next);
            const int tok2 = row.tok;
            next_row();
            issue_gates();                           // chunk c + 3
            auto contract = [&](auto wave_c, int) {
                constexpr int W8 = decltype(wave_c)::value, W = W8 & 3;
                constexpr int NQ = W / 2 + 1;                     // 32-token steps that hold causal tokens for this wave
                constexpr int t_lo = OW::start(W8), t_hi = OW::start(W8 + 1), NT_LO = t_lo / NCT, NT_HI = (t_hi - 1) / NCT;
                const int set = (c & 1) * SET;
                const uint16_t *vtr = s_v + set + (4 * g + tr_row) * VS + tr_col;
                const uint16_t *ktr = s_k + set + (4 * g + tr_row) * RS + tr_col;
                auto tr2 = [&](const uint16_t *at, int rs) {      // 32 rows of 16 columns, contracted over the rows
                    const u32x2 lo = lds_read_tr(at), hi = lds_read_tr(at + 16 * rs);
                    return u32x4{lo[0], lo[1], hi[0], hi[1]};
                };
                auto pieces = [&](const uint16_t *at) {           // a row's columns 4 g .. + 3 and 16 + 4 g .. + 3 of a 32-wide step
                    const u32x2 lo = *reinterpret_cast<const u32x2 *>(at), hi = *reinterpret_cast<const u32x2 *>(at + 16);
                    return u32x4{lo[0], lo[1], hi[0], hi[1]};
                };
                auto vpieces = [&](const uint16_t *row, int ks) { // of step ks of a value-side row (the last may be 16 wide)
                    if (2 * ks + 1 < NX) return pieces(row + 32 * ks);
                    const u32x2 lo = *reinterpret_cast<const u32x2 *>(row + 32 * ks);
                    return u32x4{lo[0], lo[1], 0u, 0u};
                };
                finish(wave_c, c);
                float fac[NCT];
                if constexpr (GS) {      // decay from the span's first step to this chunk's anchor
                    const float *t_c = s_tot + ring(c) * 16 * TS;
#pragma unroll
                    for (int ct = 0; ct < NCT; ++ct) {
                        const int at = tot_at(ct);
                        const float h0 = t_c[at] + t_c[4 * TS + at];
                        fac[ct] = exp2_fast(decay[ct] + h0);
                        decay[ct] += h0 + (t_c[8 * TS + at] + t_c[12 * TS + at]);
                    }
                }
                // ---- state tiles of this wave: P + K~^T V~ (transposed); GS: Q~^T dO~ ----
                if constexpr (t_lo < t_hi) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        u32x4 kf[2 + 2 + DT];        // hi of ct 0, 1; lo of ct 0, 1; tails
#pragma unroll
                        for (int ct = 0; ct < NCT; ++ct) {
                            bool used = false;
                            for (int t = t_lo; t < t_hi; ++t) used = used || (t % NCT == ct);
                            if (!used) continue;
                            if (ct < 2) kf[ct] = tr2(ktr + 32 * q * RS + 16 * ct, RS);
                            kf[2 + ct] = tr2(ktr + 32 * q * RS + (ct < 2 ? 32 + 16 * ct : 64 + 16 * (ct - 2)), RS);
                        }
#pragma unroll
                        for (int nt = NT_LO; nt <= NT_HI; ++nt) {
                            const u32x4 vf = tr2(vtr + 32 * q * VS + 16 * nt, VS);
#pragma unroll
                            for (int ct = 0; ct < NCT; ++ct) {
                                const int t = nt * NCT + ct;
                                if (t < t_lo || t >= t_hi) continue;
                                f32x4 a = acc[t - t_lo];
                                if (ct < 2) a = mfma(vf, kf[ct], a);
                                a = mfma(vf, kf[2 + ct], a);
                                acc[t - t_lo] = a;
                            }
                        }
                    }
                    if constexpr (GS) {
                        const uint16_t *qtr = s_q + set + (4 * g + tr_row) * RS + tr_col;
                        const uint16_t *wtr = s_w + set + (4 * g + tr_row) * VS + tr_col;
                        f32x4 part[t_hi - t_lo];
#pragma unroll
                        for (int i = 0; i < t_hi - t_lo; ++i) part[i] = zero4;
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            u32x4 qf[2 + 2 + DT];
#pragma unroll
                            for (int ct = 0; ct < NCT; ++ct) {
                                bool used = false;
                                for (int t = t_lo; t < t_hi; ++t) used = used || (t % NCT == ct);
                                if (!used) continue;
                                if (ct < 2) qf[ct] = tr2(qtr + 32 * q * RS + 16 * ct, RS);
                                qf[2 + ct] = tr2(qtr + 32 * q * RS + (ct < 2 ? 32 + 16 * ct : 64 + 16 * (ct - 2)), RS);
                            }
#pragma unroll
                            for (int nt = NT_LO; nt <= NT_HI; ++nt) {
                                const u32x4 wf = tr2(wtr + 32 * q * VS + 16 * nt, VS);
#pragma unroll
                                for (int ct = 0; ct < NCT; ++ct) {
                                    const int t = nt * NCT + ct;
                                    if (t < t_lo || t >= t_hi) continue;
                                    f32x4 a = part[t - t_lo];
                                    if (ct < 2) a = mfma(wf, qf[ct], a);
                                    a = mfma(wf, qf[2 + ct], a);
                                    part[t - t_lo] = a;
                                }
                            }
                        }
#pragma unroll
                        for (int i = 0; i < t_hi - t_lo; ++i) {
                            const int ct = (t_lo + i) % NCT;
                            f32x4 f = f32x4{fac[ct], fac[ct], fac[ct], fac[ct]};
#pragma unroll
                            for (int r = 0; r < 4; ++r) accg[i][r] = fmaf(f[r], part[i][r], accg[i][r]);
                        }
                    }
                }
                const int step = row_s0 + c * kChunk;
                const uint32_t here_k = at_k(step, tok0), here_v = at_v(step, tok0);
                if constexpr (READ) {
                // ---- Z^T = (V~ W~^T) tiles: lane (lm, g) gets Z[j = 16 W + lm][i = 16 jt + 4 g + r] ----
                u32x4 zh[NQ], zl[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q) zh[q] = zl[q] = u32x4{0, 0, 0, 0};
#pragma unroll
                for (int jt = 0; jt <= W; ++jt) {
                    f32x4 d = zero4;
#pragma unroll
                    for (int ks = 0; ks < KSV; ++ks) {
                        const u32x4 vf = vpieces(s_v + set + (16 * jt + lm) * VS + (4 * g ^ swz), ks);
                        d = mfma(vf, own.wh[ks], d);
                    }
                    if (jt == W)
                        d = f32x4{4 * g + 0 > lm ? 0.f : d[0], 4 * g + 1 > lm ? 0.f : d[1], 4 * g + 2 > lm ? 0.f : d[2], 4 * g + 3 > lm ? 0.f : d[3]};
                    const int h = 2 * (jt & 1);
                    SPLIT_PAIR(d[0], d[1], zh[jt / 2][h], zl[jt / 2][h]);
                    SPLIT_PAIR(d[2], d[3], zh[jt / 2][h + 1], zl[jt / 2][h + 1]);
                }
                // ---- R^T = P W~^T + K~^T Z^T: lane (lm, g) gets R[16 W + lm][channel 16 ct + 4 g + r] (tail: 32 + 4 e + g in r = 0 and 2) ----
                f32x4 rr[NCT];
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct) {
                    f32x4 a = zero4;
#pragma unroll
                    for (int ks = 0; ks < KSV; ++ks) {
                        if (ct < 2) {
                            const u32x4 ph = vpieces(s_p + set + (16 * ct + lm) * VS + (4 * g ^ swz), ks);
                            a = mfma(ph, own.wh[ks], a);
                        }
                        const u32x4 pl = vpieces(s_p + set + ((ct < 2 ? 32 + 16 * ct : 64 + 16 * (ct - 2)) + lm) * VS + (4 * g ^ swz), ks);
                        a = mfma(pl, own.wh[ks], a);
                    }
                    rr[ct] = a;
                }
#pragma unroll
                for (int q = 0; q < NQ; ++q)
#pragma unroll
                    for (int ct = 0; ct < NCT; ++ct) {
                        if (ct < 2) {
                            const u32x4 kh = tr2(ktr + 32 * q * RS + 16 * ct, RS);
                            rr[ct] = mfma(kh, zh[q], rr[ct]);
                            rr[ct] = mfma(kh, zl[q], rr[ct]);
                        }
                        const u32x4 kl = tr2(ktr + 32 * q * RS + (ct < 2 ? 32 + 16 * ct : 64 + 16 * (ct - 2)), RS);
                        rr[ct] = mfma(kl, zh[q], rr[ct]);
                        rr[ct] = mfma(kl, zl[q], rr[ct]);
                    }
                FRow res;
#pragma unroll
                for (int u = 0; u < 2; ++u) res.u[u] = rr[u] * own.e.u[u];
#pragma unroll
                for (int e = 0; e < DT; ++e) res.t[e] = (rr[2 + e][0] + rr[2 + e][2]) * own.e.t[e];
                put_f(br, here_k, res);
                if constexpr (DV) {
                    // ---- gate gradient, key side: x_s = q_s dq_s - k_s dk_s (in this walk the rows called k are q, those called
                    // q are k), summed inside the wave's tile ----
#pragma unroll
                        for (int u = 0; u < 2; ++u)
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                xs.u[u][2 * h] = fmaf(bf16_lo_as_float(own.raw_k.u[u][h]), r_dq.u[u][2 * h], -bf16_lo_as_float(own.raw_q.u[u][h]) * res.u[u][2 * h]);
                                xs.u[u][2 * h + 1] = fmaf(bf16_hi_as_float(own.raw_k.u[u][h]), r_dq.u[u][2 * h + 1], -bf16_hi_as_float(own.raw_q.u[u][h]) * res.u[u][2 * h + 1]);
                            }
#pragma unroll
                        for (int e = 0; e < DT; ++e) xs.t[e] = fmaf(bf16_lo_as_float(own.raw_k.t[e]), r_dq.t[e], -bf16_lo_as_float(own.raw_q.t[e]) * res.t[e]);
                        scan_rows(xs);
                        put_tot(s_x + ((c & 1) * 4 + W) * 4 * TS, xs);
                        xs_at = with_gates ? here_k : kNowhere / 2;
                }
                }
                if constexpr (!READ && DV) {
                    // ---- outputs: score tiles q~ . k~, then O^T = P^T Q~^T + V~^T A^T ----
                    u32x4 ah[NQ], al[NQ];
#pragma unroll
                    for (int q = 0; q < NQ; ++q) ah[q] = al[q] = u32x4{0, 0, 0, 0};
#pragma unroll
                    for (int jt = 0; jt <= W; ++jt) {
                        const uint16_t *krow = s_k + set + (16 * jt + lm) * RS + (4 * g ^ swz);
                        const u32x4 kh = pieces(krow), kl = pieces(krow + 32);
                        f32x4 d = zero4;
                        d = mfma(kh, own.qh, d);
                        d = mfma(kh, own.ql, d);
                        d = mfma(kl, own.qh, d);
                        d = mfma(kl, own.ql, d);
                        u32x4 kt = u32x4{0, 0, 0, 0};
#pragma unroll
                        for (int e = 0; e < DT; ++e) {
                            const u32x2 y = *reinterpret_cast<const u32x2 *>(krow + 64 + 16 * e);
                            kt[2 * e] = y[0];
                            kt[2 * e + 1] = y[1];
                        }
                        d = mfma(kt, own.qt, d);
                        if (jt == W)
                            d = f32x4{4 * g + 0 > lm ? 0.f : d[0], 4 * g + 1 > lm ? 0.f : d[1], 4 * g + 2 > lm ? 0.f : d[2], 4 * g + 3 > lm ? 0.f : d[3]};
                        const int h = 2 * (jt & 1);
                        SPLIT_PAIR(d[0], d[1], ah[jt / 2][h], al[jt / 2][h]);
                        SPLIT_PAIR(d[2], d[3], ah[jt / 2][h + 1], al[jt / 2][h + 1]);
                    }
                    const uint16_t *ptr = s_p + set + (4 * g + tr_row) * VS + tr_col;
#pragma unroll
                    for (int x = 0; x < NX; ++x) {
                        const u32x4 ph = tr2(ptr + 16 * x, VS), pl = tr2(ptr + 32 * VS + 16 * x, VS);
                        f32x4 o = zero4;
                        o = mfma(ph, own.qh, o);
                        o = mfma(ph, own.ql, o);
                        o = mfma(pl, own.qh, o);
                        o = mfma(pl, own.ql, o);
                        u32x4 pt = u32x4{0, 0, 0, 0};
#pragma unroll
                        for (int e = 0; e < DT; ++e) {
                            const u32x2 y = lds_read_tr(ptr + (64 + 16 * e) * VS + 16 * x);
                            pt[2 * e] = y[0];
                            pt[2 * e + 1] = y[1];
                        }
                        o = mfma(pt, own.qt, o);
#pragma unroll
                        for (int q = 0; q < NQ; ++q) {
                            const u32x4 vf = tr2(vtr + 32 * q * VS + 16 * x, VS);
                            o = mfma(vf, ah[q], o);
                            o = mfma(vf, al[q], o);
                        }
                        put(bo, f32_at(here_v, vcb[x]), o);
                    }
                }
                if constexpr (READ && DV) __builtin_amdgcn_sched_barrier(0);    // (registers)
                Own next;
                gate(wave_c, c + 1, next);
                publish(wave_c, c);
                own = next;
                HILO_WAVE_END(W);
            };
            per_wave(contract, c);
            r_b = b_next;
            issue_grad(walk_s - 2 * kChunk, tok1);   // chunk c + 1
            tok0 = tok1;
            tok1 = tok2;
            issue_rows(walk_s - kChunk, tok1);       // chunk c + 2
            __syncthreads();
        }
        if constexpr (DV) {
            per_wave([&](auto wave_c, int) {
                finish(wave_c, nch);
                HILO_WAVE_END(decltype(wave_c)::value);
            }, 0);
        }
        if constexpr (!DV) {
            // a bound of the reversed walk's spans: the state there
            if (p.ws_bound != nullptr && s_end < T && s_end % p.bound_len == 0) {
                float *dst = p.ws_bound + ((size_t)bh * p.bounds + s_end / p.bound_len - 1) * (size_t)(dk * dv);
                per_wave([&](auto wave_c, int) {
                    store_state(wave_c, dst, acc);
                    HILO_WAVE_END(decltype(wave_c)::value);
                }, 0);
            }
        }
        if constexpr (GS) {
            // U of the reversed walk's span, and the log of its decay: the gates of the steps a + 1 .. b (with gate_shift the
            // walk's first step decays by the gate of step b, the first one after this span)
            const size_t span = (size_t)bh * p.nspans + (p.nspans - 1 - sp);
            const uint32_t ta = (uint32_t)scan_token(p.scan_dir, min(s_end, T - 1), T, p.grid_h, p.grid_w);
            per_wave([&](auto wave_c, int) {
                store_state(wave_c, p.ws_gstate + span * (size_t)(dk * dv), accg);
                HILO_WAVE_END(decltype(wave_c)::value);
            }, 0);
            if (w8 == 0 && g == 0) {
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct) {
                    const int c = channel(ct);
                    if (c < dk && (ct < 2 || (lm & 3) == 0))
                        p.ws_glgam[span * dk + c] = decay[ct] * kLn2 + fetch<float>(bg, 2u * (ta * dk2 + 2u * (uint32_t)c));
                }
            }
        }
    };
    if (w8 < 4) walk(std::true_type{});
    else walk(std::false_type{});
}

template <bool DV, bool GS>
hipError_t launch_one(const WalkParams &p, const void *w, float *r, hipStream_t stream) {
    using L = WLayout<DV, GS>;
    auto kernel = hilo_walk_kernel<DV, GS>;
    static std::atomic<bool> configured[kMaxDevices] = {};  // per instantiation and device
    {
        hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), L::kBytes, configured);
        if (e != hipSuccess) return e;
    }
    const unsigned groups = (unsigned)(p.B * p.H * p.nspans);        // (few: launch_mfma_row_read)
    hipLaunchKernelGGL(kernel, dim3(groups), dim3(512), L::kBytes, stream, p, w, r);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_hilo_walk(const WalkParams &p, const void *w, float *r, hipStream_t stream, bool with_outputs) {
    if (with_outputs) return launch_one<true, false>(p, w, r, stream);
    return p.ws_gstate != nullptr ? launch_one<false, true>(p, w, r, stream) : launch_one<false, false>(p, w, r, stream);
}

}  // namespace gla
