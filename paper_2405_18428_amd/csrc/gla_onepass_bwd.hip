// Backward pass of the GLA recurrence on whole chunks, four waves per 64-token chunk (bf16 hi/lo MFMA operands)
// (DiG paper, Sec. 3.1 Eq. (attn_gla) rows 1-3 differentiated, in the chunk form of Sec. 3.5; heads as in gla_onepass.hip).
//
// With the mid-chunk anchor m, q~_j = q_j 2^(b_j - b_m) and k~_i = k_i 2^(b_m - b_i), S the state that enters a chunk, G the adjoint of
// the state that leaves it, P = 2^(b_m) S and Gp = 2^(b_C - b_m) G,
//     A_ji = q~_j . k~_i ,   M_ji = dO_j . v_i   (j >= i)
//     dq_j = 2^(b_j - b_m) (sum_i M_ji k~_i + P dO_j) ,   dk_i = 2^(b_m - b_i) (sum_j M_ji q~_j + Gp v_i) ,   dv_i = sum_j A_ji dO_j + k~_i Gp
//     S' = 2^(b_C) S + 2^(b_C - b_m) K~^T V ,   G' = 2^(b_C) G + 2^(b_m) Q~^T dO
//     d log alpha_s = sum_{s' >= s, in the chunk} (q dq - k dk)_s' + rowsum(S' * G)
// (the last line: all later chunks' share of the sum is what the two states at the chunk's end give), so that one pass over a
// chunk forms everything that a walk forwards and one backwards formed before, from one gating of q and k, and the gate gradient
// sums over 64 steps at most: its error is a half to a quarter of the walks' (1.4e-5 -> 7.3e-6 of its 2-norm at 4 chunks).
//
// A work-group holds a span of four chunks; wave t of a chunk owns its 16-token tile t, in either role: as queries it meets t + 1 score
// tiles, as keys 4 - t (all four are formed, and masked: straight-line code).  v and dO go straight to LDS, q~ and k~ are
// left there as hi/lo rows.  Each chunk's own states are added up there in fp32, turned by the group's threads into the split
// states P and Gp of each chunk, and read over their columns (dq, dk) and over their channels (dv).  Sequences of one span
// are one launch; else a launch of the same kernel leaves the spans' states first, and the second chains them from both sides.
//
// What bounds it on MI355X (256 sequences of 4 chunks at 36 / 72 channels: 30 us, one launch, 27 us of it a chain of dependent stages with 16 waves
// on the unit; before, a walk each way, 18 + 28 us): loads 8 us at the memory's rate, gates and scores 6, states 4, turning
// them around 3, the products with them 3, gradients 4.  A training step of that shape 59.9 -> 47.0 us.
#include <type_traits>

#include "gla_common.h"
#include "gla_onepass_util.h"

namespace gla {
namespace {

enum { kWhole, kStates, kOutputs };      // sequences of one span; the spans' states; the gradients from them

constexpr int NC = 4, NT = 256 * NC;

template <typename HD>
struct BLayout {
    static constexpr int kRow = 80;                                  // bf16 per row of k~ and q~: 32 hi, 32 lo, 4 x (hi, hi, lo, lo)
    static constexpr int kDk = 32 + 4 * HD::DT;
    static constexpr int kStateRow = 72;                             // bf16 per channel of a split state (hi rows, then lo rows)
    static constexpr int kUBytes = kDk * HD::NV * 4, kPBytes = 2 * kDk * kStateRow * 2, kKBytes = kChunk * kRow * 2;
    static constexpr int kGated = kKBytes > kUBytes ? (kKBytes > kPBytes ? kKBytes : kPBytes) : (kUBytes > kPBytes ? kUBytes : kPBytes);
    static constexpr int kRows = kChunk * HD::NV * 2;                // v and dO as they come in
    static constexpr int oQ = kGated, oV = 2 * kGated, oO = oV + kRows, kOne = oO + kRows;
    static constexpr int oDecay = NC * kOne;                         // float[NC][4][36]
    static constexpr int oZ = oDecay + NC * 4 * 36 * 4;              // float[NC][36]: sum over the columns of S G at the chunk's end
    static constexpr int oMeet = oZ + NC * 36 * 4;                   // int[4 NC]
    static constexpr int kBytes = oMeet + 4 * NC * 4;
    static_assert(kBytes <= 160 * 1024, "one group a compute unit");
};

typedef const __attribute__((address_space(4))) BackParams *Args;

// Inclusive sums over the lanes from this one to the last of its 16 (row_scan16x4 the other way round)
__device__ inline void row_suffix16x4(float &a, float &b, float &c, float &d) {
    asm volatile(
        "s_nop 4\n\t"
        "v_add_f32_dpp %0, %0, %0 row_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %1, %1, %1 row_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %2, %2, %2 row_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %3, %3, %3 row_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_shl:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %1, %1, %1 row_shl:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %2, %2, %2 row_shl:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %3, %3, %3 row_shl:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_shl:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %1, %1, %1 row_shl:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %2, %2, %2 row_shl:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %3, %3, %3 row_shl:4 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_shl:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %1, %1, %1 row_shl:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %2, %2, %2 row_shl:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_add_f32_dpp %3, %3, %3 row_shl:8 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "s_nop 1"
        : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}
__device__ inline float row_suffix16(float v) {
    v += dpp_move<0x101, 0xF, true>(v);
    v += dpp_move<0x102, 0xF, true>(v);
    v += dpp_move<0x104, 0xF, true>(v);
    v += dpp_move<0x108, 0xF, true>(v);
    return v;
}

template <typename HD, int MODE>
__global__ __launch_bounds__(NT, 4) void chunk_back_kernel(BackParams) {
    using L = BLayout<HD>;
    constexpr int DT = HD::DT, NX = HD::NX, NG = 8 + DT, NS = NX == 5 ? 3 : 2;      // NS: contraction steps over the value columns
    constexpr int RS = L::kRow, VP = HD::NV / 8, PS = L::kStateRow, US = 36;
    const Args args = (Args)__builtin_amdgcn_kernarg_segment_ptr();

    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile = w & 3;                          // of chunk w / 4
    unsigned char *mine = smem + (w >> 2) * L::kOne;
    uint16_t *s_k = reinterpret_cast<uint16_t *>(mine), *s_q = reinterpret_cast<uint16_t *>(mine + L::oQ);
    uint16_t *s_v = reinterpret_cast<uint16_t *>(mine + L::oV), *s_o = reinterpret_cast<uint16_t *>(mine + L::oO);
    float *s_decay = reinterpret_cast<float *>(smem + L::oDecay);
    float *my_decay = s_decay + (w >> 2) * 4 * US;
    float *s_z = reinterpret_cast<float *>(smem + L::oZ);

    // the four waves of a chunk wait for each other (LDS accesses of a wave are done in order)
    int *s_meet = reinterpret_cast<int *>(smem + L::oMeet);
    int met = 0;
    auto meet = [&]() {
        ++met;
        asm volatile("" ::: "memory");
        __hip_atomic_store(s_meet + w, met, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        while (!__all(__hip_atomic_load(s_meet + (w & ~3) + (threadIdx.x & 3), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >= met)) {
        }
        asm volatile("" ::: "memory");
    };
    if (tid < 4 * NC) s_meet[tid] = 0;

    // what the first loads need, all at once: a group's first access to a line of its arguments takes as long as one to memory
    int B = args->B, H = args->H, T = args->T, dk = args->dk, dv = args->dv, grid_h = args->grid_h, grid_w = args->grid_w,
        scan_dir = args->scan_dir, nspans = args->nspans, st_k = args->st_k, st_v = args->st_v;
    long long sb_k = args->sb_k, sh_k = args->sh_k, sb_v = args->sb_v, sh_v = args->sh_v;
    const void *from_v = args->v, *from_o = args->d_out, *from_k = args->k, *from_q = args->q, *from_gate = args->log_alpha;
    asm volatile("" : "+s"(B), "+s"(H), "+s"(T), "+s"(dk), "+s"(dv), "+s"(grid_h), "+s"(grid_w), "+s"(scan_dir), "+s"(nspans),
                 "+s"(st_k), "+s"(st_v), "+s"(sb_k), "+s"(sh_k), "+s"(sb_v), "+s"(sh_v), "+s"(from_v), "+s"(from_o), "+s"(from_k), "+s"(from_q), "+s"(from_gate));
    __syncthreads();           // (the counters of meet are there)
    int blk = blockIdx.x;      // contiguous ranges of spans per XCD
    {
        const int nb = B * H * nspans;
        if ((nb & 7) == 0) blk = (blk & 7) * (nb >> 3) + (blk >> 3);
    }
    const int bh = blk / nspans, sp = blk - bh * nspans;
    const int s_begin = sp * NC * kChunk, s_end = min(T, s_begin + NC * kChunk);
    const int c_begin = s_begin + (w >> 2) * kChunk;
    const int batch = bh / H, head = bh - batch * H;
    const size_t base_k = (size_t)batch * (size_t)sb_k + (size_t)head * (size_t)sh_k, base_v = (size_t)batch * (size_t)sb_v + (size_t)head * (size_t)sh_v;
    const uint32_t dk2 = 2u * (uint32_t)st_k, dv2 = 2u * (uint32_t)st_v;   // bytes from one bf16 row to the next
    const uint32_t bytes_k = (uint32_t)(T - 1) * dk2 + 2u * (uint32_t)dk, bytes_v = (uint32_t)(T - 1) * dv2 + 2u * (uint32_t)dv;
    auto view_k = [&](const void *x, uint32_t bytes) { return view(static_cast<const char *>(x) + afresh(base_k) * bytes, bytes_k / 2 * bytes); };
    auto view_v = [&](const void *x, uint32_t bytes) { return view(static_cast<const char *>(x) + afresh(base_v) * bytes, bytes_v / 2 * bytes); };

    // each lane finds one row's token (a row past the span's end repeats the last); then that of this lane's own row
    uint32_t rowk, rowv;
    auto chb = [&](int u, int g) { return 16 * u + 4 * g < dk ? 2u * (uint32_t)(16 * u + 4 * g) : kNowhere / 2; };
    auto tcb = [&](int g) { return 32 + g < dk ? 2u * (uint32_t)(32 + g) : kNowhere / 2; };
    f32x4 la[2];
    float lat = 0.f;
    u32x2 rq[2], rk[2];
    uint32_t rqt = 0, rkt = 0;
    {
        LANE;
        int tok;
        {
            const int col_len = scan_dir >= 2 ? grid_h : 1;       // (uniform)
            const int s0 = min(c_begin + lane, s_end - 1), s = (scan_dir & 1) ? T - 1 - s0 : s0;
            const int tc = s / col_len;
            tok = (s - tc * col_len) * grid_w + tc;
        }
        auto token_of = [&](int j) { return (uint32_t)__builtin_amdgcn_ds_bpermute(4 * j, tok); };
        {
            const Rsrc bv = view_v(from_v, 2), bo = view_v(from_o, 2);
#pragma unroll
            for (int i = 0; i < (VP + 3) / 4; ++i) {
                if (4 * i + tile < VP) {
                    const int at = lane + 64 * (4 * i + tile), vr = at / VP, vp = at - vr * VP;
                    const int piece = DT ? vp : vp ^ (2 * ((vr >> 1) & 3));
                    const uint32_t from = token_of(vr) * dv2 + 16u * (uint32_t)min(piece, dv / 8 - 1);
                    load_to_lds(bv, mine + L::oV + 1024 * (4 * i + tile), from);
                    load_to_lds(bo, mine + L::oO + 1024 * (4 * i + tile), from);
                }
            }
        }
        const bool there = c_begin + 16 * tile + lm < s_end;
        const uint32_t tk = token_of(16 * tile + lm);
        rowk = there ? tk * dk2 : kNowhere / 2;
        rowv = there ? tk * dv2 : kNowhere / 2;
        const Rsrc bg = view_k(from_gate, 4), bk = view_k(from_k, 2), bq = view_k(from_q, 2);
#pragma unroll
        for (int u = 0; u < 2; ++u) la[u] = fetch<f32x4>(bg, f32_at(rowk, chb(u, g)));
        if constexpr (DT) lat = fetch<float>(bg, f32_at(rowk, tcb(g)));
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            rk[u] = fetch<u32x2>(bk, rowk + chb(u, g));
            rq[u] = fetch<u32x2>(bq, rowk + chb(u, g));
        }
        if constexpr (DT) {
            rkt = fetch<uint16_t>(bk, rowk + tcb(g));
            rqt = fetch<uint16_t>(bq, rowk + tcb(g));
        }
    }
    // ---- gates: prefix sums inside the tile, totals of the tiles ----
    float ex[NG];
    {
        LANE;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) ex[4 * u + e] = la[u][e] * kLog2e;
        if constexpr (DT) ex[8] = row_scan16(fmaxf(lat * kLog2e, kLeastGate2));
        row_scan16x4_least(ex[0], ex[1], ex[2], ex[3], kLeastGate2);
        row_scan16x4_least(ex[4], ex[5], ex[6], ex[7], kLeastGate2);
        if (lm == 15) {
            float *d = my_decay + tile * US;
            *reinterpret_cast<f32x4 *>(d + 4 * g) = f32x4{ex[0], ex[1], ex[2], ex[3]};
            *reinterpret_cast<f32x4 *>(d + 16 + 4 * g) = f32x4{ex[4], ex[5], ex[6], ex[7]};
            if constexpr (DT) d[32 + g] = ex[8];
        }
    }
    meet();
    auto eq_of = [&](int i) { return exp2_fast(fminf(ex[i], kMaxExp2)); };
    auto ek_of = [&](int i) { return exp2_fast(fminf(-ex[i], kMaxExp2)); };
    u32x4 kh, kl;                // k~ of this lane's row, B operand; tail pair
    uint32_t kt = 0;
    {
        LANE;
        // relative to the anchor: -(t0 + t1), -t1, 0, t2 for the four tiles
        const float c0 = tile == 0 ? -1.f : 0.f, c1 = tile < 2 ? -1.f : 0.f, c2 = tile == 3 ? 1.f : 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const float *d = my_decay + 16 * u + 4 * g;
            const f32x4 t0 = *reinterpret_cast<const f32x4 *>(d), t1 = *reinterpret_cast<const f32x4 *>(d + US), t2 = *reinterpret_cast<const f32x4 *>(d + 2 * US);
#pragma unroll
            for (int e = 0; e < 4; ++e) ex[4 * u + e] += c0 * t0[e] + c1 * t1[e] + c2 * t2[e];
        }
        if constexpr (DT) {
            const float *d = my_decay + 32 + g;
            ex[8] += c0 * d[0] + c1 * d[US] + c2 * d[2 * US];
        }
        const int sw = 8 * (lm >> 3);
        uint16_t *krow = s_k + (16 * tile + lm) * RS, *qrow = s_q + (16 * tile + lm) * RS;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            u32x2 qh, ql;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int i = 4 * u + 2 * h;
                SPLIT_PAIR(bf16_lo_as_float(rk[u][h]) * ek_of(i), bf16_hi_as_float(rk[u][h]) * ek_of(i + 1), kh[2 * u + h], kl[2 * u + h]);
                SPLIT_PAIR(bf16_lo_as_float(rq[u][h]) * eq_of(i), bf16_hi_as_float(rq[u][h]) * eq_of(i + 1), qh[h], ql[h]);
            }
            *reinterpret_cast<u32x2 *>(krow + 16 * u + (4 * g ^ sw)) = u32x2{kh[2 * u], kh[2 * u + 1]};
            *reinterpret_cast<u32x2 *>(krow + 32 + 16 * u + (4 * g ^ sw)) = u32x2{kl[2 * u], kl[2 * u + 1]};
            *reinterpret_cast<u32x2 *>(qrow + 16 * u + (4 * g ^ sw)) = qh;
            *reinterpret_cast<u32x2 *>(qrow + 32 + 16 * u + (4 * g ^ sw)) = ql;
        }
        if constexpr (DT) {
            const float kx = bf16_lo_as_float(rkt) * ek_of(8), qx = bf16_lo_as_float(rqt) * eq_of(8);
            const uint32_t khh = pack_bf16(kx, kx), qhh = pack_bf16(qx, qx);
            const float krem = kx - bf16_lo_as_float(khh), qrem = qx - bf16_lo_as_float(qhh);
            const uint32_t kll = pack_bf16(krem, krem);
            *reinterpret_cast<u32x2 *>(krow + 64 + (4 * g ^ sw)) = u32x2{khh, kll};
            *reinterpret_cast<u32x2 *>(qrow + 64 + (4 * g ^ sw)) = u32x2{qhh, pack_bf16(qrem, qrem)};
            kt = (khh & 0xffffu) | (kll << 16);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // (v and dO are in LDS)
    }
    meet();
    {
        LANE;
        if (tile == 0 && lane < US) {        // (the totals of the tiles have been read)
            float *d = my_decay + lane;
            const float m = d[0] + d[US], e = d[2 * US] + d[3 * US];
            d[kDecay * US] = exp2_fast(m + e);
            d[kToAnchor * US] = exp2_fast(m);
            d[kFromAnchor * US] = exp2_fast(e);
            d[kLogDecay * US] = m + e;
        }
    }
    // ---- operand reads ----
#define TR_LANE \
    LANE; \
    const int tr_row = lm >> 2, tr_col = 4 * (lm & 3); \
    const int v_swz = DT ? 0 : 16 * ((2 * g + (tr_row >> 1)) & 3); \
    [[maybe_unused]] auto over_tokens = [&](const uint16_t *rows, int q32, int x) { /* columns 16 x + lm; slot (g, e) = token 32 q32 + 16 (e / 4) + 4 g + e % 4 */ \
        const uint16_t *at = rows + (32 * q32 + 4 * g + tr_row) * HD::NV + ((16 * x + tr_col) ^ v_swz); \
        const u32x2 lo = lds_read_tr(at), hi = lds_read_tr(at + 16 * HD::NV); \
        return u32x4{lo[0], lo[1], hi[0], hi[1]}; \
    }; \
    [[maybe_unused]] auto gated_over_tokens = [&](const uint16_t *rows, int q32, int col) { \
        const uint16_t *at = rows + (32 * q32 + 4 * g + tr_row) * RS + (tr_col ^ (8 * (g >> 1))) + col; \
        const u32x2 lo = lds_read_tr(at), hi = lds_read_tr(at + 16 * RS); \
        return u32x4{lo[0], lo[1], hi[0], hi[1]}; \
    }
    // 8 columns of row 16 t + lm: 8 (4 s + g) .. + 7 (of the last step, 64 .. 71 whatever g)
    auto row_piece = [&](const uint16_t *rows, int t, int s, int lm, int g) {
        const int piece = s < 2 ? 4 * s + g : 8;
        return *reinterpret_cast<const u32x4 *>(rows + (16 * t + lm) * HD::NV + 8 * (DT ? piece : piece ^ (2 * ((lm >> 1) & 3))));
    };
    // the same of this lane's own row, as the other operand: zero where there are no columns
    auto own_piece = [&](const uint16_t *rows, int s, int lm, int g) {
        const bool real = s < 2 ? 8 * (4 * s + g) < dv : (g == 0 && 64 < dv);
        const u32x4 x = row_piece(rows, tile, s, lm, g);
        return u32x4{real ? x[0] : 0, real ? x[1] : 0, real ? x[2] : 0, real ? x[3] : 0};
    };
    auto split4 = [](f32x4 x, u32x4 &h, u32x4 &l, int half) {
        const HiLo a = split_pair_val(x[0], x[1]), c = split_pair_val(x[2], x[3]);
        h[2 * half] = a.hi; h[2 * half + 1] = c.hi;
        l[2 * half] = a.lo; l[2 * half + 1] = c.lo;
    };
    const f32x4 zero4 = f32x4{0.f, 0.f, 0.f, 0.f};

    f32x4 gq[2 + DT], gk[2 + DT], gv[NX];      // dq, dk (transposed: channels 16 ct + 4 g + r of token lm; tail r = 0 hi, 2 lo) and dv (columns 16 x + 4 g + r)
    if constexpr (MODE != kStates) {
#pragma unroll
        for (int i = 0; i < 2 + DT; ++i) gq[i] = gk[i] = zero4;
#pragma unroll
        for (int x = 0; x < NX; ++x) gv[x] = zero4;
        // gradient rows from a matrix of weights over the chunk's tokens (B operand h, l) and the gated rows
        auto add_gated = [&](f32x4 (&acc)[2 + DT], auto frag, u32x4 h, u32x4 l) {
            u32x4 f[4 + DT];
#pragma unroll
            for (int i = 0; i < 4 + DT; ++i) f[i] = frag(16 * i);
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) acc[ct] = mfma(f[ct], h, acc[ct]);
            if constexpr (DT) acc[2] = mfma(f[4], h, acc[2]);
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) acc[ct] = mfma(f[ct], l, acc[ct]);
            if constexpr (DT) acc[2] = mfma(f[4], l, acc[2]);
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) acc[ct] = mfma(f[2 + ct], h, acc[ct]);
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) acc[ct] = mfma(f[2 + ct], l, acc[ct]);
        };
        {   // M_ji = dO_j . v_i of this tile's j and all i <= j: dq~_j = sum_i M_ji k~_i
            TR_LANE;
            u32x4 own[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) own[s] = own_piece(s_o, s, lm, g);
            const int past = 16 * tile + lm - 4 * g;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                u32x4 h, l;
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const int jt = 2 * q + half;
                    f32x4 d = zero4;
#pragma unroll
                    for (int s = 0; s < NS; ++s) d = mfma(row_piece(s_v, jt, s, lm, g), own[s], d);
#pragma unroll
                    for (int r = 0; r < 4; ++r) d[r] = 16 * jt + r <= past ? d[r] : 0.f;
                    split4(d, h, l, half);
                }
                add_gated(gq, [&](int col) { return gated_over_tokens(s_k, q, col); }, h, l);
            }
        }
        {   // A_ji = q~_j . k~_i of this tile's i and all j >= i: dv_i = sum_j A_ji dO_j
            TR_LANE;
            const int sw = 8 * (lm >> 3), first = 16 * tile + lm - 4 * g;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                u32x4 h, l;
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const int jt = 2 * q + half;
                    const uint16_t *row = s_q + (16 * jt + lm) * RS + (4 * g ^ sw);
                    const u32x2 h0 = *reinterpret_cast<const u32x2 *>(row), h1 = *reinterpret_cast<const u32x2 *>(row + 16);
                    const u32x2 l0 = *reinterpret_cast<const u32x2 *>(row + 32), l1 = *reinterpret_cast<const u32x2 *>(row + 48);
                    const u32x4 qh = u32x4{h0[0], h0[1], h1[0], h1[1]}, ql = u32x4{l0[0], l0[1], l1[0], l1[1]};
                    f32x4 d = mfma(qh, kh, zero4);
                    d = mfma(qh, kl, d);
                    d = mfma(ql, kh, d);
                    d = mfma(ql, kl, d);
                    if constexpr (DT) {
                        const u32x2 t = *reinterpret_cast<const u32x2 *>(row + 64);
                        d = mfma(u32x4{t[0], t[1], 0, 0}, u32x4{kt, kt, 0, 0}, d);
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) d[r] = 16 * jt + r >= first ? d[r] : 0.f;
                    split4(d, h, l, half);
                }
#pragma unroll
                for (int x = 0; x < NX; ++x) {
                    const u32x4 f = over_tokens(s_o, q, x);
                    gv[x] = mfma(f, h, gv[x]);
                    gv[x] = mfma(f, l, gv[x]);
                }
            }
        }
        {   // M_ji of this tile's i and all j >= i: dk~_i = sum_j M_ji q~_j
            TR_LANE;
            u32x4 own[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) own[s] = own_piece(s_v, s, lm, g);
            const int first = 16 * tile + lm - 4 * g;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                u32x4 h, l;
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const int jt = 2 * q + half;
                    f32x4 d = zero4;
#pragma unroll
                    for (int s = 0; s < NS; ++s) d = mfma(row_piece(s_o, jt, s, lm, g), own[s], d);
#pragma unroll
                    for (int r = 0; r < 4; ++r) d[r] = 16 * jt + r >= first ? d[r] : 0.f;
                    split4(d, h, l, half);
                }
                add_gated(gk, [&](int col) { return gated_over_tokens(s_q, q, col); }, h, l);
            }
        }
    }
    // ---- the chunk's own states, transposed: U = 2^(b_C - b_m) K~^T V and, of the adjoint recurrence, 2^(b_m) Q~^T dO.  A wave has column
    // tile `tile` of both, and of column tile 4 sixteen channels of one ----
    f32x4 acc[2][2 + DT], acc4[1 + DT];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int i = 0; i < 2 + DT; ++i) acc[m][i] = zero4;
#pragma unroll
    for (int i = 0; i < 1 + DT; ++i) acc4[i] = zero4;
    {
        TR_LANE;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const uint16_t *rows = m ? s_o : s_v, *gated = m ? s_q : s_k;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const u32x4 f = over_tokens(rows, q, tile);
#pragma unroll
                for (int ct = 0; ct < 2; ++ct) acc[m][ct] = mfma(f, gated_over_tokens(gated, q, 16 * ct), acc[m][ct]);
                if constexpr (DT) acc[m][2] = mfma(f, gated_over_tokens(gated, q, 64), acc[m][2]);
#pragma unroll
                for (int ct = 0; ct < 2; ++ct) acc[m][ct] = mfma(f, gated_over_tokens(gated, q, 32 + 16 * ct), acc[m][ct]);
            }
        }
        if constexpr (NX == 5) {
            const uint16_t *rows = tile & 2 ? s_o : s_v, *gated = tile & 2 ? s_q : s_k;
            const int col = 16 * (tile & 1);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const u32x4 f = over_tokens(rows, q, 4);
                acc4[0] = mfma(f, gated_over_tokens(gated, q, col), acc4[0]);
                if constexpr (DT) acc4[DT] = mfma(f, gated_over_tokens(gated, q, 64), acc4[DT]);
                acc4[0] = mfma(f, gated_over_tokens(gated, q, 32 + col), acc4[0]);
            }
        }
    }
    meet();      // (k~ and q~ have been read)
    {
        LANE;
        auto leave = [&](int m, int n0, int ct, f32x4 a) {
            const int c = 16 * ct + lm;
            float *u = reinterpret_cast<float *>(m ? s_q : s_k) + c * HD::NV + n0 + 4 * g;
            *reinterpret_cast<f32x4 *>(u) = a * my_decay[(m ? kToAnchor : kFromAnchor) * US + c];
        };
        auto leave_tail = [&](int m, int n0, f32x4 a) {      // columns lm: channel 32 + lm / 4, hi in lm % 4 = 0, 1, lo in 2, 3
#pragma unroll
            for (int r = 0; r < 4; ++r) a[r] += dpp_move<0x4E, 0xF, true>(a[r]);
            const int c = 32 + (lm >> 2);
            float *u = reinterpret_cast<float *>(m ? s_q : s_k) + c * HD::NV + n0 + 4 * g;
            if ((lm & 3) == 0) *reinterpret_cast<f32x4 *>(u) = a * my_decay[(m ? kToAnchor : kFromAnchor) * US + c];
        };
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            leave(m, 16 * tile, 0, acc[m][0]);
            leave(m, 16 * tile, 1, acc[m][1]);
            if constexpr (DT) leave_tail(m, 16 * tile, acc[m][2]);
        }
        if constexpr (NX == 5) {
            if (64 + 4 * g < HD::NV) {
                leave(tile >> 1, 64, tile & 1, acc4[0]);
            }
            if constexpr (DT) {
                f32x4 a = acc4[DT];
#pragma unroll
                for (int r = 0; r < 4; ++r) a[r] += dpp_move<0x4E, 0xF, true>(a[r]);
                const int c = 32 + (lm >> 2);
                float *u = reinterpret_cast<float *>(tile >> 1 ? s_q : s_k) + c * HD::NV + 64 + 4 * g;
                if ((lm & 3) == 0 && 64 + 4 * g < HD::NV && (tile & 1) == 0)
                    *reinterpret_cast<f32x4 *>(u) = a * my_decay[(tile >> 1 ? kToAnchor : kFromAnchor) * US + c];
            }
        }
    }
    __syncthreads();
    // ---- a thread's piece of the states: channel w + 16 (lane / pieces of a channel), four columns ----
    constexpr int QN = HD::NV / 4;
    int qc, qn;
    bool owns;
    {
        const int lane = recompute_per_chunk(threadIdx.x) & 63;
        const int slot = lane / QN;
        owns = slot < 3 && w + 16 * slot < L::kDk;
        qc = owns ? w + 16 * slot : w;
        qn = 4 * (lane - slot * QN);
    }
    f32x4 u[NC], h[NC];
    float dl[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        u[c] = *reinterpret_cast<const f32x4 *>(smem + c * L::kOne + 4 * (qc * HD::NV + qn));
        h[c] = *reinterpret_cast<const f32x4 *>(smem + c * L::kOne + L::oQ + 4 * (qc * HD::NV + qn));
        dl[c] = s_decay[(4 * c + kDecay) * US + qc];
    }
    const bool real = owns && qc < dk && qn < dv;
    if (!real) {       // (columns past dv hold copies of others)
#pragma unroll
        for (int c = 0; c < NC; ++c) u[c] = h[c] = zero4;
    }
    const uint32_t ne4 = 4u * (uint32_t)(dk * dv);
    const uint32_t at = real ? 4u * (uint32_t)(qc * dv + qn) : kNowhere;
    auto view_s = [&]() { return view(ARG->ws_state + (size_t)afresh(bh) * nspans * dk * dv, (uint32_t)nspans * ne4); };
    auto view_g = [&]() { return view(ARG->ws_gstate + (size_t)afresh(bh) * nspans * dk * dv, (uint32_t)nspans * ne4); };
    if constexpr (MODE == kStates) {
        f32x4 S = zero4, G = zero4;
#pragma unroll
        for (int c = 0; c < NC; ++c) S = dl[c] * S + u[c];
#pragma unroll
        for (int c = NC - 1; c >= 0; --c) G = dl[c] * G + h[c];
        const Rsrc bs = view_s(), bg = view_g();
        put(bs, at == kNowhere ? kNowhere : at + (uint32_t)sp * ne4, S);
        put(bg, at == kNowhere ? kNowhere : at + (uint32_t)sp * ne4, G);
        if (tid < dk) {
            float sum = 0.f;
#pragma unroll
            for (int c = 0; c < NC; ++c) sum += s_decay[(4 * c + kLogDecay) * US + tid];
            ARG->ws_lgam[((size_t)bh * nspans + sp) * dk + tid] = sum * kLn2;
        }
        return;
    }
    f32x4 S = zero4, G = zero4;
    if constexpr (MODE == kOutputs) {
        // the states that enter the span from either side, nearest spans first, until what is left would not show (2^-40; counted
        // from behind the nearest spans that were all zero)
        const float *lg = ARG->ws_lgam + (size_t)bh * nspans * dk + min(qc, dk - 1);
        auto chain = [&](Rsrc b, f32x4 &X, int first, int step, int count) {
            float wl = 0.f, ref = 0.f;
            constexpr int N = 4;
            for (int i = 0; i < count && __any(real && wl > ref - 40.f); i += N) {
                f32x4 x[N];
                float d[N];
#pragma unroll
                for (int n = 0; n < N; ++n) {
                    const int r = first + step * min(i + n, count - 1);
                    x[n] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(b, (int)at, (int)((uint32_t)r * ne4), 0));
                    d[n] = lg[r * dk];
                }
#pragma unroll
                for (int n = 0; n < N; ++n) {
                    if (i + n < count) {
                        X += exp2_fast(wl) * x[n];
                        wl += d[n] * kLog2e;
                        ref = X[0] == 0.f && X[1] == 0.f && X[2] == 0.f && X[3] == 0.f ? wl : ref;
                    }
                }
            }
        };
        if (sp > 0) chain(view_s(), S, sp - 1, -1, sp);
        if (sp + 1 < nspans) chain(view_g(), G, sp + 1, 1, nspans - 1 - sp);
    }
    __syncthreads();      // (all states have been read)
    {
        auto leave = [&](int region, int c, f32x4 x) {      // hi rows, then lo rows
            u32x2 a, b;
            SPLIT_PAIR(x[0], x[1], a[0], b[0]);
            SPLIT_PAIR(x[2], x[3], a[1], b[1]);
            uint16_t *p = reinterpret_cast<uint16_t *>(smem + c * L::kOne + region) + qc * PS + qn;
            if (owns) {
                *reinterpret_cast<u32x2 *>(p) = a;
                *reinterpret_cast<u32x2 *>(p + L::kDk * PS) = b;
            }
        };
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            leave(0, c, S * s_decay[(4 * c + kToAnchor) * US + qc]);
            S = dl[c] * S + u[c];
            u[c] = S;                         // the state that leaves the chunk
        }
#pragma unroll
        for (int c = NC - 1; c >= 0; --c) {
            leave(L::oQ, c, G * s_decay[(4 * c + kFromAnchor) * US + qc]);
            const f32x4 z4 = u[c] * G;
            float z = (z4[0] + z4[1]) + (z4[2] + z4[3]);
            // sum over the pieces of the channel, which neighbouring lanes hold
            if constexpr (QN == 18) {
                z += __shfl_down(z, 9);
                z += __shfl_down(z, 3) + __shfl_down(z, 6);
                z += __shfl_down(z, 1) + __shfl_down(z, 2);
            } else {
                z += __shfl_down(z, 8);
                z += __shfl_down(z, 4);
                z += __shfl_down(z, 2);
                z += __shfl_down(z, 1);
            }
            if (owns && qn == 0) s_z[c * US + qc] = z;
            G = dl[c] * G + h[c];
        }
    }
    {
        LANE;
        const Rsrc bk = view_k(ARG->k, 2), bq = view_k(ARG->q, 2);       // (again, for the gate gradient)
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            rk[x] = fetch<u32x2>(bk, rowk + chb(x, g));
            rq[x] = fetch<u32x2>(bq, rowk + chb(x, g));
        }
        if constexpr (DT) {
            rkt = fetch<uint16_t>(bk, rowk + tcb(g));
            rqt = fetch<uint16_t>(bq, rowk + tcb(g));
        }
    }
    __syncthreads();
    {
        TR_LANE;
        // ---- dq~ += P dO, dk~ += Gp v (P = 2^(b_m) S, Gp = 2^(b_C - b_m) G): rows of the split states over their columns ----
        auto state_rows = [&](const uint16_t *p, int row, int s) { return *reinterpret_cast<const u32x4 *>(p + row * PS + 8 * (s < 2 ? 4 * s + g : 8)); };
        auto add_state = [&](f32x4 (&a)[2 + DT], const uint16_t *p, const uint16_t *rows) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const u32x4 own = own_piece(rows, s, lm, g);
#pragma unroll
                for (int ct = 0; ct < 2; ++ct) a[ct] = mfma(state_rows(p, 16 * ct + lm, s), own, a[ct]);
                if constexpr (DT) a[2] = mfma(state_rows(p, 32 + (lm >> 2) + ((lm & 2) ? L::kDk : 0), s), own, a[2]);
#pragma unroll
                for (int ct = 0; ct < 2; ++ct) a[ct] = mfma(state_rows(p + L::kDk * PS, 16 * ct + lm, s), own, a[ct]);
            }
        };
        add_state(gq, s_k, s_o);
        add_state(gk, s_q, s_v);
        // ---- dv += k~ Gp: the split state over its channels (slot (g, e) = channel 16 (e / 4) + 4 g + e % 4) ----
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            auto over_channels = [&](const uint16_t *p) {
                const uint16_t *at = p + (4 * g + tr_row) * PS + 16 * x + tr_col;
                const u32x2 lo = lds_read_tr(at), hi = lds_read_tr(at + 16 * PS);
                return u32x4{lo[0], lo[1], hi[0], hi[1]};
            };
            const u32x4 ph = over_channels(s_q), pl = over_channels(s_q + L::kDk * PS);
            gv[x] = mfma(ph, kh, gv[x]);
            gv[x] = mfma(ph, kl, gv[x]);
            gv[x] = mfma(pl, kh, gv[x]);
            gv[x] = mfma(pl, kl, gv[x]);
            if constexpr (DT) {
                const uint16_t *p = s_q + (32 + g) * PS + min(16 * x + lm, HD::NV - 1);
                const uint32_t hi = p[0], lo = p[L::kDk * PS];
                gv[x] = mfma(u32x4{hi | hi << 16, lo | lo << 16, 0, 0}, u32x4{kt, kt, 0, 0}, gv[x]);
            }
        }
        const Rsrc b_dv = view_v(ARG->dv_grad, 4);
#pragma unroll
        for (int x = 0; x < NX; ++x)
            put(b_dv, 4 * g + 16 * x < dv ? f32_at(rowv, 8u * (uint32_t)g + 32u * (uint32_t)x) : kNowhere, gv[x]);
        // ---- dq = 2^(b - b_m) dq~, dk = 2^(b_m - b) dk~; d log alpha = sum of q dq - k dk from the token on ----
        float x[NG];
        const Rsrc b_dq = view_k(ARG->dq, 4), b_dk = view_k(ARG->dk_grad, 4);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            f32x4 a, b;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                a[r] = gq[c][r] * eq_of(4 * c + r);
                b[r] = gk[c][r] * ek_of(4 * c + r);
                const float qv = r & 1 ? bf16_hi_as_float(rq[c][r >> 1]) : bf16_lo_as_float(rq[c][r >> 1]);
                const float kv = r & 1 ? bf16_hi_as_float(rk[c][r >> 1]) : bf16_lo_as_float(rk[c][r >> 1]);
                x[4 * c + r] = qv * a[r] - kv * b[r];
            }
            put(b_dq, f32_at(rowk, chb(c, g)), a);
            put(b_dk, f32_at(rowk, chb(c, g)), b);
        }
        if constexpr (DT) {
            const float a = (gq[2][0] + gq[2][2]) * eq_of(8), b = (gk[2][0] + gk[2][2]) * ek_of(8);
            x[8] = bf16_lo_as_float(rqt) * a - bf16_lo_as_float(rkt) * b;
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, a), b_dq, (int)f32_at(rowk, tcb(g)), 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, b), b_dk, (int)f32_at(rowk, tcb(g)), 0, 0);
            x[8] = row_suffix16(x[8]);
        }
        row_suffix16x4(x[0], x[1], x[2], x[3]);
        row_suffix16x4(x[4], x[5], x[6], x[7]);
        if (lm == 0) {
            float *d = my_decay + tile * US;
            *reinterpret_cast<f32x4 *>(d + 4 * g) = f32x4{x[0], x[1], x[2], x[3]};
            *reinterpret_cast<f32x4 *>(d + 16 + 4 * g) = f32x4{x[4], x[5], x[6], x[7]};
            if constexpr (DT) d[32 + g] = x[8];
        }
        meet();
        // the later tiles, and what lies behind the chunk
        const float l1 = tile < 1 ? 1.f : 0.f, l2 = tile < 2 ? 1.f : 0.f, l3 = tile < 3 ? 1.f : 0.f;
        const float *z = s_z + (w >> 2) * US;
        const Rsrc b_la = view_k(ARG->dlog_alpha, 4);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float *d = my_decay + 16 * c + 4 * g;
            f32x4 a = *reinterpret_cast<const f32x4 *>(z + 16 * c + 4 * g);
            a += l3 * *reinterpret_cast<const f32x4 *>(d + 3 * US);
            a += l2 * *reinterpret_cast<const f32x4 *>(d + 2 * US);
            a += l1 * *reinterpret_cast<const f32x4 *>(d + US);
            put(b_la, f32_at(rowk, chb(c, g)), f32x4{x[4 * c], x[4 * c + 1], x[4 * c + 2], x[4 * c + 3]} + a);
        }
        if constexpr (DT) {
            const float *d = my_decay + 32 + g;
            const float a = x[8] + (((z[32 + g] + l3 * d[3 * US]) + l2 * d[2 * US]) + l1 * d[US]);
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, a), b_la, (int)f32_at(rowk, tcb(g)), 0, 0);
        }
    }
}

template <typename HD, int MODE>
hipError_t launch_one(const BackParams &p, hipStream_t stream) {
    auto kernel = chunk_back_kernel<HD, MODE>;
    static std::atomic<bool> configured[kMaxDevices] = {};  // per instantiation and device
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), BLayout<HD>::kBytes, configured);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(p.B * p.H * p.nspans)), dim3(NT), BLayout<HD>::kBytes, stream, p);
    return hipGetLastError();
}

template <typename HD>
hipError_t launch_heads(const BackParams &p, hipStream_t stream) {
    if (p.nspans == 1) return launch_one<HD, kWhole>(p, stream);
    const hipError_t e = launch_one<HD, kStates>(p, stream);
    return e != hipSuccess ? e : launch_one<HD, kOutputs>(p, stream);
}

}  // namespace

hipError_t launch_onepass_back(const BackParams &p, hipStream_t stream) {
    if (p.dk <= 32 && p.dv <= 64) return launch_heads<HeadsS>(p, stream);
    return launch_heads<HeadsXL>(p, stream);
}

}  // namespace gla
