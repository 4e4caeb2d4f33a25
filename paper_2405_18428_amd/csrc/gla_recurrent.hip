// Token-by-token fp32 engine for the spans of the GLA recurrence
// (DiG paper, Sec. 3.1 Eq. (attn_gla) rows 1-3; the value-side gate beta of Eq. (gate_gla_2) is optional).
//
// There is no factorised decay here: every step multiplies the state by the gates as they are, so any gate value
// (alpha down to 0) is exact.  The engine serves fp32 inputs, odd head sizes, and what the MFMA engines do not cover.
//
// token_span_kernel: S_s = (a_s^T b_s) * S_{s-1} + k_s^T v_s with a read along the rows (o_s = q_s S_s) or, for the
// backward pass, along the value columns (r_s[c] = sum_n S_s[c,n] w_s[n]); the second is the first on the transposed
// state, so one kernel does both: the contracted axis is called R (rows k and q, gate a), the other one C (rows v,
// gate b).  A work-group owns 16 columns of the C axis, since columns never meet, and walks its span in rounds of
// kSteps scan steps per wave:
//   1. every wave walks its steps from a zero state and leaves the local state and the product of its gates in LDS;
//   2. after a barrier every wave chains the local states of the waves before it, S = (A^T B) * S + U, walks its steps
//      again from that state and writes their results.
// A serial walk is bound by the latency of one step (LDS reads, two dependent multiply-adds): cut into waves, a round
// costs two walks of kSteps steps instead of one of all its steps.  Lane = (8 groups of the R axis) x (8 column
// pairs): a step costs one 16-byte LDS read per 4 channels and tensor for 2 * RP / 8 state elements, and the read's
// sum over R is three DPP adds among neighbouring lanes.
// Measured on MI355X, fp32 inputs, against one thread per column walking the span with a branch per channel and step:
// 2 sequences of 256 steps at 32 / 64 channels 300 us (three launches) -> 13 us (one); 16 sequences of 16384 steps at
// 36 / 72 3.0 ms -> 0.83 ms (bound by the vector units: 3 instructions per state element and step, twice); forward and
// backward of 48 sequences of 256 steps 0.79 ms -> 0.074 ms.
#include "gla_common.h"

namespace gla {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;

template <typename T> __device__ inline float load_elem(const void *base, size_t idx);
template <> __device__ inline float load_elem<float>(const void *base, size_t idx) {
    return static_cast<const float *>(base)[idx];
}
template <> __device__ inline float load_elem<uint16_t>(const void *base, size_t idx) {
    return bf16_bits_to_float(static_cast<const uint16_t *>(base)[idx]);
}
template <typename T> __device__ inline void store_elem(void *base, size_t idx, float x);
template <> __device__ inline void store_elem<float>(void *base, size_t idx, float x) {
    static_cast<float *>(base)[idx] = x;
}
template <> __device__ inline void store_elem<uint16_t>(void *base, size_t idx, float x) {
    static_cast<uint16_t *>(base)[idx] = float_to_bf16_bits(x);
}

// log gate from its pre-activation (Eqs. (gate_gla), (gate_gla_2)): logsigmoid(z) / tau
__device__ inline float log_gate(float z, float inv_tau) { return (fminf(z, 0.f) - log1pf(expf(-fabsf(z)))) * inv_tau; }

constexpr int kCols = 16;      // columns of the C axis per work-group

// The contracted axis: 8 groups of PER channels, padded to GS in LDS (8- and 16-byte reads); RP = 8 * GS positions.
// ROWREAD: that axis is the value side (backward); BETA: gates on both axes; STATE: the span-state pass (walk 1 only,
// no q).  Most waves per group: what the staged rows and the local states leave room for in 160 KB of LDS; a launch
// takes no more than its spans have steps for, so that groups of short sequences share a compute unit.
template <int GS, int PER, bool ROWREAD, bool BETA, bool STATE>
struct TokenCfg {
    static constexpr bool kGateR = ROWREAD ? BETA : true, kGateC = ROWREAD ? true : BETA;
    static constexpr int RP = 8 * GS;
    static constexpr int kMaxWaves = GS == 4 ? 16 : (GS == 16 && BETA ? 4 : 8);
    static constexpr int kSteps = GS == 16 || (GS == 4 && BETA) ? 8 : 16;
    static constexpr int kRound = kMaxWaves * kSteps;
    // LDS, in floats.  The staged rows of a wave, private to it:
    static constexpr int oA = 0;
    static constexpr int oK = oA + (kGateR ? kSteps * RP : 0);
    static constexpr int oQ = oK + kSteps * RP;
    static constexpr int oV = oQ + (STATE ? 0 : kSteps * RP);
    static constexpr int oB = oV + kSteps * kCols;
    static constexpr int kWave = oB + (kGateC ? kSteps * kCols : 0);
    // after those of all waves: local states [wave][PER][lane][2], gate products [wave][RP] and [wave][kCols], and the
    // state entering the next round [PER][lane][2]
    static constexpr int kLocal = 64 * 2 * PER;
    static constexpr int bytes(int waves) { return (waves * (kWave + kLocal + RP + kCols) + kLocal) * 4; }
    static_assert(bytes(kMaxWaves) <= 160 * 1024, "one group must fit a compute unit");
    static_assert(2 * 64 <= kLocal, "the log sums reuse the local states' room");
};

// sum over the 8 neighbouring lanes that share a column pair (all of them get it)
__device__ inline float sum_group8(float x) {
    auto mv = [](float y, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, y), decltype(ctrl)::value, 0xF, 0xF, true));
    };
    x += mv(x, std::integral_constant<int, 0xB1>{});    // quad_perm [1,0,3,2]
    x += mv(x, std::integral_constant<int, 0x4E>{});    // quad_perm [2,3,0,1]
    x += mv(x, std::integral_constant<int, 0x141>{});   // row_half_mirror: the other quad of the eight
    return x;
}

// w, r: ROWREAD only (w laid out like v, r fp32 laid out like k)
template <int GS, int PER, bool ROWREAD, bool BETA, bool STATE, typename TIn, typename TOut>
__global__ __launch_bounds__((TokenCfg<GS, PER, ROWREAD, BETA, STATE>::kMaxWaves * 64)) void token_span_kernel(Params p, const void *w, float *r_out) {
    using C = TokenCfg<GS, PER, ROWREAD, BETA, STATE>;
    constexpr int TS = C::kSteps, RP = C::RP;
    extern __shared__ __attribute__((aligned(16))) float smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cg = lane & 7, cp = lane >> 3;
    const int NW = blockDim.x >> 6, round = NW * TS;
    const int nr = ROWREAD ? p.dv : p.dk, nc = ROWREAD ? p.dk : p.dv;
    const int seq_span = blockIdx.x;          // (batch, head) and span on grid.x, whose limit is 2^31 - 1
    const int c0 = blockIdx.y * kCols;
    const int bh = seq_span / p.nspans, sp = seq_span - bh * p.nspans;
    const int s_begin = sp * p.span_len, s_end = min(p.T, s_begin + p.span_len);
    const size_t base_r = ROWREAD ? slab_v(p, bh) : slab_k(p, bh), base_c = ROWREAD ? slab_k(p, bh) : slab_v(p, bh);
    const size_t st_r = (size_t)(ROWREAD ? p.st_v : p.st_k), st_c = (size_t)(ROWREAD ? p.st_k : p.st_v);
    const void *kr = ROWREAD ? p.v : p.k, *qr = ROWREAD ? w : p.q, *vc = ROWREAD ? p.k : p.v;
    const float *gate_r = ROWREAD ? p.log_beta : p.log_alpha, *gate_c = ROWREAD ? p.log_alpha : p.log_beta;
    const void *z_r = ROWREAD ? p.z_beta : p.z_gate, *z_c = ROWREAD ? p.z_gate : p.z_beta;

    float *own = smem + wv * C::kWave;
    f32x2 *s_u = reinterpret_cast<f32x2 *>(smem + NW * C::kWave);
    float *s_gr = smem + NW * (C::kWave + C::kLocal), *s_gc = s_gr + NW * RP;
    f32x2 *s_base = reinterpret_cast<f32x2 *>(s_gc + NW * kCols);
    // this lane's PER channels of a row of RP positions
    auto read_row = [&](const float *row, float (&x)[PER]) {
#pragma unroll
        for (int i = 0; i + 4 <= PER; i += 4) {
            const f32x4 t = *reinterpret_cast<const f32x4 *>(row + cg * GS + i);
#pragma unroll
            for (int e = 0; e < 4; ++e) x[i + e] = t[e];
        }
#pragma unroll
        for (int i = PER / 4 * 4; i < PER; ++i) x[i] = row[cg * GS + i];
    };

    // state element (i, x) of a lane: R channel cg * PER + i, column c0 + 2 cp + x
    const int my_col = c0 + 2 * cp;
    auto state_index = [&](int i, int x) {
        const size_t rr = cg * PER + i, cc = my_col + x;
        return ROWREAD ? cc * nr + rr : rr * nc + cc;      // [dk][dv] either way
    };
    float base[PER][2];
    {
        const float *s0 = nullptr;
        if (!STATE) {
            if (p.nspans > 1) s0 = p.ws_state + (size_t)seq_span * p.dk * p.dv;
            else if (p.initial_state != nullptr) s0 = p.initial_state + (size_t)bh * p.dk * p.dv;
        }
#pragma unroll
        for (int i = 0; i < PER; ++i)
#pragma unroll
            for (int x = 0; x < 2; ++x)
                base[i][x] = s0 != nullptr && cg * PER + i < nr && my_col + x < nc ? s0[state_index(i, x)] : 0.f;
    }

    float S[PER][2], a[PER];
    float lsum_r = 0.f, lsum_c = 0.f;      // STATE: summed log gates of the elements this lane stages

    // one scan step of this wave's state
    auto advance = [&](int j) {
        if constexpr (C::kGateR) read_row(own + C::oA + j * RP, a);
        f32x2 b = f32x2{1.f, 1.f};
        if constexpr (C::kGateC) b = *reinterpret_cast<const f32x2 *>(own + C::oB + j * kCols + 2 * cp);
        const f32x2 v = *reinterpret_cast<const f32x2 *>(own + C::oV + j * kCols + 2 * cp);
        float k[PER];
        read_row(own + C::oK + j * RP, k);
#pragma unroll
        for (int i = 0; i < PER; ++i)
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const float g = C::kGateR ? (C::kGateC ? a[i] * b[x] : a[i]) : b[x];
                S[i][x] = fmaf(g, S[i][x], k[i] * v[x]);
            }
        return b;
    };

    for (int t0 = s_begin; t0 < s_end; t0 += round) {
        // ---- stage this wave's rows (a step past the span leaves the state alone: gates 1, k = 0) ----
        const int active = min(NW, (s_end - t0 + TS - 1) / TS);      // waves with steps in this round
        int tok = -1, tok_g = -1;
        if (lane < TS) {
            const int s = t0 + wv * TS + lane;
            if (s < s_end) {
                tok = scan_token(p.scan_dir, s, p.T, p.grid_h, p.grid_w);
                tok_g = p.gate_shift ? scan_token(p.scan_dir, max(s - 1, 0), p.T, p.grid_h, p.grid_w) : tok;
            }
        }
        if (wv < active) {
            constexpr int N = TS * RP / 64;
            float k[N], q[N], g[N];
#pragma unroll
            for (int m = 0; m < N; ++m) {
                const int idx = lane + 64 * m, j = idx / RP, pos = idx % RP, c = pos / GS * PER + pos % GS;
                const int n = __shfl(tok, j), ng = __shfl(tok_g, j);
                const bool ok = n >= 0 && pos % GS < PER && c < nr;
                const size_t e = base_r + (ok ? (size_t)n * st_r + c : 0);       // (the slab's first element otherwise)
                k[m] = load_elem<TIn>(kr, e);
                k[m] = ok ? k[m] : 0.f;
                if constexpr (!STATE) {
                    q[m] = load_elem<TIn>(qr, e);
                    q[m] = ok ? q[m] : 0.f;
                }
                if constexpr (C::kGateR) {
                    const size_t eg = base_r + (ok ? (size_t)ng * st_r + c : 0);
                    g[m] = z_r != nullptr ? log_gate(load_elem<TIn>(z_r, eg), p.inv_tau) : gate_r[eg];
                    g[m] = ok ? g[m] : 0.f;
                }
            }
            constexpr int NV = TS * kCols / 64;
            float v[NV], b[NV];
#pragma unroll
            for (int m = 0; m < NV; ++m) {
                const int idx = lane + 64 * m, j = idx / kCols, c = c0 + idx % kCols;
                const int n = __shfl(tok, j), ng = __shfl(tok_g, j);
                const bool ok = n >= 0 && c < nc;
                v[m] = load_elem<TIn>(vc, base_c + (ok ? (size_t)n * st_c + c : 0));
                v[m] = ok ? v[m] : 0.f;
                if constexpr (C::kGateC) {
                    const size_t eg = base_c + (ok ? (size_t)ng * st_c + c : 0);
                    b[m] = z_c != nullptr ? log_gate(load_elem<TIn>(z_c, eg), p.inv_tau) : gate_c[eg];
                    b[m] = ok ? b[m] : 0.f;
                }
            }
#pragma unroll
            for (int m = 0; m < N; ++m) {
                own[C::oK + lane + 64 * m] = k[m];
                if constexpr (!STATE) own[C::oQ + lane + 64 * m] = q[m];
                if constexpr (C::kGateR) {
                    if constexpr (STATE) lsum_r += g[m];
                    own[C::oA + lane + 64 * m] = expf(g[m]);
                }
            }
#pragma unroll
            for (int m = 0; m < NV; ++m) {
                own[C::oV + lane + 64 * m] = v[m];
                if constexpr (C::kGateC) {
                    if constexpr (STATE) lsum_c += b[m];
                    own[C::oB + lane + 64 * m] = expf(b[m]);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();

            // ---- 1. the local state of the wave's steps and the product of its gates ----
            if (STATE || wv + 1 < active) {
                float gr[PER], gc[2] = {1.f, 1.f};
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    gr[i] = 1.f;
                    S[i][0] = S[i][1] = 0.f;
                }
#pragma unroll 4      // (the whole walk unrolled is more code than a launch of a few groups takes time to fetch)
                for (int j = 0; j < TS; ++j) {
                    const f32x2 bj = advance(j);
                    if constexpr (C::kGateR) {
#pragma unroll
                        for (int i = 0; i < PER; ++i) gr[i] *= a[i];
                    }
                    if constexpr (C::kGateC) {
                        gc[0] *= bj[0];
                        gc[1] *= bj[1];
                    }
                }
#pragma unroll
                for (int i = 0; i < PER; ++i) s_u[(wv * PER + i) * 64 + lane] = f32x2{S[i][0], S[i][1]};
                if (C::kGateR && cp == 0) {
#pragma unroll
                    for (int i = 0; i < PER; ++i) s_gr[wv * RP + cg * GS + i] = gr[i];
                }
                if (C::kGateC && cg == 0) {
                    s_gc[wv * kCols + 2 * cp] = gc[0];
                    s_gc[wv * kCols + 2 * cp + 1] = gc[1];
                }
            }
        }
        __syncthreads();
        // ---- 2. the state entering this wave's steps; STATE: wave 0 carries the span's state over the rounds ----
        const int upto = STATE ? (wv == 0 ? active : 0) : min(wv, active);
        for (int u = 0; u < upto; ++u) {
            float gr[PER];
            f32x2 gc = f32x2{1.f, 1.f};
            if constexpr (C::kGateR) read_row(s_gr + u * RP, gr);
            if constexpr (C::kGateC) gc = *reinterpret_cast<const f32x2 *>(s_gc + u * kCols + 2 * cp);
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const f32x2 t = s_u[(u * PER + i) * 64 + lane];
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    const float g = C::kGateR ? (C::kGateC ? gr[i] * gc[x] : gr[i]) : gc[x];
                    base[i][x] = fmaf(g, base[i][x], t[x]);
                }
            }
        }
        if constexpr (!STATE) {
            if (wv < active) {
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    S[i][0] = base[i][0];
                    S[i][1] = base[i][1];
                }
                for (int j0 = 0; j0 < TS; j0 += 8) {
                    f32x2 keep = f32x2{0.f, 0.f};      // step j0 + cg of this lane's column pair
#pragma unroll 4
                    for (int j = 0; j < 8; ++j) {
                        advance(j0 + j);
                        float o0 = 0.f, o1 = 0.f, q[PER];
                        read_row(own + C::oQ + (j0 + j) * RP, q);
#pragma unroll
                        for (int i = 0; i < PER; ++i) {
                            o0 = fmaf(q[i], S[i][0], o0);
                            o1 = fmaf(q[i], S[i][1], o1);
                        }
                        o0 = sum_group8(o0);
                        o1 = sum_group8(o1);
                        keep = cg == j ? f32x2{o0, o1} : keep;
                    }
                    const int n = __shfl(tok, j0 + cg);
#pragma unroll
                    for (int x = 0; x < 2; ++x) {
                        if (n >= 0 && my_col + x < nc) {
                            const size_t e = base_c + (size_t)n * st_c + my_col + x;
                            float o = keep[x];
                            if constexpr (ROWREAD) {
                                r_out[e] = o;
                            } else {
                                if (p.accumulate) o += static_cast<const float *>(p.out)[e];   // fp32 rows (host checks)
                                store_elem<TOut>(p.out, e, o);
                            }
                        }
                    }
                }
            }
            // the state after the round's last step: for the next round, or the caller
            if (wv == active - 1) {
                if (t0 + round < s_end) {
#pragma unroll
                    for (int i = 0; i < PER; ++i) s_base[i * 64 + lane] = f32x2{S[i][0], S[i][1]};
                } else if (!ROWREAD && p.nspans == 1 && p.final_state != nullptr) {
                    float *f = p.final_state + (size_t)bh * p.dk * p.dv;
#pragma unroll
                    for (int i = 0; i < PER; ++i)
#pragma unroll
                        for (int x = 0; x < 2; ++x)
                            if (cg * PER + i < nr && my_col + x < nc) f[state_index(i, x)] = S[i][x];
                }
            }
        }
        __syncthreads();      // the local states and gate products are read, the next round's state is there
        if (!STATE && t0 + round < s_end) {
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const f32x2 t = s_base[i * 64 + lane];
                base[i][0] = t[0];
                base[i][1] = t[1];
            }
        }
    }

    if constexpr (STATE) {
        // U of this span and the log of its total decay
        if (wv == 0) {
            float *u = p.ws_state + (size_t)seq_span * p.dk * p.dv;
#pragma unroll
            for (int i = 0; i < PER; ++i)
#pragma unroll
                for (int x = 0; x < 2; ++x)
                    if (cg * PER + i < nr && my_col + x < nc) u[state_index(i, x)] = base[i][x];
        }
        // (a lane staged position lane % RP of the R axis and column lane % kCols of the C axis in every step)
        float *s_l = smem + NW * C::kWave;
        s_l[tid] = lsum_r;
        if constexpr (C::kGateC) s_l[NW * 64 + tid] = lsum_c;
        __syncthreads();
        if (c0 == 0 && tid < nr) {     // (nr <= 64 threads there are)
            float t = 0.f;
            for (int i = tid / PER * GS + tid % PER; i < NW * 64; i += RP) t += s_l[i];
            p.ws_lgam[(size_t)seq_span * p.dk + tid] = t;
        }
        if (C::kGateC && tid < kCols && c0 + tid < nc) {
            float t = 0.f;
            for (int i = tid; i < NW * 64; i += kCols) t += s_l[NW * 64 + i];
            p.ws_lgam_b[(size_t)seq_span * p.dv + c0 + tid] = t;
        }
    }
}

// Output pass with the epilogue (Eq. (attn_gla) rows 4-5 up to the projection): y = Swish(r) * LN(o) needs a token's
// whole row of o, so one work-group walks the span with thread n owning column n of the state in registers; q, k and
// alpha of a tile of tokens are staged in LDS and read as wave-wide broadcasts.  RP = padded number of key channels:
// the padding is staged as zeros, so a step has no branch per channel.  Without the epilogue it takes the sequences of a
// few steps (few_steps).
constexpr int kThreads = 128;  // >= kMaxDv
constexpr int kTile = 16;      // tokens staged per round

template <int RP, typename TIn, typename TOut, bool BETA>
__global__ __launch_bounds__(kThreads) void column_span_kernel(Params p) {
    __shared__ float s_b[BETA ? kTile : 1][BETA ? kMaxDv : 1];   // log_beta rows of the tile
    __shared__ __attribute__((aligned(16))) float s_q[kTile][RP], s_k[kTile][RP], s_a[kTile][RP];
    __shared__ float s_v[kTile][kMaxDv];
    __shared__ float s_o[kTile][kMaxDv];   // rows of o awaiting the epilogue
    __shared__ int s_tok[kTile];

    const int tid = threadIdx.x;
    const int bh = blockIdx.x / p.nspans;
    const int sp = blockIdx.x - bh * p.nspans;
    const int dk = p.dk, dv = p.dv, T = p.T;
    const int s_begin = sp * p.span_len;
    const int s_end = min(T, s_begin + p.span_len);
    const size_t base_k = slab_k(p, bh), base_v = slab_v(p, bh);
    const size_t st_k = (size_t)p.st_k, st_v = (size_t)p.st_v;
    const bool col_active = tid < dv;
    const float *lnw = p.ln_weight != nullptr ? p.ln_weight + (size_t)(bh % p.H) * dv : nullptr;
    const float *lnb = p.ln_bias != nullptr ? p.ln_bias + (size_t)(bh % p.H) * dv : nullptr;

    float S[RP];
#pragma unroll
    for (int c = 0; c < RP; ++c) S[c] = 0.f;
    // state entering the span: from the carry kernel, or (single span) the caller's initial state
    const float *s0 = nullptr;
    if (p.nspans > 1)
        s0 = p.ws_state + ((size_t)bh * p.nspans + sp) * dk * dv;
    else if (p.initial_state != nullptr)
        s0 = p.initial_state + (size_t)bh * dk * dv;
    if (s0 != nullptr && col_active) {
#pragma unroll
        for (int c = 0; c < RP; ++c)
            if (c < dk) S[c] = s0[(size_t)c * dv + tid];
    }

    for (int t0 = s_begin; t0 < s_end; t0 += kTile) {
        __syncthreads();
        if (tid < kTile) {
            int s = t0 + tid;
            s_tok[tid] = (s < s_end) ? scan_token(p.scan_dir, s, T, p.grid_h, p.grid_w) : -1;
        }
        __syncthreads();
        for (int idx = tid; idx < kTile * RP; idx += kThreads) {
            const int j = idx / RP, c = idx % RP;
            const int n = s_tok[j];
            float a = 0.f, k = 0.f, q = 0.f;
            if (n >= 0 && c < dk) {
                const size_t e = base_k + (size_t)n * st_k + c;
                a = expf(p.z_gate != nullptr ? log_gate(load_elem<TIn>(p.z_gate, e), p.inv_tau) : p.log_alpha[e]);
                k = load_elem<TIn>(p.k, e);
                q = load_elem<TIn>(p.q, e);
            }
            s_a[j][c] = a;
            s_k[j][c] = k;
            s_q[j][c] = q;
        }
        for (int idx = tid; idx < kTile * dv; idx += kThreads) {
            const int j = idx / dv, n2 = idx - j * dv;
            const int n = s_tok[j];
            if (n >= 0) {
                const size_t e = base_v + (size_t)n * st_v + n2;
                s_v[j][n2] = load_elem<TIn>(p.v, e);
                if constexpr (BETA)
                    s_b[j][n2] = p.z_beta != nullptr ? log_gate(load_elem<TIn>(p.z_beta, e), p.inv_tau) : p.log_beta[e];
            }
        }
        __syncthreads();
        if (col_active) {
            for (int j = 0; j < kTile; ++j) {
                if (s_tok[j] < 0) break;
                const float vn = s_v[j][tid];
                const float bn = BETA ? expf(s_b[j][tid]) : 1.f;
                float o = 0.f;
#pragma unroll
                for (int c = 0; c < RP; ++c) {
                    S[c] = fmaf(BETA ? s_a[j][c] * bn : s_a[j][c], S[c], s_k[j][c] * vn);
                    o = fmaf(s_q[j][c], S[c], o);
                }
                s_o[j][tid] = o;
            }
        }
        __syncthreads();
        if (p.r_pre == nullptr) {     // (uniform)
            for (int idx = tid; idx < kTile * dv; idx += kThreads) {
                const int j = idx / dv, n2 = idx - j * dv;
                const int n = s_tok[j];
                if (n < 0) break;
                const size_t e = base_v + (size_t)n * st_v + n2;
                float o = s_o[j][n2];
                if (p.accumulate) o += static_cast<const float *>(p.out)[e];   // fp32 rows (host checks)
                store_elem<TOut>(p.out, e, o);
            }
        } else {   // 8 threads per token of the tile
            const int j = tid >> 3, sub = tid & 7;
            const int n = s_tok[j];
            const float inv_n = 1.f / (float)dv;
            float sum = 0.f;
            for (int c = sub; c < dv; c += 8) sum += s_o[j][c];
            sum += __shfl_xor(sum, 1);
            sum += __shfl_xor(sum, 2);
            sum += __shfl_xor(sum, 4);
            const float mean = sum * inv_n;
            float sq = 0.f;
            for (int c = sub; c < dv; c += 8) {
                const float d = s_o[j][c] - mean;
                sq = fmaf(d, d, sq);
            }
            sq += __shfl_xor(sq, 1);
            sq += __shfl_xor(sq, 2);
            sq += __shfl_xor(sq, 4);
            const float rstd = 1.f / sqrtf(sq * inv_n + p.ln_eps);
            if (n >= 0) {
                for (int c = sub; c < dv; c += 8) {
                    const size_t e = base_v + (size_t)n * st_v + c;
                    const float r = load_elem<TIn>(p.r_pre, e);
                    const float y = (s_o[j][c] - mean) * rstd * (lnw != nullptr ? lnw[c] : 1.f) + (lnb != nullptr ? lnb[c] : 0.f);
                    store_elem<TOut>(p.out, e, y * (r / (1.f + expf(-r))));
                }
            }
        }
    }

    if (p.nspans == 1 && p.final_state != nullptr && col_active) {
        float *f = p.final_state + (size_t)bh * dk * dv;
#pragma unroll
        for (int c = 0; c < RP; ++c)
            if (c < dk) f[(size_t)c * dv + tid] = S[c];
    }
}

template <int GS, int PER, bool ROWREAD, bool BETA, bool STATE, typename TIn, typename TOut>
hipError_t launch_token(const Params &p, const void *w, float *r, hipStream_t stream) {
    using C = TokenCfg<GS, PER, ROWREAD, BETA, STATE>;
    auto kernel = token_span_kernel<GS, PER, ROWREAD, BETA, STATE, TIn, TOut>;
    static std::atomic<bool> configured[kMaxDevices] = {};
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), C::bytes(C::kMaxWaves), configured);
    if (e != hipSuccess) return e;
    const int steps = p.T < p.span_len ? p.T : p.span_len;
    int waves = (steps + C::kSteps - 1) / C::kSteps;
    if (waves > C::kMaxWaves) waves = C::kMaxWaves;
    while (waves > 1 && !launch_fits((long long)p.B * p.H * p.nspans, waves * 64)) --waves;      // (more rounds instead)
    const int cols = ((ROWREAD ? p.dk : p.dv) + kCols - 1) / kCols;
    dim3 grid((unsigned)(p.B * p.H * p.nspans), (unsigned)cols), block(waves * 64);
    hipLaunchKernelGGL(kernel, grid, block, C::bytes(waves), stream, p, w, r);
    return hipGetLastError();
}

template <bool BETA, typename TIn>
hipError_t launch_columns(const Params &p, hipStream_t stream) {
    const bool out_bf16 = p.out_dtype == GLA_DT_BF16;
    dim3 grid((unsigned)(p.B * p.H * p.nspans)), block(kThreads);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, stream, p);
        return hipGetLastError();
    };
    if (p.dk <= 32)
        return out_bf16 ? launch(column_span_kernel<32, TIn, uint16_t, BETA>) : launch(column_span_kernel<32, TIn, float, BETA>);
    return out_bf16 ? launch(column_span_kernel<64, TIn, uint16_t, BETA>) : launch(column_span_kernel<64, TIn, float, BETA>);
}

// Sequences of a few steps (a state carried on token by token): a wave of token_span_kernel walks 8 or 16 steps whether
// they are there or not and stages their rows once per 16 columns, column_span_kernel only what there is.  The less work a
// compute unit has and the fewer columns, the sooner the first is the faster one all the same.  MI355X, fp32 with an
// initial state, token_span_kernel against column_span_kernel, us a call:
//   4096 sequences at 36 / 72 channels   1 step 81.7  43.9   4 steps 83.8  60.7   6 steps 87.5  74.2   8 steps 89.9  90.2
//   3072 sequences at 32 / 64            1 step 28.0  21.3   4 steps 28.5  26.2   6 steps 29.5  30.3
//   512 sequences at 36 / 72             1 step 17.0  11.5   4 steps 17.1  15.0   5 steps 17.2  16.3
//   16 sequences at 36 / 72              2 steps 12.2 11.6   3 steps 11.9  12.3   4 steps 12.2  13.4
//   4096 sequences at 64 / 64            1 step 93.0  61.8   4 steps 94.3  79.5   6 steps 95.6  92.5
//   4096 sequences at 36 / 48            1 step 51.9  39.0   4 steps 52.4  52.4   6 steps 53.0  63.0
bool few_steps(const Params &p) {
    if (p.nspans > 1 || p.gate_shift || p.dv <= (p.dk > 32 ? 32 : 48)) return false;
    const long long sequences = (long long)p.B * p.H;
    return p.T <= 2 || (p.T <= 4 && sequences >= 512) || (p.T <= 6 && p.dk > 32 && p.dv > 64 && sequences >= 1024);
}

template <int GS, int PER, bool BETA, typename TIn>
hipError_t launch_span_class(const Params &p, SpanMode mode, hipStream_t stream) {
    if (mode == kModeState) return launch_token<GS, PER, false, BETA, true, TIn, float>(p, nullptr, nullptr, stream);
    if (p.out_dtype == GLA_DT_BF16)
        return launch_token<GS, PER, false, BETA, false, TIn, uint16_t>(p, nullptr, nullptr, stream);
    return launch_token<GS, PER, false, BETA, false, TIn, float>(p, nullptr, nullptr, stream);
}

// Channels per lane: the smallest class that holds the axis; 5 and 9 are the DiG-XL/2 head (36 / 72 channels), where
// the next power of two would do 1.6 and 1.8 times the arithmetic.
template <bool BETA, typename TIn>
hipError_t launch_span(const Params &p, SpanMode mode, hipStream_t stream) {
    if (mode == kModeOutput && (p.r_pre != nullptr || few_steps(p))) return launch_columns<BETA, TIn>(p, stream);
    if (p.dk <= 32) return launch_span_class<4, 4, BETA, TIn>(p, mode, stream);
    if (p.dk <= 40) return launch_span_class<8, 5, BETA, TIn>(p, mode, stream);
    return launch_span_class<8, 8, BETA, TIn>(p, mode, stream);
}

template <bool BETA, typename TIn>
hipError_t launch_read(const Params &p, const void *w, float *r, hipStream_t stream) {
    if (p.dv <= 32) return launch_token<4, 4, true, BETA, false, TIn, float>(p, w, r, stream);
    if (p.dv <= 64) return launch_token<8, 8, true, BETA, false, TIn, float>(p, w, r, stream);
    if (p.dv <= 72) return launch_token<16, 9, true, BETA, false, TIn, float>(p, w, r, stream);
    return launch_token<16, 16, true, BETA, false, TIn, float>(p, w, r, stream);
}

}  // namespace

hipError_t launch_recurrent_span(const Params &p, SpanMode mode, hipStream_t stream) {
    const bool bf16 = p.qkv_dtype == GLA_DT_BF16;
    if (two_sided(p))
        return bf16 ? launch_span<true, uint16_t>(p, mode, stream) : launch_span<true, float>(p, mode, stream);
    return bf16 ? launch_span<false, uint16_t>(p, mode, stream) : launch_span<false, float>(p, mode, stream);
}

hipError_t launch_row_read(const Params &p, const void *w, float *r, hipStream_t stream) {
    const bool bf16 = p.qkv_dtype == GLA_DT_BF16;
    if (two_sided(p))
        return bf16 ? launch_read<true, uint16_t>(p, w, r, stream) : launch_read<true, float>(p, w, r, stream);
    return bf16 ? launch_read<false, uint16_t>(p, w, r, stream) : launch_read<false, float>(p, w, r, stream);
}

int recurrent_chunks_per_span(const Params &p, long long max_spans) {
    const int nchunks = (p.T + kChunk - 1) / kChunk;
    // Scan steps per round of a work-group, from the span-state pass with one gate.  The output pass has as many, half
    // with both gates up to 32 key channels.  The row reads of the backward pass have 256 up to 32 value columns (128 with
    // both gates), 128 up to 64, else 64 (32 with both gates), and their columns are the key channels.  A backward call
    // keeps the forward call's plan all the same, so with long rows it is planned on up to four (both gates: eight) times
    // the steps that its rounds take: too few spans where sequences are few (8 sequences of 1024 steps at 64 / 128
    // channels, MI355X: 372 us on the one span planned, 157 us on 8).
    const int round = p.dk <= 32 ? TokenCfg<4, 4, false, false, true>::kRound : TokenCfg<8, 8, false, false, true>::kRound;
    const int chunks = round / kChunk;                                 // chunks per round
    const long long groups = (long long)p.B * p.H * ((p.dv + kCols - 1) / kCols);
    const int rounds = (nchunks + chunks - 1) / chunks;
    // Cost in rounds: the rounds a compute unit walks one after the other (one resident group each); several spans
    // walk everything twice and add the carry kernel and two launches, together about kLaunches rounds.
    constexpr int kLaunches = 4;
    long long best = (groups + 255) / 256 * rounds;
    int best_rounds = rounds;
    for (int r = 1; r < rounds; ++r) {                                 // rounds per span
        const long long spans = (rounds + r - 1) / r;
        if (spans > max_spans) continue;                               // (no room for their states)
        const long long cost = 2 * ((groups * spans + 255) / 256 * r) + kLaunches;
        if (cost < best) {
            best = cost;
            best_rounds = r;
        }
    }
    return best_rounds >= rounds ? nchunks : best_rounds * chunks;
}

}  // namespace gla
