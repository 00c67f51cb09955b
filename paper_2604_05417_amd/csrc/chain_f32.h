// Narrow fp32 models: a whole forward pass, or a whole chain of draft steps, in one launch; included after step_f32.h.
#pragma once

#include "chain_plan.h"

namespace msd {

// A layer of such a model is a few hundred KB that any compute unit reads in a microsecond, so its time is what stands between its four
// projections: a launch each (2.3 - 4.3 us with the rows it hands over, and as much of the host).  Here a few workgroups stay for the whole
// pass.  Every workgroup holds the rows in LDS; of each projection every wavefront multiplies its share of the features and publishes
// the results as tagged words (tw_put), and every workgroup collects all of them: 0.4 us from store to load between two workgroups of an idle
// chip.  Weights, gains and the cached K and V of a phase do not depend on what is awaited and are requested before it.
//   rows -> [norm, q | k | v, rotation] -> words -> [attention -> words where there are several rows -> output projection, + h] -> words -> [norm, up, activation]
//   -> words -> [down, + h] -> words -> .. -> [norm, head] -> logits; drafting: -> words -> the draw in every workgroup -> the next step
// Exchanges take four regions of words in turn; a workgroup without units in an exchange is waited for by nobody, so what keeps the others from
// writing over words that it still polls for are the exchanges in which every workgroup has units (chain_plan.h).  Positions of this launch are
// attended to from LDS (the cache rows are written as well, for later launches).  Waits are bounded: after spin_limit polls a workgroup sets *abort
// and all end; drafts that are then missing become token 0.
// What bounds it: four (several rows: five) exchanges per layer and one per step, 0.9 - 1.1 us each, the chain of each phase's few hundred
// instructions between them, 0.4 - 0.9 us (several rows: 1.0 - 1.7), and 2.2 us of attention at 60 positions.  Measured beside a launch per projection, a round of
// 4 / 15 drafts of one layer and a verification of two, d 128, F = V = 512: 16 positions 176 -> 120 us, 100 positions 206 -> 130 and 597 -> 310; d 512, F 2048,
// four layers, drafts of two, 5 drafts at 60 positions 450 -> 349.
constexpr int CH_LAYERS = 8, CH_VOCAB = AS_CH * 256;

struct ChainArgs {
    const float* w[1 + 9 * CH_LAYERS + 2];         // the model's tensors in their order
    int n_layers, D, H, KH, F, V, swiglu, max_ctx;
    float eps, scale;
    double freq[32];                               // of the rotation's pairs
    float* kv;                                     // cache planes of layer 0
    const int32_t* tok;                            // tokens of the block's rows
    int m, pos0, first;                            // rows, position of the first, first row with logits (m: none)
    int steps;                                     // 0: logits of rows first .. to out; else (one row) draft steps, logits of
    float* out;                                    // step j to out + j V
    float T;
    uint64_t seed;
    uint32_t round;
    int32_t *hist, *draft;                         // where the token of step j goes (both + j)
    unsigned long long* xw;                        // CH_REGIONS regions of `region` words
    unsigned region;
    uint32_t tag;                                  // of the first exchange; the following ones count on
    int spin_limit;
    int* abort;
};

// floats of LDS; the same on both sides of the launch
struct ChainLds { int h, x, q, kv, tab, end; };
__host__ __device__ inline ChainLds chain_lds(int m, int steps, int D, int F, int V, int KVD, int HD, int n_layers) {
    ChainLds o;
    const int rows = m + (steps > 1 ? steps - 1 : 0), wide = D > F ? D : F, x = m * wide > (steps ? V : 0) ? m * wide : V;
    o.h = 0;
    o.x = o.h + m * D;
    o.q = o.x + x;
    o.kv = o.q + m * D;
    o.tab = o.kv + (steps > 1 ? n_layers : 1) * 2 * rows * KVD;
    o.end = o.tab + rows * (HD / 2) * 4;
    return o;
}
inline int chain_exchanges(int n_layers, int steps) { return (steps > 1 ? steps : 1) * (5 * n_layers + 1); }     // at most

template <int CTRL>
__device__ __forceinline__ float ch_dpp(float v) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true)); }
// exp(t) for t <= 0 as close as expf (2^n times the hardware's 2^f, f in [-1/2, 1/2] from log2(e) as two floats), without its tests
__device__ __forceinline__ float ch_exp(float t) {
    const float x = fmaxf(t, -150.f), n = rintf(x * 1.44269504f);
    const float f = fmaf(x, 1.92596299e-8f, fmaf(x, 1.44269502162933349609375f, -n));
    return ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
}
// Sum over the wavefront, in every lane: neighbours, rows of 16, then the rows among each other.
__device__ __forceinline__ float ch_over_rows(float v) {                       // over the lanes with the same lane % 16
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_int(v), __float_as_int(v), false, false);
    v = __int_as_float((int)a[0]) + __int_as_float((int)a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_int(v), __float_as_int(v), false, false);
    return __int_as_float((int)b[0]) + __int_as_float((int)b[1]);
}
__device__ __forceinline__ float ch_rows_sum(float v) {                        // .. lane % 4
    v += ch_dpp<0x124>(v);                                                      // row_ror:4, 8
    v += ch_dpp<0x128>(v);
    return ch_over_rows(v);
}
__device__ __forceinline__ float ch_sum(float v) {
    v += ch_dpp<0xb1>(v);
    v += ch_dpp<0x4e>(v);
    return ch_rows_sum(v);
}
// Four sums at once: lane l gets that of v[l % 4].
__device__ __forceinline__ float ch_sum4(float v0, float v1, float v2, float v3, int lane) {
    const bool b0 = lane & 1, b1 = lane & 2;
    float s0 = b0 ? v0 : v1, k0 = b0 ? v1 : v0, s1 = b0 ? v2 : v3, k1 = b0 ? v3 : v2;
    k0 += ch_dpp<0xb1>(s0);
    k1 += ch_dpp<0xb1>(s1);
    const float s = b1 ? k0 : k1, k = b1 ? k1 : k0;
    return ch_rows_sum(k + ch_dpp<0x4e>(s));
}
// Sums of MR rows: lane r (and every lane with the same lane % MR) gets that of row r.
template <int MR>
__device__ __forceinline__ float ch_sum_rows(const float (&v)[MR], int lane) {
    if constexpr (MR == 1) return ch_sum(v[0]);
    else {
        const float a = ch_sum4(v[0], v[1], v[2], v[3], lane);
        if constexpr (MR == 4) return a;
        else {
            const float b = ch_sum4(v[4], v[5], v[6], v[7], lane);
            return lane & 4 ? b : a;
        }
    }
}

// n words of the exchange `tag`, handed to put(index, value).  Returns false after a timeout somewhere in the workgroup.
template <int U, typename Put>
__device__ __forceinline__ void ch_poll(const unsigned long long* words, int i0, int n, uint32_t tag, int spin_limit, int* fail, Put put) {
    unsigned long long w[U] = {};
    bool all = false;
    for (int it = 0; it < spin_limit && !all; ++it) {
        all = true;
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = __hip_atomic_load(words + min(i0 + u * CH_NT, n - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int u = 0; u < U; ++u) all = all && (uint32_t)(w[u] >> 32) == tag;
    }
    if (!all) *fail = 1;
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (i0 + u * CH_NT < n) put(i0 + u * CH_NT, __uint_as_float((uint32_t)w[u]));
}
template <int MR, typename Put>
__device__ __forceinline__ bool ch_collect(const unsigned long long* words, int n, uint32_t tag, int spin_limit, int* fail, int tid, Put put) {
    constexpr int U = MR == 1 ? 1 : 8;
    for (int i0 = tid; i0 < n; i0 += U * CH_NT) ch_poll<U>(words, i0, n, tag, spin_limit, fail, put);
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(*fail) == 0;
}

// A wavefront's share of a projection: units gw, gw + nw, .. (chain_plan.h) of NF features each, over the m rows x (LDS, ldx apart).  wptr(unit, f):
// the row of the weights; epi(unit, r0, y): y[f] holds the sum of row r0 + lane in lanes 0 .. MR - 1.  wv: weights of U units, KB float4 columns per lane,
// the first ones requested before (ch_fetch).
template <int U, int NF, int KB, typename WP>
__device__ __forceinline__ void ch_fetch(float4 (&wv)[U * NF * KB], int i0, int units, int gw, int nw, int K, int k0, int lane, WP wptr) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int unit = min(gw + (i0 + u) * nw, units - 1);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const float* w = wptr(unit, f);
#pragma unroll
            for (int j = 0; j < KB; ++j) wv[(u * NF + f) * KB + j] = *reinterpret_cast<const float4*>(w + min(k0 + (lane + 64 * j) * 4, K - 4));
        }
    }
}
template <int MR, int U, int NF, int KB, bool NORM, int KG, typename WP, typename EP>
__device__ __forceinline__ void ch_project(float4 (&wv)[U * NF * KB], const float* x, int ldx, int m, int K, const float4 (&gain)[KG], float eps, int units, int gw,
                                           int nw, int lane, WP wptr, EP epi) {
#pragma clang loop unroll(disable)
    for (int r0 = 0; r0 < m; r0 += MR) {
        float4 xv[KB][MR];
        auto rows = [&](int k0) {
#pragma unroll
            for (int j = 0; j < KB; ++j)
#pragma unroll
                for (int r = 0; r < MR; ++r) {
                    const int k = k0 + (lane + 64 * j) * 4;
                    xv[j][r] = *reinterpret_cast<const float4*>(x + min(r0 + r, m - 1) * ldx + min(k, K - 4));
                    if (k >= K) xv[j][r] = make_float4(0.f, 0.f, 0.f, 0.f);
                }
        };
        rows(0);
        if constexpr (NORM) {                          // K <= 256 KB: the whole row is here
            float ss[MR];
#pragma unroll
            for (int r = 0; r < MR; ++r) {
                ss[r] = 0.f;
#pragma unroll
                for (int j = 0; j < KB; ++j) ss[r] = dot4(xv[j][r], xv[j][r], ss[r]);
            }
            const float inv = 1.0f / sqrtf(ch_sum_rows<MR>(ss, lane) / (float)K + eps);
#pragma unroll
            for (int r = 0; r < MR; ++r) {
                const float s = MR == 1 ? inv : as_lane(inv, r);
#pragma unroll
                for (int j = 0; j < KB; ++j)
                    xv[j][r] = make_float4(xv[j][r].x * s * gain[j].x, xv[j][r].y * s * gain[j].y, xv[j][r].z * s * gain[j].z, xv[j][r].w * s * gain[j].w);
            }
        }
#pragma clang loop unroll(disable)
        for (int i0 = 0; gw + i0 * nw < units; i0 += U) {                      // wavefront-uniform
            float acc[U][NF][MR];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int r = 0; r < MR; ++r) acc[u][f][r] = 0.f;
#pragma clang loop unroll(disable)
            for (int k0 = 0; k0 < K; k0 += 256 * KB) {
                if (r0 || i0 || k0) ch_fetch<U, NF, KB>(wv, i0, units, gw, nw, K, k0, lane, wptr);
                if (!NORM && K > 256 * KB && (i0 || k0)) rows(k0);
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int f = 0; f < NF; ++f)
#pragma unroll
                        for (int j = 0; j < KB; ++j)
#pragma unroll
                            for (int r = 0; r < MR; ++r) acc[u][f][r] = dot4(wv[(u * NF + f) * KB + j], xv[j][r], acc[u][f][r]);
                if (NORM) break;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (gw + (i0 + u) * nw >= units) break;                        // wavefront-uniform
                float y[NF];
#pragma unroll
                for (int f = 0; f < NF; ++f) y[f] = ch_sum_rows<MR>(acc[u][f], lane);
                epi(gw + (i0 + u) * nw, r0, y);
            }
        }
    }
}
// Sum over the PIECES (8 or 16) neighbouring lanes that hold the pieces of a row, in each of them.
template <int PIECES>
__device__ __forceinline__ float ch_pieces_sum(float v) {
    v += ch_dpp<0xb1>(v);
    v += ch_dpp<0x4e>(v);
    v += ch_dpp<0x141>(v);                                          // row_half_mirror: quads are equal by now
    if constexpr (PIECES == 16) v += ch_dpp<0x140>(v);              // row_mirror
    return v;
}

// .. and over the lanes that hold the same piece.
template <int PIECES>
__device__ __forceinline__ float ch_classes_sum(float v) {
    if constexpr (PIECES == 8) v += ch_dpp<0x128>(v);
    return ch_over_rows(v);
}

// MR: 1, one row and its chain of draft steps (if any); 8, a block of rows without.  KJ: float4 columns of a row of D per lane (D <= 256 KJ).   grid: workgroups, block CH_NT, dynamic LDS chain_lds().end floats + 16 bytes
template <int MR, int KJ, int HD>
__global__ __launch_bounds__(CH_NT) void chain_f32_kernel(ChainArgs a) {
    extern __shared__ __align__(16) float sh[];
    constexpr int C4 = HD / 4, CLS = 64 / C4, HALF = HD / 2;                  // pieces of a row, position classes
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int tid = threadIdx.x, lane = tid & 63;
    // nothing that follows from the lane is kept in registers from one phase to the next (the loops over layers and steps invite that)
    auto fresh = [&]() { asm volatile("" : "+v"(lane), "+v"(tid)); };
    const int D = a.D, F = a.F, V = a.V, H = a.H, KH = a.KH, KVD = KH * HD, NQ = D + 2 * KVD;
    const int gw = chain_first(blockIdx.x, gridDim.x, wave, chain_side(a.D)), nw = (int)gridDim.x * CH_WAVES;
    const ChainLds o = chain_lds(a.m, a.steps, D, F, V, KVD, HD, a.n_layers);
    float *h = sh + o.h, *xb = sh + o.x, *qb = sh + o.q, *kvb = sh + o.kv;
    double2* tab = reinterpret_cast<double2*>(sh + o.tab);
    int *fail = reinterpret_cast<int*>(sh + o.end), *token = fail + 1;
    const int rows_all = a.m + max(a.steps - 1, 0);            // positions of the launch
    uint32_t tag = a.tag;
    unsigned turn = 0;
    unsigned long long* words = a.xw;
    auto next_exchange = [&]() { ++tag; turn = (turn + 1) % CH_REGIONS; words = a.xw + (size_t)turn * a.region; };
    auto give_up = [&](int step) {                     // (every workgroup ends: those that wait for this one time out too)
        if (tid == 0) *a.abort = 1;
        if (a.steps && step + tid < a.steps) { a.hist[step + tid] = 0; a.draft[step + tid] = 0; }
    };
    // weights (and gain) of the next phase, requested before what it multiplies is awaited
    float4 pre[4 * KJ], gain[KJ];
    auto fetch_gain = [&](const float* g) {
#pragma unroll
        for (int j = 0; j < KJ; ++j) gain[j] = *reinterpret_cast<const float4*>(g + min((lane + 64 * j) * 4, D - 4));
    };
    const int q_units = (H + 2 * KH) * HALF;           // a unit of q | k | v is the pair of a rotation (or of v)
    auto wQ = [&](const float* const* W, int u, int f) {
        const int head = u / HALF, i = u - head * HALF + f * HALF;
        return head < H ? W[1] + ((size_t)head * HD + i) * D : head < H + KH ? W[2] + ((size_t)(head - H) * HD + i) * D : W[3] + ((size_t)(head - H - KH) * HD + i) * D;
    };
    auto fetch_q = [&](int l) {
        const float* const* W = a.w + 1 + 9 * l;
        ch_fetch<2, 2, KJ>(pre, 0, q_units, gw, nw, D, 0, lane, [&](int u, int f) { return wQ(W, u, f); });
        fetch_gain(W[0]);
    };
    auto rotation = [&](int r, int e) {                // of row r of the launch
        double sn, cs;
        sincos((double)(a.pos0 + r) * a.freq[e], &sn, &cs);
        tab[r * HALF + e] = make_double2(cs, sn);
    };
    fetch_q(0);
    for (int i = tid; i < a.m * (D / 4); i += CH_NT) {
        const int r = i / (D / 4), c = (i - r * (D / 4)) * 4;
        *reinterpret_cast<float4*>(h + r * D + c) = *reinterpret_cast<const float4*>(a.w[0] + (size_t)min(max(a.tok[r], 0), V - 1) * D + c);
    }
    if (tid == 0) *fail = 0;
    for (int i = tid; i < a.m * HALF; i += CH_NT) rotation(i / HALF, i % HALF);
    __syncthreads();
    const size_t plane = (size_t)KH * a.max_ctx * HD;
    const int nsteps = max(a.steps, 1);
#pragma clang loop unroll(disable)
    for (int step = 0; step < nsteps; ++step) {
        const int m = MR == 1 ? 1 : a.m, rel = step, p0 = a.pos0 + step;
        auto mine = [&](int r0, int rows) { return lane < MR && r0 + lane < rows; };       // this lane has the sum of a row
        auto rows_of_h = [&](int i, float y) { h[i] = y; };
        auto add = [&](int u, int r0, const float* y) {
            const int r = r0 + lane;
            if (mine(r0, m)) tw_put(words + r * D + u, tag, __float_as_uint(h[r * D + u] + y[0]));
        };
#pragma clang loop unroll(disable)
        for (int l = 0; l < a.n_layers; ++l) {
            const float* const* W = a.w + 1 + 9 * l;
            float *kc = a.kv + (size_t)l * 2 * plane, *vc = kc + plane;
            float *kr = kvb + (a.steps > 1 ? l : 0) * 2 * rows_all * KVD, *vr = kr + rows_all * KVD;      // rows of this launch
            // ---- q | k | v
            fresh();
            ch_project<MR, 2, 2, KJ, true>(pre, h, D, m, D, gain, a.eps, q_units, gw, nw, lane, [&](int u, int f) { return wQ(W, u, f); }, [&](int u, int r0, const float* y) {
                const int head = u / HALF, i = u - head * HALF, r = r0 + lane;
                if (!mine(r0, m)) return;
                float p = y[0], q = y[1];
                if (head < H + KH) {
                    const double2 rot = tab[(rel + r) * HALF + i];
                    p = (float)((double)y[0] * rot.x - (double)y[1] * rot.y);
                    q = (float)((double)y[0] * rot.y + (double)y[1] * rot.x);
                }
                unsigned long long* dst = words + r * NQ + head * HD + i;
                tw_put(dst, tag, __float_as_uint(p));
                tw_put(dst + HALF, tag, __float_as_uint(q));
                if (head >= H) {
                    float* c = head < H + KH ? kc + ((size_t)(head - H) * a.max_ctx + p0 + r) * HD + i : vc + ((size_t)(head - H - KH) * a.max_ctx + p0 + r) * HD + i;
                    c[0] = p;
                    c[HALF] = q;
                }
            });
            fresh();
            ch_fetch<4, 1, KJ>(pre, 0, D, gw, nw, D, 0, lane, [&](int u, int) { return W[4] + (size_t)u * D; });
            if (!ch_collect<MR>(words, m * NQ, tag, a.spin_limit, fail, tid, [&](int i, float y) {
                    const int r = MR == 1 ? 0 : i / NQ, n = i - r * NQ;
                    if (n < D) qb[r * D + n] = y;
                    else if (n < D + KVD) kr[(rel + r) * KVD + n - D] = y;
                    else vr[(rel + r) * KVD + n - D - KVD] = y;
                })) { give_up(step); return; }
            next_exchange();
            // ---- attention, a head of a row per wavefront: one row in every workgroup, more of them once, handed around like a projection.  Lane
            // (class, piece) has that piece of positions class, class + CLS, ..: requests are of consecutive bytes, the pieces of a score are
            // added over neighbouring lanes, and a position's weight is where its piece of V is.  First the cached positions, then this
            // launch's from LDS
            fresh();
            const int pc = lane % C4, cls = lane / C4, old = a.pos0;
#pragma clang loop unroll(disable)
            for (int unit = MR == 1 ? wave : gw; unit < m * H; unit += MR == 1 ? CH_WAVES : nw) {     // wavefront-uniform
                const int r = MR == 1 ? 0 : unit / H, head = MR == 1 ? unit : unit - r * H, kh = head / (H / KH), n = rel + r + 1;
                const float *kp = kc + (size_t)kh * a.max_ctx * HD + 4 * pc, *vp = vc + (size_t)kh * a.max_ctx * HD + 4 * pc;
                const float *kq = kr + kh * HD + 4 * pc, *vq = vr + kh * HD + 4 * pc;
                float mx = -INFINITY, sum = 0.f;
                float4 ov = make_float4(0.f, 0.f, 0.f, 0.f);
                const float4 qv = *reinterpret_cast<const float4*>(qb + r * D + head * HD + 4 * pc);
                // the positions of a chunk from c0 on, of n; rows past the last re-read it: their weight is 0
                auto chunk = [&](auto count, int c0, int n, const float* K, const float* V, int stride) {
                    constexpr int NI = decltype(count)::value;
                    float4 k[NI], v[NI];
                    float s[NI], tm = -INFINITY;
#pragma unroll
                    for (int i = 0; i < NI; ++i) {
                        const int at = min(c0 + cls + CLS * i, n - 1) * stride;
                        k[i] = *reinterpret_cast<const float4*>(K + at);
                        v[i] = *reinterpret_cast<const float4*>(V + at);
                    }
#pragma unroll
                    for (int i = 0; i < NI; ++i) {
                        s[i] = ch_pieces_sum<C4>(dot4(k[i], qv, 0.f));
                        s[i] = c0 + cls + CLS * i < n ? s[i] * a.scale : -INFINITY;
                        tm = fmaxf(tm, s[i]);
                    }
                    const float nm = fmaxf(mx, dpp_max(tm)), alpha = ch_exp(mx - nm);      // finite: a chunk holds a position
                    mx = nm;
                    sum *= alpha;
                    ov.x *= alpha; ov.y *= alpha; ov.z *= alpha; ov.w *= alpha;
#pragma unroll
                    for (int i = 0; i < NI; ++i) {
                        const float e = ch_exp(s[i] - mx);
                        sum += e;
                        ov.x = fmaf(e, v[i].x, ov.x); ov.y = fmaf(e, v[i].y, ov.y); ov.z = fmaf(e, v[i].z, ov.z); ov.w = fmaf(e, v[i].w, ov.w);
                    }
                };
                if (old <= 4 * CLS) { if (old > 0) chunk(std::integral_constant<int, 4>(), 0, old, kp, vp, HD); }
                else {
#pragma clang loop unroll(disable)
                    for (int c0 = 0; c0 < old; c0 += 8 * CLS) chunk(std::integral_constant<int, 8>(), c0, old, kp, vp, HD);
                }
                if (n <= CLS) chunk(std::integral_constant<int, 1>(), 0, n, kq, vq, KVD);
                else {
#pragma clang loop unroll(disable)
                    for (int c0 = 0; c0 < n; c0 += 4 * CLS) chunk(std::integral_constant<int, 4>(), c0, n, kq, vq, KVD);
                }
                sum = ch_classes_sum<C4>(sum);
                ov.x = ch_classes_sum<C4>(ov.x) / sum; ov.y = ch_classes_sum<C4>(ov.y) / sum;
                ov.z = ch_classes_sum<C4>(ov.z) / sum; ov.w = ch_classes_sum<C4>(ov.w) / sum;
                const int at = r * D + head * HD + 4 * pc;
                if constexpr (MR == 1) { if (cls == 0) *reinterpret_cast<float4*>(xb + at) = ov; }
                else if (cls < 4) tw_put(words + at + cls, tag, __float_as_uint(cls == 0 ? ov.x : cls == 1 ? ov.y : cls == 2 ? ov.z : ov.w));
            }
            if constexpr (MR == 1) __syncthreads();
            else {
                if (!ch_collect<MR>(words, m * D, tag, a.spin_limit, fail, tid, [&](int i, float y) { xb[i] = y; })) { give_up(step); return; }
                next_exchange();
            }
            // ---- h + output projection
            fresh();
            ch_project<MR, 4, 1, KJ, false>(pre, xb, D, m, D, gain, 0.f, D, gw, nw, lane, [&](int u, int) { return W[4] + (size_t)u * D; }, add);
            // ---- up (and gate), activation
            fresh();
            auto wU = [&](int u, int f) { return (a.swiglu && f == 0 ? W[6] : W[7]) + (size_t)u * D; };
            if (a.swiglu) ch_fetch<2, 2, KJ>(pre, 0, F, gw, nw, D, 0, lane, wU);
            else ch_fetch<4, 1, KJ>(pre, 0, F, gw, nw, D, 0, lane, wU);
            fetch_gain(W[5]);
            if (!ch_collect<MR>(words, m * D, tag, a.spin_limit, fail, tid, rows_of_h)) { give_up(step); return; }
            next_exchange();
            if (a.swiglu)
                ch_project<MR, 2, 2, KJ, true>(pre, h, D, m, D, gain, a.eps, F, gw, nw, lane, wU, [&](int u, int r0, const float* y) {
                    if (mine(r0, m)) tw_put(words + (r0 + lane) * F + u, tag, __float_as_uint(y[0] / (1.0f + expf(-y[0])) * y[1]));
                });
            else
                ch_project<MR, 4, 1, KJ, true>(pre, h, D, m, D, gain, a.eps, F, gw, nw, lane, wU, [&](int u, int r0, const float* y) {
                    if (mine(r0, m)) tw_put(words + (r0 + lane) * F + u, tag, __float_as_uint(0.5f * y[0] * (1.0f + erff(y[0] * 0.70710678118654752f))));
                });
            // ---- h + down projection
            fresh();
            auto wD = [&](int u, int) { return W[8] + (size_t)u * F; };
            ch_fetch<2, 1, 2 * KJ>(pre, 0, D, gw, nw, F, 0, lane, wD);
            if (!ch_collect<MR>(words, m * F, tag, a.spin_limit, fail, tid, [&](int i, float y) { xb[i] = y; })) { give_up(step); return; }
            next_exchange();
            ch_project<MR, 2, 1, 2 * KJ, false>(pre, xb, F, m, F, gain, 0.f, D, gw, nw, lane, wD, add);
            fresh();
            if (l + 1 < a.n_layers) fetch_q(l + 1);
            else {
                if (a.steps == 0 && a.first >= m) return;      // no logits: nobody reads the rows (workgroup-uniform)
                const float* hw = a.w[2 + 9 * a.n_layers];
                ch_fetch<4, 1, KJ>(pre, 0, V, gw, nw, D, 0, lane, [&](int u, int) { return hw + (size_t)u * D; });
                fetch_gain(a.w[1 + 9 * a.n_layers]);
            }
            if (!ch_collect<MR>(words, m * D, tag, a.spin_limit, fail, tid, rows_of_h)) { give_up(step); return; }
            next_exchange();
        }
        // ---- head
        fresh();
        {
            const float* hw = a.w[2 + 9 * a.n_layers];
            const int first = a.steps ? m - 1 : a.first, mr = m - first;
            float* out = a.out + (size_t)step * V;
            ch_project<MR, 4, 1, KJ, true>(pre, h + first * D, D, mr, D, gain, a.eps, V, gw, nw, lane, [&](int u, int) { return hw + (size_t)u * D; },
                                           [&](int u, int r0, const float* y) {
                                               if (!mine(r0, mr)) return;
                                               out[(size_t)(r0 + lane) * V + u] = y[0];
                                               if (MR == 1 && a.steps) tw_put(words + u, tag, __float_as_uint(y[0]));
                                           });
        }
        if (MR > 1 || a.steps == 0) return;
        if constexpr (MR == 1) {
            // ---- the draw, the same in every workgroup; the next position's rotations beside it
            fresh();
            if (step + 1 < nsteps) fetch_q(0);
            if (!ch_collect<MR>(words, V, tag, a.spin_limit, fail, tid, [&](int i, float y) { xb[i] = y; })) { give_up(step); return; }
            next_exchange();
            if (wave == CH_WAVES - 1 && step + 1 < nsteps && lane < HALF) rotation(step + 1, lane);
            if (wave == 0) {
                auto draw = [&](auto& x) {
#pragma unroll
                    for (int c = 0; c < (int)(sizeof(x) / sizeof(x[0])); ++c) {
                        const int i = c * 256 + lane * 4;
                        const float4 y = *reinterpret_cast<const float4*>(xb + min(i, V - 4));
                        const bool in = i < V;
                        x[c][0] = in ? y.x : -INFINITY; x[c][1] = in ? y.y : -INFINITY; x[c][2] = in ? y.z : -INFINITY; x[c][3] = in ? y.w : -INFINITY;
                    }
                    if (a.T <= 0.f) return as_wave_argmax(x, V, lane);
                    const float u = philox_uniform(a.seed, 0u, a.round, (uint32_t)step, 2u);
                    return a.T == 1.0f ? as_wave_draw<true>(x, a.T, u, V, lane) : as_wave_draw<false>(x, a.T, u, V, lane);
                };
                int tok;
                if (V <= 512) { float x[2][4]; tok = draw(x); }
                else { float x[AS_CH][4]; tok = draw(x); }
                if (lane == 0) {
                    *token = tok;
                    if (blockIdx.x == 0) { a.hist[step] = tok; a.draft[step] = tok; }
                }
            }
            __syncthreads();
            if (step + 1 < nsteps)
                for (int i = tid * 4; i < D; i += CH_NT * 4) *reinterpret_cast<float4*>(h + i) = *reinterpret_cast<const float4*>(a.w[0] + (size_t)*token * D + i);
            __syncthreads();
        }
    }
}

}  // namespace msd
