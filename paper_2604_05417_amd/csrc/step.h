// Skinny GEMM of short blocks (at most 16 rows) whose K range is reduced inside the workgroup; included after kernels.h.
#pragma once

namespace msd {

// One workgroup of 16 wavefronts per CU.  T feature tiles are multiplied at a time, the K range of a tile dealt out to S = 16 / T
// wavefronts; the partial tiles are added through LDS.  The launch leaves finished sums, so the next kernel reads one array instead of
// up to eight split-K partials, and what follows the projection (activation, residual add) happens in its epilogue.
//   STEP_NORM   the input rows are h (+ the partials of the projection before): every workgroup forms h * gain itself, stages it in
//               LDS as two bf16 terms and scales its sums by 1/rms at the end (RMSNorm's scale commutes with the product)
//   STEP_TERMS  the input is given as two bf16 arrays (store_split4); each wavefront loads the operands of its slice straight into registers
//   STEP_OUT    out[r][n] = sum          STEP_ADD  out[r][n] += sum (the residual stream)
//   STEP_ACT    out = SiLU(gate) * up or GELU(up) as two bf16 arrays; with SwiGLU units 2 j and 2 j + 1 are gate and up of 16 features
//   STEP_ROPE   q | k | v projection: q rotated into out (two bf16 arrays; one of floats when head_dim < 64), the rotated k and the v
//               rows rounded into the cache.  The packed tiles keep both members of a rotary pair in one lane.  What was a launch of
//               its own behind the projection (4.3 us of a 7B layer at 6 rows, 3.1 of a 1B one).
// What bounds it: bytes of weights per CU at about 25 GB/s, and the chain launch - input - multiply - LDS - store in front of and behind
// them (2.9 us for a kernel that does nothing else with one wide workgroup per CU, 4.5 us with 256 threads).  So the input is requested
// first and the first group of weights before it is waited for: per wavefront 4 or 8 KiB with STEP_NORM, 4 with STEP_TERMS, 3 with half
// tiles (48 - 128 KiB per CU).  The hi and lo term of a row
// are columns r and 8 + r of one MFMA operand: one multiply per KiB instead of two.
// HALF: a unit is half a feature tile (8 features), so that a projection of d_model features has enough units for all CUs: one load
// brings the 8 features of two neighbouring chunks, multiplied with the inputs of either one (two MFMAs, each good for 8 of its rows).
enum { STEP_NORM = 0, STEP_TERMS = 1 };
enum { STEP_OUT = 0, STEP_ADD = 1, STEP_ACT = 2, STEP_ROPE = 3 };
constexpr int STEP_ROWS = 16;

struct StepArgs {
    const float* h;                  // NORM: residual rows [m][K]
    const float* part;               // NORM, PART: partials [s][m][K] added to them (split stride sstride, 1 <= ns <= 8)
    float* h_out;                    // NORM, PART: the updated rows (another buffer: other workgroups still read h)
    const bf16_t* gain;              // NORM
    size_t sstride;
    int ns;
    float eps;
    const bf16_t* x;                 // TERMS: hi array [m][K]; the lo array follows x_lo elements behind it
    size_t x_lo;
    const bf16_t *W0, *W1, *W2;      // packed weights, concatenated at tiles t0 <= t1 <= ntiles
    int t0, t1, ntiles;
    float* out;
    int N;                           // row length of out (ACT: d_ffn)
    int swiglu;                      // ACT
    int m, K, T, S, passes;          // T * S <= 16; a workgroup works through passes * T units (ADD: one pass)
    const double2* tab;              // ROPE: rotations [m][hd / 2]
    bf16_t *kc, *vc;                 // ROPE: cache planes of the layer, row r goes to position pos0 + r
    int H, KH, hd, pos0, max_ctx;    // ROPE
    const long long* rowkv;          // ROPE, rows of several sequences: where row r goes in a K/V head's plane (elements), -1: nowhere
};

// LDS of a launch: NORM [2 (hi, lo)][m][rs] 16-byte pieces and 16 sums of squares, then [16][64] partial tiles.
__host__ __device__ inline int step_rs(int K) { return K / 8 + 1; }
inline size_t step_lds(bool norm, int m, int K) { return (norm ? (size_t)2 * m * step_rs(K) * 16 + 64 : 0) + (size_t)16 * 64 * 16; }

// J: float4 columns of a row per lane (NORM).  U: loads of weights per group; two groups in flight.
// NR: 8, or 16 for blocks of 9 - 16 rows, whose terms are two operands.  Measured at 12 rows beside the split-K kernel with the launches behind
// it: q | k | v of 2048 inputs and 3072 outputs 13.3 -> 8.1 us, gate | up (16384) 18.7 -> 15.1, output projection 12.3 -> 8.7.  Rows of
// 4096 inputs do not fit: staged in two parts, q | k | v took 29.9 against 23.8 us, gate | up 39.6 against 38.2.
template <int PRO, int EPI, bool PART, int J, int U, bool HALF, int NR>
__global__ __launch_bounds__(1024) void gemm_step_kernel(StepArgs a) {
    extern __shared__ uint4 xs[];
    constexpr int XT = NR / 8;                                            // operands per chunk of K
    constexpr int XN = PRO == STEP_TERMS ? (HALF ? 2 * U : U) : 1;        // chunks whose operands travel with a group of weights
    struct Group { u32x4 w[U], x[XT * XN]; };
    const int m = a.m, K = a.K, kchunks = K >> 5, rs = step_rs(K), S = a.S, T = a.T;
    float* ssp = reinterpret_cast<float*>(xs + 2 * m * rs);
    f32x4* red = reinterpret_cast<f32x4*>(PRO == STEP_NORM ? ssp + 16 : reinterpret_cast<float*>(xs));
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int col = lane & 15, g = lane >> 4;
    const int tp = wave / S, sl = wave - tp * S;                          // wavefronts from T S on have no tile
    int cps = (kchunks + S - 1) / S;
    if (HALF) cps = (cps + 1) & ~1;
    const int nc = tp < T ? max(0, min(cps, kchunks - sl * cps)) : 0, c0 = min(sl * cps, kchunks - (HALF ? 2 : 1));
    const int nl = HALF ? nc >> 1 : nc, last = max(nl, 1) - 1;            // loads of a unit
    const int ngroups = (nl + U - 1) / U;
    const bool pairs = EPI == STEP_ACT && a.swiglu;
    const int nunits = HALF ? 2 * a.ntiles : a.ntiles;
    auto unit_of = [&](int p, int t) { return ((int)blockIdx.x * a.passes + p) * T + t; };
    auto unit_base = [&](int p) -> const u32x4* {
        const int u = min(unit_of(p, min(tp, T - 1)), nunits - 1);
        const int t = HALF ? u >> 1 : pairs ? (u & 1) * a.t0 + (u >> 1) : u;
        const bf16_t* W = t < a.t0 ? a.W0 : t < a.t1 ? a.W1 : a.W2;
        const int tl = t < a.t0 ? t : t < a.t1 ? t - a.t0 : t - a.t1;
        const int piece = HALF ? ((lane >> 3) & 1) * 64 + ((lane & 48) | (u & 1) * 8 | (lane & 7)) : lane;
        return reinterpret_cast<const u32x4*>(W) + ((size_t)tl * kchunks + c0) * 64 + piece;
    };
    // operand column: term col / 8 of row col % 8, or row col of either term (columns past m repeat the last row and are never stored)
    const int xr = min(col & (NR - 1), m - 1), xt = NR == 8 ? col >> 3 : 0;
    const u32x4* xg = reinterpret_cast<const u32x4*>(a.x + xt * a.x_lo + (size_t)xr * K + c0 * 32 + g * 8);           // TERMS
    const u32x4* xl = reinterpret_cast<const u32x4*>(xs) + (xt * m + xr) * rs + g + c0 * 4;                           // NORM
    const char *xhi = reinterpret_cast<const char*>(a.x), *xlo = xhi + a.x_lo * 2;       // TERMS, NR = 16: the same by bytes
    const uint32_t xg_at = (uint32_t)(xr * K + c0 * 32 + g * 8) * 2;
    const int xl_lo = m * rs;
    // every load is unconditional and clamped into the slice, so that each wait counts exactly the requests it needs
    auto issue = [&](Group& b, const u32x4* wp, int gi) {
        if constexpr (PRO == STEP_TERMS) {
#pragma unroll
            for (int u = 0; u < XN; ++u) {
                const int ch = min(gi * XN + u, HALF ? 2 * last + 1 : last);
                if constexpr (NR == 16) {
                    b.x[2 * u] = *reinterpret_cast<const u32x4*>(xhi + (xg_at + (uint32_t)ch * 64));
                    b.x[2 * u + 1] = *reinterpret_cast<const u32x4*>(xlo + (xg_at + (uint32_t)ch * 64));
                } else {
                    b.x[u] = xg[(size_t)ch * 4];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) b.w[u] = __builtin_nontemporal_load(wp + (size_t)min(gi * U + u, last) * (HALF ? 128 : 64));
    };
    Group ba, bb;
    const u32x4* wp = unit_base(0);
    float4 h_pre = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (EPI == STEP_ADD) {               // the epilogue's input first of all (one pass per workgroup)
        const int u = min(unit_of(0, min(wave, T - 1)), nunits - 1), q = HALF ? g & 1 : g;
        h_pre = *reinterpret_cast<const float4*>(a.out + (size_t)min(col, m - 1) * a.N + (HALF ? u * 8 : u * 16) + q * 4);
    }
    const int lw = NR == 16 ? 4 : m <= 1 ? 0 : m <= 2 ? 1 : m <= 4 ? 2 : 3, wpr = 16 >> lw;     // wavefronts per row
    if constexpr (PRO == STEP_NORM) {
        const int row = wave >> (4 - lw), rl = min(row, m - 1), li = (wave & (wpr - 1)) * 64 + lane;
        float4 v[J], pp[PART ? J : 1][8];
        uint2 gn[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int cc = min((li + j * 64 * wpr) * 4, K - 4);
            v[j] = *reinterpret_cast<const float4*>(a.h + (size_t)rl * K + cc);
            gn[j] = *reinterpret_cast<const uint2*>(a.gain + cc);
            if constexpr (PART) {
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    pp[j][u] = *reinterpret_cast<const float4*>(a.part + (size_t)min(u, a.ns - 1) * a.sstride + (size_t)rl * K + cc);
            }
        }
        issue(ba, wp, 0);
        float ss = 0.f;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int cj = (li + j * 64 * wpr) * 4;
            if constexpr (PART) {
                float4 y = make_float4(0.f, 0.f, 0.f, 0.f);        // added in the order s = 0, 1, ..
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const bool on = u < a.ns;
                    y.x += on ? pp[j][u].x : 0.f; y.y += on ? pp[j][u].y : 0.f; y.z += on ? pp[j][u].z : 0.f; y.w += on ? pp[j][u].w : 0.f;
                }
                v[j].x += y.x; v[j].y += y.y; v[j].z += y.z; v[j].w += y.w;
            }
            if (row < m && cj < K) {
                if (PART && blockIdx.x == 0) *reinterpret_cast<float4*>(a.h_out + (size_t)row * K + cj) = v[j];
                ss += v[j].x * v[j].x + v[j].y * v[j].y + v[j].z * v[j].z + v[j].w * v[j].w;
                const float4 hg = make_float4(v[j].x * bf2f((bf16_t)(gn[j].x & 0xffffu)), v[j].y * bf2f((bf16_t)(gn[j].x >> 16)),
                                              v[j].z * bf2f((bf16_t)(gn[j].y & 0xffffu)), v[j].w * bf2f((bf16_t)(gn[j].y >> 16)));
                store_split4(reinterpret_cast<float*>(xs + row * rs), (size_t)m * rs * 8, cj, hg);
            }
        }
        ss = wave_sum(ss);
        if (lane == 0) ssp[wave] = ss;
        __syncthreads();
    } else {
        issue(ba, wp, 0);
    }
    f32x4 acc0, acc1;                              // even and odd chunks; NR = 16: hi and lo terms (HALF: even and odd chunks)
    auto mul = [&](const u32x4& w, const u32x4& x, f32x4& acc) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), acc, 0, 0, 0);
    };
    auto mul1 = [&](const Group& b, int u, int i) {
        if constexpr (PRO == STEP_NORM && NR == 16) { mul(b.w[u], xl[i * 4], acc0); mul(b.w[u], xl[xl_lo + i * 4], acc1); }
        else if constexpr (NR == 16 && HALF) {
            mul(b.w[u], b.x[4 * u], acc0); mul(b.w[u], b.x[4 * u + 2], acc1);
            mul(b.w[u], b.x[4 * u + 1], acc0); mul(b.w[u], b.x[4 * u + 3], acc1);
        }
        else if constexpr (NR == 16) { mul(b.w[u], b.x[2 * u], acc0); mul(b.w[u], b.x[2 * u + 1], acc1); }
        else if constexpr (PRO == STEP_NORM) mul(b.w[u], xl[i * 4], (u & 1) ? acc1 : acc0);
        else if constexpr (HALF) { mul(b.w[u], b.x[2 * u], acc0); mul(b.w[u], b.x[2 * u + 1], acc1); }
        else mul(b.w[u], b.x[u], (u & 1) ? acc1 : acc0);
    };
    auto multiply = [&](const Group& b, int gi) {
        if (gi * U + U <= nl) {
#pragma unroll
            for (int u = 0; u < U; ++u) mul1(b, u, gi * U + u);
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (gi * U + u < nl) mul1(b, u, gi * U + u);
        }
    };
    double2 rot0 = make_double2(1.0, 0.0), rot1 = rot0;        // ROPE: rotations of this lane's two pairs
    long long kv_at = 0;                                       // .. and its row's place in a plane of the cache
    for (int p = 0; p < a.passes; ++p) {
        acc0 = f32x4{0.f, 0.f, 0.f, 0.f};
        acc1 = acc0;
        if (nl > 0) {
            int gi = 0;
            for (; gi + 2 < ngroups; gi += 2) {
                issue(bb, wp, gi + 1);
                multiply(ba, gi);
                issue(ba, wp, gi + 2);
                multiply(bb, gi + 1);
            }
            if (gi + 2 == ngroups) {
                issue(bb, wp, gi + 1);
                multiply(ba, gi);
                multiply(bb, gi + 1);
            } else {
                multiply(ba, gi);
            }
        }
        if (p + 1 < a.passes) { wp = unit_base(p + 1); issue(ba, wp, 0); }
        if constexpr (EPI == STEP_ROPE) {          // arrives while the partial tiles are gathered
            const int n = min(unit_of(p, min(wave, T - 1)), nunits - 1) * 16, half = a.hd >> 1;
            const double2* t = a.tab + min(col, m - 1) * half + min(((n % a.hd) >> 1) + 2 * g, half - 2);
            rot0 = t[0]; rot1 = t[1];
            kv_at = a.rowkv ? a.rowkv[min(col, m - 1)] : (long long)(a.pos0 + col) * a.hd;
        }
        if (p > 0) __syncthreads();                // the partial tiles of the pass before are read
        if constexpr (HALF) red[wave * 64 + lane] = g < 2 ? acc0 : acc1;
        else red[wave * 64 + lane] = acc0 + acc1;
        __syncthreads();
        float inv = 1.f;
        if constexpr (PRO == STEP_NORM) {
            float tot = 0.f;
            for (int i = 0; i < wpr; ++i) tot += ssp[xr * wpr + i];
            inv = 1.0f / sqrtf(tot / (float)K + a.eps);
        }
        auto unit_sum = [&](int t) {                // sums of unit t: features 4 g .. of row col (both terms added)
            f32x4 y = red[t * S * 64 + lane];
            for (int s = 1; s < S; ++s) y += red[(t * S + s) * 64 + lane];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (NR == 8) y[e] += __shfl_xor(y[e], 8, 64);
                if constexpr (HALF) y[e] += __shfl_xor(y[e], 32, 64);
            }
            return y;
        };
        if (wave < (pairs ? T >> 1 : T)) {
            if constexpr (EPI == STEP_ACT) {
                f32x4 gt = unit_sum(pairs ? 2 * wave : wave), up = gt;
                if (pairs) up = unit_sum(2 * wave + 1);
                const int ft = unit_of(p, pairs ? 2 * wave : wave) >> (pairs ? 1 : 0);
                float y[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float gg = gt[e] * inv, uu = up[e] * inv;
                    y[e] = pairs ? gg / (1.0f + expf(-gg)) * uu : 0.5f * gg * (1.0f + erff(gg * 0.70710678118654752f));
                }
                if (col < m && ft * 16 < a.N)
                    store_split4(a.out, (size_t)m * a.N, (size_t)col * a.N + ft * 16 + g * 4, make_float4(y[0], y[1], y[2], y[3]));
            } else if constexpr (EPI == STEP_ROPE) {
                const f32x4 y = unit_sum(wave);
                const int n = unit_of(p, wave) * 16, hd = a.hd, half = hd >> 1, head = n / hd, c = n - head * hd;
                if (col < m && unit_of(p, wave) < nunits) {
                    const float v[4] = {y[0] * inv, y[1] * inv, y[2] * inv, y[3] * inv};
                    // packed columns c + 4 g .. are the pairs i, i + 1 (first and second member, hd / 2 apart)
                    const int i = (c >> 1) + 2 * g;
                    const float a0 = (float)((double)v[0] * rot0.x - (double)v[1] * rot0.y), b0 = (float)((double)v[0] * rot0.y + (double)v[1] * rot0.x);
                    const float a1 = (float)((double)v[2] * rot1.x - (double)v[3] * rot1.y), b1 = (float)((double)v[2] * rot1.y + (double)v[3] * rot1.x);
                    const uint32_t ah = f2bf2(a0, a1), bh = f2bf2(b0, b1);
                    if (head >= a.H) {
                        if (kv_at >= 0) {
                            const size_t plane = (size_t)a.max_ctx * hd;
                            if (head >= a.H + a.KH) {
                                *reinterpret_cast<uint2*>(a.vc + (size_t)(head - a.H - a.KH) * plane + kv_at + c + 4 * g) = make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
                            } else {
                                bf16_t* k = a.kc + (size_t)(head - a.H) * plane + kv_at + i;
                                *reinterpret_cast<uint32_t*>(k) = ah;
                                *reinterpret_cast<uint32_t*>(k + half) = bh;
                            }
                        }
                    } else if (hd >= 64) {
                        bf16_t* qh = reinterpret_cast<bf16_t*>(a.out) + ((size_t)col * a.H + head) * hd + i;
                        bf16_t* ql = qh + (size_t)m * a.H * hd;
                        *reinterpret_cast<uint32_t*>(qh) = ah;
                        *reinterpret_cast<uint32_t*>(qh + half) = bh;
                        *reinterpret_cast<uint32_t*>(ql) = f2bf2(a0 - __uint_as_float(ah << 16), a1 - __uint_as_float(ah & 0xffff0000u));
                        *reinterpret_cast<uint32_t*>(ql + half) = f2bf2(b0 - __uint_as_float(bh << 16), b1 - __uint_as_float(bh & 0xffff0000u));
                    } else {
                        float* q = a.out + ((size_t)col * a.H + head) * hd + i;
                        *reinterpret_cast<float2*>(q) = make_float2(a0, a1);
                        *reinterpret_cast<float2*>(q + half) = make_float2(b0, b1);
                    }
                }
            } else {
                const f32x4 y = unit_sum(wave);
                const int u = unit_of(p, wave);
                if (col < m && u < nunits && (!HALF || g < 2)) {
                    float4* o = reinterpret_cast<float4*>(a.out + (size_t)col * a.N + (HALF ? u * 8 : u * 16) + g * 4);
                    if constexpr (EPI == STEP_ADD) *o = make_float4(h_pre.x + y[0], h_pre.y + y[1], h_pre.z + y[2], h_pre.w + y[3]);
                    else *o = make_float4(y[0] * inv, y[1] * inv, y[2] * inv, y[3] * inv);
                }
            }
        }
    }
}

}  // namespace msd
