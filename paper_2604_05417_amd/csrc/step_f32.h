// fp32 models, blocks of rows of at most STEP_F32_K inputs: GEMMs with what stands before and behind them; included after kernels.h.
#pragma once

namespace msd {

// A layer of a narrow fp32 model moves a few hundred KB, so its time is its launches: 2 - 4 us each, ten of them, of which six (norms,
// rotation, merge, activation, residual) only hand rows from one GEMM to the next.  Here the GEMM that reads a row normalises it and the
// GEMM that makes it rotates, activates or adds it: five launches per layer, four where the context is short enough for attention and output
// projection in one (below).
// One wavefront per unit = NF output features: one, or the pair a rotation or a SwiGLU needs; lanes stride over K.  Everything a wavefront
// reads is requested before anything is waited for; NORM: every workgroup normalises all m rows into LDS itself (they are few and short).
// Sums: lane partials in fp32, then over the lanes; the norm is 1/sqrt(mean of squares + eps) of the rows in fp32 as in addnorm_kernel.
//   grid ceil(units / 4), block 256, dynamic LDS (NORM) m * K * 4 bytes
enum { F32_OUT = 0, F32_ADD = 1, F32_ACT = 2, F32_ROPE = 3 };
constexpr int STEP_F32_K = 512;                    // two float4 columns per lane of a normalised row

struct F32Args {
    const float* x;                                // [m][K]: residual rows (NORM) or activations
    const float* gain;                             // NORM
    float eps;
    const float *W0, *W1, *W2;                     // rows of K inputs; ROPE: q | k | v, ACT with pairs: gate | up
    float* out;                                    // OUT / ADD / ACT: row stride ldo
    int ldo, m, K, units;
    const double2* tab;                            // ROPE: rotations [m][hd / 2]; q to out, k and v to the cache planes at pos0 + r
    float *kc, *vc;
    int pos0, H, KH, hd, max_ctx;
};

__device__ __forceinline__ float dpp_sum(float v) {
    v += dpp_move<0x111, 0xf>(0.f, v);
    v += dpp_move<0x112, 0xf>(0.f, v);
    v += dpp_move<0x114, 0xf>(0.f, v);
    v += dpp_move<0x118, 0xf>(0.f, v);
    v += dpp_move<0x142, 0xa>(0.f, v);
    v += dpp_move<0x143, 0xc>(0.f, v);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float dot4(const float4& a, const float4& b, float c) { return fmaf(a.w, b.w, fmaf(a.z, b.z, fmaf(a.y, b.y, fmaf(a.x, b.x, c)))); }

// MR: rows the loops are unrolled for (rows past m repeat the last one and are dropped)
template <int MR, int NF, bool NORM, int EPI>
__global__ __launch_bounds__(256) void gemm_f32_step_kernel(F32Args a) {
    extern __shared__ float xn[];                  // NORM: [m][K]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = a.m, K = a.K, half = a.hd >> 1;
    const int unit = blockIdx.x * 4 + wave, u = min(unit, a.units - 1);
    const int head = EPI == F32_ROPE ? u / half : 0, pi = EPI == F32_ROPE ? u - head * half : 0;
    const float* w[NF];
    if constexpr (EPI == F32_ROPE) {
        const int kind = head < a.H ? 0 : head < a.H + a.KH ? 1 : 2, hh = kind == 0 ? head : kind == 1 ? head - a.H : head - a.H - a.KH;
        const float* W = kind == 0 ? a.W0 : kind == 1 ? a.W1 : a.W2;
        w[0] = W + ((size_t)hh * a.hd + pi) * K;
        w[NF - 1] = w[0] + (size_t)half * K;
    } else {
        w[0] = a.W0 + (size_t)u * K;
        if constexpr (NF == 2) w[1] = a.W1 + (size_t)u * K;
    }
    const int rl = min(lane, m - 1);
    float pre = 0.f;
    double2 rot = make_double2(1.0, 0.0);
    if constexpr (EPI == F32_ADD) pre = a.out[(size_t)rl * a.ldo + u];
    if constexpr (EPI == F32_ROPE) rot = a.tab[rl * half + pi];
    float acc[NF][MR];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int r = 0; r < MR; ++r) acc[f][r] = 0.f;
    if constexpr (NORM) {
        constexpr int KJ = STEP_F32_K / 256, RW = (MR + 3) / 4;
        float4 v[RW][KJ], gn[KJ], wv[NF][KJ];
#pragma unroll
        for (int j = 0; j < KJ; ++j) {
            const int k = min((lane + 64 * j) * 4, K - 4);
#pragma unroll
            for (int i = 0; i < RW; ++i) v[i][j] = *reinterpret_cast<const float4*>(a.x + (size_t)min(wave + 4 * i, m - 1) * K + k);
            gn[j] = *reinterpret_cast<const float4*>(a.gain + k);
#pragma unroll
            for (int f = 0; f < NF; ++f) wv[f][j] = *reinterpret_cast<const float4*>(w[f] + k);
        }
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const int r = wave + 4 * i;
            float ss = 0.f;
#pragma unroll
            for (int j = 0; j < KJ; ++j)
                if ((lane + 64 * j) * 4 < K) ss = dot4(v[i][j], v[i][j], ss);
            const float inv = 1.0f / sqrtf(dpp_sum(ss) / (float)K + a.eps);
#pragma unroll
            for (int j = 0; j < KJ; ++j) {
                const int k = (lane + 64 * j) * 4;
                if (r < m && k < K)
                    *reinterpret_cast<float4*>(xn + (size_t)r * K + k) = make_float4(v[i][j].x * inv * gn[j].x, v[i][j].y * inv * gn[j].y,
                                                                                     v[i][j].z * inv * gn[j].z, v[i][j].w * inv * gn[j].w);
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < KJ; ++j) {
            const int k = (lane + 64 * j) * 4;
            if (k < K) {
#pragma unroll
                for (int r = 0; r < MR; ++r) {
                    const float4 x = *reinterpret_cast<const float4*>(xn + (size_t)min(r, m - 1) * K + k);
#pragma unroll
                    for (int f = 0; f < NF; ++f) acc[f][r] = dot4(wv[f][j], x, acc[f][r]);
                }
            }
        }
    } else {
        constexpr int XJ = MR > 8 ? 1 : 2;         // columns of 256 inputs in flight
        for (int k0 = 0; k0 < K; k0 += 256 * XJ) {
            float4 wv[NF][XJ], x[MR][XJ];
#pragma unroll
            for (int j = 0; j < XJ; ++j) {
                const int k = min(k0 + (lane + 64 * j) * 4, K - 4);
#pragma unroll
                for (int r = 0; r < MR; ++r) x[r][j] = *reinterpret_cast<const float4*>(a.x + (size_t)min(r, m - 1) * K + k);
#pragma unroll
                for (int f = 0; f < NF; ++f) wv[f][j] = *reinterpret_cast<const float4*>(w[f] + k);
            }
#pragma unroll
            for (int j = 0; j < XJ; ++j)
                if (k0 + (lane + 64 * j) * 4 < K) {
#pragma unroll
                    for (int r = 0; r < MR; ++r)
#pragma unroll
                        for (int f = 0; f < NF; ++f) acc[f][r] = dot4(wv[f][j], x[r][j], acc[f][r]);
                }
        }
    }
    float y[NF];                                   // lane r: the sums of row r
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        y[f] = 0.f;
#pragma unroll
        for (int r = 0; r < MR; ++r) {
            const float s = dpp_sum(acc[f][r]);
            y[f] = lane == r ? s : y[f];
        }
    }
    if (lane >= m || unit >= a.units) return;
    const size_t row = (size_t)lane * a.ldo;
    if constexpr (EPI == F32_OUT) a.out[row + u] = y[0];
    else if constexpr (EPI == F32_ADD) a.out[row + u] = pre + y[0];
    else if constexpr (EPI == F32_ACT) a.out[row + u] = NF == 2 ? y[0] / (1.0f + expf(-y[0])) * y[NF - 1] : 0.5f * y[0] * (1.0f + erff(y[0] * 0.70710678118654752f));
    else {
        float p = y[0], q = y[NF - 1];
        if (head < a.H + a.KH) {
            const float rp = (float)((double)p * rot.x - (double)q * rot.y);
            q = (float)((double)p * rot.y + (double)q * rot.x);
            p = rp;
        }
        float* dst = head < a.H ? a.out + row + (size_t)head * a.hd
                     : head < a.H + a.KH ? a.kc + ((size_t)(head - a.H) * a.max_ctx + a.pos0 + lane) * a.hd
                                         : a.vc + ((size_t)(head - a.H - a.KH) * a.max_ctx + a.pos0 + lane) * a.hd;
        dst[pi] = p;
        dst[pi + half] = q;
    }
}

// Attention over a short context and the output projection behind it, h += attention(q) Wo^T, in one launch: such a context is a few
// KB per head, so every workgroup attends for itself and multiplies its output features from LDS.  What bounds it is the chain request -
// scores - sums over the lanes - products; as two launches (attention through LDS behind four barriers, then the projection) it ran
// twice.  60 positions, 4 heads of 32: 1 row 6.8 + 2.4 -> 4.4 us, 5 rows 6.8 + 3.0 -> 7.1 us.  (Several rows in the one-row form, every
// wavefront reading K for itself: 10.7 us with 4 wavefronts, 11.6 with 16 - a lane per position touches 64 lines per request.)
// One row: wavefront w takes heads w, w + 4, ..; contexts of up to 64 P positions.
//   scores      lane = position (P of them), its K row in registers, q broadcast from LDS
//   products    lane = (piece of four columns, one of 256 / HD position classes), P broadcast from LDS, V rows in registers
//   grid ceil(D / 4), block 256; K = H * HD <= STEP_F32_K
__device__ __forceinline__ void f32_out_product(const float4 (&wv)[STEP_F32_K / 256], const float* xo, int K, int lane, float& y) {
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < STEP_F32_K / 256; ++j)
        if ((lane + 64 * j) * 4 < K) acc = dot4(wv[j], *reinterpret_cast<const float4*>(xo + (lane + 64 * j) * 4), acc);
    y = dpp_sum(acc);
}
template <int HD, int P>
__global__ __launch_bounds__(256) void attn_out_f32_kernel(const float* __restrict__ q, const float* __restrict__ kc, const float* __restrict__ vc,
                                                           const float* __restrict__ W, float* __restrict__ h, int pos0, int H, int KH,
                                                           int max_ctx, float scale, int D, TreeBlk tb) {
    constexpr int C4 = HD / 4, CLS = 64 / C4, NV = 64 * P / CLS;     // pieces per row, position classes, V rows per lane
    __shared__ __align__(16) float xo[STEP_F32_K], qs[4][HD];        // attention output, q of the head in hand
    __shared__ float ps[4][64 * P];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int K = H * HD, L = pos0 + 1, u = min((int)blockIdx.x * 4 + wave, D - 1);
    // what the projection needs, requested ahead
    float4 wv[STEP_F32_K / 256];
#pragma unroll
    for (int j = 0; j < STEP_F32_K / 256; ++j) wv[j] = *reinterpret_cast<const float4*>(W + (size_t)u * K + min((lane + 64 * j) * 4, K - 4));
    const float pre = h[u];
    const int pc = lane % C4, cls = lane / C4;
    for (int hd0 = wave; hd0 < H; hd0 += 4) {
        const size_t plane = (size_t)(hd0 / (H / KH)) * max_ctx * HD;
        float4 k[P][C4], v[NV];
#pragma unroll
        for (int a = 0; a < P; ++a)
#pragma unroll
            for (int c = 0; c < C4; ++c) k[a][c] = *reinterpret_cast<const float4*>(kc + plane + (size_t)min(lane + 64 * a, L - 1) * HD + 4 * c);
        const float qv = q[hd0 * HD + min(lane, HD - 1)];
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] = *reinterpret_cast<const float4*>(vc + plane + (size_t)min(cls + CLS * i, L - 1) * HD + 4 * pc);
        if (lane < HD) qs[wave][lane] = qv;
        float s[P], mx = -INFINITY, sum = 0.f;
#pragma unroll
        for (int a = 0; a < P; ++a) {
            s[a] = 0.f;
#pragma unroll
            for (int c = 0; c < C4; ++c) s[a] = dot4(k[a][c], *reinterpret_cast<const float4*>(qs[wave] + 4 * c), s[a]);
            const int p = lane + 64 * a;
            const bool see = p < L && (!tb.on || tree_allowed(tb, p, 0, pos0));
            s[a] = see ? s[a] * scale : -INFINITY;
            mx = fmaxf(mx, s[a]);
        }
        mx = dpp_max(mx);                              // finite: a row sees its own position
#pragma unroll
        for (int a = 0; a < P; ++a) {
            const float e = expf(s[a] - mx);
            ps[wave][lane + 64 * a] = e;
            sum += e;
        }
        sum = dpp_sum(sum);
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const float e = ps[wave][cls + CLS * i];   // positions past the end carry weight 0
            o.x = fmaf(e, v[i].x, o.x); o.y = fmaf(e, v[i].y, o.y); o.z = fmaf(e, v[i].z, o.z); o.w = fmaf(e, v[i].w, o.w);
        }
#pragma unroll
        for (int x = C4; x < 64; x <<= 1) {
            o.x += __shfl_xor(o.x, x, 64); o.y += __shfl_xor(o.y, x, 64); o.z += __shfl_xor(o.z, x, 64); o.w += __shfl_xor(o.w, x, 64);
        }
        if (cls == 0) *reinterpret_cast<float4*>(xo + hd0 * HD + 4 * pc) = make_float4(o.x / sum, o.y / sum, o.z / sum, o.w / sum);
    }
    __syncthreads();
    float y;
    f32_out_product(wv, xo, K, lane, y);
    if (lane == 0 && (int)blockIdx.x * 4 + wave < D) h[u] = pre + y;
}

// Two to MR rows over up to 64 positions, head_dim 32: four heads at a time are staged in LDS once for all rows, and the (head, row)
// pairs are dealt out to 16 wavefronts.   grid ceil(D / 16), block 1024
template <int MR>
__global__ __launch_bounds__(1024) void attn_out_rows_f32_kernel(const float* __restrict__ q, const float* __restrict__ kc, const float* __restrict__ vc,
                                                                 const float* __restrict__ W, float* __restrict__ h, int m, int pos0, int H, int KH,
                                                                 int max_ctx, float scale, int D, TreeBlk tb) {
    constexpr int HD = 32, C4 = 8, RS = HD + 4;        // RS: row stride in LDS
    __shared__ __align__(16) float xo[MR * STEP_F32_K], ks[4][64 * RS], vs[4][64 * RS], qs[MR * 4 * HD];
    __shared__ float ps[16][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), tid = threadIdx.x;
    const int K = H * HD, L = pos0 + m, u = min((int)blockIdx.x * 16 + wave, D - 1);
    float4 wv[STEP_F32_K / 256];
#pragma unroll
    for (int j = 0; j < STEP_F32_K / 256; ++j) wv[j] = *reinterpret_cast<const float4*>(W + (size_t)u * K + min((lane + 64 * j) * 4, K - 4));
    const float pre = h[(size_t)min(lane, m - 1) * D + u];
    const int pc = lane & 7, cls = lane >> 3;
    for (int h0 = 0; h0 < H; h0 += 4) {
        if (h0) __syncthreads();                       // the heads before are done with the buffers
        float4 kr[2], vr[2], qr;
#pragma unroll
        for (int j = 0; j < 2; ++j) {                  // 4 heads x 64 positions x 8 pieces
            const int i = tid + 1024 * j, hh = min(h0 + (i >> 9), H - 1), p = min((i >> 3) & 63, L - 1);
            const size_t at = ((size_t)(hh / (H / KH)) * max_ctx + p) * HD + (i & 7) * 4;
            kr[j] = *reinterpret_cast<const float4*>(kc + at);
            vr[j] = *reinterpret_cast<const float4*>(vc + at);
        }
        {
            const int i = min(tid, m * 32 - 1), r = i >> 5, c = i & 31;            // m rows x 4 heads x 8 pieces
            qr = *reinterpret_cast<const float4*>(q + (size_t)r * K + min(h0 * HD + c * 4, K - 4));
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int i = tid + 1024 * j;
            *reinterpret_cast<float4*>(ks[i >> 9] + ((i >> 3) & 63) * RS + (i & 7) * 4) = kr[j];
            *reinterpret_cast<float4*>(vs[i >> 9] + ((i >> 3) & 63) * RS + (i & 7) * 4) = vr[j];
        }
        if (tid < m * 32) *reinterpret_cast<float4*>(qs + tid * 4) = qr;
        __syncthreads();
        for (int pr = wave; pr < 4 * m; pr += 16) {    // wavefront-uniform
            const int hl = pr & 3, r = pr >> 2;
            if (h0 + hl >= H) continue;
            float s = 0.f;
#pragma unroll
            for (int c = 0; c < C4; ++c) s = dot4(*reinterpret_cast<const float4*>(ks[hl] + lane * RS + 4 * c), *reinterpret_cast<const float4*>(qs + (r * 4 + hl) * HD + 4 * c), s);
            const bool see = lane < L && (tb.on ? tree_allowed(tb, lane, r, pos0) : lane <= pos0 + r);
            s = see ? s * scale : -INFINITY;
            const float e = expf(s - dpp_max(s));      // the maximum is finite: a row sees its own position
            ps[wave][lane] = e;
            const float sum = dpp_sum(e);
            float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float w = ps[wave][cls + 8 * i];
                const float4 v = *reinterpret_cast<const float4*>(vs[hl] + (cls + 8 * i) * RS + 4 * pc);
                o.x = fmaf(w, v.x, o.x); o.y = fmaf(w, v.y, o.y); o.z = fmaf(w, v.z, o.z); o.w = fmaf(w, v.w, o.w);
            }
#pragma unroll
            for (int x = 8; x < 64; x <<= 1) {
                o.x += __shfl_xor(o.x, x, 64); o.y += __shfl_xor(o.y, x, 64); o.z += __shfl_xor(o.z, x, 64); o.w += __shfl_xor(o.w, x, 64);
            }
            if (cls == 0) *reinterpret_cast<float4*>(xo + (size_t)r * K + (h0 + hl) * HD + 4 * pc) = make_float4(o.x / sum, o.y / sum, o.z / sum, o.w / sum);
        }
    }
    __syncthreads();
    float y = 0.f;                                     // lane r: the sum of row r
#pragma unroll
    for (int r = 0; r < MR; ++r) {
        float t;
        f32_out_product(wv, xo + (size_t)min(r, m - 1) * K, K, lane, t);
        y = lane == r ? t : y;
    }
    if (lane < m && (int)blockIdx.x * 16 + wave < D) h[(size_t)lane * D + u] = pre + y;
}

}  // namespace msd
