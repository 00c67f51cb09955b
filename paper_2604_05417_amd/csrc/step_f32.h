// fp32 models, blocks of rows of at most STEP_F32_K inputs: GEMMs with what stands before and behind them; included after kernels.h.
#pragma once

namespace msd {

// A layer of a narrow fp32 model moves a few hundred KB, so its time is its launches: 2 - 4 us each, ten of them, of which six (norms,
// rotation, merge, activation, residual) only hand rows from one GEMM to the next.  Here the GEMM that reads a row normalises it and the
// GEMM that makes it rotates, activates or adds it: five launches per layer.
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

}  // namespace msd
