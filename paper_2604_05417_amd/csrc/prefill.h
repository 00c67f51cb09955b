// Kernels for long blocks of consecutive rows of one sequence: the prefill of a prompt, and a drafter's catch-up over a
// backlog of committed tokens.  Included after kernels.h and batch.h.
#pragma once

namespace msd {

typedef short s16x4 __attribute__((ext_vector_type(4)));

// the two-term form of a pair: hi = bf16(x), lo = bf16(x - hi)
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& hi, uint32_t& lo) {
    hi = f2bf2(a, b);
    lo = f2bf2(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xffff0000u));
}
// Transposing LDS read: the 16 lanes of a group give the addresses of a 4 x 16 block of 16-bit elements (lane i: row i / 4,
// columns 4 (i % 4) .. + 3); lane i receives column i (rows 0 .. 3).
__device__ __forceinline__ s16x4 lds_read_tr(const bf16_t* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
}

// ------------------------------------------------------------------------------------------
// Causal attention of m consecutive rows (positions pos0 .. pos0 + m - 1; their K/V are in the cache already) over the cache.
// A workgroup of 4 wavefronts takes 64 rows of one head, a wavefront 16 of them, and walks the positions in tiles of 64
// with a running (max, sum, O) per row:
//   S^T[pos][row] = K . q^T   A = K rows from LDS, B = q as two bf16 terms in registers;
//   O^T[hd][row] += V^T . P^T A = V read through the transposing LDS read, B = P as two bf16 terms - straight from the registers
//                             that held S^T: an MFMA sums over k in whatever order its two operands agree on, so slot 8 g + j
//                             of a 32-position chunk stands for position 4 g + j (j < 4) or 16 + 4 g + j - 4, which is where
//                             the lanes of group g already hold the scores.
// What bounds it: the chain of a tile - barrier, scores, maximum, exponentials, products - with two (head_dim 64: four) workgroups of a
// CU to cover it.  Tiles alternate between two buffers in LDS, so a tile has one barrier; while it is multiplied the next is written from
// registers and the one after requested.  Heads are dealt out over the 8 XCDs (workgroup id mod 8) so that the row blocks of one head share
// that XCD's L2, the longest row blocks first.  Measured: 1499 rows x 32 heads of 128: 74 us per layer (18.4 GFLOP causal, twice
// that with the second terms: 0.5 PFLOP/s); 113 us with 128 rows per workgroup, one buffer and two barriers per tile; 1400 rows x 32 heads
// of 64 on 8 K/V heads 42 us (62), 511 rows 11.8 (12.4).  Tiles of 32 positions with twice the workgroups per CU: 78 us.
//   grid (ceil(m / 64) * H), block 256.   out: [m][H HD] as two bf16 terms (split: see store_terms4).
template <int HD>
__global__ __launch_bounds__(256, HD == 128 ? 2 : 4) void attn_prefill_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ kc,
                                                              const bf16_t* __restrict__ vc, int m, int pos0, int H, int KH, int max_ctx,
                                                              float scale, float* __restrict__ out, int split) {
    constexpr int TP = 64, KC = HD / 32, NT = HD / 16, VPR = HD / 8;
    constexpr int RSV = HD + 16;                       // V row stride (elements): 8 consecutive rows fall into different banks
    constexpr int IT = TP * VPR / 256;                 // 16-byte pieces of a tile per thread
    __shared__ __align__(16) bf16_t kbuf[2][TP * HD];  // piece p of row r in position p ^ (r & 7)
    __shared__ __align__(16) bf16_t vbuf[2][TP * RSV];
    const int nblk = (m + 63) / 64;
    int h, blk;
    if ((H & 7) == 0) {
        const int idx = blockIdx.x >> 3;
        h = (blockIdx.x & 7) + 8 * (idx / nblk);
        blk = nblk - 1 - idx % nblk;
    } else {
        h = blockIdx.x / nblk;
        blk = nblk - 1 - blockIdx.x % nblk;
    }
    const int kh = h / (H / KH);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, row = lane & 15, g = lane >> 4;
    const int r0 = blk * 64 + wave * 16;     // this wavefront's first row
    const size_t q_lo = (size_t)m * H * HD;
    uint4 qh[KC], ql[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        const bf16_t* src = q + (size_t)min(r0 + row, m - 1) * H * HD + (size_t)h * HD + k * 32 + g * 8;
        qh[k] = *reinterpret_cast<const uint4*>(src);
        ql[k] = *reinterpret_cast<const uint4*>(src + q_lo);
    }
    f32x4 o[NT];
    float mx = -INFINITY, ls = 0.f;
#pragma unroll
    for (int t = 0; t < NT; ++t) o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int L = pos0 + min(m, (blk + 1) * 64);       // positions this workgroup's rows can see
    const int last_pos = pos0 + min(r0 + 16, m) - 1;   // .. and this wavefront's
    const bf16_t* kb = kc + (size_t)kh * max_ctx * HD;
    const bf16_t* vb = vc + (size_t)kh * max_ctx * HD;
    u32x4 kr[IT], vr[IT];
    auto request = [&](int p0) {                       // rows past the end re-read the last row: their weight is zero
        // byte offsets of 32 bits (addresses of 64 bits per piece do not fit in the registers) against the base of the tile, which is uniform:
        // a whole plane can be longer than 4 GiB
        const char *kt = reinterpret_cast<const char*>(kb) + (size_t)p0 * (HD * 2), *vt = reinterpret_cast<const char*>(vb) + (size_t)p0 * (HD * 2);
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const uint32_t at = (uint32_t)min(it * (256 / VPR) + tid / VPR, L - 1 - p0) * (HD * 2) + (tid % VPR) * 16;
            kr[it] = *reinterpret_cast<const u32x4*>(kt + at);
            vr[it] = *reinterpret_cast<const u32x4*>(vt + at);
        }
    };
    auto stage = [&](int b) {
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int p = it * (256 / VPR) + tid / VPR, v = tid % VPR;
            *reinterpret_cast<u32x4*>(kbuf[b] + p * HD + ((v ^ (p & 7)) * 8)) = kr[it];
            *reinterpret_cast<u32x4*>(vbuf[b] + p * RSV + v * 8) = vr[it];
        }
    };
    request(0);
    stage(0);
    request(min(TP, L - 1));
    const float sc = scale * 1.44269504088896341f;     // scores in units of log2
    for (int p0 = 0, b = 0; p0 < L; p0 += TP, b ^= 1) {
        lds_barrier();                                 // this tile is staged, and the readers of the one before are done
        if (p0 + TP < L) {
            stage(b ^ 1);
            request(min(p0 + 2 * TP, L - 1));
        }
        const bf16_t *ks = kbuf[b], *vs = vbuf[b];
        if (p0 > last_pos) continue;                   // wavefront-uniform: nothing of this tile is visible to its rows
        f32x4 s[TP / 16];
#pragma unroll
        for (int t = 0; t < TP / 16; ++t) {
            s[t] = f32x4{0.f, 0.f, 0.f, 0.f};
            const int p = t * 16 + row;
#pragma unroll
            for (int k = 0; k < KC; ++k) {
                const bf16x8 kf = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(ks + p * HD + (((k * 4 + g) ^ (p & 7)) * 8)));
                s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, __builtin_bit_cast(bf16x8, qh[k]), s[t], 0, 0, 0);
                s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, __builtin_bit_cast(bf16x8, ql[k]), s[t], 0, 0, 0);
            }
        }
        const bool edge = p0 + TP - 1 > pos0 + r0;     // some row of the wavefront does not see the whole tile
        uint4 ph[TP / 32], pl[TP / 32];
        const int lim = pos0 + r0 + row - p0 - 4 * g;      // this lane's row sees element (t, v) iff 16 t + v <= lim
        float tm = -INFINITY;
#pragma unroll
        for (int t = 0; t < TP / 16; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float x = (edge && 16 * t + v > lim) ? -INFINITY : s[t][v] * sc;
                s[t][v] = x;
                tm = fmaxf(tm, x);
            }
        tm = fmaxf(tm, __shfl_xor(tm, 16, 64));
        tm = fmaxf(tm, __shfl_xor(tm, 32, 64));
        const float nm = fmaxf(mx, tm);         // finite: every row sees position 0, in the first tile
        const float alpha = __builtin_amdgcn_exp2f(mx - nm);
        mx = nm;
        float sum = 0.f;
#pragma unroll
        for (int t = 0; t < TP / 16; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float e = __builtin_amdgcn_exp2f(s[t][v] - nm);
                s[t][v] = e;
                sum += e;
            }
        ls = ls * alpha + sum;
#pragma unroll
        for (int t = 0; t < NT; ++t) o[t] *= alpha;
#pragma unroll
        for (int c = 0; c < TP / 32; ++c) {
            split_pair(s[2 * c][0], s[2 * c][1], ph[c].x, pl[c].x);
            split_pair(s[2 * c][2], s[2 * c][3], ph[c].y, pl[c].y);
            split_pair(s[2 * c + 1][0], s[2 * c + 1][1], ph[c].z, pl[c].z);
            split_pair(s[2 * c + 1][2], s[2 * c + 1][3], ph[c].w, pl[c].w);
        }
#pragma unroll
        for (int c = 0; c < TP / 32; ++c)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const bf16_t* src = vs + (c * 32 + 4 * g + (row >> 2)) * RSV + t * 16 + (row & 3) * 4;
                const s16x4 a0 = lds_read_tr(src), a1 = lds_read_tr(src + 16 * RSV);
                const bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7));
                o[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, __builtin_bit_cast(bf16x8, ph[c]), o[t], 0, 0, 0);
                o[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, __builtin_bit_cast(bf16x8, pl[c]), o[t], 0, 0, 0);
            }
    }
    float sum = ls;
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    const float inv = 1.0f / sum;
    const int r = r0 + row;
    if (r < m) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
            store_terms4(out, split, q_lo, (size_t)r * H * HD + (size_t)h * HD + t * 16 + 4 * g,
                         make_float4(o[t][0] * inv, o[t][1] * inv, o[t][2] * inv, o[t][3] * inv));
    }
}

}  // namespace msd
