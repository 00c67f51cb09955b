// Kernels for blocks of rows that belong to several sequences (batch > 1), and the bf16 GEMM for
// more than 16 rows.  Included after kernels.h; the single-sequence kernels there stay as they are.
//
// A block is a list of segments: segment s holds rows [s*ms, s*ms + m[s]) - the tokens of sequence
// seq[s] at positions pos0[s] .. pos0[s] + m[s] - 1.  All segments are ms rows apart (ms = the longest
// segment of the block, <= 16); rows j >= m[s] of a segment are padding: they are computed like the
// segment's last row, write no K/V and are never read back.  A verification block has m[s] = gamma + 1
// for every sequence (no padding), a draft step m[s] = 1; only catch-up blocks are ragged.
#pragma once

#include <type_traits>

namespace msd {

constexpr int MAX_SEGS = 32;

struct Segs {
    int n, ms;
    int seq[MAX_SEGS], m[MAX_SEGS], pos0[MAX_SEGS];
};

struct SeqTab { int v[MAX_SEGS]; };
static_assert(MAX_SEGS == ROUND_TAB, "one round word per sequence of a batch");

// Blocks whose segments run through different models of one shape (the drafter step of a batched round: every
// sequence advances by one token in the drafter its bandit chose).  Segments are ordered by model, so the rows of a
// model are contiguous: group g holds rows [r0[g], r0[g] + m[g]).  Kernels that touch weights or caches take one
// pointer per segment (SegPtrs) or per group (RowGroups).
constexpr int MAX_GROUPS = 8;
struct SegPtrs { const void* p[MAX_SEGS]; };
struct RowGroups {
    int n;
    int r0[MAX_GROUPS], m[MAX_GROUPS];
    const bf16_t* W[MAX_GROUPS][3];
};

// Workgroup barrier that orders LDS accesses only (global loads stay in flight).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// h[r] = E[token of row r]; tokens come from the per-sequence histories hist[seq][max_ctx].   grid (R), block 256
template <typename T>
__global__ void embed_seg_kernel(const int32_t* __restrict__ hist, int max_ctx, const T* __restrict__ E, int d,
                                 float* __restrict__ h, Segs sg) {
    const int r = blockIdx.x, s = r / sg.ms, j = min(r - s * sg.ms, sg.m[s] - 1);
    const size_t t = (size_t)hist[(size_t)sg.seq[s] * max_ctx + sg.pos0[s] + j];
    for (int i = threadIdx.x; i < d; i += blockDim.x) h[(size_t)r * d + i] = El<T>::ld(E[t * d + i]);
}

// The same with one embedding table per segment.
template <typename T>
__global__ void embed_segp_kernel(const int32_t* __restrict__ hist, int max_ctx, SegPtrs E, int d, float* __restrict__ h, Segs sg) {
    const int r = blockIdx.x, s = r / sg.ms, j = min(r - s * sg.ms, sg.m[s] - 1);
    const size_t t = (size_t)hist[(size_t)sg.seq[s] * max_ctx + sg.pos0[s] + j];
    const T* Es = static_cast<const T*>(E.p[s]);
    for (int i = threadIdx.x; i < d; i += blockDim.x) h[(size_t)r * d + i] = El<T>::ld(Es[t * d + i]);
}

// add + RMSNorm with one gain vector per segment (row r belongs to segment r / ms).   grid (R), block 1024
template <typename T>
__global__ __launch_bounds__(1024) void addnorm_segp_kernel(float* __restrict__ h, const float* __restrict__ part, int nsplit,
                                                            size_t sstride, int d, SegPtrs gain, int ms, float eps,
                                                            float* __restrict__ xn, int split) {
    addnorm_body<T>(h, part, nsplit, sstride, d, static_cast<const T*>(gain.p[blockIdx.x / ms]), eps, xn, split);
}

// Rotation table per block row: tab[r][i] = (cos, sin)(position of row r * theta^(-2i/hd)), in fp64.  rowkv != nullptr: also where row r
// goes in a K/V head's plane (elements behind the plane of sequence 0; -1: padding).   grid (R), block hd/2
__global__ void rope_table_seg_kernel(Segs sg, int hd, float theta, double2* __restrict__ tab, long long* __restrict__ rowkv, size_t kv_seq_stride) {
    const int r = blockIdx.x, i = threadIdx.x, half = hd >> 1;
    if (i >= half) return;
    const int s = r / sg.ms, j = min(r - s * sg.ms, sg.m[s] - 1);
    if (rowkv && i == 0) rowkv[r] = r - s * sg.ms < sg.m[s] ? (long long)((size_t)sg.seq[s] * kv_seq_stride + (size_t)(sg.pos0[s] + j) * hd) : -1;
    const double freq = pow((double)theta, -2.0 * (double)i / (double)hd);
    double sn, cs;
    sincos((double)(sg.pos0[s] + j) * freq, &sn, &cs);
    tab[r * half + i] = make_double2(cs, sn);
}

// RoPE + K/V append per block row; kc / vc are the planes of sequence 0, sequence b's are kv_seq_stride
// elements further.   grid (H + 2KH, R), block 64
template <typename T>
__global__ void rope_kv_seg_kernel(const float* __restrict__ part, int nsplit, size_t sstride, int N, Segs sg, int H, int KH,
                                   int hd, const double2* __restrict__ tab, float* __restrict__ q, T* __restrict__ kc,
                                   T* __restrict__ vc, size_t kv_seq_stride, int max_ctx, int interleaved, int q_split) {
    const int r = blockIdx.y, s = r / sg.ms, j = r - s * sg.ms;
    const bool valid = j < sg.m[s];
    const size_t so = (size_t)sg.seq[s] * kv_seq_stride;
    rope_kv_body<T>(part, nsplit, sstride, N, sg.pos0[s] + min(j, sg.m[s] - 1), H, KH, hd, tab, q, kc + so, vc + so, max_ctx,
                    interleaved, q_split, nullptr, valid);
}

// grid (ceil(N / 1024), R)
__global__ __launch_bounds__(256) void rope_kv4_seg_kernel(const float* __restrict__ part, int nsplit, size_t sstride, int N, Segs sg, int H, int KH, int hd,
                                                           const double2* __restrict__ tab, bf16_t* __restrict__ q, bf16_t* __restrict__ kc,
                                                           bf16_t* __restrict__ vc, size_t kv_seq_stride, int max_ctx) {
    const int r = blockIdx.y, s = r / sg.ms, j = r - s * sg.ms;
    const size_t so = (size_t)sg.seq[s] * kv_seq_stride;
    rope_kv4_body(part, nsplit, sstride, N, r, gridDim.y, H, KH, hd, tab, q, kc + so, vc + so, max_ctx, (size_t)sg.pos0[s] + min(j, sg.m[s] - 1), j < sg.m[s]);
}

// The same with the cache planes of each segment given directly (kc.p[s], vc.p[s]: the planes of the segment's
// sequence in its model, at the layer in hand).
template <typename T>
__global__ void rope_kv_segp_kernel(const float* __restrict__ part, int nsplit, size_t sstride, int N, Segs sg, int H, int KH,
                                    int hd, const double2* __restrict__ tab, float* __restrict__ q, SegPtrs kc, SegPtrs vc,
                                    int max_ctx, int interleaved, int q_split) {
    const int r = blockIdx.y, s = r / sg.ms, j = r - s * sg.ms;
    const bool valid = j < sg.m[s];
    rope_kv_body<T>(part, nsplit, sstride, N, sg.pos0[s] + min(j, sg.m[s] - 1), H, KH, hd, tab, q,
                    static_cast<T*>(const_cast<void*>(kc.p[s])), static_cast<T*>(const_cast<void*>(vc.p[s])), max_ctx, interleaved,
                    q_split, nullptr, valid);
}

// Attention partials per (chunk, head, segment); records of segment s start s * H * nch_max chunk records
// into part.   grid (nch_max, H, segments), block 256
template <typename T, int HD>
__global__ __launch_bounds__(256) void attn_partial_seg_kernel(const float* __restrict__ q, const T* __restrict__ kc,
                                                               const T* __restrict__ vc, size_t kv_seq_stride, Segs sg, int H,
                                                               int KH, int max_ctx, float scale, float* __restrict__ part,
                                                               int nch_max) {
    const int s = blockIdx.z, m = sg.m[s], pos0 = sg.pos0[s], c = blockIdx.x;
    if (c * ATT_CH >= pos0 + m) return;                 // workgroup-uniform
    const size_t so = (size_t)sg.seq[s] * kv_seq_stride;
    attn_partial_body<T, HD>(q + (size_t)s * sg.ms * H * HD, kc + so, vc + so, m, pos0, H, KH, max_ctx, scale,
                             part + (size_t)s * H * nch_max * 16 * (HD + 2), nch_max, c, (int)blockIdx.y);
}

// singles: the rows of segments with one record are to be written too (attn_seg_kernel leaves them finished).   grid (H, R), block HD
template <int HD>
__global__ void attn_combine_seg_kernel(const float* __restrict__ part, int nch_max, int H, float* __restrict__ out, int split,
                                        Segs sg, int cpw, int singles) {
    const int r = blockIdx.y, s = r / sg.ms, j = min(r - s * sg.ms, sg.m[s] - 1);
    const int nch = ((sg.pos0[s] + sg.m[s] + ATT_CH - 1) / ATT_CH + cpw - 1) / cpw;    // records: one per cpw * ATT_CH positions
    if (nch == 1 && !singles) return;
    attn_combine_body<HD>(part + (size_t)s * H * nch_max * 16 * (HD + 2), nch, nch_max, H, out, split, (int)blockIdx.x, j, r,
                          (size_t)gridDim.y * H * HD);
}

// out[dst row][n] = sum of split-K partials of block row r, for the rows that carry logits:
//   dst row = seq * out_seq_rows + out_row0 + (last_only ? 0 : j);  last_only: only the last valid row of a segment.
// grid (ceil(N / 256), R), block 256
__global__ void sum_partials_seg_kernel(const float* __restrict__ part, int nsplit, size_t sstride, int N, float* __restrict__ out,
                                        Segs sg, int out_seq_rows, int out_row0, int last_only) {
    const int r = blockIdx.y, s = r / sg.ms, j = r - s * sg.ms;
    const int n = blockIdx.x * 256 + threadIdx.x;
    if (j >= sg.m[s] || (last_only && j != sg.m[s] - 1) || n >= N) return;
    float y = 0.f;
    for (int k = 0; k < nsplit; ++k) y += part[(size_t)k * sstride + (size_t)r * N + n];
    out[((size_t)sg.seq[s] * out_seq_rows + out_row0 + (last_only ? 0 : j)) * N + n] = y;
}

// Draft token of every sequence b from its row of logits (logits + b * row_stride):
//   hist[b * max_ctx + at.v[b]] = token, draft[b * draft_stride] = token.   grid (batch), block 512
__global__ __launch_bounds__(AK_NT) void sample_seq_kernel(const float* __restrict__ logits, size_t row_stride, int V, float T,
                                                           uint64_t seed, RoundTab rt, uint32_t pos,
                                                           int32_t* __restrict__ hist, int max_ctx, SeqTab at,
                                                           int32_t* __restrict__ draft, int draft_stride) {
    __shared__ AkShared sm;
    const int b = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float xp[AK_CH][4];
    ak_load(logits + (size_t)b * row_stride, V, wave, lane, xp);
    int token;
    if (T <= 0.f) {
        token = ak_argmax(xp, sm, wave, lane);
    } else {
        const float u = philox_uniform(seed, (uint32_t)b, rt.v[b], pos, 2u);
        token = T == 1.0f ? sample_rows_body<true>(xp, V, T, u, sm, wave, lane) : sample_rows_body<false>(xp, V, T, u, sm, wave, lane);
    }
    if (threadIdx.x == 0) {
        hist[(size_t)b * max_ctx + at.v[b]] = token;
        draft[(size_t)b * draft_stride] = token;
    }
}

// Commit of the emitted tokens: hist[b][l_b + n_acc[b]] = token[b].   grid (1), block 64
__global__ void commit_tokens_kernel(const int32_t* __restrict__ n_acc, const int32_t* __restrict__ token, int32_t* __restrict__ hist,
                                     int max_ctx, SeqTab l, int batch) {
    const int b = threadIdx.x;
    if (b >= batch) return;
    const int tok = token[b];
    if (tok >= 0) hist[(size_t)b * max_ctx + l.v[b] + n_acc[b]] = tok;
}

// ------------------------------------------------------------------------------------------
// addnorm_kernel's arithmetic (same order of additions, same results) for many rows of d = 1024 COLS columns (COLS = 1: at most 1024, a
// multiple of 4): one 256-thread workgroup per row, every thread COLS float4 columns, the row of h and all partials of a group of NS
// requested at once (up to 36 requests in flight per thread instead of 9: with one workgroup per CU the time goes with the
// number of requests a CU keeps in flight).  NS: the smallest of 2, 4 and 8 that takes all partials at once; with eight slots whatever their
// number (the others re-read the last one) and two barriers per column group 1499 rows of 4096 with two partials took 27.5 us, now 22.0
// (123 MB), 256 rows with four 8.4, now 7.8.       grid (rows), block 256
template <typename T, int COLS, int NS>
__global__ __launch_bounds__(256) void addnorm_rows_kernel(float* __restrict__ h, const float* __restrict__ part, int nsplit, size_t sstride,
                                                           const T* __restrict__ gain, float eps, float* __restrict__ xn, int split, int d1) {
    __shared__ float red[COLS][4];
    const int d = COLS == 1 ? d1 : 1024 * COLS;
    const bool mine = COLS > 1 || (int)threadIdx.x * 4 < d;
    const int r = blockIdx.x;
    float* hr = h + (size_t)r * d;
    const float* pr = part + (size_t)r * d;
    float4 v[COLS], gn[COLS];
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
        const int i = COLS == 1 ? min((int)threadIdx.x * 4, d - 4) : (int)threadIdx.x * 4 + 1024 * c;
        v[c] = *reinterpret_cast<const float4*>(hr + i);
        if constexpr (sizeof(T) == 2) {
            const uint2 w = *reinterpret_cast<const uint2*>(gain + i);
            gn[c] = make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u), __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xffff0000u));
        } else gn[c] = *reinterpret_cast<const float4*>(gain + i);
    }
    if (nsplit > 0) {
        float4 y[COLS];
#pragma unroll
        for (int c = 0; c < COLS; ++c) y[c] = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int s0 = 0; s0 < nsplit; s0 += NS) {
            float4 p[NS][COLS];
#pragma unroll
            for (int u = 0; u < NS; ++u)
#pragma unroll
                for (int c = 0; c < COLS; ++c)
                    p[u][c] = *reinterpret_cast<const float4*>(pr + (size_t)min(s0 + u, nsplit - 1) * sstride + (COLS == 1 ? min((int)threadIdx.x * 4, d - 4) : (int)threadIdx.x * 4 + 1024 * c));
#pragma unroll
            for (int u = 0; u < NS; ++u) {
                const bool on = s0 + u < nsplit;
#pragma unroll
                for (int c = 0; c < COLS; ++c) {
                    y[c].x += on ? p[u][c].x : 0.f; y[c].y += on ? p[u][c].y : 0.f; y[c].z += on ? p[u][c].z : 0.f; y[c].w += on ? p[u][c].w : 0.f;
                }
            }
        }
#pragma unroll
        for (int c = 0; c < COLS; ++c) {
            v[c].x += y[c].x; v[c].y += y[c].y; v[c].z += y[c].z; v[c].w += y[c].w;
            if (mine) *reinterpret_cast<float4*>(hr + threadIdx.x * 4 + 1024 * c) = v[c];
        }
    }
    // sum of squares in addnorm_kernel's order: a thread of its 1024-thread workgroup holds one column per 4096, i.e. the
    // columns c of this thread belong to threads tid + 256 c there - different wavefronts, summed per wavefront first
    float tot = 0.f;
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
        float ss = v[c].x * v[c].x + v[c].y * v[c].y + v[c].z * v[c].z + v[c].w * v[c].w;
        if (!mine) ss = 0.f;
        ss = wave_sum(ss);
        if ((threadIdx.x & 63) == 0) red[c][threadIdx.x >> 6] = ss;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < COLS; ++c)
#pragma unroll
        for (int w = 0; w < 4; ++w) tot += red[c][w];
    const float inv = 1.0f / sqrtf(tot / (float)d + eps);
    if (xn && mine) {
#pragma unroll
        for (int c = 0; c < COLS; ++c) {
            const int i = threadIdx.x * 4 + 1024 * c;
            float4 o;
            o.x = v[c].x * inv * gn[c].x;
            o.y = v[c].y * inv * gn[c].y;
            o.z = v[c].z * inv * gn[c].z;
            o.w = v[c].w * inv * gn[c].w;
            if (split) store_terms4(xn, split, (size_t)gridDim.x * d, (size_t)r * d + i, o);
            else *reinterpret_cast<float4*>(xn + (size_t)r * d + i) = o;
        }
    }
}

}  // namespace msd
