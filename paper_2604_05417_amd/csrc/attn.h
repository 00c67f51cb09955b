// Attention of short blocks (at most 16 rows of a sequence) over a bf16 cache with head_dim 64 or 128; included after kernels.h,
// batch.h and prefill.h.
#pragma once

#include "attn_plan.h"

namespace msd {

static_assert(ATT_SEGS == MAX_SEGS, "sequences of a launch");

// One workgroup of 4 wavefronts per (span of positions, query heads, sequence).  The rows of hp query heads that share a K/V head
// (hp m <= 16) are the columns of one MFMA operand, so K and V are read once for all of them.  A wavefront walks its sub-blocks of 32
// positions (every fourth of the span) on its own, with a running (maximum, sum, O) per row and no barrier:
//   S^T[pos][row] = K . q^T    A = K rows straight from the cache, B = q as two bf16 terms
//   O^T[hd][row] += V^T . P^T  A = V rows staged in a private piece of LDS and read transposed, B = P as two bf16 terms straight from the
//                              registers that held S^T (slot 8 g + j of the 32 positions stands for 4 g + j or 16 + 4 g + j - 4)
// K and V of the next sub-block are requested as soon as the registers of the current one are free (16 KiB per wavefront at head_dim
// 128, up to 192 KiB per CU); at the end the wavefronts merge through LDS.  One record per workgroup, merged by attn_combine_kernel; a
// span that is the whole context of its sequence needs no merge and the workgroup writes the rows itself.
// What bounds it: HBM (6.6 TB/s with 1024 workgroups or more), for short contexts the chain request - scores - products - merge.
// Measured beside the kernel it replaced (one chunk of 128 positions per workgroup, V staged behind two workgroup barriers and gathered
// element by element), with the merge: 32 heads of 128, 6 rows, 2054 positions 15.5 -> 11.8 us; 12 rows, 8012 positions 42.0 -> 26.1 us
// (8 records per head instead of 63); 32 sequences of 2056 positions (1.05 GB) 211 -> 160 us.
template <int HD>
struct AttnShared {
    static constexpr int RSV = HD + 16;                // V row stride (elements)
    __align__(16) bf16_t v[ATT_NW][32 * RSV];          // .. and at the end the O tile of each wavefront
    float mx[ATT_NW][16], sum[ATT_NW][16];
};

struct AttnOut {
    float* part;       // records [head][nrec][16][HD + 2] (O, maximum, sum per row) of the sequence
    int nrec, rec;
    int direct;        // one record holds the whole context: the rows are written instead of it, to
    float* out;        // [.][H HD] as two bf16 terms (split: see store_terms4)
    int split;
    size_t lo_off;     // elements of the whole block
    int row0, rows;    // first row of the sequence in out and rows to write (past m: padding, copies of the last one)
};

// q: rows of this sequence (lo terms q_lo elements behind the hi terms); h0: first of hp query heads; kb / vb: K and V rows of their K/V
// head; sub-blocks s0 .. s1 - 1.  SHARED: other workgroups read the same K and V rows.
template <int HD, bool SHARED>
__device__ __forceinline__ void attn_body(AttnShared<HD>& sm, const bf16_t* __restrict__ q, size_t q_lo, int H, int h0, int hp,
                                          const bf16_t* __restrict__ kb, const bf16_t* __restrict__ vb, int m, int pos0, float scale, int s0, int s1,
                                          const AttnOut& ao, const TreeBlk* tb) {
    constexpr int KC = HD / 32, NT = HD / 16, VPR = HD / 8, VIT = 32 * VPR / 64, RSV = AttnShared<HD>::RSV;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, g = lane >> 4, L = pos0 + m;
    const bool colok = col < hp * m;
    const int hh = colok ? col / m : hp - 1, row = colok ? col - hh * m : m - 1;      // columns past the last one repeat it
    u32x4 qh[KC], ql[KC];
    {
        const bf16_t* src = q + ((size_t)row * H + h0 + hh) * HD + g * 8;
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            qh[k] = *reinterpret_cast<const u32x4*>(src + k * 32);
            ql[k] = *reinterpret_cast<const u32x4*>(src + q_lo + k * 32);
        }
    }
    // what this lane's row sees of a tree block (tree_allowed): everything below v0, and from there on the nodes of a mask (mode 1) or the
    // positions from v1 on (mode 2), up to its own
    const bool stream = tb && tb->on == 2;
    const int v0 = tb ? (stream ? tb->sink : tb->base) : 0, v1 = stream ? max(tb->base, pos0 + row - tb->i0 + 1) : v0;
    const uint32_t nodes = tb && !stream ? tb->anc[tb->i0 + row] : 0;
    auto next = [&](int s) {                           // streaming caches: sub-blocks no row attends to are passed over
        if (stream)
            while (s < s1 && stream_skips(*tb, s * 32, 32, pos0)) s += ATT_NW;
        return s;
    };
    u32x4 kf[2][KC], vr[VIT];
    // byte offsets of 32 bits against the first row of the span (a span is at most 4 GiB long, a plane can be longer); positions past the
    // end re-read the last one: their weight is zero
    const char *kspan = reinterpret_cast<const char*>(kb) + (size_t)s0 * (32 * HD * 2), *vspan = reinterpret_cast<const char*>(vb) + (size_t)s0 * (32 * HD * 2);
    const int last = L - 1 - s0 * 32;
    auto request_k = [&](int s) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint32_t at = (uint32_t)min((s - s0) * 32 + t * 16 + col, last) * (HD * 2) + g * 16;
#pragma unroll
            for (int k = 0; k < KC; ++k) kf[t][k] = *reinterpret_cast<const u32x4*>(kspan + at + k * 64);
        }
    };
    auto request_v = [&](int s) {
#pragma unroll
        for (int it = 0; it < VIT; ++it) {
            const uint32_t at = (uint32_t)min((s - s0) * 32 + it * (64 / VPR) + lane / VPR, last) * (HD * 2) + (lane % VPR) * 16;
            const u32x4* vp = reinterpret_cast<const u32x4*>(vspan + at);
            vr[it] = SHARED ? *vp : __builtin_nontemporal_load(vp);
        }
    };
    f32x4 o[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    float mx = -INFINITY, sum = 0.f;
    constexpr float L2E = 1.44269504088896341f;
    bf16_t* vs = sm.v[wave];
    int s = next(s0 + wave);
    if (s < s1) { request_k(s); request_v(s); }
    while (s < s1) {
        const int p0 = s * 32, sn = next(s + ATT_NW), sq = min(sn, s1 - 1);    // past the end the last sub-block is requested: no branch around requests
        f32x4 sc[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
#pragma unroll
            for (int k = 0; k < KC; ++k) {
                a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[t][k]), __builtin_bit_cast(bf16x8, qh[k]), a, 0, 0, 0);
                b = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[t][k]), __builtin_bit_cast(bf16x8, ql[k]), b, 0, 0, 0);
            }
            sc[t] = a + b;
        }
        request_k(sq);
        float tm = -INFINITY;
        const bool edge = tb ? stream || p0 + 32 > v0 : p0 + 32 > pos0;    // some row may not see all 32 positions
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float x = sc[t][v] * scale;
                if (edge) {
                    const int p = p0 + t * 16 + g * 4 + v;
                    bool see = p <= pos0 + row;
                    if (tb) see = stream ? see && (p < v0 || p >= v1) : p < v0 || (p - v0 < TREE_MAX && (nodes >> (p - v0)) & 1);
                    x = see && p < L ? x : -INFINITY;
                }
                sc[t][v] = x;
                tm = fmaxf(tm, x);
            }
        tm = fmaxf(tm, __shfl_xor(tm, 16, 64));
        tm = fmaxf(tm, __shfl_xor(tm, 32, 64));
        const float nm = fmaxf(mx, tm), base = nm == -INFINITY ? 0.f : nm;
        const float alpha = __builtin_amdgcn_exp2f((mx - base) * L2E);
        mx = nm;
        float part = 0.f;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float e = __builtin_amdgcn_exp2f((sc[t][v] - base) * L2E);
                sc[t][v] = e;
                part += e;
            }
        sum = sum * alpha + part;
        uint4 ph, pl;
        split_pair(sc[0][0], sc[0][1], ph.x, pl.x);
        split_pair(sc[0][2], sc[0][3], ph.y, pl.y);
        split_pair(sc[1][0], sc[1][1], ph.z, pl.z);
        split_pair(sc[1][2], sc[1][3], ph.w, pl.w);
#pragma unroll
        for (int it = 0; it < VIT; ++it)
            *reinterpret_cast<u32x4*>(vs + (lane / VPR) * RSV + (lane % VPR) * 8 + it * (64 / VPR) * RSV) = vr[it];
        request_v(sq);
        asm volatile("" ::: "memory");                 // a wavefront's own LDS accesses are carried out in program order
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const bf16_t* src = vs + (4 * g + (col >> 2)) * RSV + t * 16 + (col & 3) * 4;
            const s16x4 a0 = lds_read_tr(src), a1 = lds_read_tr(src + 16 * RSV);
            const bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7));
            o[t] *= alpha;
            o[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, __builtin_bit_cast(bf16x8, ph), o[t], 0, 0, 0);
            o[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, __builtin_bit_cast(bf16x8, pl), o[t], 0, 0, 0);
        }
        asm volatile("" ::: "memory");
        s = sn;
    }
    // ---- merge the wavefronts
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    if (g == 0) { sm.mx[wave][col] = mx; sm.sum[wave][col] = sum; }
    constexpr int OS = HD + 4;
    float* ow = reinterpret_cast<float*>(vs);
#pragma unroll
    for (int t = 0; t < NT; ++t) *reinterpret_cast<f32x4*>(ow + col * OS + t * 16 + 4 * g) = o[t];
    __syncthreads();
    const int rows = ao.direct ? ao.rows : m;
    for (int i = tid; i < hp * rows * (HD / 4); i += ATT_NW * 64) {
        const int hr = i / (HD / 4), c4 = (i - hr * (HD / 4)) * 4, hi = hr / rows, r = hr - hi * rows, c = hi * m + min(r, m - 1), h = h0 + hi;
        float M = sm.mx[0][c];
#pragma unroll
        for (int w = 1; w < ATT_NW; ++w) M = fmaxf(M, sm.mx[w][c]);
        f32x4 y = {0.f, 0.f, 0.f, 0.f};
        float tot = 0.f;
#pragma unroll
        for (int w = 0; w < ATT_NW; ++w) {
            const float f = sm.mx[w][c] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((sm.mx[w][c] - M) * L2E);
            y += *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(sm.v[w]) + c * OS + c4) * f;
            tot += sm.sum[w][c] * f;
        }
        if (ao.direct) {
            store_terms4(ao.out, ao.split, ao.lo_off, ((size_t)(ao.row0 + r) * H + h) * HD + c4, make_float4(y[0] / tot, y[1] / tot, y[2] / tot, y[3] / tot));
        } else {
            float* dst = ao.part + (((size_t)h * ao.nrec + ao.rec) * 16 + r) * (HD + 2);
            *reinterpret_cast<float2*>(dst + c4) = make_float2(y[0], y[1]);
            *reinterpret_cast<float2*>(dst + c4 + 2) = make_float2(y[2], y[3]);
            if (c4 == 0) *reinterpret_cast<float2*>(dst + HD) = make_float2(M, tot);
        }
    }
}

// The workgroups of a launch: u = (item, group of query heads).  Groups that share a K/V head and a span are 8 workgroup ids apart and so on
// one XCD, whose L2 they share; the items of a sequence follow each other over the XCDs.
__device__ __forceinline__ int attn_unit(int id, int groups, int& group) {
    const int j = id >> 3;
    group = j % groups;
    return (j / groups) * 8 + (id & 7);
}

// A block of one sequence; spw sub-blocks per workgroup.   grid: attn_grid, block 256
template <int HD, bool TREE, bool SHARED>
__global__ __launch_bounds__(64 * ATT_NW, HD == 128 ? 3 : 4) void attn_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ kc,
                                                                            const bf16_t* __restrict__ vc, int m, int pos0, int H, int KH, int hp,
                                                                            int max_ctx, float scale, int spw, AttnOut ao, TreeBlk tb) {
    __shared__ AttnShared<HD> sm;
    int gi;
    const int u = attn_unit(blockIdx.x, H / (KH * hp), gi), kh = u / ao.nrec;
    if (kh >= KH) return;                              // workgroup-uniform
    const size_t at = (size_t)kh * max_ctx * HD;
    ao.rec = u - kh * ao.nrec;
    ao.direct = ao.nrec == 1;
    attn_body<HD, SHARED>(sm, q, (size_t)m * H * HD, H, kh * (H / KH) + gi * hp, hp, kc + at, vc + at, m, pos0, scale, ao.rec * spw,
                          min((pos0 + m + 31) >> 5, (ao.rec + 1) * spw), ao, TREE ? &tb : nullptr);
}

// Blocks of several sequences: K and V planes of segment s at kc.p[s], vc.p[s] (PTRS) or kv_seq_stride elements per sequence behind
// kc0, vc0; q_lo: elements of the whole block's q.  The records of a segment follow those of the one before; a segment that needs only one
// gets its rows written here and leaves none.  EVEN: every sequence has ao.nrec records, so that an item needs no look-up (0.3 - 0.5 us of
// a launch, 6.7 us for 5 sequences of 333 positions).
template <int HD, bool SHARED, bool PTRS, bool EVEN>
__global__ __launch_bounds__(64 * ATT_NW, HD == 128 ? 3 : 4) void attn_seg_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ kc0,
                                                                                const bf16_t* __restrict__ vc0, size_t kv_seq_stride, SegPtrs kc,
                                                                                SegPtrs vc, Segs sg, int H, int KH, int hp, int max_ctx, float scale,
                                                                                size_t q_lo, int spw, AttnOut ao, AttnItems items) {
    __shared__ AttnShared<HD> sm;
    int gi;
    const int u = attn_unit(blockIdx.x, H / (KH * hp), gi);
    int s, kh, nrec;                                   // sequence and K/V head of the item, records of the sequence
    if constexpr (EVEN) {
        nrec = ao.nrec;
        const int head = u / nrec;
        ao.rec = u - head * nrec;
        s = head / KH;
        kh = head - s * KH;
        if (s >= sg.n) return;                         // workgroup-uniform
    } else {
        if (u >= items.n) return;
        s = 0;
        int r = u;                                     // .. and its place in the sequence
#pragma unroll
        for (int i = 1; i < ATT_SEGS; ++i)
            if (items.first[i] <= u) { s = i; r = u - items.first[i]; }
        nrec = (((sg.pos0[s] + sg.m[s] + 31) >> 5) + spw - 1) / spw;
        kh = r / nrec;
        ao.rec = r - kh * nrec;
    }
    const int m = sg.m[s], pos0 = sg.pos0[s], nsub = (pos0 + m + 31) >> 5;
    const size_t at = (size_t)kh * max_ctx * HD, so = (size_t)sg.seq[s] * kv_seq_stride;
    ao.direct = nrec == 1;
    ao.part += (size_t)s * H * ao.nrec * 16 * (HD + 2);
    ao.row0 = s * sg.ms;
    ao.rows = sg.ms;
    attn_body<HD, SHARED>(sm, q + (size_t)s * sg.ms * H * HD, q_lo, H, kh * (H / KH) + gi * hp, hp, (PTRS ? static_cast<const bf16_t*>(kc.p[s]) : kc0 + so) + at,
                          (PTRS ? static_cast<const bf16_t*>(vc.p[s]) : vc0 + so) + at, m, pos0, scale, ao.rec * spw, min(nsub, (ao.rec + 1) * spw),
                          ao, nullptr);
}

}  // namespace msd
