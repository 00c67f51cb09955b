// Many-row GEMM on MFMA: prefill blocks and the verification of a batch.  Included after kernels.h and batch.h.
#pragma once

namespace msd {

// ------------------------------------------------------------------------------------------
//   out[ks][r][n] = sum over K-slice ks of x[r][k] W[n][k],  W in streaming-tile order (1 KiB: 16 features x 32 inputs),
//   x interleaved (store_il4): per row and 32-wide chunk one 128-byte line, 32 hi terms, then 32 lo terms.
// A workgroup of 8 wavefronts, four along the rows and two along the features, owns 64 RB rows x 2 TB tiles of one K-slice;
// a wavefront multiplies 16 RB rows with TB tiles, both terms.  The slice advances one 32-wide chunk per stage: a stage - the
// rows' lines and the tiles' KiBs - goes from memory straight into LDS (global_load_lds_dwordx4, no staging registers), NS
// stages ahead, and a wavefront waits only for the requests of the stage it needs (vmcnt counts), so the stream runs on
// through the barriers.  Both operands are read from LDS: per stage and wavefront 2 RB + TB KiB for 2 RB TB MFMAs.
//   LDS layout of a stage: row r: its 8 pieces of 16 bytes, piece q in position q ^ ((r >> 1) & 7) (conflict-free fragment
// reads); then the tiles as they are.
//   Fragments are held twice: while a stage is multiplied from one set of registers, the next is read from LDS into the other, so one
// barrier per stage is enough, neither the reads nor the waits for them stand between MFMAs, and a stage's buffer is free as soon as it
// has been read - its next request is made NS stages ahead.  The first row block is multiplied before the requests and reads are issued,
// so that the matrix cores start right behind the barrier.
//   What bounds it: from about 500 rows on the quantum of whole tiles per CU and power.  Gate | up of the 7B shape at 1499 rows (192 x 256
// tiles) 391 us with random values, 1.38 PFLOP/s with both terms counted, 331 us with zeros.
// Two groups of wavefronts taking turns between reading and multiplying, two barriers per stage and one register set, were here before;
// on the same card and with the same tiles, 7B shape at 1499 rows: gate | up 457 -> 430 us, q | k | v 268 -> 260, output and down 141 -> 132
// (mean); 511 rows of the 1B shape: gate | up 62.5 -> 56.5, down 37.3 -> 36.2.  Large tiles gained most (192 x 256 9 %, 128 x 256 8,
// 256 x 192 7 over all shapes and splits), small ones lost some (64 x 256 4 %, 128 x 96 3, 64 x 192 2): q | k | v at 256 rows in two
// halves of K 54.5 -> 47.8 with 128 x 256 tiles, 44.1 -> 44.5 with 128 x 192.
//   Workgroup ids are dealt out so that the row blocks of one feature group run on one XCD one after the other (its L2 then
// serves the weights to all of them).
//   grid nrb * ngroups * ksplit, block 512, dynamic LDS NS * (8192 RB + 2048 TB) bytes;
//   nrb = ceil(R / (64 RB)), ngroups = ceil(ntiles / (2 TB)).
// What stands behind the product where K is not split (the sums are finished in the registers of one workgroup):
//   TILES_ACT   out = SiLU(gate) * up (swiglu: local tiles 2 j and 2 j + 1 are gate and up of the same 16 features; TB even) or GELU(up),
//               interleaved terms of rows N long.  Written: 8 bytes per feature instead of 8 + 8 read + 4 by a launch of its own.
//   TILES_ROPE  q | k | v: q rotated as two bf16 arrays, k rotated and v rounded into the cache at position pos0 + row
//   TILES_ADD   out[row][n] += sum (the residual stream)
// Measured at 1499 rows of the 7B shape, per layer: rotation 37 and activation 31 us as launches of their own, gone.
enum { TILES_PART = 0, TILES_ACT = 1, TILES_ROPE = 2, TILES_ADD = 3 };
struct TilesEpi {
    int swiglu;                      // ACT
    int row0;                        // ACT: rows of out in front of this group's
    const double2* tab;              // ROPE: rotations [row][hd / 2]
    bf16_t *kc, *vc;                 // ROPE: cache planes of the layer
    int H, KH, hd, pos0, max_ctx;    // ROPE
};
template <int RB, int TB, int NS, int EPI>
__device__ __forceinline__ void gemm_tiles_body(const bf16_t* __restrict__ x, int R, int kchunks, const bf16_t* __restrict__ W0,
                                                const bf16_t* __restrict__ W1, const bf16_t* __restrict__ W2, int t0, int t1, int ntiles,
                                                float* __restrict__ out, size_t out_sstride, int N, int cps, int nrb, const TilesEpi& ep) {
    extern __shared__ uint4 lds[];
    constexpr int BM = 64 * RB, NT = 2 * TB;
    constexpr int STAGE = BM * 8 + NT * 64;            // 16-byte pieces per stage
    constexpr int NREQ = 8 * RB + NT;                  // requests of 1 KiB per stage: 8 rows each, then one tile each
    constexpr int PER = NREQ / 8, REM = NREQ % 8;      // wavefront w issues PER (w < REM: one more)
    const int n8 = gridDim.x >> 3, r8 = gridDim.x & 7, xcd = blockIdx.x & 7;
    int id = xcd * n8 + min(xcd, r8) + (blockIdx.x >> 3);
    const int rb = id % nrb;
    id /= nrb;
    const int ngroups = (ntiles + NT - 1) / NT, tg = id % ngroups, ks = id / ngroups;
    if (rb * BM >= R) return;                          // a smaller row group (workgroup-uniform, before any barrier)
    const int c0 = ks * cps, nst = min(cps, kchunks - c0);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 1, wc = wave & 1, row16 = lane & 15, g = lane >> 4;
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)lds;

    // this wavefront's requests: id w, w + 8, ..: source (uniform base, advancing with the stage; per-lane offset) and place
    unsigned voff[PER + 1];
    const char* base[PER + 1];
    unsigned step[PER + 1];
#pragma unroll
    for (int j = 0; j <= PER; ++j) {
        const int q = wave + 8 * j;
        if (j < RB) {                                  // (8 RB row requests: j < RB for every wavefront)
            const int row = 8 * q + (lane >> 3), piece = (lane & 7) ^ ((row >> 1) & 7);
            base[j] = reinterpret_cast<const char*>(x) + ((size_t)rb * BM * kchunks + c0) * 128;
            voff[j] = (unsigned)min(row, R - 1 - rb * BM) * (unsigned)kchunks * 128u + (unsigned)piece * 16u;
            step[j] = 128;
        } else {
            int t = min(tg * NT + min(q - 8 * RB, NT - 1), ntiles - 1);
            if (EPI == TILES_ACT && ep.swiglu) t = (t & 1) * t0 + (t >> 1);
            const bf16_t* W;
            int tt;
            if (t < t0) { W = W0; tt = t; }
            else if (t < t1) { W = W1; tt = t - t0; }
            else { W = W2; tt = t - t1; }
            base[j] = reinterpret_cast<const char*>(W) + ((size_t)tt * kchunks + c0) * 1024;
            voff[j] = lane * 16;
            step[j] = 1024;
        }
    }
    auto request = [&](int buf) {                      // the next stage's requests into buffer buf
#pragma unroll
        for (int j = 0; j <= PER; ++j)
            if (j < PER || wave < REM) {
                const unsigned dst = __builtin_amdgcn_readfirstlane(lds0 + (unsigned)(buf * STAGE * 16 + (wave + 8 * j) * 1024));
                const unsigned long long b = (unsigned long long)base[j];
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(voff[j]), "s"(b) : "memory", "m0");
                base[j] += step[j];
            }
    };
    // all but the youngest NS - 2 stages of this wavefront's requests have landed
    auto wait_stage = [&]() {
        if (REM && wave < REM) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((PER + (REM ? 1 : 0)) * (NS - 2)) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER * (NS - 2)) : "memory");
    };
    static_assert((PER + 1) * (NS - 1) < 64, "vmcnt counts to 63");
    f32x4 acc[RB][TB];
#pragma unroll
    for (int a = 0; a < RB; ++a)
#pragma unroll
        for (int i = 0; i < TB; ++i) acc[a][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int xrow = wr * 16 * RB + row16, sw = (xrow >> 1) & 7;     // the same for all row blocks of the wavefront (16 rows apart)
    const int xat_h = xrow * 8 + (g ^ sw), xat_l = xrow * 8 + ((g ^ sw) ^ 4), wat = BM * 8 + wc * TB * 64 + lane;
#pragma unroll
    for (int u = 0; u < NS; ++u)
        if (u < nst) request(u);
    struct Frag { u32x4 w[TB], fh[RB], fl[RB]; };
    auto fetch = [&](Frag& f, int buf) {
        const u32x4* sb = reinterpret_cast<const u32x4*>(lds) + (size_t)buf * STAGE;
#pragma unroll
        for (int i = 0; i < TB; ++i) f.w[i] = sb[wat + 64 * i];
#pragma unroll
        for (int a = 0; a < RB; ++a) { f.fh[a] = sb[xat_h + 128 * a]; f.fl[a] = sb[xat_l + 128 * a]; }
    };
    auto mult = [&](const Frag& f, int a0, int a1) {
#pragma unroll
        for (int a = 0; a < RB; ++a) {
            if (a < a0 || a >= a1) continue;
#pragma unroll
            for (int i = 0; i < TB; ++i)
                acc[a][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f.w[i]), __builtin_bit_cast(bf16x8, f.fh[a]), acc[a][i], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < TB; ++i)
                acc[a][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f.w[i]), __builtin_bit_cast(bf16x8, f.fl[a]), acc[a][i], 0, 0, 0);
        }
    };
    // top of stage st: its fragments are in registers (every wavefront's, behind the barrier: its buffer is free) and stage st + 1 has landed
    auto top = [&](int st) {
        __builtin_amdgcn_sched_barrier(0);
        if (st + NS - 1 < nst) wait_stage();           // stages st + 1 .. st + NS - 1 are on their way
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    Frag fa, fb;
    // the prologue asked for stages 0 .. NS - 1
    if (NS - 1 < nst) {
        if (REM && wave < REM) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((PER + (REM ? 1 : 0)) * (NS - 1)) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER * (NS - 1)) : "memory");
    } else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
    fetch(fa, 0);
    int buf = 0;
    auto stage = [&](int st, const Frag& now, Frag& nxt) {
        top(st);
        const int nb = buf + 1 == NS ? 0 : buf + 1;
        mult(now, 0, 1);
        __builtin_amdgcn_sched_barrier(0);
        if (st + NS < nst) request(buf);
        if (st + 1 < nst) fetch(nxt, nb);
        mult(now, 1, RB);
        buf = nb;
    };
    for (int st = 0; st < nst; st += 2) {
        stage(st, fa, fb);
        if (st + 1 < nst) stage(st + 1, fb, fa);
    }
    if constexpr (EPI == TILES_ROPE) {
        // A lane holds two pairs of a tile, four bytes of each of its results.  They pass through a piece of LDS of this wavefront (the stages
        // are read: every wavefront is behind its last barrier), so that up to TB 16-byte pieces of a row leave side by side: stored
        // from the registers, in pieces of four bytes, q | k | v of the 7B shape at 1499 rows took 263 us, now 246 (without any stores 234).
        constexpr int RS = 4 * (TB | 1), PLANE = 16 * RS;   // words of a row and of the 16 rows; the rows of a store fall into different banks
        static_assert(8 * 4 * PLANE * 4 <= NS * STAGE * 16, "LDS of the results");
        uint32_t* const ws = reinterpret_cast<uint32_t*>(lds) + wave * 4 * PLANE;
        const int half = ep.hd >> 1, sh = 31 - __clz(ep.hd), tw = tg * NT + wc * TB;   // head_dim 64 or 128
#pragma unroll
        for (int a = 0; a < RB; ++a) {
            const int row0 = rb * BM + (wr * RB + a) * 16;
            if (row0 >= R) break;                           // wavefront-uniform
            const double2* tab = ep.tab + (size_t)min(row0 + row16, R - 1) * half + 2 * g;
            uint32_t* const wl = ws + row16 * RS;
#pragma unroll
            for (int i = 0; i < TB; ++i) {
                const f32x4 v = acc[a][i];
                const int n = (tw + i) * 16, head = n >> sh;
                if (head >= ep.H + ep.KH) {                 // wavefront-uniform
                    *reinterpret_cast<uint2*>(wl + (g >> 1) * PLANE + i * 4 + (g & 1) * 2) = make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
                    continue;
                }
                // packed columns 4 g .. are the pairs i, i + 1 (first and second member, hd / 2 apart)
                const int pi = (n & (ep.hd - 1)) >> 1;
                const double2 r0 = tab[pi], r1 = tab[pi + 1];
                const float a0 = (float)((double)v[0] * r0.x - (double)v[1] * r0.y), b0 = (float)((double)v[0] * r0.y + (double)v[1] * r0.x);
                const float a1 = (float)((double)v[2] * r1.x - (double)v[3] * r1.y), b1 = (float)((double)v[2] * r1.y + (double)v[3] * r1.x);
                const uint32_t ah = f2bf2(a0, a1), bh = f2bf2(b0, b1);
                wl[i * 4 + g] = ah;
                wl[PLANE + i * 4 + g] = bh;
                if (head < ep.H) {
                    wl[2 * PLANE + i * 4 + g] = f2bf2(a0 - __uint_as_float(ah << 16), a1 - __uint_as_float(ah & 0xffff0000u));
                    wl[3 * PLANE + i * 4 + g] = f2bf2(b0 - __uint_as_float(bh << 16), b1 - __uint_as_float(bh & 0xffff0000u));
                }
            }
            asm volatile("" ::: "memory");                  // a wavefront's own LDS accesses are carried out in program order
#pragma unroll
            for (int j = 0; j < TB; ++j) {
                // piece: plane (q: first and second members, hi then lo terms; k: first and second members; v: columns 0 - 7 and 8 - 15), row, tile
                const int q = lane + 64 * j, tile = q % TB, r = (q / TB) & 15, kind = q / (16 * TB), t = tw + tile, row = row0 + r;
                const uint4 y = *reinterpret_cast<const uint4*>(ws + kind * PLANE + r * RS + tile * 4);
                const int n = t * 16, head = n >> sh, c = n & (ep.hd - 1);
                const bool isq = head < ep.H, isv = head >= ep.H + ep.KH;
                bf16_t* dst;
                if (isq) dst = reinterpret_cast<bf16_t*>(out) + ((size_t)(kind >> 1) * R + row) * ep.H * ep.hd + n - c;
                else dst = (isv ? ep.vc : ep.kc) + ((size_t)(head - ep.H - (isv ? ep.KH : 0)) * ep.max_ctx + ep.pos0 + row) * ep.hd;
                dst += isv ? c + 8 * (kind & 1) : (c >> 1) + (kind & 1) * half;
                if (row < R && t < ntiles && (isq || kind < 2)) *reinterpret_cast<uint4*>(dst) = y;
            }
            asm volatile("" ::: "memory");
        }
        return;
    }
#pragma unroll
    for (int a = 0; a < RB; ++a) {
        const int row = rb * BM + (wr * RB + a) * 16 + row16;
        if (row >= R) continue;
        if constexpr (EPI == TILES_ACT) {
            bf16_t* orow = reinterpret_cast<bf16_t*>(out);
            auto put = [&](int f, const float (&y)[4]) {        // features f + 4 g ..
                store_terms4(reinterpret_cast<float*>(orow), 2, 0, (size_t)(ep.row0 + row) * N + f + g * 4, make_float4(y[0], y[1], y[2], y[3]));
            };
            float y[4];
            if (ep.swiglu) {
                if constexpr (TB % 2 == 0) {
#pragma unroll
                    for (int i = 0; i < TB; i += 2) {
                        const int t = tg * NT + wc * TB + i;
#pragma unroll
                        for (int e = 0; e < 4; ++e) y[e] = acc[a][i][e] / (1.0f + expf(-acc[a][i][e])) * acc[a][i + 1][e];
                        if (t < ntiles) put(t * 8, y);
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < TB; ++i) {
                    const int t = tg * NT + wc * TB + i;
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] = 0.5f * acc[a][i][e] * (1.0f + erff(acc[a][i][e] * 0.70710678118654752f));
                    if (t < ntiles) put(t * 16, y);
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < TB; ++i) {
                const int t = tg * NT + wc * TB + i;
                if (t >= ntiles) continue;
                const f32x4 v = acc[a][i];
                float4* o = reinterpret_cast<float4*>(out + (EPI == TILES_PART ? (size_t)ks * out_sstride : 0) + (size_t)row * N + (size_t)t * 16 + g * 4);
                if constexpr (EPI == TILES_ADD) {
                    const float4 h = *o;
                    *o = make_float4(h.x + v[0], h.y + v[1], h.z + v[2], h.w + v[3]);
                } else *o = make_float4(v[0], v[1], v[2], v[3]);
            }
        }
    }
}

template <int RB, int TB, int NS, int EPI>
__global__ __launch_bounds__(512) void gemm_tiles_kernel(const bf16_t* __restrict__ x, int R, int kchunks, const bf16_t* __restrict__ W0,
                                                         const bf16_t* __restrict__ W1, const bf16_t* __restrict__ W2, int t0, int t1,
                                                         int ntiles, float* __restrict__ out, size_t out_sstride, int N, int cps, int nrb, TilesEpi ep) {
    gemm_tiles_body<RB, TB, NS, EPI>(x, R, kchunks, W0, W1, W2, t0, t1, ntiles, out, out_sstride, N, cps, nrb, ep);
}

// One launch for several row groups with weights of their own (same shapes): blockIdx.y is the group; its rows [r0, r0 + m) of
// x are multiplied with its matrices into the same rows of out.   grid (as above with the largest m, groups)
template <int RB, int TB, int NS, int EPI>
__global__ __launch_bounds__(512) void gemm_tiles_grouped_kernel(const bf16_t* __restrict__ x, int kchunks, int t0, int t1, int ntiles,
                                                                 float* __restrict__ out, size_t out_sstride, int N, int cps, int nrb,
                                                                 RowGroups gg, TilesEpi ep) {
    static_assert(EPI == TILES_PART || EPI == TILES_ACT, "row groups have partials or activations");
    const int g = blockIdx.y;
    ep.row0 = gg.r0[g];
    gemm_tiles_body<RB, TB, NS, EPI>(x + (size_t)gg.r0[g] * kchunks * 64, gg.m[g], kchunks, gg.W[g][0], gg.W[g][1], gg.W[g][2], t0, t1, ntiles,
                                     EPI == TILES_PART ? out + (size_t)gg.r0[g] * N : out, out_sstride, N, cps, nrb, ep);
}

}  // namespace msd
