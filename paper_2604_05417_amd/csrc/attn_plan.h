// How the attention of a short block is split over workgroups (attn.h).  Host code that needs nothing of HIP.
#pragma once

#include <algorithm>
#include <cstddef>

namespace msd {

constexpr int ATT_NW = 4;      // wavefronts of a workgroup; each takes every fourth sub-block of 32 positions

// How a block is split.  hp: as many query heads of a K/V head as fit into 16 rows.  All records of a launch span the same number of passes,
// so what decides is the work of the whole block in units of its longest context (wgs; for sequences of one length their number times the
// head groups): a long context among short ones is split as if it were alone.  Records per head: none to merge (one workgroup sees the
// whole context) where that fills the CUs - 32 sequences x 32 heads 160 us against 180 + 10 with three records, 8 x 32 heads 43 against
// 47 + 4 - also nearly (7/8 of them: 12 sequences, half of 3000 and half of 500 positions, a layer 227 against 236 us with two records) or
// with contexts a quarter shorter on average than the longest (8 sequences, half of them half as long, 218 against 224); or where several
// sequences with fewer workgroups than CUs are done sooner so: one workgroup alone on its CU walks 35 GB/s, the full chip does 25 per CU, and
// a merge and the records cost 5.5 us (7B shape, a layer, without and with records: 2 sequences of 333 positions 91.6 / 93.9 us, of 900 100.3 /
// 96.9; 4 of 500 105.3 / 107.5, of 1600 122.3 / 121.0; 5 of 333 118.6 / 124.9, of 1600 136.5 / 139.7; drafter steps of 20 of 1600 66.8 / 72.0);
// or where the context is short (128 KiB of K and V); otherwise up to 8, the most the merge takes in its shortest form, each a whole number
// of passes of its
// wavefronts (65 sub-blocks x 32 heads: 6 records of 3 passes 11.8 us, 8 of 2.25 12.4), and two passes where that still gives half the
// CUs a workgroup (3 sequences of 500 positions: 11.5 against 13.7 us).  Up to 16 where few heads walk a long context (12 heads x 8012
// positions: 11.6 against 13.1 us).
// Per layer, one record per head of every sequence against this rule: 32 sequences, one of 8000 positions and 31 of 64, 256 verification rows of
// the 7B shape 335 -> 284 us, a drafter step (12 heads of 64) 97 -> 66; 8 sequences with one of 8000 232 -> 175; 64 .. 8000 in even
// steps, a drafter step 152 -> 138.
constexpr int ATT_MAX_PASSES = 1 << 16;     // a span's K or V rows of 128: 2 GiB, so that the kernel's byte offsets in it fit into 32 bits
constexpr int ATT_SEGS = 32;   // most sequences of a launch
// The workgroup items of a launch - (sequence, K/V head, record) - without gaps: those of sequence s are first[s] .. first[s + 1] - 1, of n in all
// (past the last sequence: first[s] = n).
struct AttnItems { int n, first[ATT_SEGS + 1]; };
struct AttnPlan {
    int hp, spw, nrec, grid;     // spw: sub-blocks per record; nrec: records of the longest context
    bool even;                   // every sequence has nrec records
    AttnItems items;
};
// len: positions that the sequences see
inline AttnPlan plan_attn(const int* len, int nseg, int H, int KH, int hd, int m, int n_cu, int force_passes) {
    AttnPlan p{};
    const int G = H / KH;
    p.hp = 1;
    for (int t = 2; t <= G && t * m <= 16; ++t)
        if (G % t == 0) p.hp = t;
    int max_len = 1;
    long total = 0;
    for (int s = 0; s < nseg; ++s) { max_len = std::max(max_len, len[s]); total += (len[s] + 31) / 32; }
    const int nsub = (max_len + 31) / 32, all = nseg * (H / p.hp), wgs = (int)std::max(1L, total * (H / p.hp) / nsub);
    auto passes_of = [&](int records) { return (nsub + ATT_NW * records - 1) / (ATT_NW * records); };
    int passes = force_passes;
    if (passes <= 0) {
        const bool full = all >= n_cu && (wgs * 8 >= n_cu * 7 || wgs * 4 >= all * 3);
        const double kv = (double)max_len * hd * 4;       // bytes
        const bool few = nseg > 1 && all < n_cu && kv * (1 / 35e3 - wgs / (25e3 * n_cu)) <= 5.5;
        if (full || few || kv <= 128 * 1024) passes = passes_of(1);
        else {
            passes = passes_of(std::min(8, (3 * n_cu / 2 + wgs - 1) / wgs));
            if (passes == 1 && wgs * ((nsub + 2 * ATT_NW - 1) / (2 * ATT_NW)) >= n_cu / 2) passes = 2;
            if (passes > 4 && wgs * 8 <= n_cu / 2) passes = passes_of(16);
        }
    }
    p.spw = ATT_NW * std::min(passes, ATT_MAX_PASSES);
    p.nrec = (nsub + p.spw - 1) / p.spw;
    for (int s = 0; s < ATT_SEGS; ++s) p.items.first[s + 1] = p.items.first[s] + (s < nseg ? KH * (((len[s] + 31) / 32 + p.spw - 1) / p.spw) : 0);
    p.items.n = p.items.first[nseg];
    p.even = p.items.n == nseg * KH * p.nrec;
    p.grid = 8 * ((p.items.n + 7) / 8) * (G / p.hp);
    return p;
}

}  // namespace msd
