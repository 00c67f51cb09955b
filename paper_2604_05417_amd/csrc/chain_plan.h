// How a pass of a narrow fp32 model (chain_f32.h) is dealt out over workgroups, and where the words that they exchange go.  Needs nothing of HIP.
#pragma once

#include <algorithm>

namespace msd {

constexpr int CH_NT = 512, CH_WAVES = CH_NT / 64;

// The phases of a pass whose results are exchanged, in their order.  CH_ATTN: blocks of several rows only; CH_HEAD: drafting (one row) only.
enum { CH_QKV, CH_ATTN, CH_OUT, CH_UP, CH_DOWN, CH_HEAD, CH_PHASES };
struct ChainShape { int m, D, H, KH, HD, F, V; };

// Workgroups of a launch: a unit or four per wavefront; more of them wait longer for each other (d 128: 16 of them 120 us, 8 139, 32 126; 256: 32
// 244, 16 271, 64 292; 512: 64 351, 32 376; below 128, a round of 4 drafts: 16 of them 128 - 130 us, d / 8 135 - 137).
constexpr int chain_groups(int D) { return D <= 128 ? 16 : D < 512 ? D / 8 : 64; }

// Units of a phase, dealt out to the workgroups `side` neighbouring ones at a time, as many as leave no workgroup without a unit where there are D:
// 8, all wavefronts, from D 128 on, 2 or 4 below (D is a multiple of 32).  Wavefront w of workgroup g has units chain_first(g, w) + i wavefronts.
constexpr int chain_units(const ChainShape& s, int phase) {
    return phase == CH_QKV ? (s.H + 2 * s.KH) * (s.HD / 2) : phase == CH_ATTN ? s.m * s.H : phase == CH_UP ? s.F : phase == CH_HEAD ? s.V : s.D;
}
constexpr int chain_side(int D) { return D < 64 ? 2 : D < 128 ? 4 : CH_WAVES; }
constexpr int chain_first(int group, int groups, int wave, int side) { return group * side + wave % side + wave / side * side * groups; }
// Words of its results
constexpr int chain_values(const ChainShape& s, int phase) {
    return phase == CH_QKV ? s.m * (s.D + 2 * s.KH * s.HD) : phase == CH_UP ? s.m * s.F : phase == CH_HEAD ? s.V : s.m * s.D;
}

// Exchanges take the regions of the words in turn.  A workgroup writes over the words of exchange e with those of e + CH_REGIONS, and by then
// all must have collected e, or one that still polls for e would never see its tag.  What says so is an exchange between the two in which every
// workgroup has published something: each did so after it collected e, and the writer has collected all of it.  CH_OUT and CH_DOWN are such
// exchanges; the others need not be (20 units of attention for 128 wavefronts, 300 tokens for 512), and at most two of these follow each other: q | k | v
// and attention, or head and q | k | v.  So of any three consecutive exchanges one is complete, and four regions will do.
constexpr int CH_REGIONS = 4;

// Words of a region.  vocab: of the longest vocabulary that is drawn from.
inline unsigned chain_words(const ChainShape& s, int vocab) {
    return (unsigned)std::max(std::max(chain_values(s, CH_QKV), chain_values(s, CH_UP)), std::min(s.V, vocab));
}

}  // namespace msd
