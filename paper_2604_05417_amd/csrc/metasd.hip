// Host side of the MetaSD hot-path library: C ABI (include/metasd.h), launch plans, bandit.
// Device memory is never allocated here; every buffer comes from the caller.
#include "../../include/metasd.h"

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "kernels.h"
#include "batch.h"
#include "prefill.h"
#include "attn.h"
#include "gemm_tiles.h"
#include "step.h"
#include "step_f32.h"
#include "chain_f32.h"

using namespace msd;

// Scratch of metasd_accept_logits_noalloc: candidates and exchange words of up to METASD_ACCEPT_NOALLOC_MAX_ITEMS
// (row, position) items.  Every GPU the library runs on holds its own copy at its own address; host code reaches it
// only through the per-device pointer that noalloc_scratch() asks the runtime for.
static __device__ __align__(256) unsigned char scratch[(size_t)METASD_ACCEPT_NOALLOC_MAX_ITEMS * 336];

namespace {

thread_local std::string g_err = "";

int fail_global(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

constexpr int PER_LAYER = 9;
constexpr int MAX_ROWS = 16;
constexpr int BIG_ROWS = 2048;                // most rows of one sequence that go through a model in one pass (forward_big)
constexpr size_t ALIGN = 256;
constexpr int LDS_BUDGET = 60 * 1024;
constexpr size_t FULLK_LDS_MAX = 150 * 1024;   // gemm_fullk_residual_kernel: the whole activation block in LDS

size_t align_up(size_t x) { return (x + ALIGN - 1) / ALIGN * ALIGN; }
size_t elem_size(const metasd_model_desc& d) { return d.dtype == METASD_BF16 ? 2 : 4; }

struct Model {
    metasd_model_desc d{};
    std::vector<const void*> w;
    void* kv = nullptr;
    bool shared_kv = false;  // an early-exit drafter whose layers are the target's first n_layers and whose cache IS the target's
    int kv_layers = 0;       // layers of the cache buffer behind kv (the target's count for a shared cache): sequence stride
    int hd = 0;
    std::vector<int> kvl;   // positions valid in the KV cache, per sequence
    bool head = false;      // a drafter head on the target's hidden states (metasd_set_drafter_head): see forward_rows
    const void* fc = nullptr;   // its input projection W_fc [d][2 d]
    bool stream = false;    // a drafter with a streaming cache (cfg.stream_sink, cfg.stream_window): see forward()
    int tail = 0;           // streaming cache: first position of the contiguous tail (what lies between the sinks and it was skipped)
    const void** d_table = nullptr;   // device copy of w
    const void* layer_w(int L, int i) const { return w[1 + PER_LAYER * L + i]; }
    const void* final_norm() const { return w[1 + PER_LAYER * d.n_layers]; }
    const void* lm_head() const { return w[2 + PER_LAYER * d.n_layers]; }
};

// split of one GEMM launch
struct Split {
    int ksplit, cps, tpb;
    size_t lds;
};

int env_int(const char* name, int dflt) { const char* e = getenv(name); return e ? atoi(e) : dflt; }
// Launch epoch of tagged exchange words (see tw_put in kernels.h): unique per launch in this process, never 0.
// Epochs 0 (a zero-filled buffer) and 1 (the accept flag the one-workgroup accept path leaves in the upper half of a
// candidate word) are never handed out.
std::atomic<uint32_t>& epoch_counter() {
    static std::atomic<uint32_t> e{1};
    return e;
}
uint32_t next_epoch() {
    std::atomic<uint32_t>& e = epoch_counter();
    uint32_t v = ++e;
    while (v < 2) v = ++e;
    return v;
}
// n consecutive ones
uint32_t next_epochs(uint32_t n) {
    std::atomic<uint32_t>& e = epoch_counter();
    uint32_t v = e.fetch_add(n) + 1;
    while (v < 2 || v + n < v) v = e.fetch_add(n) + 1;
    return v;
}
// Polls after which a workgroup gives up a wait for another one.  Split-K siblings are neighbours in the order of dispatch and wait for one
// another's product: 2^18, a few tenths of a second.  The workgroups of a chain (chain_f32.h) need all of them resident and may wait for one that
// has no place yet behind another stream's kernels: 2^22.
int gemm_spin_limit(int dflt) { return std::max(0, env_int("METASD_GEMM_SPIN_LIMIT", dflt)); }
constexpr int KS_CAP = 8;            // split-K siblings wanted for parallelism (LDS capacity can ask for more)
constexpr int ks_cap() { return KS_CAP; }

Split choose_split(int m, int ntiles, int kchunks) {
    constexpr int target_units = 3072, align = 8;   // wavefront work units aimed for; slices are multiples of 8 chunks (whole load groups)
    const int cps_max = std::max(1, ((LDS_BUDGET / 32 / m) - 1) / 4);   // two bf16 terms per activation
    int want = target_units / ntiles;                             // aim for about 3072 wavefront work units, never fewer tiles' worth
    want = std::max(1, std::min(want, ks_cap()));
    want = std::min(want, std::max(1, kchunks / 8));              // at least 8 chunks per slice
    int ks = std::max(want, (kchunks + cps_max - 1) / cps_max);   // LDS capacity wins
    int cps = (kchunks + ks - 1) / ks;
    if (align > 1 && (cps + align - 1) / align * align <= cps_max) cps = (cps + align - 1) / align * align;
    ks = (kchunks + cps - 1) / cps;
    Split s;
    s.ksplit = ks;
    s.cps = cps;
    s.tpb = 4;
    s.lds = (size_t)2 * m * (cps * 4 + 1) * 16;
    return s;
}

// Many-row GEMM (gemm_tiles.h; more than 16 rows): workgroup tile (64 rb rows x 2 tb feature tiles, ns stages of LDS) and K
// split.  The launch runs in rounds of 256 workgroups.  A stage of 32 inputs takes 0.158 + 0.0374 rb tb us, a round 1.1 us besides, a launch
// some 4 us whatever the plan (left out of the cost); few rows are bound by the weight stream, 6.1 TB/s; a set of partials costs 1.93 times
// its traffic at 5 TB/s (written and read again).  The constants are those whose choice loses least over every tile and split of the 7B
// and 1B projections at 17 .. 2048 rows, each timed with the launch that reads its partials (which costs 2 us more among a layer's launches
// than in that loop): 1.2 % to the best plan on average, 12.5 at most (a rotation behind 160 rows of 3072 x 2048, 17.5 against 15.5 us);
// with those fitted to the kernel before (0.115 + 0.044 rb tb, 5.6 TB/s, 1.2) 2.3 and 27 %: gate | up of the 7B shape at 777 rows 312 us in
// tiles of 64 x 192 instead of 245, of the 1B shape at 20 rows with whole K 21.0 instead of 18.7, q | k | v of the 7B shape at 256 rows with
// whole K 60.4 instead of 52.5.
// A split whose partials exceed PARTIALS_MAX never pays (50 us of traffic).
struct RowsPlan { int rb, tb, ksplit, cps, nrb, ngroups; };
constexpr size_t PARTIALS_MAX = (size_t)128 << 20;
// (of two that cost the same the first is taken: 3 x 8 is 4 - 8 % faster than 4 x 6, gate | up of the 7B shape at 1499 rows 384 against 404 us)
constexpr int ROWS_TILES[][2] = {{3, 8}, {4, 6}, {3, 6}, {3, 4}, {2, 8}, {2, 6}, {2, 4}, {2, 3}, {1, 8}, {1, 6}, {1, 4}, {1, 2}};
// Stages of LDS of a tile: three of 40 KiB and more, else four or six (144 KiB at most); four for the two smallest, so that several
// workgroups share a CU.
constexpr int rows_stages(int rb, int tb) {
    return rb * 8 + tb * 2 >= 40 ? 3 : rb * 8 + tb * 2 >= 28 || (rb == 2 && tb == 4) || (rb == 1 && tb <= 4) ? 4 : 6;
}

//   behind: what is done with the sums besides storing them, in the launch itself where K is whole (TILES_ACT: pairs of tiles for SwiGLU;
// TILES_ROPE: 1.43 times the sums' traffic in all), else in a launch of its own, 3.2 us and the traffic of its results.  These
// are the same for every split, so that of the plans with partials the cheapest is the one that BEHIND_NONE would give.
enum { BEHIND_NONE = 0, BEHIND_ACT = 1, BEHIND_PAIRS = 2, BEHIND_ROPE = 3 };
RowsPlan plan_rows(int ntiles, int kchunks, int R, int groups, int forced_tpb, int forced_rb, int behind) {
    RowsPlan best{};
    double best_cost = 1e30;
    const double stream = (double)groups * ntiles * kchunks * 1024 / 6.1e6;
    for (const auto& t : ROWS_TILES) {
        const int rb = t[0], tb = t[1];
        if ((forced_tpb && 2 * tb != forced_tpb) || (forced_rb && rb != forced_rb)) continue;
        if (!forced_rb && rb > 1 && 64 * (rb - 1) >= R) continue;
        const int nrb = (R + 64 * rb - 1) / (64 * rb), ng = (ntiles + 2 * tb - 1) / (2 * tb);
        for (int ks = 1; ks <= 8 && (ks == 1 || (kchunks / ks >= 8 && (size_t)ks * R * groups * ntiles * 64 <= PARTIALS_MAX)); ++ks) {
            const int cps = (kchunks + ks - 1) / ks, k2 = (kchunks + cps - 1) / cps;
            const double rounds = (nrb * ng * k2 * groups + 255) / 256;
            const double mult = rounds * (cps * (0.158 + 0.0374 * rb * tb) + 1.1);
            const double sums = (double)R * groups * ntiles * 64 / 5e6;      // R: rows of a group
            const bool whole = k2 == 1 && (behind != BEHIND_PAIRS || tb % 2 == 0);
            const double cost = std::max(mult, stream) + 0.27 * std::min(mult, stream) +
                                (behind == BEHIND_NONE ? 1.93 * k2 * sums : whole ? 1.43 * sums : 1.93 * k2 * sums + 3.2 + 0.29 * sums);
            if (cost < best_cost) { best_cost = cost; best = RowsPlan{rb, tb, k2, cps, nrb, ng}; }
        }
    }
    return best.rb ? best : plan_rows(ntiles, kchunks, R, groups, 0, 0, behind);   // a forced pair that is no tile
}

const char* check_model(const metasd_model_desc& d, const char* who, char* buf, size_t n) {
    auto bad = [&](const char* what) { snprintf(buf, n, "%s: %s", who, what); return buf; };
    if (d.n_layers < 1 || d.d_model < 1 || d.n_heads < 1 || d.n_kv_heads < 1 || d.d_ffn < 1 || d.vocab < 1) return bad("non-positive dimension");
    if (d.d_model % d.n_heads) return bad("d_model not divisible by n_heads");
    if (d.n_heads % d.n_kv_heads) return bad("n_heads not divisible by n_kv_heads");
    const int hd = d.d_model / d.n_heads;
    if (hd != 32 && hd != 64 && hd != 128) return bad("head_dim must be 32, 64 or 128");
    if (d.act != METASD_GELU && d.act != METASD_SWIGLU) return bad("act");
    if (d.dtype != METASD_F32 && d.dtype != METASD_BF16) return bad("dtype");
    if (d.dtype == METASD_F32 && hd > 64) return bad("fp32 models support head_dim <= 64");
    if (d.vocab % 4 || d.vocab > AK_WAVES * AK_SEG) return bad("vocab must be a multiple of 4 and <= 32768");
    if (d.dtype == METASD_BF16) {
        if (d.d_model % 32 || d.d_ffn % 32) return bad("bf16: d_model and d_ffn must be multiples of 32");
        if (d.vocab % 16) return bad("bf16: vocab must be a multiple of 16");
    } else if (d.d_model % 4 || d.d_ffn % 4) return bad("fp32: d_model and d_ffn must be multiples of 4");
    if (!(d.rms_eps > 0.f) || !(d.rope_theta > 0.f)) return bad("rms_eps / rope_theta must be positive");
    return nullptr;
}

// Models whose long blocks take forward_big, and the rows such a block can have in a context.
bool big_ok(const metasd_model_desc& d) { return d.dtype == METASD_BF16 && d.d_model / d.n_heads >= 64; }
int big_rows(const metasd_config& c) { return std::min(BIG_ROWS, c.max_ctx); }

// Whether n rows (more than MAX_ROWS) from position pos0 on are faster through forward_big than in blocks of 16, which nseq sequences
// share.  Few rows leave attn_prefill_kernel one workgroup per head, which walks all positions before it: 1.0 (head_dim 64) or 1.6 us
// per 64 positions and layer but the last, where the 16-row kernels deal the positions out over the chip (7.2 TB/s, at least 0.03 us).
// Otherwise a layer takes its weights' time (7 TB/s) and 25 us against 54 us per 16-row block.  Measured after 18 .. 192 rows behind 500 ..
// 32000 positions, 2 to 6 layers, 768 x 12 heads of 64 to 4096 x 32 of 128: the choice costs 0.06 % on average, 5.5 % at most.  Draft step of two
// layers at context 32000, big / small: 768 x 12 heads after 48 rows 642 / 551 us, 4096 x 32 1249 / 1505; of six, 768 x 12 after 64 2937 / 2033.
// From position 0 the big block always wins.
bool big_pays(const metasd_model_desc& d, int pos0, int n, int nseq) {
    const double hd = d.d_model / d.n_heads, D = d.d_model, walk = (pos0 + n) / 64.0;
    const double w = (2 * D * D + 2 * D * d.n_kv_heads * hd + (d.act == METASD_SWIGLU ? 3 : 2) * D * d.d_ffn) * 2 / 7e6;
    const double small = (double)n / (MAX_ROWS * nseq) * (54 + w + std::max(0.03, d.n_kv_heads * hd * 256 / 7.2e6) * walk);
    return small >= 25 + w + (hd > 64 ? 1.6 : 1.0) * walk * (d.n_layers - 1) / d.n_layers;
}

// Narrow fp32 models whose forward passes are one launch (chain_f32.h), and the words of an exchange region of 16 rows.
bool chain_model(const metasd_model_desc& d) {
    return d.dtype == METASD_F32 && d.d_model <= STEP_F32_K && d.d_ffn <= 4 * STEP_F32_K && d.d_model / d.n_heads <= 64 && d.n_layers <= CH_LAYERS;
}
size_t chain_region(const metasd_model_desc& d) {
    return chain_model(d) ? chain_words({MAX_ROWS, d.d_model, d.n_heads, d.n_kv_heads, d.d_model / d.n_heads, d.d_ffn, d.vocab}, CH_VOCAB) : 0;
}

// Word the split-K siblings of a residual GEMM set when their bounded wait for each other runs out (read back with
// the results of every accept).
struct GridBar { int abort; int pad[3]; };

// Workspace layout shared by metasd_workspace_bytes and metasd_create.
constexpr size_t INV_BYTES = 128;       // 1/rms of 16 rows; places of 16 rows in a plane of the cache
struct Layout {
    size_t hist, h, h2, xn, part, gx, ssq, inv, q, ao, act, apart, rope, P, Q, cand, bd, res, draft, tstep, feat, fest, bar, xchg, chain, tables, table_stride, total;
};

Layout make_layout(const metasd_config& c, const metasd_model_desc& t, const metasd_model_desc* dr) {
    int dmax = t.d_model, fmax = t.d_ffn, vmax = t.vocab, hmax = t.n_heads, hdmax = t.d_model / t.n_heads;
    size_t partmax = 0, gxmax = ALIGN;   // split-K partials of the largest block
    auto acc = [&](const metasd_model_desc& d) {
        // sibling exchange of the residual GEMMs (N = d_model; K = attention width or d_ffn): ksplit - 1 published
        // partial tiles of m rows, for the split choose_split really takes at every block height (LDS capacity
        // can push it past ks_cap())
        if (d.dtype == METASD_BF16)
            for (int m = 1; m <= MAX_ROWS; ++m)
                for (int K : {d.d_model, d.d_ffn})
                    gxmax = std::max(gxmax, (size_t)(choose_split(m, d.d_model / 16, K / 32).ksplit - 1) * m * d.d_model * 8);
        dmax = std::max(dmax, d.d_model); fmax = std::max(fmax, d.d_ffn); vmax = std::max(vmax, d.vocab);
        hmax = std::max(hmax, d.n_heads); hdmax = std::max(hdmax, d.d_model / d.n_heads);
        const int hd = d.d_model / d.n_heads;
        const int ns[5] = {(d.n_heads + 2 * d.n_kv_heads) * hd, d.d_model, (d.act == METASD_SWIGLU ? 2 : 1) * d.d_ffn, d.d_model, d.vocab};
        const int ks[5] = {d.d_model, d.d_model, d.d_model, d.d_ffn, d.d_model};
        if (c.feature_heads && d.dtype == METASD_BF16)   // a drafter head's input projection: N = d, K = 2 d
            partmax = std::max(partmax, (size_t)std::max(choose_split(MAX_ROWS, d.d_model / 16, 2 * d.d_model / 32).ksplit, ks_cap()) *
                                            MAX_ROWS * d.d_model * sizeof(float));
        // the many-row GEMM: one set of partials of the largest block, or any split of it within PARTIALS_MAX
        auto rows_part = [&](int n, size_t rows) {
            return std::max(rows * n * sizeof(float), std::min(PARTIALS_MAX, 8 * rows * n * sizeof(float)));
        };
        if (c.feature_heads && big_ok(d)) partmax = std::max(partmax, rows_part(d.d_model, big_rows(c)));
        for (int i = 0; i < 5; ++i) {
            int ksplit = 1;
            if (d.dtype == METASD_BF16) ksplit = choose_split(MAX_ROWS, ns[i] / 16, ks[i] / 32).ksplit;
            // a smaller m never needs more splits for LDS, but may use up to 8 for parallelism
            ksplit = std::max(ksplit, ks_cap());
            partmax = std::max(partmax, (size_t)ksplit * MAX_ROWS * ns[i] * sizeof(float));
            if (big_ok(d) && i < 4) partmax = std::max(partmax, rows_part(ns[i], big_rows(c)));
            if (c.batch > 1) partmax = std::max(partmax, rows_part(ns[i], (size_t)MAX_ROWS * c.batch));
        }
    };
    acc(t);
    for (int k = 0; k < c.K; ++k) acc(dr[k]);
    const int nchunks = (c.max_ctx + ATT_CH - 1) / ATT_CH;
    Layout L{};
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o += align_up(bytes); return at; };
    bool big = big_ok(t);
    for (int k = 0; k < c.K; ++k) big = big || big_ok(dr[k]);
    const size_t B = (size_t)c.batch, RM = std::max((size_t)MAX_ROWS * B, big ? (size_t)big_rows(c) : 0);   // sequences, rows of the largest block
    L.hist = take(B * c.max_ctx * 4);
    L.h = take(RM * dmax * 4);
    L.h2 = take((size_t)MAX_ROWS * dmax * 4);
    L.xn = take(RM * dmax * 4);
    L.part = take(partmax);
    L.gx = take(gxmax);                                            // tagged partial sums of the residual GEMMs
    L.ssq = take((size_t)(dmax / 16 + 1) * 16 * 4);              // per tile group (or per tile) and row
    L.inv = take(INV_BYTES);
    L.q = take(RM * dmax * 4);
    L.ao = take(RM * dmax * 4);
    L.act = take(RM * std::max(fmax, c.feature_heads ? 2 * dmax : 0) * 4);   // a drafter head's input rows, 2 d wide, are staged here too
    L.apart = take(B * hmax * nchunks * 16 * (hdmax + 2) * 4);
    L.rope = take(RM * (hdmax / 2) * sizeof(double2));
    L.P = take(B * (c.gamma_max + 1) * vmax * 4);
    L.Q = take(B * c.gamma_max * vmax * 4);
    L.cand = take(B * (c.gamma_max + 1) * 2 * sizeof(int2));       // two words per position
    L.bd = take(B * c.gamma_max * sizeof(double));
    L.res = take(std::max<size_t>(128, B * 12));                   // batch 1: also the path of a tree round (2 + 15 words)
    L.draft = take(std::max<size_t>(64, B * (c.gamma_max + 1) * 4)); // chain: gamma tokens per sequence; tree: one per node
    L.tstep = take(TREE_MAX * sizeof(int2));                       // sampled tree rounds: the decision of every node
    L.bar = take(sizeof(GridBar));                                 // bd .. bar: the span read back after every round, kept small
    L.xchg = take(B * (c.gamma_max + 1) * AS_XCHG_BYTES);
    size_t words = chain_region(t);                                // regions of tagged words of the narrow fp32 models
    for (int k = 0; k < c.K; ++k) words = std::max(words, chain_region(dr[k]));
    L.chain = take(c.batch == 1 ? CH_REGIONS * words * 8 : 0);
    // drafter heads: the target's feature of every processed position, and the head's estimate of the latest one
    L.feat = take(c.feature_heads ? (size_t)c.max_ctx * t.d_model * 4 : 0);
    L.fest = take(c.feature_heads ? (size_t)TREE_MAX * t.d_model * 4 : 0);   // one row per tree node (a chain uses row 0)
    int lmax = t.n_layers;
    for (int k = 0; k < c.K; ++k) lmax = std::max(lmax, dr[k].n_layers);
    L.table_stride = align_up((size_t)(1 + PER_LAYER * lmax + 2) * sizeof(void*));
    L.tables = take(L.table_stride * (size_t)(c.K + 1));
    L.total = o;
    return L;
}

// uniform in [0,1) at Philox counter (seq, round, pos, stream): the host twin of philox_uniform
float host_philox_uniform(uint64_t seed, uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3) {
    uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0, n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
        c0 = n0; c1 = (uint32_t)p1; c2 = n2; c3 = (uint32_t)p0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return (float)(c0 >> 8) * (1.0f / 16777216.0f);
}

// Drafter-selection state of one sequence.  UCB is Alg. 2; the others are the algorithms of the
// paper's appendix on switching costs and non-stationary rewards, and its EXP3 / random baselines.
struct Bandit {
    int K = 0, t = 0, policy = METASD_POLICY_UCB, window = 0;
    double beta = 1.0, param = 1.0;
    uint64_t seed = 0;
    uint32_t seq = 0;           // sequence id: first Philox counter word of this bandit's draws
    std::vector<double> mu;     // reported estimate per arm
    std::vector<int> n;         // reported count per arm
    std::vector<double> aux;    // D-UCB: discounted reward sums; EXP3: weights; SH: reward sums of the phase
    std::vector<int> last;      // D-UCB: round of the arm's latest pull
    std::vector<double> prob;   // EXP3: probabilities of the latest select
    std::vector<std::pair<int, double>> recent;   // SW-UCB: (arm, reward) of the rounds in the window, oldest first
    std::vector<int> alive;     // SH: surviving arms, ascending
    int sh_phases = 0, sh_pos = 0;

    void init(const metasd_config& c) {
        K = c.K; beta = c.ucb_beta; policy = c.policy; param = c.policy_param; window = c.policy_window; seed = c.seed;
        reset();
    }
    void reset() {
        t = 0;
        mu.assign(K, 0.0); n.assign(K, 0);
        aux.assign(K, policy == METASD_POLICY_EXP3 ? 1.0 : 0.0);
        last.assign(K, 0);
        prob.assign(K, 1.0 / std::max(K, 1));
        recent.clear();
        alive.resize(K);
        for (int i = 0; i < K; ++i) alive[i] = i;
        sh_phases = 0;
        for (int v = 1; v < K; v <<= 1) ++sh_phases;   // ceil(log2 K)
        sh_pos = 0;
    }
    int ucb_argmax() const {
        int best = 0;
        double bs = -INFINITY;
        for (int i = 0; i < K; ++i) {
            const double s = mu[i] + beta * std::sqrt(2.0 * std::log((double)t) / (double)n[i]);
            if (s > bs) { bs = s; best = i; }
        }
        return best;
    }
    static int draw(const std::vector<double>& p, double u) {   // first arm whose cumulative probability exceeds u
        double c = 0.0;
        for (size_t i = 0; i < p.size(); ++i) {
            c += p[i];
            if (c > u) return (int)i;
        }
        return (int)p.size() - 1;
    }
    int sh_pulls() const { return std::max(1, window / ((int)alive.size() * std::max(sh_phases, 1))); }

    int select() {
        switch (policy) {
            case METASD_POLICY_UCB:
            case METASD_POLICY_DUCB:
                return t < K ? t : ucb_argmax();
            case METASD_POLICY_SWUCB:
                if (t < K) return t;
                for (int i = 0; i < K; ++i)
                    if (n[i] == 0) return i;            // no pull left in the window: no estimate, try it
                return ucb_argmax();
            case METASD_POLICY_EXP3: {
                double tot = 0.0;
                for (double w : aux) tot += w;
                for (int i = 0; i < K; ++i) prob[i] = (1.0 - param) * (aux[i] / tot) + param / (double)K;
                return draw(prob, (double)host_philox_uniform(seed, seq, (uint32_t)t, 0u, 3u));
            }
            case METASD_POLICY_SH:
                return alive.size() == 1 ? alive[0] : alive[sh_pos / sh_pulls()];
            default: {                                   // METASD_POLICY_RANDOM
                std::vector<double> p(K, 1.0 / (double)K);
                return draw(p, (double)host_philox_uniform(seed, seq, (uint32_t)t, 0u, 3u));
            }
        }
    }

    void plain_mean(int k, double r) { mu[k] = (mu[k] * (double)n[k] + r) / (double)(n[k] + 1); n[k] += 1; }

    void update(int k, double r) {
        switch (policy) {
            case METASD_POLICY_DUCB:
                // discounted sum carried from the arm's latest pull: S <- S gamma^(t - t_last) + r
                aux[k] = (n[k] > 0 ? aux[k] * std::pow(param, (double)(t - last[k])) : 0.0) + r;
                last[k] = t;
                n[k] += 1;
                mu[k] = aux[k] / (double)n[k];
                break;
            case METASD_POLICY_SWUCB: {
                recent.emplace_back(k, r);
                if ((int)recent.size() > window) recent.erase(recent.begin());
                std::vector<double> s(K, 0.0);
                std::fill(n.begin(), n.end(), 0);
                for (const auto& e : recent) { s[e.first] += e.second; n[e.first] += 1; }
                for (int i = 0; i < K; ++i) mu[i] = n[i] ? s[i] / (double)n[i] : 0.0;
                break;
            }
            case METASD_POLICY_EXP3: {
                aux[k] *= std::exp(param * (r / prob[k]) / (double)K);
                const double big = *std::max_element(aux.begin(), aux.end());
                if (big > 1e100) {                       // exact power-of-two rescale, probabilities unchanged
                    int e;
                    std::frexp(big, &e);
                    for (double& w : aux) w = std::ldexp(w, -e);
                }
                plain_mean(k, r);
                break;
            }
            case METASD_POLICY_SH:
                plain_mean(k, r);
                if (alive.size() > 1) {
                    aux[k] += r;
                    if (++sh_pos == (int)alive.size() * sh_pulls()) {   // phase over: keep the better half
                        std::vector<int> order = alive;
                        std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return aux[a] > aux[b]; });
                        order.resize((alive.size() + 1) / 2);
                        std::sort(order.begin(), order.end());
                        alive = order;
                        std::fill(aux.begin(), aux.end(), 0.0);
                        sh_pos = 0;
                    }
                }
                break;
            default:                                     // UCB (Alg. 2 mean update), RANDOM
                plain_mean(k, r);
                break;
        }
        t += 1;
    }
};


enum Phase { PH_NONE = 0, PH_READY, PH_DRAFTED, PH_VERIFIED, PH_TREE_DRAFTED, PH_TREE_VERIFIED };

}  // namespace

struct metasd_ctx {
    metasd_config cfg{};
    Model target;
    std::vector<Model> drafters;
    hipStream_t stream = nullptr;
    char* ws = nullptr;
    Layout lay{};
    struct SeqState {
        std::vector<int32_t> hist;   // host mirror of committed tokens
        int l = 0;                   // committed tokens
        int cur_k = -1;              // drafter of the running round
        int round = 0;               // rounds completed since this sequence's context was set: the round word of its Philox counters
        bool ready = false;          // a context has been set
        Bandit bandit;
    };
    std::vector<SeqState> sq;        // one per sequence (cfg.batch)
    int cur_gamma = 0;
    Phase phase = PH_NONE;
    // Pinned host mirror of the workspace span [lay.bd, lay.bar + sizeof(GridBar)): the BD terms, the result words
    // (n_acc, token, mask per sequence), the draft tokens and the abort flag come back in one copy per accept.
    char* hspan = nullptr;
    size_t span_bytes() const { return lay.bar + sizeof(GridBar) - lay.bd; }
    template <typename U> const U* mirror(size_t ws_offset) const { return reinterpret_cast<const U*>(hspan + (ws_offset - lay.bd)); }
    int fetch_results() {          // copy the span and wait for it (the only synchronisation of a round)
        hipError_t e = hipMemcpyAsync(hspan, ws + lay.bd, span_bytes(), hipMemcpyDeviceToHost, stream);
        if (e == hipSuccess) e = hipStreamSynchronize(stream);
        if (e != hipSuccess) return fail(METASD_E_HIP, "reading back the accept results: %s", hipGetErrorString(e));
        return 0;
    }
    std::string err;
    // optional per-launch timing of the three bandwidth-bound kernels (metasd_profile)
    struct ProfRec { hipEvent_t a, b; int kind; double bytes; int n, k, m, model; };   // GEMM launches: N, K, rows, model (-1 target, else drafter)
    bool prof_on = false;
    bool fullk = true;               // residual GEMMs whose input fits in LDS run without split-K (METASD_GEMM_FULLK=0: off)
    bool grouped_on = true;          // batched drafting: one forward per step for all arms (METASD_DRAFT_GROUPED=0: one per arm)
    int att_cpw = 0;                 // attention of short blocks: passes of 128 positions per workgroup, 0 = plan_attn (METASD_ATT_CPW=1..64 forces them)
    int rows_tpb = 0;                // many-row GEMM: feature tiles per workgroup, 0 = by the cost model (METASD_ROWS_TPB=4|6|8|12|16 forces one)
    int rows_rb = 0;                 // .. and its rows in units of 64 (METASD_ROWS_RB=1..4)
    struct { int ntiles, kchunks, R, groups, behind; RowsPlan plan; } plans[64] = {};   // rows_plan
    bool fullk_roll = true;          // .. and larger inputs with rolling private staging (METASD_GEMM_ROLL=0: sibling reduction instead)
    bool gemm_reduce = true;         // bf16 models: residual GEMMs reduce their split-K partials themselves (METASD_GEMM_REDUCE=0: off)
    float cur_eps = 1e-5f;           // rms_eps of the model whose forward is being launched
    bool fuse_small = true;          // short blocks of narrow bf16 models use the GEMMs with fused prologues (METASD_FUSE_SMALL=0: off)
    int n_cu = 0;
    const TreeBlk* tree = nullptr;   // set while a block of draft-tree nodes is being launched (positions and mask of its rows)
    bool embedded = false;           // the one row of the forward being launched is in d_h and its rotations in d_rope already (NextRow)
    bool head_est = false;           // a drafter head's forward takes its own estimates (d_fest) as the feature input (draft steps after the first)
    FeatSrc fsrc{};                  // .. row r the estimate fsrc.idx[r] (chain steps: 0; tree levels: the parent node's)
    TreeShape tshape{};              // the tree of the running round (metasd_draft_tree)
    int tdepth[TREE_MAX] = {};       // depth of every node, tlevel[d] = first node of depth d (tlevel[max depth + 1] = n)
    int tlevel[TREE_MAX + 2] = {};
    int tmaxdepth = 0;
    uint16_t tanc[TREE_MAX] = {};
    int accept_fallbacks = 0;        // accept steps taken again with one workgroup per position after an exchange timeout
    std::vector<ProfRec> prof;       // event pool
    size_t prof_used = 0;
    // Next free record, or nullptr when profiling is off / the pool is used up.  The launcher hands
    // the record's two events to the dispatch itself (hipExtLaunchKernelGGL), so they carry the
    // kernel's own begin and end times rather than those of marker packets around it.
    int cur_model = -1;              // model whose forward is being launched (-1 target, k drafter k): label of the timing records
    ProfRec* prof_take(int kind, double bytes, int n = 0, int k = 0, int m = 0) {
        if (!prof_on || prof_used >= prof.size()) return nullptr;
        ProfRec* r = &prof[prof_used++];
        r->kind = kind;
        r->bytes = bytes;
        r->n = n; r->k = k; r->m = m; r->model = cur_model;
        return r;
    }
    // for launches that cannot carry events (cooperative): marker events on the stream around them
    bool prof_begin(int kind, double bytes) {
        if (!prof_on || prof_used >= prof.size()) return false;
        prof[prof_used].kind = kind;
        prof[prof_used].bytes = bytes;
        return hipEventRecord(prof[prof_used].a, stream) == hipSuccess;
    }
    void prof_end() { (void)hipEventRecord(prof[prof_used].b, stream); ++prof_used; }

    int32_t* d_hist() const { return reinterpret_cast<int32_t*>(ws + lay.hist); }
    float* d_h() const { return reinterpret_cast<float*>(ws + lay.h); }
    void* d_xn() const { return ws + lay.xn; }
    float* d_part() const { return reinterpret_cast<float*>(ws + lay.part); }
    unsigned long long* d_gx() const { return reinterpret_cast<unsigned long long*>(ws + lay.gx); }
    float* d_ssq() const { return reinterpret_cast<float*>(ws + lay.ssq); }
    float* d_inv() const { return reinterpret_cast<float*>(ws + lay.inv); }
    unsigned long long* d_chain() const { return reinterpret_cast<unsigned long long*>(ws + lay.chain); }
    unsigned long long* d_xchg() const { return reinterpret_cast<unsigned long long*>(ws + lay.xchg); }
    float* d_h_pp(int i) const { return reinterpret_cast<float*>(ws + (i ? lay.h2 : lay.h)); }
    void* d_q() const { return ws + lay.q; }
    void* d_ao() const { return ws + lay.ao; }
    void* d_act() const { return ws + lay.act; }
    float* d_apart() const { return reinterpret_cast<float*>(ws + lay.apart); }
    double2* d_rope() const { return reinterpret_cast<double2*>(ws + lay.rope); }
    float* d_P() const { return reinterpret_cast<float*>(ws + lay.P); }
    float* d_Q() const { return reinterpret_cast<float*>(ws + lay.Q); }
    int2* d_cand() const { return reinterpret_cast<int2*>(ws + lay.cand); }
    int2* d_tstep() const { return reinterpret_cast<int2*>(ws + lay.tstep); }
    float* d_feat() const { return reinterpret_cast<float*>(ws + lay.feat); }
    float* d_fest() const { return reinterpret_cast<float*>(ws + lay.fest); }
    double* d_bd() const { return reinterpret_cast<double*>(ws + lay.bd); }
    int32_t* d_res() const { return reinterpret_cast<int32_t*>(ws + lay.res); }
    int32_t* d_draft() const { return reinterpret_cast<int32_t*>(ws + lay.draft); }
    GridBar* d_bar() const { return reinterpret_cast<GridBar*>(ws + lay.bar); }

    int fail(int code, const char* fmt, ...) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        err = buf;
        return code;
    }
};

namespace {

#define HIP_TRY(ctx, expr)                                                                              \
    do {                                                                                                \
        hipError_t e_ = (expr);                                                                         \
        if (e_ != hipSuccess) return (ctx)->fail(METASD_E_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

#define LAUNCH_CHECK(ctx, name)                                                                              \
    do {                                                                                                     \
        hipError_t e_ = hipGetLastError();                                                                   \
        if (e_ != hipSuccess) return (ctx)->fail(METASD_E_HIP, "launch %s: %s", name, hipGetErrorString(e_)); \
    } while (0)

// ---- GEMM launcher: out[.][r][n] over up to three matrices concatenated along n.
// Returns the number of split-K partials written to `part` (their split stride is m*N);
// when direct_out != nullptr the summed result is written there instead and 0 is returned.
template <typename T>
int gemm(metasd_ctx* c, const void* x, int ldx, int m, int K, const void* W0, int n0, const void* W1, int n1,
         const void* W2, int n2, float* direct_out, int* nsplit_out, size_t x_lo_off = 0, const float* ssq = nullptr,
         int ntg = 0, float* inv_out = nullptr, int inv_row0 = 0);

template <>
int gemm<float>(metasd_ctx* c, const void* x, int ldx, int m, int K, const void* W0, int n0, const void* W1, int n1,
                const void* W2, int n2, float* direct_out, int* nsplit_out, size_t, const float*, int, float*, int) {
    const int N = n0 + n1 + n2;
    float* out = direct_out ? direct_out : c->d_part();
    hipLaunchKernelGGL(gemm_f32_kernel, dim3((N + 3) / 4), dim3(256), 0, c->stream, (const float*)x, ldx, m, K,
                       (const float*)W0, (const float*)W1, (const float*)W2, n0, n0 + n1, N, out);
    LAUNCH_CHECK(c, "gemm_f32");
    *nsplit_out = direct_out ? 0 : 1;
    return 0;
}

template <>
// x: the activations as two bf16 arrays, hi at x and lo x_lo_off elements behind it (see store_split4).
// ssq != nullptr: x is h * gain of a residual epilogue, not yet normalised; workgroup 0 writes 1/rms per row
// to inv_out (rows inv_row0 ..) for the consumers of this GEMM's output, and a direct result is scaled by it.
int gemm<bf16_t>(metasd_ctx* c, const void* x, int ldx, int m, int K, const void* W0, int n0, const void* W1, int n1,
                 const void* W2, int n2, float* direct_out, int* nsplit_out, size_t x_lo_off, const float* ssq, int ntg,
                 float* inv_out, int inv_row0) {
    const int N = n0 + n1 + n2;
    const int ntiles = N / 16, kchunks = K / 32;
    const Split s = choose_split(m, ntiles, kchunks);
    const bool direct = direct_out && s.ksplit == 1 && !ssq;     // a scaled result always goes through sum_partials
    float* out = direct ? direct_out : c->d_part();
    const int groups = (ntiles + s.tpb - 1) / s.tpb;
    // algorithmic bytes: every weight once, the activations once, the result once
    metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_GEMM, (double)N * K * 2 + (double)m * K * 4 + (double)m * N * 4, N, K, m);
    GemmPro plain{};
    plain.sstride = x_lo_off;
    if (ssq) { plain.src = ssq; plain.row0 = inv_row0; plain.ns = ntg; plain.h_out = inv_out + inv_row0; plain.eps = c->cur_eps; }
    hipExtLaunchKernelGGL(gemm_bf16_kernel<PRO_PLAIN>, dim3(groups * s.ksplit), dim3(256), (uint32_t)s.lds, c->stream,
                          pr ? pr->a : nullptr, pr ? pr->b : nullptr, 0u, (const float*)x, ldx, m, K, (const bf16_t*)W0,
                          (const bf16_t*)W1, (const bf16_t*)W2, n0 / 16, (n0 + n1) / 16, ntiles, out, N, s.ksplit, s.cps, s.tpb,
                          plain, GemmEpi{});
    LAUNCH_CHECK(c, "gemm_bf16");
    if (direct_out && !direct) {
        const size_t n = (size_t)m * N;
        hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, c->d_part(),
                           s.ksplit, n, n, direct_out, ssq ? (const float*)(inv_out + inv_row0) : nullptr, N);
        LAUNCH_CHECK(c, "sum_partials");
    }
    *nsplit_out = direct_out ? 0 : s.ksplit;
    return 0;
}

// The same projection without split-K (gemm_fullk_residual_kernel): used when the input block fits in LDS
// and there are enough tiles to occupy the CUs.
bool fullk_ok(const metasd_ctx* c, int m, int K, int ntiles, size_t* lds_out) {
    const int cpw = (K / 32 + 7) / 8;
    const size_t lds = (size_t)2 * 8 * m * (cpw * 4 + 1) * 16 + (size_t)8 * 64 * 16;
    *lds_out = lds;
    return c->fullk && lds <= FULLK_LDS_MAX && ntiles * 4 >= c->n_cu * 3;
}

// bf16 GEMM into the residual stream (attention output / FFN down projection): the split-K siblings reduce
// among themselves and the last one updates h, writes h * gain in the two-bf16 form for the next GEMM and the
// per-tile-group sums of squares (EPI_RESIDUAL in kernels.h).  N = d_model.
int gemm_residual(metasd_ctx* c, const void* x, int ldx, int m, int K, const void* W, int N, size_t x_lo_off, float* h,
                  const void* gain_next, float* xsplit, float* ssq, int* ntg_out) {
    const int ntiles = N / 16, kchunks = K / 32;
    size_t lds_full = 0;
    if (fullk_ok(c, m, K, ntiles, &lds_full)) {
        metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_GEMM, (double)N * K * 2 + (double)m * K * 4 + (double)m * N * 4, N, K, m);
        hipExtLaunchKernelGGL(gemm_fullk_residual_kernel, dim3(ntiles), dim3(512), (uint32_t)lds_full, c->stream, pr ? pr->a : nullptr,
                              pr ? pr->b : nullptr, 0u, (const bf16_t*)x, x_lo_off, ldx, m, K, (const bf16_t*)W, ntiles, N, h,
                              (const bf16_t*)gain_next, xsplit, ssq);
        LAUNCH_CHECK(c, "gemm_bf16 (full-K residual)");
        *ntg_out = ntiles;
        return 0;
    }
    // up to 8 rows: two private staging buffers per wavefront; 9 .. 16 rows: one (see the kernel)
    const size_t lds_roll = (size_t)8 * (m <= 8 ? 4 : 2) * m * (GEMM_U * 4 + 1) * 16 + (size_t)8 * 64 * 16;
    if (c->fullk && c->fullk_roll && m <= 16 && ntiles * 4 >= c->n_cu * 3 && kchunks >= 8 * GEMM_U && lds_roll <= FULLK_LDS_MAX) {
        metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_GEMM, (double)N * K * 2 + (double)m * K * 4 + (double)m * N * 4, N, K, m);
        hipEvent_t ea = pr ? pr->a : nullptr, eb = pr ? pr->b : nullptr;
#define ROLL_GO(XB, DB) hipExtLaunchKernelGGL((gemm_fullk_roll_residual_kernel<XB, DB>), dim3(ntiles), dim3(512), (uint32_t)lds_roll, c->stream, ea, eb, 0u, \
                                              (const bf16_t*)x, x_lo_off, ldx, m, K, (const bf16_t*)W, ntiles, N, h, (const bf16_t*)gain_next, xsplit, ssq)
        if (m <= 6) ROLL_GO(3, true);
        else if (m <= 8) ROLL_GO(4, true);
        else if (m <= 10) ROLL_GO(5, false);
        else if (m <= 12) ROLL_GO(6, false);
        else if (m <= 14) ROLL_GO(7, false);
        else ROLL_GO(8, false);
#undef ROLL_GO
        LAUNCH_CHECK(c, "gemm_bf16 (full-K residual, rolling staging)");
        *ntg_out = ntiles;
        return 0;
    }
    const Split s = choose_split(m, ntiles, kchunks);
    const int groups = (ntiles + s.tpb - 1) / s.tpb;
    if ((size_t)(s.ksplit - 1) * m * N * 8 > c->lay.ssq - c->lay.gx)
        return c->fail(METASD_E_WORKSPACE, "residual GEMM (m %d, K %d, N %d): %d split-K siblings exceed the exchange area of the workspace", m, K, N, s.ksplit);
    metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_GEMM, (double)N * K * 2 + (double)m * K * 4 + (double)m * N * 4, N, K, m);
    GemmPro plain{};
    plain.sstride = x_lo_off;
    GemmEpi epi{};
    epi.xw = c->d_gx(); epi.h = h; epi.gain = (const bf16_t*)gain_next; epi.xsplit = xsplit; epi.ssq = ssq;
    epi.abort = &reinterpret_cast<GridBar*>(c->d_bar())->abort;
    epi.epoch = next_epoch();
    epi.spin_limit = gemm_spin_limit(1 << 18);
    hipExtLaunchKernelGGL((gemm_bf16_kernel<PRO_PLAIN, EPI_RESIDUAL>), dim3(groups * s.ksplit), dim3(256), (uint32_t)s.lds, c->stream,
                          pr ? pr->a : nullptr, pr ? pr->b : nullptr, 0u, (const float*)x, ldx, m, K, (const bf16_t*)W,
                          (const bf16_t*)W, (const bf16_t*)W, ntiles, ntiles, ntiles, (float*)nullptr, N, s.ksplit, s.cps, s.tpb,
                          plain, epi);
    LAUNCH_CHECK(c, "gemm_bf16 (residual epilogue)");
    *ntg_out = groups;
    return 0;
}

// bf16 GEMM of the merged attention output, merged from the per-chunk records in its prologue (PRO_COMBINE, see kernels.h): partials
// to part_out (split stride m*N).
int gemm_combine(metasd_ctx* c, const GemmPro& pro, int m, int K, const void* W, int N, float* part_out, int* nsplit_out) {
    const int ntiles = N / 16;
    const Split s = choose_split(m, ntiles, K / 32);
    const int groups = (ntiles + s.tpb - 1) / s.tpb;
    if (s.ksplit > 8) return c->fail(METASD_E_INVALID, "output projection: %d partials for a consumer of at most 8", s.ksplit);
    metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_GEMM, (double)N * K * 2 + (double)m * K * 4 + (double)m * N * 4, N, K, m);
    hipExtLaunchKernelGGL(gemm_bf16_kernel<PRO_COMBINE>, dim3(groups * s.ksplit), dim3(256), (uint32_t)s.lds, c->stream, pr ? pr->a : nullptr,
                          pr ? pr->b : nullptr, 0u, (const float*)nullptr, K, m, K, (const bf16_t*)W, (const bf16_t*)W, (const bf16_t*)W,
                          ntiles, ntiles, ntiles, part_out, N, s.ksplit, s.cps, s.tpb, pro, GemmEpi{});
    LAUNCH_CHECK(c, "gemm_bf16 (attention combine)");
    *nsplit_out = s.ksplit;
    return 0;
}

// Launch of gemm_step_kernel: units (feature tiles, gate and up tiles of a pair, or half tiles) to workgroups.
// A CU runs one workgroup of 16 wavefronts and pulls about 25 GB/s whatever the wavefronts do, so the time is the largest number of
// tiles a CU has to stream; among the plans with the least of that the one with the fewest passes (each ends in a reduction).
struct StepPlan { int T, S, passes, grid, loads; bool half; };

StepPlan plan_step(int ntiles, int kchunks, bool pairs, bool add, int n_cu) {
    StepPlan best{};
    long best_cost = 1L << 60;
    for (int half = 0; half <= (add && kchunks % 2 == 0 ? 1 : 0); ++half) {
        const int units = half ? 2 * ntiles : ntiles;
        for (int T = pairs ? 2 : 1; T <= 16; T += pairs ? 2 : 1) {
            const int passes = add ? 1 : (units + T * n_cu - 1) / (T * n_cu), grid = (units + T * passes - 1) / (T * passes);
            const int rounds = (grid + n_cu - 1) / n_cu, S = 16 / T;
            const long cost = (long)rounds * passes * T * (half ? 1 : 2) * 64 + passes;
            const int cps = (kchunks + S - 1) / S;
            if (cost < best_cost) { best_cost = cost; best = StepPlan{T, S, passes, grid, half ? (cps + 1) / 2 : cps, half != 0}; }
        }
    }
    return best;
}

template <int PRO, int EPI, bool PART, int J, int U, bool HALF, int NR>
hipError_t step_allow_lds() {
    return hipFuncSetAttribute((const void*)gemm_step_kernel<PRO, EPI, PART, J, U, HALF, NR>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)FULLK_LDS_MAX);
}
template <int PRO, int EPI, bool PART, int J, bool HALF, int NR>
int launch_step(metasd_ctx* c, const StepArgs& a, const StepPlan& pl) {
    const int N = a.ntiles * 16;
    metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_GEMM, (double)N * a.K * 2 + (double)a.m * a.K * 4 + (double)a.m * N * 4, N, a.K, a.m);
    const uint32_t lds = (uint32_t)step_lds(PRO == STEP_NORM, a.m, a.K);
    constexpr int BIG = PRO == STEP_NORM ? 8 : (HALF ? 3 : 4) - (NR == 16 ? 1 : 0), FEW = std::min(BIG, 4);   // TERMS: the operands share the registers
    if (pl.loads <= FEW) hipExtLaunchKernelGGL((gemm_step_kernel<PRO, EPI, PART, J, FEW, HALF, NR>), dim3(pl.grid), dim3(1024), lds, c->stream, pr ? pr->a : nullptr, pr ? pr->b : nullptr, 0u, a);
    else hipExtLaunchKernelGGL((gemm_step_kernel<PRO, EPI, PART, J, BIG, HALF, NR>), dim3(pl.grid), dim3(1024), lds, c->stream, pr ? pr->a : nullptr, pr ? pr->b : nullptr, 0u, a);
    LAUNCH_CHECK(c, "gemm_step");
    return 0;
}
// the forms that stage their input may use more than 64 KiB of LDS
template <int EPI, bool PART, int J, int NR>
bool step_init_one() {
    return step_allow_lds<STEP_NORM, EPI, PART, J, 4, false, NR>() == hipSuccess && step_allow_lds<STEP_NORM, EPI, PART, J, 8, false, NR>() == hipSuccess;
}
template <int J, int NR>
bool step_init_j() { return step_init_one<STEP_OUT, false, J, NR>() && step_init_one<STEP_ROPE, false, J, NR>() && step_init_one<STEP_ACT, false, J, NR>(); }
bool step_init() {
    const bool ok = step_init_j<1, 8>() && step_init_j<2, 8>() && step_init_j<4, 8>() && step_init_j<8, 8>() && step_init_j<4, 16>() && step_init_j<8, 16>() &&
                    step_init_one<STEP_ACT, true, 1, 8>() && step_init_one<STEP_ACT, true, 2, 8>();
    if (!ok) (void)hipGetLastError();
    return ok;
}

int step_cols(int m, int K) {           // float4 columns of a row per lane
    const int wpr = m <= 1 ? 16 : m <= 2 ? 8 : m <= 4 ? 4 : m <= 8 ? 2 : 1;
    return (K + 256 * wpr - 1) / (256 * wpr);
}
bool step_ok(int m, int K) { return m <= STEP_ROWS && step_cols(m, K) <= 8 && step_lds(true, m, K) <= FULLK_LDS_MAX; }

// The projections of normalised rows; a: everything but the weights and the split.
template <int EPI, bool PART>
int gemm_step_norm(metasd_ctx* c, StepArgs a, const void* W0, int n0, const void* W1, int n1, const void* W2, int n2) {
    a.W0 = (const bf16_t*)W0; a.W1 = (const bf16_t*)W1; a.W2 = (const bf16_t*)W2;
    a.t0 = n0 / 16; a.t1 = (n0 + n1) / 16; a.ntiles = (n0 + n1 + n2) / 16;
    const StepPlan pl = plan_step(a.ntiles, a.K / 32, EPI == STEP_ACT && a.swiglu, false, c->n_cu);
    a.T = pl.T; a.S = pl.S; a.passes = pl.passes;
    const int J = step_cols(a.m, a.K);
    if (!step_ok(a.m, a.K) || (PART && (a.m > 8 || J > 2 || a.ns < 1 || a.ns > 8)))
        return c->fail(METASD_E_INVALID, "step GEMM: %d rows of %d, %d partials do not fit", a.m, a.K, a.ns);
    if constexpr (!PART) {
        if (a.m > 8) return J <= 4 ? launch_step<STEP_NORM, EPI, PART, 4, false, 16>(c, a, pl) : launch_step<STEP_NORM, EPI, PART, 8, false, 16>(c, a, pl);
    }
    if (J == 1) return launch_step<STEP_NORM, EPI, PART, 1, false, 8>(c, a, pl);
    if (PART || J == 2) return launch_step<STEP_NORM, EPI, PART, 2, false, 8>(c, a, pl);
    if constexpr (!PART) {
        if (J <= 4) return launch_step<STEP_NORM, EPI, PART, 4, false, 8>(c, a, pl);
        return launch_step<STEP_NORM, EPI, PART, 8, false, 8>(c, a, pl);
    }
    return 0;
}
// h += x W^T, x as two bf16 arrays
int gemm_step_add(metasd_ctx* c, const void* x, int m, int K, const void* W, int N, float* h) {
    StepArgs a{};
    a.x = (const bf16_t*)x; a.x_lo = (size_t)m * K;
    a.W0 = a.W1 = a.W2 = (const bf16_t*)W;
    a.t0 = a.t1 = a.ntiles = N / 16;
    a.out = h; a.N = N; a.m = m; a.K = K;
    const StepPlan pl = plan_step(a.ntiles, K / 32, false, true, c->n_cu);
    a.T = pl.T; a.S = pl.S; a.passes = 1;
    if (m > STEP_ROWS) return c->fail(METASD_E_INVALID, "step GEMM: %d rows", m);
    if (m > 8) return pl.half ? launch_step<STEP_TERMS, STEP_ADD, false, 1, true, 16>(c, a, pl) : launch_step<STEP_TERMS, STEP_ADD, false, 1, false, 16>(c, a, pl);
    return pl.half ? launch_step<STEP_TERMS, STEP_ADD, false, 1, true, 8>(c, a, pl) : launch_step<STEP_TERMS, STEP_ADD, false, 1, false, 8>(c, a, pl);
}

// q, k and v of layer L: q rotated in d_q, the block's K / V rows (positions pos0 ..) rotated and rounded in the cache
int gemm_step_qkv(metasd_ctx* c, const Model& M, int L, int pos0, StepArgs a) {
    const metasd_model_desc& d = M.d;
    const int DQ = d.n_heads * M.hd, DKV = d.n_kv_heads * M.hd;
    const size_t plane = (size_t)d.n_kv_heads * c->cfg.max_ctx * M.hd;
    a.out = (float*)c->d_q(); a.N = DQ;
    a.tab = (const double2*)c->d_rope();
    a.kc = (bf16_t*)M.kv + (size_t)L * 2 * plane; a.vc = a.kc + plane;
    a.H = d.n_heads; a.KH = d.n_kv_heads; a.hd = M.hd; a.pos0 = pos0; a.max_ctx = c->cfg.max_ctx;
    return gemm_step_norm<STEP_ROPE, false>(c, a, M.layer_w(L, 1), DQ, M.layer_w(L, 2), DKV, M.layer_w(L, 3), DKV);
}

// nrec_out != nullptr: the records are left to the consumer, which merges them itself (*nrec_out of them; 1: the rows are in d_ao)
template <typename T, int HD>
int attention_hd(metasd_ctx* c, const Model& M, int L, int pos0, int m, int* nrec_out) {
    const metasd_model_desc& d = M.d;
    const size_t plane = (size_t)d.n_kv_heads * c->cfg.max_ctx * HD;
    const T* kc = (const T*)M.kv + (size_t)L * 2 * plane;
    const T* vc = kc + plane;
    const int nchunks = (pos0 + m + ATT_CH - 1) / ATT_CH;
    const float scale = 1.0f / sqrtf((float)HD);
    // algorithmic bytes: K and V of every cached position once per KV head, q in, partials out
    metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_ATTN, 2.0 * d.n_kv_heads * (double)(pos0 + m) * HD * sizeof(T) +
                                                                 (double)m * d.n_heads * HD * 4);
    hipEvent_t ea = pr ? pr->a : nullptr, eb = pr ? pr->b : nullptr;
    int nrec = nchunks;
    bool combine = true;
    if constexpr (sizeof(T) == 2 && HD >= 64) {
        const int len = pos0 + m;
        const AttnPlan pl = plan_attn(&len, 1, d.n_heads, d.n_kv_heads, HD, m, c->n_cu, c->att_cpw);
        const AttnOut ao{c->d_apart(), pl.nrec, 0, 0, (float*)c->d_ao(), 1, (size_t)m * d.n_heads * HD, 0, m};
        nrec = pl.nrec;
        if (nrec == 1) combine = false;
#define ATTN_GO(TREE, SHARED) hipExtLaunchKernelGGL((attn_kernel<HD, TREE, SHARED>), dim3(pl.grid), dim3(64 * ATT_NW), 0u, c->stream, ea, eb, 0u, (const bf16_t*)c->d_q(), \
                                                kc, vc, m, pos0, d.n_heads, d.n_kv_heads, pl.hp, c->cfg.max_ctx, scale, pl.spw, ao, c->tree ? *c->tree : TreeBlk{})
        const bool shared = d.n_heads > d.n_kv_heads * pl.hp;
        if (c->tree) { if (shared) ATTN_GO(true, true); else ATTN_GO(true, false); }
        else { if (shared) ATTN_GO(false, true); else ATTN_GO(false, false); }
#undef ATTN_GO
    } else {
        // a context of one chunk needs no merge (fp32: nothing but the division is left of it)
        float* direct = sizeof(T) == 4 && combine && nchunks == 1 ? (float*)c->d_ao() : nullptr;
        if (direct) combine = false;
        if (c->tree)
            hipExtLaunchKernelGGL((attn_partial_tree_kernel<T, HD>), dim3(nchunks, d.n_heads), dim3(256), 0u, c->stream, ea, eb, 0u,
                                  (const float*)c->d_q(), kc, vc, m, pos0, d.n_heads, d.n_kv_heads, c->cfg.max_ctx, scale,
                                  c->d_apart(), nchunks, *c->tree, direct);
        else
            hipExtLaunchKernelGGL((attn_partial_kernel<T, HD>), dim3(nchunks, d.n_heads), dim3(256), 0u, c->stream, ea, eb, 0u,
                                  (const float*)c->d_q(), kc, vc, m, pos0, d.n_heads, d.n_kv_heads, c->cfg.max_ctx, scale,
                                  c->d_apart(), nchunks, direct);
    }
    LAUNCH_CHECK(c, "attn_partial");
    if (nrec_out) *nrec_out = combine ? nrec : 1;
    if (!combine || nrec_out) return 0;
    hipLaunchKernelGGL((attn_combine_kernel<T, HD>), dim3(d.n_heads, m), dim3(HD), 0, c->stream, c->d_apart(), nrec,
                       d.n_heads, (float*)c->d_ao(), sizeof(T) == 2 ? 1 : 0);
    LAUNCH_CHECK(c, "attn_combine");
    return 0;
}

template <typename T>
int attention(metasd_ctx* c, const Model& M, int L, int pos0, int m, int* nrec_out = nullptr) {
    switch (M.hd) {
        case 32: return attention_hd<T, 32>(c, M, L, pos0, m, nrec_out);
        case 64: return attention_hd<T, 64>(c, M, L, pos0, m, nrec_out);
        default:
            if constexpr (sizeof(T) == 2) return attention_hd<T, 128>(c, M, L, pos0, m, nrec_out);
            return c->fail(METASD_E_INVALID, "fp32 head_dim 128 unsupported");
    }
}

// Residual rows of a block from its tokens, and its table of rotations.  A drafter head starts from
// W_fc . [embedding ; feature of the position before] instead of the embedding.
template <typename T>
int embed_rows(metasd_ctx* c, Model& M, int pos0, int m, float* h) {
    const metasd_model_desc& d = M.d;
    const int D = d.d_model;
    if (!c->embedded) {
        hipLaunchKernelGGL(embed_rope_kernel<T>, dim3(m), dim3(320), 0, c->stream, c->d_hist() + pos0, (const T*)M.w[0], D, h, pos0, M.hd, d.rope_theta,
                           c->d_rope(), c->tree ? *c->tree : TreeBlk{});
        LAUNCH_CHECK(c, "embed + rope table");
    }
    if (!M.head) return 0;
    float* cat = (float*)c->d_act();
    hipLaunchKernelGGL(feat_cat_kernel, dim3(m), dim3(256), 0, c->stream, (const float*)h, (const float*)c->d_feat(),
                       c->head_est ? (const float*)c->d_fest() : (const float*)nullptr, c->fsrc, pos0, D, cat, sizeof(T) == 2 ? 1 : 0);
    LAUNCH_CHECK(c, "feat_cat");
    int dummy;
    return gemm<T>(c, cat, 2 * D, m, 2 * D, M.fc, D, nullptr, 0, nullptr, 0, h, &dummy, (size_t)m * 2 * D);
}

// Forward of m <= 16 rows whose tokens are hist[pos0 .. pos0+m) at positions pos0..; appends K/V.
// logits: nullptr = none; otherwise rows [first_row, m) of the block get logits, written
// consecutively to `logits` (row stride V).
template <typename T>
int forward_rows(metasd_ctx* c, Model& M, int pos0, int m, float* logits, int first_row) {
    const metasd_model_desc& d = M.d;
    const int D = d.d_model, H = d.n_heads, KH = d.n_kv_heads, hd = M.hd, F = d.d_ffn, V = d.vocab;
    const int DQ = H * hd, DKV = KH * hd;
    hipStream_t st = c->stream;
    float* h = c->d_h();
    float* xn = (float*)c->d_xn();
    float* part = c->d_part();
    int ns = 0, rc;
    constexpr int split = sizeof(T) == 2 ? 1 : 0;   // bf16 models: activations for the GEMM are stored as two bf16 arrays
    if ((rc = embed_rows<T>(c, M, pos0, m, h))) return rc;
    for (int L = 0; L < d.n_layers; ++L) {
        // h += previous FFN output (split partials); xn = norm(h)
        hipLaunchKernelGGL(addnorm_kernel<T>, dim3(m), dim3(1024), 0, st, h, part, ns, (size_t)m * D, D, (const T*)M.layer_w(L, 0),
                           d.rms_eps, xn, split);
        LAUNCH_CHECK(c, "addnorm");
        if ((rc = gemm<T>(c, xn, D, m, D, M.layer_w(L, 1), DQ, M.layer_w(L, 2), DKV, M.layer_w(L, 3), DKV, nullptr, &ns, (size_t)m * D))) return rc;
        const int NQKV = DQ + 2 * DKV;
        const size_t plane = (size_t)KH * c->cfg.max_ctx * hd;
        T* kc = (T*)M.kv + (size_t)L * 2 * plane;
        hipLaunchKernelGGL(rope_kv_kernel<T>, dim3((H + 2 * KH + 3) / 4, m), dim3(256), 0, st, part, ns, (size_t)m * NQKV, NQKV, pos0, H, KH,
                           hd, (const double2*)c->d_rope(), (float*)c->d_q(), kc, kc + plane, c->cfg.max_ctx, sizeof(T) == 2 ? 1 : 0,
                           (sizeof(T) == 2 && hd >= 64) ? 1 : 0, (const float*)nullptr);
        LAUNCH_CHECK(c, "rope_kv");
        if ((rc = attention<T>(c, M, L, pos0, m))) return rc;
        if ((rc = gemm<T>(c, c->d_ao(), DQ, m, DQ, M.layer_w(L, 4), D, nullptr, 0, nullptr, 0, nullptr, &ns, (size_t)m * DQ))) return rc;
        hipLaunchKernelGGL(addnorm_kernel<T>, dim3(m), dim3(1024), 0, st, h, part, ns, (size_t)m * D, D, (const T*)M.layer_w(L, 5),
                           d.rms_eps, xn, split);
        LAUNCH_CHECK(c, "addnorm");
        if (d.act == METASD_SWIGLU) {
            if ((rc = gemm<T>(c, xn, D, m, D, M.layer_w(L, 6), F, M.layer_w(L, 7), F, nullptr, 0, nullptr, &ns, (size_t)m * D))) return rc;
        } else {
            if ((rc = gemm<T>(c, xn, D, m, D, M.layer_w(L, 7), F, nullptr, 0, nullptr, 0, nullptr, &ns, (size_t)m * D))) return rc;
        }
        const size_t nact = (size_t)m * F;
        const int NF = (d.act == METASD_SWIGLU ? 2 : 1) * F;
        hipLaunchKernelGGL(ffn_act4_kernel, dim3((unsigned)((nact / 4 + 255) / 256)), dim3(256), 0, st, part, ns, (size_t)m * NF, m, F,
                           d.act, (float*)c->d_act(), split, (const float*)nullptr);
        LAUNCH_CHECK(c, "ffn_act");
        if ((rc = gemm<T>(c, c->d_act(), F, m, F, M.layer_w(L, 8), D, nullptr, 0, nullptr, 0, nullptr, &ns, (size_t)m * F))) return rc;
    }
    if (logits || c->cfg.feature_heads) {          // with drafter heads the finished residual rows are wanted in any case
        hipLaunchKernelGGL(addnorm_kernel<T>, dim3(m), dim3(1024), 0, st, h, part, ns, (size_t)m * D, D, (const T*)M.final_norm(),
                           d.rms_eps, xn, split);
        LAUNCH_CHECK(c, "addnorm");
    }
    if (logits) {
        int dummy;
        const void* xrow = split ? (const void*)((const bf16_t*)xn + (size_t)first_row * D) : (const void*)(xn + (size_t)first_row * D);
        if ((rc = gemm<T>(c, xrow, D, m - first_row, D, M.lm_head(), V, nullptr, 0, nullptr, 0, logits, &dummy, (size_t)m * D)))
            return rc;
    }
    return 0;
}

// fp32 models of narrow rows (step_f32.h): four launches per layer instead of ten while the context is short, then five, six when it has
// more than one chunk.
bool f32_step_ok(const Model& M) { return M.d.dtype == METASD_F32 && M.d.d_model <= STEP_F32_K; }

template <int NF, bool NORM, int EPI>
int launch_f32_step(metasd_ctx* c, const F32Args& a, const char* what) {
    const dim3 grid((a.units + 3) / 4);
    const uint32_t lds = NORM ? (uint32_t)(a.m * a.K * 4) : 0u;
    if (a.m <= 1) hipLaunchKernelGGL((gemm_f32_step_kernel<1, NF, NORM, EPI>), grid, dim3(256), lds, c->stream, a);
    else if (a.m <= 4) hipLaunchKernelGGL((gemm_f32_step_kernel<4, NF, NORM, EPI>), grid, dim3(256), lds, c->stream, a);
    else if (a.m <= 8) hipLaunchKernelGGL((gemm_f32_step_kernel<8, NF, NORM, EPI>), grid, dim3(256), lds, c->stream, a);
    else hipLaunchKernelGGL((gemm_f32_step_kernel<16, NF, NORM, EPI>), grid, dim3(256), lds, c->stream, a);
    LAUNCH_CHECK(c, what);
    return 0;
}

// Contexts short enough for attention and output projection in one launch, h += ..: one row over 128 positions (head_dim 64: 64), several
// rows over 64 (head_dim 32).
bool f32_attn_out_ok(const Model& M, int m, int len) {
    return M.d.n_heads * M.hd <= STEP_F32_K && len <= (m == 1 && M.hd == 32 ? 128 : 64) && (m == 1 || M.hd == 32);
}
int launch_f32_attn_out(metasd_ctx* c, const Model& M, int L, int pos0, int m, const float* W, float* h) {
    const metasd_model_desc& d = M.d;
    const size_t plane = (size_t)d.n_kv_heads * c->cfg.max_ctx * M.hd;
    const float* kc = (const float*)M.kv + (size_t)L * 2 * plane;
    const float scale = 1.0f / sqrtf((float)M.hd);
    const int len = pos0 + m;
    metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_ATTN, 2.0 * d.n_kv_heads * (double)len * M.hd * 4 + (double)m * d.n_heads * M.hd * 4);
#define AO_GO(KERNEL, NW, ...) hipExtLaunchKernelGGL(KERNEL, dim3((d.d_model + NW - 1) / NW), dim3(64 * NW), 0u, c->stream, pr ? pr->a : nullptr, pr ? pr->b : nullptr, 0u, \
                                                     (const float*)c->d_q(), kc, kc + plane, W, h, __VA_ARGS__, d.n_heads, d.n_kv_heads, c->cfg.max_ctx, scale, d.d_model, \
                                                     c->tree ? *c->tree : TreeBlk{})
    if (m == 1) {
        if (M.hd == 64) AO_GO((attn_out_f32_kernel<64, 1>), 4, pos0);
        else if (len <= 64) AO_GO((attn_out_f32_kernel<32, 1>), 4, pos0);
        else AO_GO((attn_out_f32_kernel<32, 2>), 4, pos0);
    } else if (m <= 8) AO_GO((attn_out_rows_f32_kernel<8>), 16, m, pos0);
    else AO_GO((attn_out_rows_f32_kernel<16>), 16, m, pos0);
#undef AO_GO
    LAUNCH_CHECK(c, "attention and output projection");
    return 0;
}

int forward_rows_f32(metasd_ctx* c, Model& M, int pos0, int m, float* logits, int first_row) {
    typedef float T;
    const metasd_model_desc& d = M.d;
    const int D = d.d_model, H = d.n_heads, KH = d.n_kv_heads, hd = M.hd, F = d.d_ffn;
    float* h = c->d_h();
    int rc;
    if ((rc = embed_rows<T>(c, M, pos0, m, h))) return rc;
    F32Args base{};
    base.eps = d.rms_eps; base.m = m;
    base.tab = (const double2*)c->d_rope(); base.pos0 = pos0; base.H = H; base.KH = KH; base.hd = hd; base.max_ctx = c->cfg.max_ctx;
    for (int L = 0; L < d.n_layers; ++L) {
        const size_t plane = (size_t)KH * c->cfg.max_ctx * hd;
        auto W = [&](int i) { return (const float*)M.layer_w(L, i); };
        F32Args a = base;                           // q, and k and v in the cache
        a.x = h; a.gain = W(0); a.W0 = W(1); a.W1 = W(2); a.W2 = W(3); a.K = D;
        a.out = (float*)c->d_q(); a.ldo = H * hd; a.units = (H + 2 * KH) * (hd / 2);
        a.kc = (float*)M.kv + (size_t)L * 2 * plane; a.vc = a.kc + plane;
        if ((rc = launch_f32_step<2, true, F32_ROPE>(c, a, "gemm_f32 (q, k, v)"))) return rc;
        if (f32_attn_out_ok(M, m, pos0 + m)) {
            if ((rc = launch_f32_attn_out(c, M, L, pos0, m, W(4), h))) return rc;
        } else {
            if ((rc = attention<T>(c, M, L, pos0, m))) return rc;
            a = base;                               // h += output projection
            a.x = (const float*)c->d_ao(); a.W0 = W(4); a.K = H * hd; a.out = h; a.ldo = D; a.units = D;
            if ((rc = launch_f32_step<1, false, F32_ADD>(c, a, "gemm_f32 (output)"))) return rc;
        }
        a = base;                                   // activation of the FFN
        a.x = h; a.gain = W(5); a.K = D; a.out = (float*)c->d_act(); a.ldo = F; a.units = F;
        if (d.act == METASD_SWIGLU) { a.W0 = W(6); a.W1 = W(7); rc = launch_f32_step<2, true, F32_ACT>(c, a, "gemm_f32 (gate, up)"); }
        else { a.W0 = W(7); rc = launch_f32_step<1, true, F32_ACT>(c, a, "gemm_f32 (up)"); }
        if (rc) return rc;
        a = base;                                   // h += down projection
        a.x = (const float*)c->d_act(); a.W0 = W(8); a.K = F; a.out = h; a.ldo = D; a.units = D;
        if ((rc = launch_f32_step<1, false, F32_ADD>(c, a, "gemm_f32 (down)"))) return rc;
    }
    if (!logits) return 0;
    F32Args a = base;
    a.x = h + (size_t)first_row * D; a.m = m - first_row; a.gain = (const float*)M.final_norm(); a.W0 = (const float*)M.lm_head();
    a.K = D; a.out = logits; a.ldo = d.vocab; a.units = d.vocab;
    return launch_f32_step<1, true, F32_OUT>(c, a, "gemm_f32 (head)");
}

// A forward pass, or a chain of draft steps, in one launch.  Contexts: a wavefront walks a head's positions alone, so that the separate launches, which
// deal them out, overtake it - with heads of 32, at most one per wavefront, between 900 positions (round of 4 drafts 192 against 222 us) and
// 1800 (266 / 208), with 16 heads between 60 (349 / 450) and 450 (514 / 460), with heads of 64 before 450 (565 / 537).  Not while launches
// are timed one by one (metasd_profile).
bool chain_ok(const metasd_ctx* c, const Model& M, int m, int steps, int len) {
    const metasd_model_desc& d = M.d;
    return c->fuse_small && c->cfg.batch == 1 && !c->tree && !M.head && !c->cfg.feature_heads && !c->prof_on && chain_model(d) && m <= MAX_ROWS &&
           len * ((d.n_heads + CH_WAVES - 1) / CH_WAVES) * (M.hd / 32) <= 512 && (steps == 0 || d.vocab <= CH_VOCAB) &&
           (size_t)chain_lds(m, steps, d.d_model, d.d_ffn, d.vocab, d.n_kv_heads * M.hd, M.hd, d.n_layers).end * 4 + 16 <= FULLK_LDS_MAX;
}
template <int MR, int KJ, int HD>
int launch_chain_as(metasd_ctx* c, const ChainArgs& a, int groups, uint32_t lds) {
    static const hipError_t attr = hipFuncSetAttribute((const void*)chain_f32_kernel<MR, KJ, HD>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)FULLK_LDS_MAX);
    if (attr != hipSuccess) return c->fail(METASD_E_HIP, "chain_f32_kernel: cannot reserve %zu bytes of LDS", FULLK_LDS_MAX);
    hipLaunchKernelGGL((chain_f32_kernel<MR, KJ, HD>), dim3(groups), dim3(CH_NT), lds, c->stream, a);
    LAUNCH_CHECK(c, "chain_f32");
    return 0;
}
// rows pos0 .. pos0 + m - 1 of the history; steps = 0: logits of rows first .. to out (first = m: none), else draft steps with their logits there
int launch_chain(metasd_ctx* c, const Model& M, int pos0, int m, int first, int steps, float* out) {
    const metasd_model_desc& d = M.d;
    const int KVD = d.n_kv_heads * M.hd;
    ChainArgs a{};
    for (size_t i = 0; i < M.w.size(); ++i) a.w[i] = (const float*)M.w[i];
    a.n_layers = d.n_layers; a.D = d.d_model; a.H = d.n_heads; a.KH = d.n_kv_heads; a.F = d.d_ffn; a.V = d.vocab; a.swiglu = d.act == METASD_SWIGLU;
    a.max_ctx = c->cfg.max_ctx; a.eps = d.rms_eps; a.scale = 1.0f / sqrtf((float)M.hd);
    for (int i = 0; i < M.hd / 2; ++i) a.freq[i] = std::pow((double)d.rope_theta, -2.0 * (double)i / (double)M.hd);
    a.kv = (float*)M.kv; a.tok = c->d_hist() + pos0; a.m = m; a.pos0 = pos0; a.first = first; a.steps = steps; a.out = out;
    a.T = c->cfg.temperature; a.seed = c->cfg.seed; a.round = (uint32_t)c->sq[0].round; a.hist = c->d_hist() + pos0 + m; a.draft = c->d_draft();
    a.xw = c->d_chain(); a.region = chain_words({m, d.d_model, d.n_heads, d.n_kv_heads, M.hd, d.d_ffn, d.vocab}, CH_VOCAB);
    a.tag = next_epochs(chain_exchanges(d.n_layers, steps)); a.spin_limit = gemm_spin_limit(1 << 22); a.abort = &c->d_bar()->abort;
    const uint32_t lds = (uint32_t)chain_lds(m, steps, d.d_model, d.d_ffn, d.vocab, KVD, M.hd, d.n_layers).end * 4 + 16;
    const int groups = chain_groups(d.d_model);
#define CHAIN_GO(KJ, HD) return m == 1 ? launch_chain_as<1, KJ, HD>(c, a, groups, lds) : launch_chain_as<8, KJ, HD>(c, a, groups, lds)
    if (d.d_model <= 256) { if (M.hd == 32) CHAIN_GO(1, 32); CHAIN_GO(1, 64); }
    if (M.hd == 32) CHAIN_GO(2, 32);
    CHAIN_GO(2, 64);
#undef CHAIN_GO
}

// bf16 models, general case: the two projections into the residual stream reduce their split-K partials
// inside the GEMM and hand the next GEMM h * gain directly (EPI_RESIDUAL); the kernels that consume a
// projection of such an input scale by 1/rms.  8 launches per layer instead of 10 (no add+norm kernels).
int forward_rows_residual(metasd_ctx* c, Model& M, int pos0, int m, float* logits, int first_row) {
    typedef bf16_t T;
    const metasd_model_desc& d = M.d;
    const int D = d.d_model, H = d.n_heads, KH = d.n_kv_heads, hd = M.hd, F = d.d_ffn, V = d.vocab;
    const int DQ = H * hd, DKV = KH * hd, NQKV = DQ + 2 * DKV;
    hipStream_t st = c->stream;
    float* h = c->d_h();
    float* xn = (float*)c->d_xn();
    float* part = c->d_part();
    float* ssq = c->d_ssq();
    float* inv = c->d_inv();
    int ns = 0, rc, ntg = 0;
    c->cur_eps = d.rms_eps;
    if ((rc = embed_rows<T>(c, M, pos0, m, h))) return rc;
    // first norm: a plain RMSNorm of the embedding rows (normalised x, no scaling downstream)
    hipLaunchKernelGGL(addnorm_kernel<T>, dim3(m), dim3(1024), 0, st, h, part, 0, (size_t)m * D, D, (const T*)M.layer_w(0, 0), d.rms_eps,
                       xn, 1);
    LAUNCH_CHECK(c, "addnorm");
    bool scaled = false;            // does xn hold h * gain (true) or the normalised rows (false)?
    for (int L = 0; L < d.n_layers; ++L) {
        if ((rc = gemm<T>(c, xn, D, m, D, M.layer_w(L, 1), DQ, M.layer_w(L, 2), DKV, M.layer_w(L, 3), DKV, nullptr, &ns, (size_t)m * D,
                          scaled ? ssq : nullptr, ntg, inv, 0))) return rc;
        const size_t plane = (size_t)KH * c->cfg.max_ctx * hd;
        T* kc = (T*)M.kv + (size_t)L * 2 * plane;
        hipLaunchKernelGGL(rope_kv_kernel<T>, dim3((H + 2 * KH + 3) / 4, m), dim3(256), 0, st, part, ns, (size_t)m * NQKV, NQKV, pos0, H, KH, hd,
                           (const double2*)c->d_rope(), (float*)c->d_q(), kc, kc + plane, c->cfg.max_ctx, 1, hd >= 64 ? 1 : 0,
                           scaled ? (const float*)inv : nullptr);
        LAUNCH_CHECK(c, "rope_kv");
        if ((rc = attention<T>(c, M, L, pos0, m))) return rc;
        if ((rc = gemm_residual(c, c->d_ao(), DQ, m, DQ, M.layer_w(L, 4), D, (size_t)m * DQ, h, M.layer_w(L, 5), xn, ssq, &ntg))) return rc;
        if (d.act == METASD_SWIGLU) {
            if ((rc = gemm<T>(c, xn, D, m, D, M.layer_w(L, 6), F, M.layer_w(L, 7), F, nullptr, 0, nullptr, &ns, (size_t)m * D, ssq, ntg, inv, 0))) return rc;
        } else {
            if ((rc = gemm<T>(c, xn, D, m, D, M.layer_w(L, 7), F, nullptr, 0, nullptr, 0, nullptr, &ns, (size_t)m * D, ssq, ntg, inv, 0))) return rc;
        }
        const size_t nact = (size_t)m * F;
        const int NF = (d.act == METASD_SWIGLU ? 2 : 1) * F;
        hipLaunchKernelGGL(ffn_act4_kernel, dim3((unsigned)((nact / 4 + 255) / 256)), dim3(256), 0, st, part, ns, (size_t)m * NF, m, F, d.act,
                           (float*)c->d_act(), 1, (const float*)inv);
        LAUNCH_CHECK(c, "ffn_act");
        const void* gain_next = L + 1 < d.n_layers ? M.layer_w(L + 1, 0) : M.final_norm();
        if ((rc = gemm_residual(c, c->d_act(), F, m, F, M.layer_w(L, 8), D, (size_t)m * F, h, gain_next, xn, ssq, &ntg))) return rc;
        scaled = true;
    }
    if (logits) {
        int dummy;
        const void* xrow = (const void*)((const bf16_t*)xn + (size_t)first_row * D);
        if ((rc = gemm<T>(c, xrow, D, m - first_row, D, M.lm_head(), V, nullptr, 0, nullptr, 0, logits, &dummy, (size_t)m * D, ssq, ntg, inv,
                          first_row))) return rc;
    }
    return 0;
}

// Short blocks of narrow bf16 models (drafter steps; d_model <= 2048): the same forward with the add+norm, the rotation and cache append,
// the FFN activation, the residual add and the attention merge folded into the GEMMs before or behind them (step.h) - 5 launches per
// layer instead of 10.  The residual stream ping-pongs between two buffers where the gate | up projection adds the output projection's
// partials to it, because its workgroups read the old rows while one writes the new ones; attention that leaves finished rows (one
// record) needs neither the merge nor the partials: the output projection adds to the stream itself.
constexpr int fused_max_rows() { return 4; }
bool fused_small_ok(const Model& M, int m) {
    const metasd_model_desc& d = M.d;
    // d_model: the gate | up form that adds the output projection's partials exists for two float4 columns per lane, which at four rows
    // is 2048.  d_ffn: no launch needs the limit; it is the widest FFN these blocks were measured with, wider ones take forward_rows_step.
    constexpr int dmax = 2048;
    return d.dtype == METASD_BF16 && m <= fused_max_rows() && d.d_model <= dmax && d.d_ffn <= 4 * dmax && M.hd >= 64;
}

int forward_rows_fused(metasd_ctx* c, Model& M, int pos0, int m, float* logits, int first_row) {
    typedef bf16_t T;
    const metasd_model_desc& d = M.d;
    const int D = d.d_model, H = d.n_heads, hd = M.hd, F = d.d_ffn, V = d.vocab;
    const int DQ = H * hd;
    int hp = 0, rc;                     // current residual buffer
    if ((rc = embed_rows<T>(c, M, pos0, m, c->d_h_pp(0)))) return rc;
    auto norm_in = [&](const void* gain, int row0) {
        StepArgs a{};
        a.h = c->d_h_pp(hp) + (size_t)row0 * D;
        a.gain = (const bf16_t*)gain;
        a.eps = d.rms_eps;
        a.m = m - row0; a.K = D;
        return a;
    };
    for (int L = 0; L < d.n_layers; ++L) {
        // q, and the new K / V rows in the cache, from the QKV projection of norm(h)
        StepArgs a = norm_in(M.layer_w(L, 0), 0);
        if ((rc = gemm_step_qkv(c, M, L, pos0, a))) return rc;
        int nrec = 0;
        if ((rc = attention<T>(c, M, L, pos0, m, &nrec))) return rc;
        if (nrec > 1) {
            // output projection of the attention output, merged in its prologue; the gate | up projection adds its partials to h
            int ns = 0;
            GemmPro pro{};
            pro.src = c->d_apart(); pro.nchunks = nrec; pro.hd = hd;
            if ((rc = gemm_combine(c, pro, m, DQ, M.layer_w(L, 4), D, c->d_part(), &ns))) return rc;
            a = norm_in(M.layer_w(L, 5), 0);
            a.part = c->d_part(); a.sstride = (size_t)m * D; a.ns = ns; a.h_out = c->d_h_pp(hp ^ 1);
            hp ^= 1;
        } else {
            if ((rc = gemm_step_add(c, c->d_ao(), m, DQ, M.layer_w(L, 4), D, c->d_h_pp(hp)))) return rc;
            a = norm_in(M.layer_w(L, 5), 0);
        }
        // activation of the gate | up projection of norm(h + attention output)
        a.out = (float*)c->d_act(); a.N = F; a.swiglu = d.act == METASD_SWIGLU;
        const void *w0 = M.layer_w(L, a.swiglu ? 6 : 7), *w1 = a.swiglu ? M.layer_w(L, 7) : nullptr;
        rc = nrec > 1 ? gemm_step_norm<STEP_ACT, true>(c, a, w0, F, w1, w1 ? F : 0, nullptr, 0)
                      : gemm_step_norm<STEP_ACT, false>(c, a, w0, F, w1, w1 ? F : 0, nullptr, 0);
        if (rc) return rc;
        // h += down projection
        if ((rc = gemm_step_add(c, c->d_act(), m, F, M.layer_w(L, 8), D, c->d_h_pp(hp)))) return rc;
    }
    if (logits) {
        StepArgs a = norm_in(M.final_norm(), first_row);
        a.out = logits; a.N = V;
        if ((rc = gemm_step_norm<STEP_OUT, false>(c, a, M.lm_head(), V, nullptr, 0, nullptr, 0))) return rc;
    }
    return 0;
}

// 9 - 16 rows: the operands of a tile (16 rows of both terms, 64 bytes per input) pass through every CU beside its weights, so that a long K
// takes longer than a split over CUs with an exchange between them.  At 12 rows: K 2048 8.7 against 12.3 us, 3072 11.5 against 13.2, 8192 18.5
// against 14.8, 11008 28.7 against 23 (with the normalised rows and their sums of squares that the split-K kernel also writes: they go to
// scratch that nothing reads here - the next step GEMM normalises h - and gain_next is only there to be multiplied with).
constexpr int STEP_ADD_K = 4096;
int residual_add(metasd_ctx* c, const void* x, int m, int K, const void* W, int N, float* h, const void* gain_next) {
    if (m <= 8 || K <= STEP_ADD_K) return gemm_step_add(c, x, m, K, W, N, h);
    int ntg;
    return gemm_residual(c, x, K, m, K, W, N, (size_t)m * K, h, gain_next, (float*)c->d_xn(), c->d_ssq(), &ntg);
}

// Short blocks whose normalised rows fit in LDS, in general (8 rows of 4096 columns, 16 of 2048; verification, drafter heads, models wider than
// the path above takes): 6 launches per layer (5 where attention needs no merge), none of which leaves partial sums.  12 rows, 1B shape, per layer:
// 67 -> 55 us against forward_rows_residual.
constexpr int STEP_DMIN = 512;      // from here on each of the 16 wavefronts has a chunk of the input
int forward_rows_step(metasd_ctx* c, Model& M, int pos0, int m, float* logits, int first_row) {
    typedef bf16_t T;
    const metasd_model_desc& d = M.d;
    const int D = d.d_model, F = d.d_ffn, V = d.vocab, DQ = d.n_heads * M.hd;
    float* h = c->d_h();
    int rc;
    if ((rc = embed_rows<T>(c, M, pos0, m, h))) return rc;
    auto norm_in = [&](const void* gain, int row0) {
        StepArgs a{};
        a.h = h + (size_t)row0 * D;
        a.gain = (const bf16_t*)gain;
        a.eps = d.rms_eps;
        a.m = m - row0; a.K = D;
        return a;
    };
    for (int L = 0; L < d.n_layers; ++L) {
        StepArgs a = norm_in(M.layer_w(L, 0), 0);
        if ((rc = gemm_step_qkv(c, M, L, pos0, a))) return rc;
        if ((rc = attention<T>(c, M, L, pos0, m))) return rc;
        if ((rc = residual_add(c, c->d_ao(), m, DQ, M.layer_w(L, 4), D, h, M.layer_w(L, 5)))) return rc;
        a = norm_in(M.layer_w(L, 5), 0);
        a.out = (float*)c->d_act(); a.N = F; a.swiglu = d.act == METASD_SWIGLU;
        if (a.swiglu) rc = gemm_step_norm<STEP_ACT, false>(c, a, M.layer_w(L, 6), F, M.layer_w(L, 7), F, nullptr, 0);
        else rc = gemm_step_norm<STEP_ACT, false>(c, a, M.layer_w(L, 7), F, nullptr, 0, nullptr, 0);
        if (rc) return rc;
        if ((rc = residual_add(c, c->d_act(), m, F, M.layer_w(L, 8), D, h, M.layer_w(L, 5)))) return rc;
    }
    if (logits) {
        StepArgs a = norm_in(M.final_norm(), first_row);
        a.out = logits; a.N = V;
        if ((rc = gemm_step_norm<STEP_OUT, false>(c, a, M.lm_head(), V, nullptr, 0, nullptr, 0))) return rc;
    }
    return 0;
}

int upload_table(metasd_ctx* c, Model& M) {
    HIP_TRY(c, hipMemcpyAsync((void*)M.d_table, M.w.data(), M.w.size() * sizeof(void*), hipMemcpyHostToDevice, c->stream));
    return 0;
}

// Forward over tokens hist[pos0 .. pos0+n) in blocks of <= 16 rows (later blocks see the KV of
// earlier ones).  logits (optional): want_all ? all n rows (n <= 16) : the last row only.
int model_index(const metasd_ctx* c, const Model& M) { return &M == &c->target ? -1 : (int)(&M - c->drafters.data()); }

int forward_blocks(metasd_ctx* c, Model& M, int pos0, int n, float* logits, bool want_all);
int forward_big(metasd_ctx* c, Model& M, int seq, int pos0, int n);

// A drafter with a streaming cache attends to the sinks and to the last stream_window positions of its cache's tail: the
// block mask of the attention kernels (TreeBlk, on == 2) carries that for the duration of its forward passes.
int forward(metasd_ctx* c, Model& M, int pos0, int n, float* logits, bool want_all) {
    if (!M.stream || c->tree) return forward_blocks(c, M, pos0, n, logits, want_all);
    TreeBlk wb{};
    wb.on = 2; wb.base = M.tail; wb.i0 = c->cfg.stream_window; wb.sink = c->cfg.stream_sink;
    c->tree = &wb;
    const int rc = forward_blocks(c, M, pos0, n, logits, want_all);
    c->tree = nullptr;
    return rc;
}

int forward_blocks(metasd_ctx* c, Model& M, int pos0, int n, float* logits, bool want_all) {
    c->cur_model = model_index(c, M);
    if (pos0 + n > c->cfg.max_ctx) return c->fail(METASD_E_OVERFLOW, "positions %d..%d exceed max_ctx %d", pos0, pos0 + n, c->cfg.max_ctx);
    int done = 0;
    // long blocks: everything but the row that carries logits goes through in big blocks
    const int rows = n - (logits ? 1 : 0);
    if (big_ok(M.d) && !c->tree && rows > MAX_ROWS && big_pays(M.d, pos0, rows, 1)) {
        done = rows;
        if (int rc = forward_big(c, M, 0, pos0, done)) return rc;
    }
    while (done < n) {
        const int m = std::min(MAX_ROWS, n - done);
        const bool last = done + m == n;
        float* lg = (last && logits) ? logits : nullptr;
        const int first_row = want_all ? 0 : m - 1;
        int rc;
        const bool is_target = &M == &c->target;
        // the short-block path may leave the finished rows in the second residual buffer, which the feature copy below does not read: not
        // for the target when its features are wanted
        const bool fused = c->fuse_small && fused_small_ok(M, m) && !(is_target && c->cfg.feature_heads);
        if (chain_ok(c, M, m, 0, pos0 + done + m)) rc = launch_chain(c, M, pos0 + done, m, lg ? first_row : m, 0, lg);
        else if (c->fuse_small && f32_step_ok(M)) rc = forward_rows_f32(c, M, pos0 + done, m, lg, first_row);
        else if (M.d.dtype != METASD_BF16) rc = forward_rows<float>(c, M, pos0 + done, m, lg, first_row);
        else if (fused && !M.head) rc = forward_rows_fused(c, M, pos0 + done, m, lg, first_row);       // (the others carry the head's input projection)
        // (a switch that names one of the split-K forms of the residual projections asks for the path that has them)
        else if (c->fuse_small && c->gemm_reduce && c->fullk_roll && M.d.d_model >= STEP_DMIN && step_ok(m, M.d.d_model))
            rc = forward_rows_step(c, M, pos0 + done, m, lg, first_row);
        else if (c->gemm_reduce) rc = forward_rows_residual(c, M, pos0 + done, m, lg, first_row);
        else rc = forward_rows<bf16_t>(c, M, pos0 + done, m, lg, first_row);
        if (rc) return rc;
        const int D = M.d.d_model;
        if (is_target && c->cfg.feature_heads) {        // the target's features of the block's positions
            const unsigned n4 = (unsigned)((size_t)m * D / 4);
            hipLaunchKernelGGL(copy_f4_kernel, dim3((n4 + 255) / 256), dim3(256), 0, c->stream, (const float4*)c->d_h(),
                               (float4*)(c->d_feat() + (size_t)(pos0 + done) * D), n4);
            LAUNCH_CHECK(c, "feature rows");
        }
        if (M.head && c->tree && c->tree->on == 1) {     // a tree level (one block): the estimates at its nodes, for their children
            const unsigned n4 = (unsigned)((size_t)m * D / 4);
            hipLaunchKernelGGL(copy_f4_kernel, dim3((n4 + 255) / 256), dim3(256), 0, c->stream, (const float4*)c->d_h(),
                               (float4*)(c->d_fest() + (size_t)c->tree->i0 * D), n4);
            LAUNCH_CHECK(c, "feature estimates");
        } else if (M.head && last) {                     // the head's estimate of the last row's feature: input of its next step
            hipLaunchKernelGGL(copy_f4_kernel, dim3((D / 4 + 255) / 256), dim3(256), 0, c->stream,
                               (const float4*)(c->d_h() + (size_t)(m - 1) * D), (float4*)c->d_fest(), (unsigned)(D / 4));
            LAUNCH_CHECK(c, "feature estimate");
        }
        done += m;
    }
    M.kvl[0] = pos0 + n;
    return 0;
}


// ================================================================================================
// Blocks of rows from several sequences (cfg.batch > 1): the plain step-by-step forward on the
// segment-aware kernels of batch.h.  Rows R = sg.n * sg.ms; row-wise kernels (add+norm, activation)
// are the single-sequence ones launched over R rows.

// GEMM over R rows into split-K partials part[s][R][N] (split stride R*N).
template <typename T>
int gemm_rows(metasd_ctx* c, const void* x, int ldx, int R, int K, const void* W0, int n0, const void* W1, int n1, const void* W2,
              int n2, int* nsplit_out);

template <>
int gemm_rows<float>(metasd_ctx* c, const void* x, int ldx, int R, int K, const void* W0, int n0, const void* W1, int n1,
                     const void* W2, int n2, int* nsplit_out) {
    const int N = n0 + n1 + n2;
    for (int r0 = 0; r0 < R; r0 += MAX_ROWS) {
        hipLaunchKernelGGL(gemm_f32_kernel, dim3((N + 3) / 4), dim3(256), 0, c->stream, (const float*)x + (size_t)r0 * ldx, ldx,
                           std::min(MAX_ROWS, R - r0), K, (const float*)W0, (const float*)W1, (const float*)W2, n0, n0 + n1, N,
                           c->d_part() + (size_t)r0 * N);
        LAUNCH_CHECK(c, "gemm_f32");
    }
    *nsplit_out = 1;
    return 0;
}

// The plan of a many-row launch, kept per shape (a forward repeats a handful of them; the search takes a microsecond or two).
const RowsPlan& rows_plan(metasd_ctx* c, int ntiles, int kchunks, int R, int groups, int behind = BEHIND_NONE) {
    auto& e = c->plans[(unsigned)(ntiles * 31 + kchunks * 17 + R * 5 + groups + behind) % (sizeof c->plans / sizeof c->plans[0])];
    if (e.ntiles != ntiles || e.kchunks != kchunks || e.R != R || e.groups != groups || e.behind != behind) {
        e.ntiles = ntiles; e.kchunks = kchunks; e.R = R; e.groups = groups; e.behind = behind;
        e.plan = plan_rows(ntiles, kchunks, R, groups, c->rows_tpb, c->rows_rb, behind);
    }
    return e.plan;
}

// One launch of the many-row GEMM.  out, N: partials [ks][R][N] or what the epilogue writes.
struct TilesLaunch {
    const bf16_t* x;
    int R, K;
    const void *W0, *W1, *W2;
    int t0, t1, ntiles;
    const RowGroups* gg;
    float* out;
    int N;
    TilesEpi ep;
};

// more than 64 KiB of dynamic LDS needs the function attribute (set once per variant)
template <int RB, int TB, int EPI>
int launch_gemm_tiles(metasd_ctx* c, const TilesLaunch& a, const RowsPlan& s, metasd_ctx::ProfRec* pr) {
    constexpr int NS = rows_stages(RB, TB);
    constexpr int lds = NS * (8192 * RB + 2048 * TB);
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    const hipEvent_t ea = pr ? pr->a : nullptr, eb = pr ? pr->b : nullptr;
    const dim3 grid(s.nrb * s.ngroups * s.ksplit, a.gg ? a.gg->n : 1);
    // forms that do not exist (the callers' plans avoid them): a wavefront with an odd number of tiles has no pairs of gate and up, and row
    // groups have neither rotations nor residual rows
    if (EPI == TILES_ACT && TB % 2 && a.ep.swiglu) return c->fail(METASD_E_INVALID, "many-row GEMM: SwiGLU behind %d tiles per wavefront", TB);
    if (a.gg) {
        if constexpr (EPI != TILES_PART && EPI != TILES_ACT) return c->fail(METASD_E_INVALID, "many-row GEMM: row groups with epilogue %d", EPI);
        else {
            static const hipError_t attr = hipFuncSetAttribute((const void*)gemm_tiles_grouped_kernel<RB, TB, NS, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (attr != hipSuccess) return c->fail(METASD_E_HIP, "gemm_tiles_grouped_kernel: cannot reserve %d bytes of LDS", lds);
            hipExtLaunchKernelGGL((gemm_tiles_grouped_kernel<RB, TB, NS, EPI>), grid, dim3(512), (uint32_t)lds, c->stream, ea, eb, 0u, a.x, a.K / 32, a.t0,
                                  a.t1, a.ntiles, a.out, (size_t)a.R * a.N, a.N, s.cps, s.nrb, *a.gg, a.ep);
        }
    } else {
        static const hipError_t attr = hipFuncSetAttribute((const void*)gemm_tiles_kernel<RB, TB, NS, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (attr != hipSuccess) return c->fail(METASD_E_HIP, "gemm_tiles_kernel: cannot reserve %d bytes of LDS", lds);
        hipExtLaunchKernelGGL((gemm_tiles_kernel<RB, TB, NS, EPI>), grid, dim3(512), (uint32_t)lds, c->stream, ea, eb, 0u, a.x, a.R, a.K / 32,
                              (const bf16_t*)a.W0, (const bf16_t*)a.W1, (const bf16_t*)a.W2, a.t0, a.t1, a.ntiles, a.out, (size_t)a.R * a.N, a.N, s.cps,
                              s.nrb, a.ep);
    }
    LAUNCH_CHECK(c, "gemm_tiles");
    return 0;
}

template <int EPI>
int launch_gemm_tiles_any(metasd_ctx* c, const TilesLaunch& a, const RowsPlan& s, metasd_ctx::ProfRec* pr) {
#define TILES_GO(RB, TB) if (s.rb == RB && s.tb == TB) return launch_gemm_tiles<RB, TB, EPI>(c, a, s, pr)
    TILES_GO(4, 6); TILES_GO(3, 8); TILES_GO(3, 6); TILES_GO(3, 4); TILES_GO(2, 8); TILES_GO(2, 6);
    TILES_GO(2, 4); TILES_GO(2, 3); TILES_GO(1, 8); TILES_GO(1, 6); TILES_GO(1, 4); TILES_GO(1, 2);
#undef TILES_GO
    return c->fail(METASD_E_INVALID, "many-row GEMM: no tile of %d x %d", s.rb, s.tb);
}

// R > MAX_ROWS: x interleaved (store_terms4, split = 2); R <= MAX_ROWS: two arrays (split = 1)
int rows_split(int R) { return R > MAX_ROWS ? 2 : 1; }

template <>
int gemm_rows<bf16_t>(metasd_ctx* c, const void* x, int ldx, int R, int K, const void* W0, int n0, const void* W1, int n1,
                      const void* W2, int n2, int* nsplit_out) {
    if (R <= MAX_ROWS) return gemm<bf16_t>(c, x, ldx, R, K, W0, n0, W1, n1, W2, n2, nullptr, nsplit_out, (size_t)R * ldx);
    const int N = n0 + n1 + n2;
    const RowsPlan& s = rows_plan(c, N / 16, K / 32, R, 1);
    metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_GEMM, (double)N * K * 2 + (double)R * K * 4 + (double)R * N * 4 * s.ksplit, N, K, R);
    *nsplit_out = s.ksplit;
    return launch_gemm_tiles_any<TILES_PART>(c, TilesLaunch{(const bf16_t*)x, R, K, W0, W1, W2, n0 / 16, (n0 + n1) / 16, N / 16, nullptr, c->d_part(), N, {}}, s, pr);
}

// h += x W^T where the plan leaves K whole (*nsplit_out = 0: nothing is left to add), else the partials
template <typename T>
int gemm_rows_add(metasd_ctx* c, const void* x, int R, int K, const void* W, int N, float* h, int* nsplit_out) {
    if constexpr (sizeof(T) == 2) {
        if (R > MAX_ROWS && rows_plan(c, N / 16, K / 32, R, 1).ksplit == 1) {
            const RowsPlan& s = rows_plan(c, N / 16, K / 32, R, 1);
            metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_GEMM, (double)N * K * 2 + (double)R * K * 4 + (double)R * N * 4, N, K, R);
            *nsplit_out = 0;
            return launch_gemm_tiles_any<TILES_ADD>(c, TilesLaunch{(const bf16_t*)x, R, K, W, W, W, N / 16, N / 16, N / 16, nullptr, h, N, {}}, s, pr);
        }
    }
    return gemm_rows<T>(c, x, K, R, K, W, N, nullptr, 0, nullptr, 0, nsplit_out);
}

// The activations of layer L's FFN from the normalised rows x (d_act; split as the rows are): in the projection's own launch where
// its plan leaves K whole, else from its partials.
template <typename T>
int gemm_rows_act(metasd_ctx* c, const Model& M, int L, const void* x, int R, int split) {
    const metasd_model_desc& d = M.d;
    const int D = d.d_model, F = d.d_ffn, sw = d.act == METASD_SWIGLU, NF = (sw ? 2 : 1) * F;
    const void *w0 = M.layer_w(L, sw ? 6 : 7), *w1 = sw ? M.layer_w(L, 7) : nullptr;
    if constexpr (sizeof(T) == 2) {
        if (R > MAX_ROWS) {
            const RowsPlan& s = rows_plan(c, NF / 16, D / 32, R, 1, sw ? BEHIND_PAIRS : BEHIND_ACT);
            if (s.ksplit == 1 && (!sw || s.tb % 2 == 0)) {
                metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_GEMM, (double)NF * D * 2 + (double)R * D * 4 + (double)R * F * 4, NF, D, R);
                TilesEpi ep{};
                ep.swiglu = sw;
                return launch_gemm_tiles_any<TILES_ACT>(c, TilesLaunch{(const bf16_t*)x, R, D, w0, w1, w1, F / 16, NF / 16, NF / 16, nullptr, (float*)c->d_act(), F, ep}, s, pr);
            }
        }
    }
    int ns = 0;
    if (int rc = gemm_rows<T>(c, x, D, R, D, w0, F, w1, sw ? F : 0, nullptr, 0, &ns)) return rc;
    const size_t nact = (size_t)R * F;
    hipLaunchKernelGGL(ffn_act4_kernel, dim3((unsigned)((nact / 4 + 255) / 256)), dim3(256), 0, c->stream, (const float*)c->d_part(), ns, (size_t)R * NF, R, F, d.act,
                       (float*)c->d_act(), split, (const float*)nullptr);
    LAUNCH_CHECK(c, "ffn_act");
    return 0;
}

// What the attention of a block is launched with, the same in every layer.
struct SegAttn {
    AttnPlan pl;       // bf16, head_dim 64 and 128
    int nch_max;       // chunks of ATT_CH positions of the longest context
    double kvpos;      // positions of all sequences
};
SegAttn plan_segs(const metasd_ctx* c, const metasd_model_desc& d, int hd, const Segs& sg) {
    SegAttn a{};
    int len[ATT_SEGS], max_len = 1;
    for (int s = 0; s < sg.n; ++s) {
        len[s] = sg.pos0[s] + sg.m[s];
        max_len = std::max(max_len, len[s]);
        a.kvpos += (double)len[s];
    }
    a.nch_max = (max_len + ATT_CH - 1) / ATT_CH;
    if (d.dtype == METASD_BF16 && hd >= 64) a.pl = plan_attn(len, sg.n, d.n_heads, d.n_kv_heads, hd, sg.ms, c->n_cu, c->att_cpw);
    return a;
}

template <typename T, int HD>
int attention_seg_hd(metasd_ctx* c, const Model& M, int L, const Segs& sg, const SegAttn& at) {
    const metasd_model_desc& d = M.d;
    const int R = sg.n * sg.ms;
    const size_t plane = (size_t)d.n_kv_heads * c->cfg.max_ctx * HD;
    const size_t seq_stride = (size_t)M.kv_layers * 2 * plane;
    const T* kc = (const T*)M.kv + (size_t)L * 2 * plane;
    const T* vc = kc + plane;
    const float scale = 1.0f / sqrtf((float)HD);
    metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_ATTN, 2.0 * d.n_kv_heads * at.kvpos * HD * sizeof(T) + (double)R * d.n_heads * HD * 4);
    hipEvent_t ea = pr ? pr->a : nullptr, eb = pr ? pr->b : nullptr;
    int nrec = at.nch_max, passes = 1;
    if constexpr (sizeof(T) == 2 && HD >= 64) {
        const AttnPlan& pl = at.pl;
        const AttnOut ao{c->d_apart(), pl.nrec, 0, 0, (float*)c->d_ao(), rows_split(R), (size_t)R * d.n_heads * HD, 0, 0};
        nrec = pl.nrec;
        passes = pl.spw / ATT_NW;
#define ATTN_GO(SHARED, EVEN) hipExtLaunchKernelGGL((attn_seg_kernel<HD, SHARED, false, EVEN>), dim3(pl.grid), dim3(64 * ATT_NW), 0u, c->stream, ea, eb, 0u, \
                                                   (const bf16_t*)c->d_q(), kc, vc, seq_stride, SegPtrs{}, SegPtrs{}, sg, d.n_heads, d.n_kv_heads, pl.hp, \
                                                   c->cfg.max_ctx, scale, (size_t)R * d.n_heads * HD, pl.spw, ao, pl.items)
        if (d.n_heads > d.n_kv_heads * pl.hp) { if (pl.even) ATTN_GO(true, true); else ATTN_GO(true, false); }
        else { if (pl.even) ATTN_GO(false, true); else ATTN_GO(false, false); }
#undef ATTN_GO
        if (nrec == 1) { LAUNCH_CHECK(c, "attn (segments)"); return 0; }
    } else {
        hipExtLaunchKernelGGL((attn_partial_seg_kernel<T, HD>), dim3(at.nch_max, d.n_heads, sg.n), dim3(256), 0u, c->stream, ea, eb, 0u,
                              (const float*)c->d_q(), kc, vc, seq_stride, sg, d.n_heads, d.n_kv_heads, c->cfg.max_ctx, scale,
                              c->d_apart(), at.nch_max);
    }
    LAUNCH_CHECK(c, "attn_partial (segments)");
    hipLaunchKernelGGL((attn_combine_seg_kernel<HD>), dim3(d.n_heads, R), dim3(HD), 0, c->stream, c->d_apart(), nrec, d.n_heads,
                       (float*)c->d_ao(), sizeof(T) == 2 ? rows_split(R) : 0, sg, passes, sizeof(T) == 2 && HD >= 64 ? 0 : 1);
    LAUNCH_CHECK(c, "attn_combine (segments)");
    return 0;
}

template <typename T>
int attention_seg(metasd_ctx* c, const Model& M, int L, const Segs& sg, const SegAttn& at) {
    switch (M.hd) {
        case 32: return attention_seg_hd<T, 32>(c, M, L, sg, at);
        case 64: return attention_seg_hd<T, 64>(c, M, L, sg, at);
        default:
            if constexpr (sizeof(T) == 2) return attention_seg_hd<T, 128>(c, M, L, sg, at);
            return c->fail(METASD_E_INVALID, "fp32 head_dim 128 unsupported");
    }
}

// Causal attention of the m rows of a long block (q in d_q, result in d_ao), 64 rows of a head per workgroup.
int attention_big(metasd_ctx* c, const metasd_model_desc& d, int hd, const bf16_t* kc, const bf16_t* vc, int pos0, int m) {
    const float scale = 1.0f / sqrtf((float)hd);
    metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_ATTN, 2.0 * d.n_kv_heads * (double)(pos0 + m) * hd * 2 + (double)m * d.n_heads * hd * 4);
    hipEvent_t ea = pr ? pr->a : nullptr, eb = pr ? pr->b : nullptr;
#define BIG_GO(HD) hipExtLaunchKernelGGL((attn_prefill_kernel<HD>), dim3((m + 63) / 64 * d.n_heads), dim3(256), 0u, c->stream, ea, eb, 0u, \
                                         (const bf16_t*)c->d_q(), kc, vc, m, pos0, d.n_heads, d.n_kv_heads, c->cfg.max_ctx, scale, (float*)c->d_ao(), rows_split(m))
    if (hd == 128) BIG_GO(128);
    else BIG_GO(64);
#undef BIG_GO
    LAUNCH_CHECK(c, "attn_prefill");
    return 0;
}

// add the split-K partials to the residual rows and normalise: many rows of 2048, 4096 or at most 1024 columns go through the form that
// keeps more requests in flight per CU (same arithmetic in the same order; other widths, which are no models of this library's own workloads,
// have not been measured and keep the general form); rows of 768 columns, of whose
// 1024 threads a workgroup of the general form uses 192: 32 rows 6.6 -> 4.2 us, 288 rows 17.4 -> 4.7, 1499 rows 19.8 -> 5.7
template <typename T>
void launch_addnorm_many(metasd_ctx* c, int R, float* h, const float* part, int ns, int D, const T* gain, float eps, float* xn, int split) {
#define ROWS_GO(COLS, NS) hipLaunchKernelGGL((addnorm_rows_kernel<T, COLS, NS>), dim3(R), dim3(256), 0, c->stream, h, part, ns, (size_t)R * D, gain, eps, xn, split, D)
    if (R > MAX_ROWS && D == 4096) { if (ns <= 2) ROWS_GO(4, 2); else if (ns <= 4) ROWS_GO(4, 4); else ROWS_GO(4, 8); }
    else if (R > MAX_ROWS && D == 2048) { if (ns <= 2) ROWS_GO(2, 2); else if (ns <= 4) ROWS_GO(2, 4); else ROWS_GO(2, 8); }
    else if (R > MAX_ROWS && D <= 1024 && D % 4 == 0) { if (ns <= 2) ROWS_GO(1, 2); else if (ns <= 4) ROWS_GO(1, 4); else ROWS_GO(1, 8); }
#undef ROWS_GO
    else
        hipLaunchKernelGGL(addnorm_kernel<T>, dim3(R), dim3(1024), 0, c->stream, h, part, ns, (size_t)R * D, D, gain, eps, xn, split);
}

// Forward of the block sg through model M; appends K/V of the valid rows.  logits == nullptr: none.
// Otherwise the rows that carry logits are written to logits[(seq * out_seq_rows + out_row0 + j) * V]
// (last_only: only the last valid row of each segment, at j = 0).
template <typename T>
int forward_segs_t(metasd_ctx* c, Model& M, const Segs& sg, float* logits, int out_seq_rows, int out_row0, int last_only) {
    const metasd_model_desc& d = M.d;
    const int D = d.d_model, H = d.n_heads, KH = d.n_kv_heads, hd = M.hd, F = d.d_ffn, V = d.vocab;
    const int DQ = H * hd, DKV = KH * hd, NQKV = DQ + 2 * DKV;
    const int R = sg.n * sg.ms;
    hipStream_t st = c->stream;
    float* h = c->d_h();
    float* xn = (float*)c->d_xn();
    float* part = c->d_part();
    int ns = 0, rc;
    const int split = sizeof(T) == 2 ? rows_split(R) : 0;
    const size_t plane = (size_t)KH * c->cfg.max_ctx * hd;
    const size_t seq_stride = (size_t)M.kv_layers * 2 * plane;
    hipLaunchKernelGGL(embed_seg_kernel<T>, dim3(R), dim3(256), 0, st, (const int32_t*)c->d_hist(), c->cfg.max_ctx, (const T*)M.w[0], D, h, sg);
    LAUNCH_CHECK(c, "embed (segments)");
    hipLaunchKernelGGL(rope_table_seg_kernel, dim3(R), dim3(hd / 2), 0, st, sg, hd, d.rope_theta, c->d_rope(), (long long*)nullptr, (size_t)0);
    LAUNCH_CHECK(c, "rope_table (segments)");
    const SegAttn at = plan_segs(c, d, hd, sg);
    for (int L = 0; L < d.n_layers; ++L) {
        launch_addnorm_many<T>(c, R, h, part, ns, D, (const T*)M.layer_w(L, 0), d.rms_eps, xn, split);
        LAUNCH_CHECK(c, "addnorm");
        if ((rc = gemm_rows<T>(c, xn, D, R, D, M.layer_w(L, 1), DQ, M.layer_w(L, 2), DKV, M.layer_w(L, 3), DKV, &ns))) return rc;
        T* kc = (T*)M.kv + (size_t)L * 2 * plane;
        if (sizeof(T) == 2 && R >= ROPE4_ROWS && hd >= 64)
            hipLaunchKernelGGL(rope_kv4_seg_kernel, dim3((NQKV + 1023) / 1024, R), dim3(256), 0, st, part, ns, (size_t)R * NQKV, NQKV, sg, H, KH, hd,
                               (const double2*)c->d_rope(), (bf16_t*)c->d_q(), (bf16_t*)kc, (bf16_t*)(kc + plane), seq_stride, c->cfg.max_ctx);
        else
            hipLaunchKernelGGL(rope_kv_seg_kernel<T>, dim3(H + 2 * KH, R), dim3(64), 0, st, part, ns, (size_t)R * NQKV, NQKV, sg, H, KH, hd,
                               (const double2*)c->d_rope(), (float*)c->d_q(), kc, kc + plane, seq_stride, c->cfg.max_ctx, sizeof(T) == 2 ? 1 : 0,
                               (split && hd >= 64) ? 1 : 0);
        LAUNCH_CHECK(c, "rope_kv (segments)");
        if ((rc = attention_seg<T>(c, M, L, sg, at))) return rc;
        if ((rc = gemm_rows_add<T>(c, c->d_ao(), R, DQ, M.layer_w(L, 4), D, h, &ns))) return rc;
        launch_addnorm_many<T>(c, R, h, part, ns, D, (const T*)M.layer_w(L, 5), d.rms_eps, xn, split);
        LAUNCH_CHECK(c, "addnorm");
        if ((rc = gemm_rows_act<T>(c, M, L, xn, R, split))) return rc;
        if ((rc = gemm_rows_add<T>(c, c->d_act(), R, F, M.layer_w(L, 8), D, h, &ns))) return rc;
    }
    if (logits) {
        launch_addnorm_many<T>(c, R, h, part, ns, D, (const T*)M.final_norm(), d.rms_eps, xn, split);
        LAUNCH_CHECK(c, "addnorm");
        if ((rc = gemm_rows<T>(c, xn, D, R, D, M.lm_head(), V, nullptr, 0, nullptr, 0, &ns))) return rc;
        hipLaunchKernelGGL(sum_partials_seg_kernel, dim3((V + 255) / 256, R), dim3(256), 0, st, (const float*)part, ns, (size_t)R * V, V,
                           logits, sg, out_seq_rows, out_row0, last_only);
        LAUNCH_CHECK(c, "sum_partials (segments)");
    }
    for (int s = 0; s < sg.n; ++s) M.kvl[sg.seq[s]] = sg.pos0[s] + sg.m[s];
    return 0;
}

// At most 8 rows (16 of at most 2048 columns) of several sequences (the drafter steps of a small batch, its verification): the step GEMMs of
// forward_rows_step with the rows' places in their caches taken from a table - 5 launches per layer (6 where attention leaves records)
// instead of 10.  One row in each of 5 sequences, 1B shape, per layer: 60 -> 43 us.
bool segs_step_ok(const metasd_ctx* c, const Model& M, int R) {
    return c->fuse_small && c->gemm_reduce && c->fullk_roll && M.d.dtype == METASD_BF16 && M.hd >= 64 && M.d.d_model >= STEP_DMIN && step_ok(R, M.d.d_model);
}
int forward_segs_step(metasd_ctx* c, Model& M, const Segs& sg, float* logits, int out_seq_rows, int out_row0, int last_only) {
    typedef bf16_t T;
    const metasd_model_desc& d = M.d;
    const int D = d.d_model, F = d.d_ffn, V = d.vocab, hd = M.hd, DQ = d.n_heads * hd, R = sg.n * sg.ms;
    hipStream_t st = c->stream;
    float* h = c->d_h();
    long long* rowkv = reinterpret_cast<long long*>(c->d_inv());       // the 1/rms table, which this path does not use
    static_assert(STEP_ROWS * sizeof(long long) <= INV_BYTES, "row table");
    int rc;
    hipLaunchKernelGGL(embed_seg_kernel<T>, dim3(R), dim3(256), 0, st, (const int32_t*)c->d_hist(), c->cfg.max_ctx, (const T*)M.w[0], D, h, sg);
    LAUNCH_CHECK(c, "embed (segments)");
    hipLaunchKernelGGL(rope_table_seg_kernel, dim3(R), dim3(hd / 2), 0, st, sg, hd, d.rope_theta, c->d_rope(), rowkv,
                       (size_t)M.kv_layers * 2 * d.n_kv_heads * c->cfg.max_ctx * hd);
    LAUNCH_CHECK(c, "rope_table (segments)");
    auto norm_in = [&](const void* gain) {
        StepArgs a{};
        a.h = h; a.gain = (const bf16_t*)gain; a.eps = d.rms_eps; a.m = R; a.K = D;
        return a;
    };
    const SegAttn at = plan_segs(c, d, hd, sg);
    for (int L = 0; L < d.n_layers; ++L) {
        StepArgs a = norm_in(M.layer_w(L, 0));
        a.rowkv = rowkv;
        if ((rc = gemm_step_qkv(c, M, L, 0, a))) return rc;
        if ((rc = attention_seg<T>(c, M, L, sg, at))) return rc;
        if ((rc = residual_add(c, c->d_ao(), R, DQ, M.layer_w(L, 4), D, h, M.layer_w(L, 5)))) return rc;
        a = norm_in(M.layer_w(L, 5));
        a.out = (float*)c->d_act(); a.N = F; a.swiglu = d.act == METASD_SWIGLU;
        if (a.swiglu) rc = gemm_step_norm<STEP_ACT, false>(c, a, M.layer_w(L, 6), F, M.layer_w(L, 7), F, nullptr, 0);
        else rc = gemm_step_norm<STEP_ACT, false>(c, a, M.layer_w(L, 7), F, nullptr, 0, nullptr, 0);
        if (rc) return rc;
        if ((rc = residual_add(c, c->d_act(), R, F, M.layer_w(L, 8), D, h, M.layer_w(L, 5)))) return rc;
    }
    if (logits) {
        StepArgs a = norm_in(M.final_norm());
        a.out = c->d_part(); a.N = V;
        if ((rc = gemm_step_norm<STEP_OUT, false>(c, a, M.lm_head(), V, nullptr, 0, nullptr, 0))) return rc;
        hipLaunchKernelGGL(sum_partials_seg_kernel, dim3((V + 255) / 256, R), dim3(256), 0, st, (const float*)c->d_part(), 1, (size_t)R * V, V, logits, sg,
                           out_seq_rows, out_row0, last_only);
        LAUNCH_CHECK(c, "sum_partials (segments)");
    }
    for (int s = 0; s < sg.n; ++s) M.kvl[sg.seq[s]] = sg.pos0[s] + sg.m[s];
    return 0;
}

// n consecutive tokens of one sequence, hist[seq][pos0 .. pos0 + n), through model M in blocks of up to BIG_ROWS rows: what
// they leave is their K/V (and, with drafter heads, the target's features).  bf16 models with head_dim >= 64; no tree or
// streaming mask.  Every weight is read once per pass instead of once per 16 rows: a 1500-token query start on the 7B shape
// took 362 ms in 16-row blocks and takes 41 ms, 512 tokens on the 1B shape 40.7 and 4.3 ms.  The last layer ends with its K/V: nothing
// reads what follows, unless the features are wanted.
int forward_big(metasd_ctx* c, Model& M, int seq, int pos0, int n) {
    typedef bf16_t T;
    const metasd_model_desc& d = M.d;
    const int D = d.d_model, H = d.n_heads, KH = d.n_kv_heads, hd = M.hd, F = d.d_ffn;
    const int DQ = H * hd, DKV = KH * hd, NQKV = DQ + 2 * DKV;
    hipStream_t st = c->stream;
    float* h = c->d_h();
    float* xn = (float*)c->d_xn();
    float* part = c->d_part();
    const size_t plane = (size_t)KH * c->cfg.max_ctx * hd;
    T* kv = (T*)M.kv + (size_t)seq * M.kv_layers * 2 * plane;
    const bool features = &M == &c->target && c->cfg.feature_heads;
    if (pos0 + n > c->cfg.max_ctx) return c->fail(METASD_E_OVERFLOW, "positions %d..%d exceed max_ctx %d", pos0, pos0 + n, c->cfg.max_ctx);
    c->cur_model = model_index(c, M);
    for (int done = 0; done < n;) {
        const int m = std::min(big_rows(c->cfg), n - done), p0 = pos0 + done, split = rows_split(m);
        int ns = 0, rc;
        hipLaunchKernelGGL(embed_rope_kernel<T>, dim3(m), dim3(320), 0, st, c->d_hist() + (size_t)seq * c->cfg.max_ctx + p0, (const T*)M.w[0], D,
                           h, p0, hd, d.rope_theta, c->d_rope(), TreeBlk{});
        LAUNCH_CHECK(c, "embed + rope table");
        if (M.head) {   // W_fc . [embedding ; the target's feature of the position before]
            float* cat = (float*)c->d_act();
            hipLaunchKernelGGL(feat_cat_kernel, dim3(m), dim3(256), 0, st, (const float*)h, (const float*)c->d_feat(), (const float*)nullptr,
                               FeatSrc{}, p0, D, cat, split);
            LAUNCH_CHECK(c, "feat_cat");
            if ((rc = gemm_rows<T>(c, cat, 2 * D, m, 2 * D, M.fc, D, nullptr, 0, nullptr, 0, &ns))) return rc;
            const size_t nh = (size_t)m * D;
            hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)((nh + 255) / 256)), dim3(256), 0, st, (const float*)part, ns, nh, nh, h,
                               (const float*)nullptr, D);
            LAUNCH_CHECK(c, "sum_partials");
            ns = 0;
        }
        for (int L = 0; L < d.n_layers; ++L) {
            launch_addnorm_many<T>(c, m, h, part, ns, D, (const T*)M.layer_w(L, 0), d.rms_eps, xn, split);
            LAUNCH_CHECK(c, "addnorm");
            T* kc = kv + (size_t)L * 2 * plane;
            const RowsPlan* pl = m > MAX_ROWS ? &rows_plan(c, NQKV / 16, D / 32, m, 1, BEHIND_ROPE) : nullptr;
            if (pl && pl->ksplit == 1) {
                metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_GEMM, (double)NQKV * D * 2 + (double)m * D * 4 + (double)m * NQKV * 4, NQKV, D, m);
                const TilesEpi ep{0, 0, (const double2*)c->d_rope(), kc, kc + plane, H, KH, hd, p0, c->cfg.max_ctx};
                if ((rc = launch_gemm_tiles_any<TILES_ROPE>(c, TilesLaunch{(const bf16_t*)xn, m, D, M.layer_w(L, 1), M.layer_w(L, 2), M.layer_w(L, 3), DQ / 16,
                                                                          (DQ + DKV) / 16, NQKV / 16, nullptr, (float*)c->d_q(), DQ, ep}, *pl, pr))) return rc;
            } else {
                if ((rc = gemm_rows<T>(c, xn, D, m, D, M.layer_w(L, 1), DQ, M.layer_w(L, 2), DKV, M.layer_w(L, 3), DKV, &ns))) return rc;
                if (m >= ROPE4_ROWS)
                    hipLaunchKernelGGL(rope_kv4_kernel, dim3((NQKV + 1023) / 1024, m), dim3(256), 0, st, part, ns, (size_t)m * NQKV, NQKV, p0, H, KH, hd,
                                       (const double2*)c->d_rope(), (bf16_t*)c->d_q(), kc, kc + plane, c->cfg.max_ctx);
                else
                    hipLaunchKernelGGL(rope_kv_kernel<T>, dim3((H + 2 * KH + 3) / 4, m), dim3(256), 0, st, part, ns, (size_t)m * NQKV, NQKV, p0, H, KH, hd,
                                       (const double2*)c->d_rope(), (float*)c->d_q(), kc, kc + plane, c->cfg.max_ctx, 1, 1, (const float*)nullptr);
                LAUNCH_CHECK(c, "rope_kv");
            }
            if (L + 1 == d.n_layers && !features) break;
            if ((rc = attention_big(c, d, hd, kc, kc + plane, p0, m))) return rc;
            if ((rc = gemm_rows_add<T>(c, c->d_ao(), m, DQ, M.layer_w(L, 4), D, h, &ns))) return rc;
            launch_addnorm_many<T>(c, m, h, part, ns, D, (const T*)M.layer_w(L, 5), d.rms_eps, xn, split);
            LAUNCH_CHECK(c, "addnorm");
            if ((rc = gemm_rows_act<T>(c, M, L, xn, m, split))) return rc;
            if ((rc = gemm_rows_add<T>(c, c->d_act(), m, F, M.layer_w(L, 8), D, h, &ns))) return rc;
        }
        if (features) {
            launch_addnorm_many<T>(c, m, h, part, ns, D, (const T*)M.final_norm(), d.rms_eps, xn, split);   // finishes the residual rows
            LAUNCH_CHECK(c, "addnorm");
            const unsigned n4 = (unsigned)((size_t)m * D / 4);
            hipLaunchKernelGGL(copy_f4_kernel, dim3((n4 + 255) / 256), dim3(256), 0, st, (const float4*)h, (float4*)(c->d_feat() + (size_t)p0 * D), n4);
            LAUNCH_CHECK(c, "feature rows");
        }
        done += m;
    }
    M.kvl[seq] = pos0 + n;
    return 0;
}

int forward_segs(metasd_ctx* c, Model& M, const Segs& sg, float* logits, int out_seq_rows, int out_row0, int last_only) {
    c->cur_model = model_index(c, M);
    for (int s = 0; s < sg.n; ++s)
        if (sg.pos0[s] + sg.m[s] > c->cfg.max_ctx)
            return c->fail(METASD_E_OVERFLOW, "sequence %d: positions %d..%d exceed max_ctx %d", sg.seq[s], sg.pos0[s], sg.pos0[s] + sg.m[s], c->cfg.max_ctx);
    if (segs_step_ok(c, M, sg.n * sg.ms)) return forward_segs_step(c, M, sg, logits, out_seq_rows, out_row0, last_only);
    if (M.d.dtype == METASD_BF16) return forward_segs_t<bf16_t>(c, M, sg, logits, out_seq_rows, out_row0, last_only);
    return forward_segs_t<float>(c, M, sg, logits, out_seq_rows, out_row0, last_only);
}

// ---- one drafter step of a batched round as a single forward: every sequence advances by one token in the drafter
// its bandit chose.  All drafters must have the same shape (bf16, head_dim >= 64); segments are ordered by arm, each
// kernel that touches weights or caches takes them per segment / per group (25 launches per step instead of 25 per
// arm in use - the draft phase of a batch is bound by the host's launch rate otherwise).

bool same_shape(const metasd_model_desc& a, const metasd_model_desc& b) {
    return a.n_layers == b.n_layers && a.d_model == b.d_model && a.n_heads == b.n_heads && a.n_kv_heads == b.n_kv_heads &&
           a.d_ffn == b.d_ffn && a.vocab == b.vocab && a.act == b.act && a.dtype == b.dtype && a.rms_eps == b.rms_eps &&
           a.rope_theta == b.rope_theta;
}

bool grouped_step_supported(const metasd_ctx* c) {
    if (!c->grouped_on || c->cfg.K > MAX_GROUPS) return false;
    const metasd_model_desc& d0 = c->drafters[0].d;
    if (d0.dtype != METASD_BF16 || c->drafters[0].hd < 64) return false;
    for (int a = 1; a < c->cfg.K; ++a)
        if (!same_shape(d0, c->drafters[a].d)) return false;
    return true;
}

// x: R rows, interleaved (store_terms4, split = 2); gg: the row groups and their matrices.
// act >= 0 (METASD_GELU, METASD_SWIGLU): the activations in d_act instead of partials where the plan leaves K whole (*nsplit_out = 0).
int gemm_rows_grouped(metasd_ctx* c, const void* x, int R, int K, const RowGroups& gg, int n0, int n1, int n2, int* nsplit_out, int act = -1) {
    const int N = n0 + n1 + n2;
    int mmax = 1;
    for (int g = 0; g < gg.n; ++g) mmax = std::max(mmax, gg.m[g]);
    const RowsPlan& s = rows_plan(c, N / 16, K / 32, mmax, gg.n, act < 0 ? BEHIND_NONE : act == METASD_SWIGLU ? BEHIND_PAIRS : BEHIND_ACT);
    metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_GEMM, (double)gg.n * N * K * 2 + (double)R * K * 4 + (double)R * N * 4 * s.ksplit, N, K, R);
    TilesLaunch a{(const bf16_t*)x, R, K, nullptr, nullptr, nullptr, n0 / 16, (n0 + n1) / 16, N / 16, &gg, c->d_part(), N, {}};
    if (act >= 0 && s.ksplit == 1 && (act != METASD_SWIGLU || s.tb % 2 == 0)) {
        a.out = (float*)c->d_act(); a.N = n0; a.ep.swiglu = act == METASD_SWIGLU;
        *nsplit_out = 0;
        return launch_gemm_tiles_any<TILES_ACT>(c, a, s, pr);
    }
    *nsplit_out = s.ksplit;
    return launch_gemm_tiles_any<TILES_PART>(c, a, s, pr);
}

// sg: the segments ordered by arm (ms <= 16 rows each, at most 256 rows per arm); arm[s]: the drafter of segment s.
// The logits of each segment's last valid row go to logits[(seq * out_seq_rows + out_row0) * V].
template <int HD>
int forward_step_grouped(metasd_ctx* c, const Segs& sg, const int* arm, float* logits, int out_seq_rows, int out_row0) {
    typedef bf16_t T;
    c->cur_model = arm[0];
    const metasd_model_desc& d = c->drafters[arm[0]].d;
    const int D = d.d_model, H = d.n_heads, KH = d.n_kv_heads, hd = HD, F = d.d_ffn, V = d.vocab;
    const int DQ = H * hd, DKV = KH * hd, NQKV = DQ + 2 * DKV;
    const int R = sg.n * sg.ms;
    hipStream_t st = c->stream;
    float* h = c->d_h();
    float* xn = (float*)c->d_xn();
    float* part = c->d_part();
    int ns = 0, rc;
    const size_t plane = (size_t)KH * c->cfg.max_ctx * hd;
    // groups of consecutive segments with one arm
    RowGroups gg{};
    for (int s0 = 0; s0 < sg.n;) {
        int s1 = s0;
        while (s1 < sg.n && arm[s1] == arm[s0]) ++s1;
        gg.r0[gg.n] = s0 * sg.ms; gg.m[gg.n] = (s1 - s0) * sg.ms; ++gg.n;
        s0 = s1;
    }
    auto seg_ptrs = [&](auto&& of_model) {
        SegPtrs p{};
        for (int s = 0; s < sg.n; ++s) p.p[s] = of_model(c->drafters[arm[s]], s);
        return p;
    };
    auto weights = [&](int L, int i0, int i1, int i2) {
        RowGroups g = gg;
        for (int q = 0; q < g.n; ++q) {
            const Model& M = c->drafters[arm[g.r0[q] / sg.ms]];
            g.W[q][0] = (const bf16_t*)(L < 0 ? M.lm_head() : M.layer_w(L, i0));
            g.W[q][1] = i1 >= 0 ? (const bf16_t*)M.layer_w(L, i1) : nullptr;
            g.W[q][2] = i2 >= 0 ? (const bf16_t*)M.layer_w(L, i2) : nullptr;
        }
        return g;
    };
    hipLaunchKernelGGL(embed_segp_kernel<T>, dim3(R), dim3(256), 0, st, (const int32_t*)c->d_hist(), c->cfg.max_ctx,
                       seg_ptrs([](const Model& M, int) { return (const void*)M.w[0]; }), D, h, sg);
    LAUNCH_CHECK(c, "embed (grouped)");
    hipLaunchKernelGGL(rope_table_seg_kernel, dim3(R), dim3(hd / 2), 0, st, sg, hd, d.rope_theta, c->d_rope(), (long long*)nullptr, (size_t)0);
    LAUNCH_CHECK(c, "rope_table (segments)");
    const SegAttn at = plan_segs(c, d, HD, sg);
    const AttnPlan& pl = at.pl;
    const AttnOut ao{c->d_apart(), pl.nrec, 0, 0, (float*)c->d_ao(), 2, (size_t)R * H * HD, 0, 0};
    const float scale = 1.0f / sqrtf((float)HD);
    for (int L = 0; L < d.n_layers; ++L) {
        hipLaunchKernelGGL(addnorm_segp_kernel<T>, dim3(R), dim3(1024), 0, st, h, part, ns, (size_t)R * D, D,
                           seg_ptrs([&](const Model& M, int) { return (const void*)M.layer_w(L, 0); }), sg.ms, d.rms_eps, xn, 2);
        LAUNCH_CHECK(c, "addnorm (grouped)");
        if ((rc = gemm_rows_grouped(c, xn, R, D, weights(L, 1, 2, 3), DQ, DKV, DKV, &ns))) return rc;
        const SegPtrs kcs = seg_ptrs([&](const Model& M, int s) { return (const void*)((const T*)M.kv + (size_t)L * 2 * plane + (size_t)sg.seq[s] * M.kv_layers * 2 * plane); });
        const SegPtrs vcs = seg_ptrs([&](const Model& M, int s) { return (const void*)((const T*)M.kv + (size_t)L * 2 * plane + plane + (size_t)sg.seq[s] * M.kv_layers * 2 * plane); });
        hipLaunchKernelGGL(rope_kv_segp_kernel<T>, dim3(H + 2 * KH, R), dim3(64), 0, st, part, ns, (size_t)R * NQKV, NQKV, sg, H, KH, hd,
                           (const double2*)c->d_rope(), (float*)c->d_q(), kcs, vcs, c->cfg.max_ctx, 1, 1);
        LAUNCH_CHECK(c, "rope_kv (grouped)");
        {
            metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_ATTN, 2.0 * KH * at.kvpos * HD * sizeof(T) + (double)R * H * HD * 4);
#define ATTN_GO(SHARED, EVEN) hipExtLaunchKernelGGL((attn_seg_kernel<HD, SHARED, true, EVEN>), dim3(pl.grid), dim3(64 * ATT_NW), 0u, st, pr ? pr->a : nullptr, \
                                                   pr ? pr->b : nullptr, 0u, (const bf16_t*)c->d_q(), (const bf16_t*)nullptr, (const bf16_t*)nullptr, (size_t)0, \
                                                   kcs, vcs, sg, H, KH, pl.hp, c->cfg.max_ctx, scale, (size_t)R * H * HD, pl.spw, ao, pl.items)
            if (H > KH * pl.hp) { if (pl.even) ATTN_GO(true, true); else ATTN_GO(true, false); }
            else { if (pl.even) ATTN_GO(false, true); else ATTN_GO(false, false); }
#undef ATTN_GO
            LAUNCH_CHECK(c, "attn (grouped)");
            if (pl.nrec > 1) {
                hipLaunchKernelGGL((attn_combine_seg_kernel<HD>), dim3(H, R), dim3(HD), 0, st, c->d_apart(), pl.nrec, H, (float*)c->d_ao(), 2, sg, pl.spw / ATT_NW, 0);
                LAUNCH_CHECK(c, "attn_combine (segments)");
            }
        }
        if ((rc = gemm_rows_grouped(c, c->d_ao(), R, DQ, weights(L, 4, -1, -1), D, 0, 0, &ns))) return rc;
        hipLaunchKernelGGL(addnorm_segp_kernel<T>, dim3(R), dim3(1024), 0, st, h, part, ns, (size_t)R * D, D,
                           seg_ptrs([&](const Model& M, int) { return (const void*)M.layer_w(L, 5); }), sg.ms, d.rms_eps, xn, 2);
        LAUNCH_CHECK(c, "addnorm (grouped)");
        const int sw = d.act == METASD_SWIGLU, NF = (sw ? 2 : 1) * F;
        if ((rc = gemm_rows_grouped(c, xn, R, D, sw ? weights(L, 6, 7, -1) : weights(L, 7, -1, -1), F, sw ? F : 0, 0, &ns, d.act))) return rc;
        if (ns) {
            const size_t nact = (size_t)R * F;
            hipLaunchKernelGGL(ffn_act4_kernel, dim3((unsigned)((nact / 4 + 255) / 256)), dim3(256), 0, st, part, ns, (size_t)R * NF, R, F, d.act,
                               (float*)c->d_act(), 2, (const float*)nullptr);
            LAUNCH_CHECK(c, "ffn_act");
        }
        if ((rc = gemm_rows_grouped(c, c->d_act(), R, F, weights(L, 8, -1, -1), D, 0, 0, &ns))) return rc;
    }
    hipLaunchKernelGGL(addnorm_segp_kernel<T>, dim3(R), dim3(1024), 0, st, h, part, ns, (size_t)R * D, D,
                       seg_ptrs([](const Model& M, int) { return (const void*)M.final_norm(); }), sg.ms, d.rms_eps, xn, 2);
    LAUNCH_CHECK(c, "addnorm (grouped)");
    if ((rc = gemm_rows_grouped(c, xn, R, D, weights(-1, 0, -1, -1), V, 0, 0, &ns))) return rc;
    hipLaunchKernelGGL(sum_partials_seg_kernel, dim3((V + 255) / 256, R), dim3(256), 0, st, (const float*)part, ns, (size_t)R * V, V,
                       logits, sg, out_seq_rows, out_row0, 1);
    LAUNCH_CHECK(c, "sum_partials (segments)");
    for (int s = 0; s < sg.n; ++s) c->drafters[arm[s]].kvl[sg.seq[s]] = sg.pos0[s] + sg.m[s];
    return 0;
}

// Model M processes, for every listed sequence, the tokens at positions [M.kvl[seq], upto[seq]) in blocks of
// at most 16 rows per sequence.  logits (optional): the logits of each sequence's last token go to
// logits[(seq * out_seq_rows + out_row0) * V].
int catch_up(metasd_ctx* c, Model& M, const std::vector<int>& seqs, const std::vector<int>& upto, float* logits, int out_seq_rows,
             int out_row0) {
    for (;;) {
        Segs sg{};
        int pend_max = 0;
        bool more = false;
        for (size_t i = 0; i < seqs.size(); ++i) {
            const int b = seqs[i], pend = upto[i] - M.kvl[b];
            if (pend <= 0) continue;
            const int s = sg.n++;
            sg.seq[s] = b; sg.pos0[s] = M.kvl[b]; sg.m[s] = std::min(MAX_ROWS, pend);
            pend_max = std::max(pend_max, sg.m[s]);
            more = more || pend > MAX_ROWS;
        }
        if (sg.n == 0) return 0;
        sg.ms = pend_max;
        // logits are only needed from a sequence's last block; every block that ends a sequence computes them
        bool ends = false;
        for (int s = 0; s < sg.n; ++s) {
            size_t i = 0;
            while (seqs[i] != sg.seq[s]) ++i;
            ends = ends || sg.pos0[s] + sg.m[s] == upto[i];
        }
        if (int rc = forward_segs(c, M, sg, (logits && ends) ? logits : nullptr, out_seq_rows, out_row0, 1)) return rc;
        if (!more) return 0;
    }
}

int launch_sample(hipStream_t st, const float* logits, int rows, int V, float T, uint64_t seed, uint32_t round, uint32_t pos,
                  uint32_t seq0, int32_t* tok, int stride, int32_t* tok_copy, const NextRow& next = NextRow{}) {
    hipLaunchKernelGGL(sample_rows_kernel, dim3(rows), dim3(AK_NT), 0, st, logits, V, T, seed, round, pos, seq0, tok, stride,
                       tok_copy, next);
    return hipGetLastError() == hipSuccess ? 0 : METASD_E_HIP;
}

bool accept_split_enabled() { return env_int("METASD_ACCEPT_SPLIT", 1) != 0; }   // read per launch: tests toggle it

// xchg != nullptr: four workgroups per (row, position) (accept_split_kernel); else one (accept_rows_kernel).
// rounds: the round word of the Philox counters, one per row (rt.n == rows) or the same for every row (rt.n == 0: rt.v[0]).
int launch_accept(hipStream_t st, const float* P, const float* Q, const int32_t* d, int rows, int gamma, int V, float T,
                  uint64_t seed, const RoundTab& rt, uint32_t seq0, int2* cand, double* bd, int32_t* n_acc, int32_t* token,
                  uint32_t* mask, int32_t* hist, int l, unsigned long long* xchg, hipEvent_t ev_begin = nullptr,
                  hipEvent_t ev_end = nullptr) {
    if (xchg && accept_split_enabled()) {   // one launch: the kernel also writes N_acc, the token and the mask
        // as many quarters as the vocabulary reaches into (one: no meeting at all), and as many groups of them as the chip holds at once, so
        // that a group requests its next item while it finishes one: 64 rows, gamma 5 24.4 against 26.1 us, 700 rows x 2 of 4096 17.5 / 19.2.
        // Past four items each the groups no longer end together and one item per group is faster (250 rows, gamma 7 96.8 / 93.4, 1000 x 2 of
        // 16000 47.3 / 49.9); greedy ones, whose items are one read, always have one (64 rows 13.3 us with several, 12.9 with
        // one and the loop over items, 12.3 without it).
        const int nq = (V + AS_QSEG - 1) / AS_QSEG, items = rows * (gamma + 1), slots = AS_SLOTS / nq;
        const int groups = T > 0.f && items <= 4 * slots ? std::min(items, slots) : items;
        const AsArgs a{P, Q, d, gamma, V, T, seed, seq0, (unsigned long long*)cand, bd, xchg, next_epoch(), std::max(0, env_int("METASD_ACCEPT_SPIN_LIMIT", 1 << 18)),
                       nq, items / groups, items % groups, n_acc, token, mask, hist, l};
#define ACCEPT_GO(KIND) hipExtLaunchKernelGGL((accept_split_kernel<KIND>), dim3(nq * groups), dim3(AS_NT), 0u, st, ev_begin, ev_end, 0u, a, rt)
        if (T <= 0.f) ACCEPT_GO(2);
        else if (T == 1.0f) ACCEPT_GO(0);
        else ACCEPT_GO(1);
#undef ACCEPT_GO
        return hipGetLastError() == hipSuccess ? 0 : METASD_E_HIP;
    }
    hipExtLaunchKernelGGL(accept_rows_kernel, dim3(gamma + 1, rows), dim3(AK_NT), 0u, st, ev_begin, ev_end, 0u, P, Q, d, gamma, V,
                          T, seed, rt, seq0, cand, bd);
    if (hipGetLastError() != hipSuccess) return METASD_E_HIP;
    hipLaunchKernelGGL(accept_finalize_kernel, dim3((rows + 63) / 64), dim3(64), 0, st, cand, rows, gamma, n_acc, token, mask,
                       hist, l);
    return hipGetLastError() == hipSuccess ? 0 : METASD_E_HIP;
}

bool valid_vocab(int V) { return V >= 4 && V % 4 == 0 && V <= AK_WAVES * AK_SEG; }

// ---- one round over a batch of independent sequences (cfg.batch > 1): every sequence drafts with its own
// arm (sequences that share an arm share that drafter's forward), one verification block over all
// batch x (gamma + 1) rows, one accept launch over all rows.

// A drafter that shares the target's cache has, by definition, processed exactly what the target has.
void sync_shared_kv(metasd_ctx* c) {
    for (auto& D : c->drafters)
        if (D.shared_kv) D.kvl = c->target.kvl;
}

RoundTab seq_rounds(const metasd_ctx* c) {
    RoundTab rt{};
    rt.n = c->cfg.batch;
    for (int b = 0; b < rt.n; ++b) rt.v[b] = (uint32_t)c->sq[b].round;
    return rt;
}
RoundTab one_round(uint32_t round) {
    RoundTab rt{};
    rt.v[0] = round;
    return rt;
}

int draft_batch(metasd_ctx* c, const int32_t* k, int gamma) {
    const int B = c->cfg.batch, V = c->target.d.vocab;
    for (int b = 0; b < B; ++b) {
        if (k[b] < 0 || k[b] >= c->cfg.K) return c->fail(METASD_E_INVALID, "draft: drafter index of sequence %d out of range", b);
        if (c->sq[b].l + gamma + 1 > c->cfg.max_ctx)
            return c->fail(METASD_E_OVERFLOW, "draft: sequence %d: l + gamma + 1 = %d exceeds max_ctx %d", b, c->sq[b].l + gamma + 1, c->cfg.max_ctx);
    }
    sync_shared_kv(c);
    SeqTab at{};
    const bool can_group = grouped_step_supported(c);
    // A drafter that has a long backlog in some sequences reads all but its last token in big blocks, sequence by sequence.  A
    // big block costs about as many launches as one 16-row block over all the sequences of the arm, so it wins once
    // the backlog has more such blocks than the arm has sequences.
    for (int b = 0; b < B; ++b) {
        Model& D = c->drafters[k[b]];
        const int pend = c->sq[b].l - D.kvl[b], nseq = (int)std::count(k, k + B, k[b]);
        if (big_ok(D.d) && pend > MAX_ROWS && pend > MAX_ROWS * nseq && big_pays(D.d, D.kvl[b], pend - 1, nseq))
            if (int rc = forward_big(c, D, b, D.kvl[b], pend - 1)) return rc;
    }
    for (int j = 0; j < gamma; ++j) {
        // one forward for all arms when more than one arm is in use and every sequence has 1..16 tokens to process in its
        // drafter (always so after the first step; in the first step unless a drafter was idle for many rounds)
        bool grouped = can_group;
        int arms_used = 0, pend_max = 0, rows_max = 0;
        for (int a = 0; a < c->cfg.K && grouped; ++a) {
            int nseq = 0;
            for (int b = 0; b < B; ++b)
                if (k[b] == a) {
                    ++nseq;
                    const int pend = c->sq[b].l + j - c->drafters[a].kvl[b];
                    if (pend < 1 || pend > MAX_ROWS) grouped = false;
                    pend_max = std::max(pend_max, pend);
                }
            arms_used += nseq > 0;
            rows_max = std::max(rows_max, nseq);
        }
        if (grouped && arms_used > 1 && rows_max * pend_max <= 256) {
            Segs sg{};
            int arm[MAX_SEGS];
            sg.ms = pend_max;
            for (int a = 0; a < c->cfg.K; ++a)
                for (int b = 0; b < B; ++b)
                    if (k[b] == a) {
                        const int s = sg.n++;
                        sg.seq[s] = b; sg.pos0[s] = c->drafters[a].kvl[b]; sg.m[s] = c->sq[b].l + j - c->drafters[a].kvl[b];
                        arm[s] = a;
                    }
            for (int s = 0; s < sg.n; ++s)
                if (sg.pos0[s] + sg.m[s] > c->cfg.max_ctx) return c->fail(METASD_E_OVERFLOW, "draft: sequence %d exceeds max_ctx", sg.seq[s]);
            const int rc = c->drafters[0].hd == 64 ? forward_step_grouped<64>(c, sg, arm, c->d_Q(), gamma, j)
                                                    : forward_step_grouped<128>(c, sg, arm, c->d_Q(), gamma, j);
            if (rc) return rc;
        } else
        for (int a = 0; a < c->cfg.K; ++a) {
            std::vector<int> seqs, upto;
            for (int b = 0; b < B; ++b)
                if (k[b] == a) { seqs.push_back(b); upto.push_back(c->sq[b].l + j); }
            if (seqs.empty()) continue;
            // j = 0: every committed token the drafter has not seen (ends with the last committed one);
            // j > 0: the draft token d_j at position l + j - 1
            if (int rc = catch_up(c, c->drafters[a], seqs, upto, c->d_Q(), gamma, j)) return rc;
        }
        for (int b = 0; b < B; ++b) at.v[b] = c->sq[b].l + j;
        hipLaunchKernelGGL(sample_seq_kernel, dim3(B), dim3(AK_NT), 0, c->stream, (const float*)c->d_Q() + (size_t)j * V, (size_t)gamma * V, V,
                           c->cfg.temperature, c->cfg.seed, seq_rounds(c), (uint32_t)j, c->d_hist(), c->cfg.max_ctx, at,
                           c->d_draft() + j, gamma);
        LAUNCH_CHECK(c, "sample (batch)");
    }
    for (int b = 0; b < B; ++b) c->sq[b].cur_k = k[b];
    return 0;
}

int verify_batch(metasd_ctx* c, int gamma) {
    Segs sg{};
    sg.n = c->cfg.batch;
    sg.ms = gamma + 1;
    for (int b = 0; b < sg.n; ++b) { sg.seq[b] = b; sg.m[b] = gamma + 1; sg.pos0[b] = c->sq[b].l - 1; }
    return forward_segs(c, c->target, sg, c->d_P(), gamma + 1, 0, 0);
}

int accept_batch(metasd_ctx* c, int gamma, int32_t* n_acc_out, int32_t* token_out, uint32_t* mask_out, double* bd_out) {
    const int B = c->cfg.batch, V = c->target.d.vocab, gm = c->cfg.gamma_max;
    int32_t* res = c->d_res();
    metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_ACCEPT, (double)B * (2 * gamma + 1) * V * 4);
    if (launch_accept(c->stream, c->d_P(), c->d_Q(), c->d_draft(), B, gamma, V, c->cfg.temperature, c->cfg.seed, seq_rounds(c), 0u,
                      c->d_cand(), c->d_bd(), res, res + B, (uint32_t*)(res + 2 * B), nullptr, 0, c->d_xchg(), pr ? pr->a : nullptr,
                      pr ? pr->b : nullptr))
        return c->fail(METASD_E_HIP, "launch accept kernels failed");
    SeqTab lt{};
    for (int b = 0; b < B; ++b) lt.v[b] = c->sq[b].l;
    hipLaunchKernelGGL(commit_tokens_kernel, dim3(1), dim3(64), 0, c->stream, (const int32_t*)res, (const int32_t*)(res + B), c->d_hist(),
                       c->cfg.max_ctx, lt, B);
    LAUNCH_CHECK(c, "commit_tokens");
    if (int rc = c->fetch_results()) return rc;
    (void)gm;
    const int32_t* hn = c->mirror<int32_t>(c->lay.res);
    bool timed_out = false;
    for (int b = 0; b < B; ++b) timed_out = timed_out || hn[B + b] == -2;
    if (timed_out && !c->mirror<GridBar>(c->lay.bar)->abort) {
        // some position's workgroups did not meet within their bounded wait: nothing of those rows was committed and the
        // logits are untouched - take the whole step again with one workgroup per position
        if (launch_accept(c->stream, c->d_P(), c->d_Q(), c->d_draft(), B, gamma, V, c->cfg.temperature, c->cfg.seed, seq_rounds(c), 0u,
                          c->d_cand(), c->d_bd(), res, res + B, (uint32_t*)(res + 2 * B), nullptr, 0, nullptr))
            return c->fail(METASD_E_HIP, "launch accept kernels failed");
        hipLaunchKernelGGL(commit_tokens_kernel, dim3(1), dim3(64), 0, c->stream, (const int32_t*)res, (const int32_t*)(res + B), c->d_hist(),
                           c->cfg.max_ctx, lt, B);
        LAUNCH_CHECK(c, "commit_tokens");
        if (int rc = c->fetch_results()) return rc;
        c->accept_fallbacks += 1;
    }
    const int32_t* ht = hn + B;
    const uint32_t* hm = (const uint32_t*)(hn + 2 * B);
    const int32_t* hd = c->mirror<int32_t>(c->lay.draft);
    const double* hbd = c->mirror<double>(c->lay.bd);
    if (c->mirror<GridBar>(c->lay.bar)->abort) {
        (void)hipMemsetAsync(c->d_bar(), 0, sizeof(GridBar), c->stream);
        c->phase = PH_NONE;
        for (auto& q : c->sq) q.ready = false;
        return c->fail(METASD_E_HIP, "a bounded device-side wait between workgroups timed out; call metasd_set_context (for every sequence) to start over");
    }
    for (int b = 0; b < B; ++b) {
        if (ht[b] == -2) { c->phase = PH_NONE; for (auto& q : c->sq) q.ready = false; return c->fail(METASD_E_HIP, "accept: the workgroups of a position did not meet (exchange timed out); call metasd_set_context to start over"); }
        if (hn[b] < 0 || hn[b] > gamma || ht[b] < 0 || ht[b] >= V) return c->fail(METASD_E_HIP, "accept: device returned n_acc %d token %d for sequence %d", hn[b], ht[b], b);
    }
    for (int b = 0; b < B; ++b) {
        metasd_ctx::SeqState& S = c->sq[b];
        const int l = S.l, n = hn[b];
        for (int j = 0; j < n; ++j) S.hist[l + j] = hd[(size_t)b * gamma + j];
        S.hist[l + n] = ht[b];
        S.l = l + n + 1;
        S.round += 1;
        c->target.kvl[b] = l + n;
        c->drafters[S.cur_k].kvl[b] = std::min(l + n, l + gamma - 1);
        if (n_acc_out) n_acc_out[b] = n;
        if (token_out) token_out[b] = ht[b];
        if (mask_out) mask_out[b] = hm[b];
        if (bd_out) {
            double sum = 0.0;
            for (int j = 0; j < gamma; ++j) sum += hbd[(size_t)b * gamma + j];
            bd_out[b] = sum / (double)gamma;
        }
    }
    sync_shared_kv(c);
    c->phase = PH_READY;
    return METASD_OK;
}

}  // namespace

namespace {
template <typename T>
int compact_kv(metasd_ctx* c, Model& M, int base, int limit) {
    const int planes = M.d.n_layers * 2 * M.d.n_kv_heads;
    const size_t total = (size_t)planes * M.hd;
    hipLaunchKernelGGL(kv_compact_kernel<T>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, c->stream, (T*)M.kv, planes, c->cfg.max_ctx, M.hd,
                       base, (const int32_t*)c->d_res(), limit, c->tshape.n);
    LAUNCH_CHECK(c, "kv_compact");
    return 0;
}

}  // namespace

// ================================================================================================ C ABI

extern "C" {

const char* metasd_last_error(const metasd_ctx* c) { return c ? c->err.c_str() : g_err.c_str(); }

int32_t metasd_kv_bytes(const metasd_model_desc* m, int32_t max_ctx, size_t* bytes_out) {
    if (!m || !bytes_out || max_ctx < 1) return fail_global(METASD_E_INVALID, "metasd_kv_bytes: bad argument");
    char buf[256];
    if (const char* e = check_model(*m, "model", buf, sizeof buf)) return fail_global(METASD_E_INVALID, "%s", e);
    *bytes_out = (size_t)m->n_layers * 2 * m->n_kv_heads * (size_t)max_ctx * (m->d_model / m->n_heads) * elem_size(*m);
    return METASD_OK;
}

static int check_config(const metasd_config* cfg, const metasd_model_desc* target, const metasd_model_desc* drafters) {
    if (!cfg || !target || !drafters) return fail_global(METASD_E_INVALID, "NULL config or descriptor");
    if (cfg->K < 1 || cfg->K > METASD_MAX_K) return fail_global(METASD_E_INVALID, "K must be in 1..%d", METASD_MAX_K);
    if (cfg->gamma_max < 1 || cfg->gamma_max > METASD_MAX_GAMMA) return fail_global(METASD_E_INVALID, "gamma_max must be in 1..%d", METASD_MAX_GAMMA);
    if (cfg->batch < 1 || cfg->batch > METASD_MAX_BATCH) return fail_global(METASD_E_INVALID, "batch must be in 1..%d", METASD_MAX_BATCH);
    if (cfg->max_ctx < cfg->gamma_max + 2) return fail_global(METASD_E_INVALID, "max_ctx too small");
    if (!(cfg->temperature >= 0.f)) return fail_global(METASD_E_INVALID, "temperature must be >= 0");
    if (cfg->reward != METASD_REWARD_BE && cfg->reward != METASD_REWARD_BD) return fail_global(METASD_E_INVALID, "reward");
    if (!(cfg->ucb_beta >= 0.0)) return fail_global(METASD_E_INVALID, "ucb_beta must be >= 0");
    switch (cfg->policy) {
        case METASD_POLICY_UCB: case METASD_POLICY_RANDOM: break;
        case METASD_POLICY_DUCB: case METASD_POLICY_EXP3:
            if (!(cfg->policy_param > 0.0 && cfg->policy_param <= 1.0)) return fail_global(METASD_E_INVALID, "policy_param must be in (0, 1] for this policy");
            break;
        case METASD_POLICY_SWUCB: case METASD_POLICY_SH:
            if (cfg->policy_window < 1) return fail_global(METASD_E_INVALID, "policy_window must be >= 1 for this policy");
            break;
        default: return fail_global(METASD_E_INVALID, "unknown policy %d", cfg->policy);
    }
    if (cfg->stream_window < 0 || cfg->stream_sink < 0) return fail_global(METASD_E_INVALID, "stream_sink and stream_window must be >= 0");
    if (cfg->stream_window > 0 && cfg->batch > 1) return fail_global(METASD_E_INVALID, "streaming drafter caches: contexts with one sequence only");
    if (cfg->feature_heads != 0 && cfg->feature_heads != 1) return fail_global(METASD_E_INVALID, "feature_heads must be 0 or 1");
    if (cfg->feature_heads && cfg->batch > 1) return fail_global(METASD_E_INVALID, "drafter heads on the target's hidden states: contexts with one sequence only");
    char buf[256];
    if (const char* e = check_model(*target, "target", buf, sizeof buf)) return fail_global(METASD_E_INVALID, "%s", e);
    for (int k = 0; k < cfg->K; ++k) {
        char who[32];
        snprintf(who, sizeof who, "drafter %d", k);
        if (const char* e = check_model(drafters[k], who, buf, sizeof buf)) return fail_global(METASD_E_INVALID, "%s", e);
        if (drafters[k].vocab != target->vocab) return fail_global(METASD_E_INVALID, "%s: vocab differs from the target's", who);
    }
    return METASD_OK;
}

int32_t metasd_workspace_bytes(const metasd_config* cfg, const metasd_model_desc* target, const metasd_model_desc* drafters,
                               size_t* bytes_out) {
    if (!bytes_out) return fail_global(METASD_E_INVALID, "NULL bytes_out");
    if (int rc = check_config(cfg, target, drafters)) return rc;
    *bytes_out = make_layout(*cfg, *target, drafters).total;
    return METASD_OK;
}

int32_t metasd_pack_weight(void* dst, const void* src, int32_t n_out, int32_t n_in, int32_t rope_head_dim, void* hip_stream) {
    if (!dst || !src || dst == src) return fail_global(METASD_E_INVALID, "metasd_pack_weight: NULL or aliased pointers");
    if (n_out < 16 || n_in < 32 || n_out % 16 || n_in % 32) return fail_global(METASD_E_INVALID, "metasd_pack_weight: n_out %% 16 and n_in %% 32 must be 0");
    if (rope_head_dim != 0 && (rope_head_dim < 32 || rope_head_dim % 32 || n_out % rope_head_dim))
        return fail_global(METASD_E_INVALID, "metasd_pack_weight: rope_head_dim must be 0 or a multiple of 32 dividing n_out");
    const size_t total = (size_t)n_out * n_in / 8;
    hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)hip_stream,
                       (const uint4*)src, (uint4*)dst, n_out, n_in, rope_head_dim);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail_global(METASD_E_HIP, "pack_weight: %s", hipGetErrorString(e));
    return METASD_OK;
}

int32_t metasd_create(metasd_ctx** out, const metasd_config* cfg, const metasd_model_desc* target,
                      const metasd_model_desc* drafters, const void* const* target_weights,
                      const void* const* const* drafter_weights, void* target_kv, void* const* drafter_kv, void* workspace,
                      size_t workspace_bytes, void* hip_stream) {
    if (!out) return fail_global(METASD_E_INVALID, "NULL out");
    *out = nullptr;
    if (int rc = check_config(cfg, target, drafters)) return rc;
    if (!target_weights || !drafter_weights || !target_kv || !drafter_kv || !workspace) return fail_global(METASD_E_INVALID, "NULL pointer argument");
    if ((uintptr_t)workspace % ALIGN) return fail_global(METASD_E_INVALID, "workspace must be 256-byte aligned");
    const Layout lay = make_layout(*cfg, *target, drafters);
    if (workspace_bytes < lay.total) return fail_global(METASD_E_WORKSPACE, "workspace too small: need %zu bytes, got %zu", lay.total, workspace_bytes);
    auto fill = [&](Model& M, const metasd_model_desc& d, const void* const* w, void* kv, const char* who) -> int {
        M.d = d;
        M.hd = d.d_model / d.n_heads;
        M.kv = kv;
        M.kv_layers = d.n_layers;
        M.kvl.assign(cfg->batch, 0);
        const int nw = 1 + PER_LAYER * d.n_layers + 2;
        M.w.assign(w, w + nw);
        for (int i = 0; i < nw; ++i) {
            const bool gate = i >= 1 && i < nw - 2 && (i - 1) % PER_LAYER == 6;
            if (!M.w[i] && !(gate && d.act == METASD_GELU)) return fail_global(METASD_E_INVALID, "%s: weight %d is NULL", who, i);
            if ((uintptr_t)M.w[i] % 16) return fail_global(METASD_E_INVALID, "%s: weight %d is not 16-byte aligned", who, i);
        }
        if (!kv || (uintptr_t)kv % 16) return fail_global(METASD_E_INVALID, "%s: KV cache NULL or misaligned", who);
        return 0;
    };
    metasd_ctx* c = new (std::nothrow) metasd_ctx();
    if (!c) return fail_global(METASD_E_INVALID, "out of host memory");
    c->cfg = *cfg;
    c->stream = (hipStream_t)hip_stream;
    c->ws = (char*)workspace;
    c->lay = lay;
    int rc = fill(c->target, *target, target_weights, target_kv, "target");
    c->drafters.resize(cfg->K);
    for (int k = 0; k < cfg->K && !rc; ++k) {
        if (!drafter_weights[k]) rc = fail_global(METASD_E_INVALID, "drafter %d: NULL weight table", k);
        else {
            char who[32];
            snprintf(who, sizeof who, "drafter %d", k);
            rc = fill(c->drafters[k], drafters[k], drafter_weights[k], drafter_kv[k], who);
            if (!rc && drafter_kv[k] == target_kv) {
                // shared cache: the drafter must be the target's first layers, tensor for tensor, or its K/V would not be the target's
                Model& D = c->drafters[k];
                const metasd_model_desc &a = D.d, &b = *target;
                bool same = a.n_layers <= b.n_layers && a.d_model == b.d_model && a.n_heads == b.n_heads && a.n_kv_heads == b.n_kv_heads &&
                            a.d_ffn == b.d_ffn && a.act == b.act && a.dtype == b.dtype && a.rms_eps == b.rms_eps && a.rope_theta == b.rope_theta;
                for (int i = 0; same && i < 1 + PER_LAYER * a.n_layers; ++i) same = D.w[i] == c->target.w[i];
                if (!same) rc = fail_global(METASD_E_INVALID, "%s: shares the target's KV cache but its layers are not the target's first %d layers (same shapes and weight pointers required)", who, a.n_layers);
                D.shared_kv = true;
                D.kv_layers = b.n_layers;
            }
            if (!rc) c->drafters[k].stream = cfg->stream_window > 0 && !c->drafters[k].shared_kv;
        }
    }
    if (rc) { delete c; return rc; }
    c->sq.resize(cfg->batch);
    for (int b = 0; b < cfg->batch; ++b) {
        c->sq[b].hist.assign(cfg->max_ctx, 0);
        c->sq[b].bandit.init(*cfg);
        c->sq[b].bandit.seq = (uint32_t)b;
    }
    hipError_t e = hipHostMalloc((void**)&c->hspan, c->span_bytes(), hipHostMallocDefault);
    if (e != hipSuccess) {
        rc = fail_global(METASD_E_HIP, "hipHostMalloc: %s", hipGetErrorString(e));
        delete c;
        return rc;
    }
    {
        int dev = 0, ncu = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1) {
            rc = fail_global(METASD_E_HIP, "cannot query the device");
            (void)hipHostFree(c->hspan);
            delete c;
            return rc;
        }
        if (const char* ev = getenv("METASD_FUSE_SMALL")) c->fuse_small = ev[0] != '0';
        if (const char* ev = getenv("METASD_GEMM_REDUCE")) c->gemm_reduce = ev[0] != '0';
        if (const char* ev = getenv("METASD_GEMM_ROLL")) c->fullk_roll = ev[0] != '0';
        if (const char* ev = getenv("METASD_DRAFT_GROUPED")) c->grouped_on = ev[0] != '0';
        if (const char* ev = getenv("METASD_ATT_CPW")) { const int v = atoi(ev); c->att_cpw = (v >= 1 && v <= 64) ? v : 0; }
        if (const char* ev = getenv("METASD_ROWS_TPB")) { const int v = atoi(ev); c->rows_tpb = (v == 4 || v == 6 || v == 8 || v == 12 || v == 16) ? v : 0; }
        if (const char* ev = getenv("METASD_ROWS_RB")) { const int v = atoi(ev); c->rows_rb = v >= 1 && v <= 4 ? v : 0; }
        {
            const int roll_lds = (int)FULLK_LDS_MAX;
            if (hipFuncSetAttribute((const void*)gemm_fullk_roll_residual_kernel<3, true>, hipFuncAttributeMaxDynamicSharedMemorySize, roll_lds) != hipSuccess ||
                hipFuncSetAttribute((const void*)gemm_fullk_roll_residual_kernel<4, true>, hipFuncAttributeMaxDynamicSharedMemorySize, roll_lds) != hipSuccess ||
                hipFuncSetAttribute((const void*)gemm_fullk_roll_residual_kernel<5, false>, hipFuncAttributeMaxDynamicSharedMemorySize, roll_lds) != hipSuccess ||
                hipFuncSetAttribute((const void*)gemm_fullk_roll_residual_kernel<6, false>, hipFuncAttributeMaxDynamicSharedMemorySize, roll_lds) != hipSuccess ||
                hipFuncSetAttribute((const void*)gemm_fullk_roll_residual_kernel<7, false>, hipFuncAttributeMaxDynamicSharedMemorySize, roll_lds) != hipSuccess ||
                hipFuncSetAttribute((const void*)gemm_fullk_roll_residual_kernel<8, false>, hipFuncAttributeMaxDynamicSharedMemorySize, roll_lds) != hipSuccess) {
                c->fullk_roll = false;
                (void)hipGetLastError();
            }
        }
        if (hipFuncSetAttribute((const void*)gemm_fullk_residual_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)FULLK_LDS_MAX) != hipSuccess) { c->fullk = false; (void)hipGetLastError(); }
        if (!step_init()) c->fuse_small = false;
        c->n_cu = ncu;
    }
    c->target.d_table = (const void**)(c->ws + lay.tables);
    for (int k = 0; k < cfg->K; ++k) c->drafters[k].d_table = (const void**)(c->ws + lay.tables + lay.table_stride * (size_t)(k + 1));
    e = hipMemsetAsync(c->d_bar(), 0, sizeof(GridBar), c->stream);
    if (e == hipSuccess) e = hipMemsetAsync(c->d_gx(), 0, c->lay.ssq - c->lay.gx, c->stream);
    if (e == hipSuccess) e = hipMemsetAsync(c->d_xchg(), 0, (size_t)cfg->batch * (cfg->gamma_max + 1) * AS_XCHG_BYTES, c->stream);
    if (e == hipSuccess) e = hipMemsetAsync(c->d_chain(), 0, c->lay.feat - c->lay.chain, c->stream);
    if (e == hipSuccess) e = hipMemsetAsync(c->d_cand(), 0, (size_t)cfg->batch * (cfg->gamma_max + 1) * 2 * sizeof(int2), c->stream);
    if (e == hipSuccess) e = hipMemcpyAsync((void*)c->target.d_table, c->target.w.data(), c->target.w.size() * sizeof(void*), hipMemcpyHostToDevice, c->stream);
    for (int k = 0; k < cfg->K && e == hipSuccess; ++k)
        e = hipMemcpyAsync((void*)c->drafters[k].d_table, c->drafters[k].w.data(), c->drafters[k].w.size() * sizeof(void*), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) {
        rc = fail_global(METASD_E_HIP, "context set-up: %s", hipGetErrorString(e));
        (void)hipHostFree(c->hspan);
        delete c;
        return rc;
    }
    *out = c;
    return METASD_OK;
}

int32_t metasd_destroy(metasd_ctx* c) {
    if (!c) return METASD_OK;
    if (c->hspan) (void)hipHostFree(c->hspan);
    for (auto& r : c->prof) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
    delete c;
    return METASD_OK;
}

int32_t metasd_set_context(metasd_ctx* c, int32_t seq, const int32_t* tokens, int32_t n, int32_t kv_prefilled) {
    if (!c) return fail_global(METASD_E_INVALID, "NULL ctx");
    if (seq < 0 || seq >= c->cfg.batch || !tokens || n < 1) return c->fail(METASD_E_INVALID, "set_context: bad seq / tokens / n");
    if (n + c->cfg.gamma_max + 1 > c->cfg.max_ctx) return c->fail(METASD_E_OVERFLOW, "set_context: n + gamma_max + 1 = %d exceeds max_ctx %d", n + c->cfg.gamma_max + 1, c->cfg.max_ctx);
    for (int i = 0; i < n; ++i)
        if (tokens[i] < 0 || tokens[i] >= c->target.d.vocab) return c->fail(METASD_E_INVALID, "set_context: token %d out of range at %d", tokens[i], i);
    if (c->phase == PH_DRAFTED || c->phase == PH_VERIFIED || c->phase == PH_TREE_DRAFTED || c->phase == PH_TREE_VERIFIED)
        return c->fail(METASD_E_ORDER, "set_context: a round is in flight (finish it with metasd_accept first)");
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    metasd_ctx::SeqState& S = c->sq[seq];
    std::copy(tokens, tokens + n, S.hist.begin());
    HIP_TRY(c, hipMemcpyAsync(c->d_hist() + (size_t)seq * c->cfg.max_ctx, S.hist.data(), (size_t)n * 4, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    S.l = n;
    S.bandit.reset();
    S.ready = true;
    S.round = 0;                    // this sequence's Philox round word restarts with its query; the others carry on
    bool all = true;
    for (const auto& q : c->sq) all = all && q.ready;
    c->phase = all ? PH_READY : PH_NONE;
    c->target.kvl[seq] = kv_prefilled ? n - 1 : 0;
    for (auto& d : c->drafters) { d.kvl[seq] = (kv_prefilled || d.shared_kv) ? n - 1 : 0; d.tail = 0; }
    if (!kv_prefilled && n > 1) {
        if (c->cfg.batch == 1) { if (int rc = forward(c, c->target, 0, n - 1, nullptr, false)) return rc; }
        else if (big_ok(c->target.d) && n - 1 > MAX_ROWS) { if (int rc = forward_big(c, c->target, seq, 0, n - 1)) return rc; }
        else if (int rc = catch_up(c, c->target, std::vector<int>{seq}, std::vector<int>{n - 1}, nullptr, 0, 0)) return rc;
    }
    return METASD_OK;
}

int32_t metasd_swap_weight(metasd_ctx* c, int32_t model, int32_t index, const void* dev_ptr) {
    if (!c) return fail_global(METASD_E_INVALID, "NULL ctx");
    if (model < -1 || model >= c->cfg.K) return c->fail(METASD_E_INVALID, "swap_weight: model %d out of range", model);
    Model& M = model < 0 ? c->target : c->drafters[model];
    if (index < 0 || index >= (int)M.w.size() || !dev_ptr || (uintptr_t)dev_ptr % 16) return c->fail(METASD_E_INVALID, "swap_weight: bad index or pointer");
    M.w[index] = dev_ptr;
    HIP_TRY(c, hipStreamSynchronize(c->stream));        // no launch in flight reads the old table
    if (int rc = upload_table(c, M)) return rc;
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return METASD_OK;
}

// ---- bandit

int32_t metasd_bandit_select(metasd_ctx* c, int32_t seq, int32_t* k_out) {
    if (!c) return fail_global(METASD_E_INVALID, "NULL ctx");
    if (seq < 0 || seq >= c->cfg.batch || !k_out) return c->fail(METASD_E_INVALID, "bandit_select: bad argument");
    *k_out = c->sq[seq].bandit.select();
    return METASD_OK;
}

int32_t metasd_bandit_update(metasd_ctx* c, int32_t seq, int32_t k, int32_t n_acc, int32_t gamma, double bd_reward) {
    if (!c) return fail_global(METASD_E_INVALID, "NULL ctx");
    if (seq < 0 || seq >= c->cfg.batch || k < 0 || k >= c->cfg.K || gamma < 1 || n_acc < 0 || n_acc > gamma) return c->fail(METASD_E_INVALID, "bandit_update: bad argument");
    double r = (double)n_acc / (double)gamma;
    if (c->cfg.reward == METASD_REWARD_BD) {
        if (!(bd_reward >= 0.0 && bd_reward <= 1.0 + 1e-9)) return c->fail(METASD_E_INVALID, "bandit_update: BD reward %g not in [0,1]", bd_reward);
        r = bd_reward;
    }
    c->sq[seq].bandit.update(k, r);
    return METASD_OK;
}

int32_t metasd_bandit_state(const metasd_ctx* c, int32_t seq, double* mu, int32_t* n, int32_t* t) {
    if (!c || seq < 0 || seq >= c->cfg.batch) return fail_global(METASD_E_INVALID, "bandit_state: bad argument");
    const Bandit& B = c->sq[seq].bandit;
    if (mu) std::copy(B.mu.begin(), B.mu.end(), mu);
    if (n) std::copy(B.n.begin(), B.n.end(), n);
    if (t) *t = B.t;
    return METASD_OK;
}

// ---- round

int32_t metasd_set_drafter_head(metasd_ctx* c, int32_t k, const void* w_fc) {
    if (!c) return fail_global(METASD_E_INVALID, "NULL ctx");
    if (!c->cfg.feature_heads) return c->fail(METASD_E_INVALID, "set_drafter_head: the context was created without metasd_config.feature_heads");
    if (k < 0 || k >= c->cfg.K || !w_fc) return c->fail(METASD_E_INVALID, "set_drafter_head: bad drafter index or NULL weight");
    if (c->phase != PH_NONE) return c->fail(METASD_E_ORDER, "set_drafter_head: call it before the first metasd_set_context");
    Model& D = c->drafters[k];
    const metasd_model_desc& t = c->target.d;
    if (D.d.d_model != t.d_model || D.d.dtype != t.dtype) return c->fail(METASD_E_INVALID, "set_drafter_head: the head must have the target's width and dtype");
    if (D.shared_kv) return c->fail(METASD_E_INVALID, "set_drafter_head: a head keeps a cache of its own");
    if (t.d_ffn < t.d_model) return c->fail(METASD_E_INVALID, "set_drafter_head: needs d_ffn >= d_model (the input block is staged in the FFN buffer)");
    D.head = true;
    D.fc = w_fc;
    D.stream = false;
    return METASD_OK;
}

int32_t metasd_draft(metasd_ctx* c, const int32_t* k, int32_t gamma) {
    if (!c) return fail_global(METASD_E_INVALID, "NULL ctx");
    if (!k || k[0] < 0 || k[0] >= c->cfg.K) return c->fail(METASD_E_INVALID, "draft: drafter index out of range");
    if (gamma < 1 || gamma > c->cfg.gamma_max) return c->fail(METASD_E_INVALID, "draft: gamma %d not in 1..%d", gamma, c->cfg.gamma_max);
    if (c->phase != PH_READY) return c->fail(METASD_E_ORDER, "draft: call set_context first (for every sequence) / finish the previous round with accept");
    if (c->cfg.batch > 1) {
        if (int rc = draft_batch(c, k, gamma)) return rc;
        c->cur_gamma = gamma;
        c->phase = PH_DRAFTED;
        return METASD_OK;
    }
    if (c->sq[0].l + gamma + 1 > c->cfg.max_ctx) return c->fail(METASD_E_OVERFLOW, "draft: l + gamma + 1 = %d exceeds max_ctx %d", c->sq[0].l + gamma + 1, c->cfg.max_ctx);
    sync_shared_kv(c);
    Model& D = c->drafters[k[0]];
    const int V = D.d.vocab, l = c->sq[0].l;
    const float T = c->cfg.temperature;
    // the whole chain in one launch, behind a backlog of more than the last token
    const bool chained = !D.stream && chain_ok(c, D, 1, gamma, l + gamma);
    if (chained) {
        if (l - 1 > D.kvl[0])
            if (int rc = forward(c, D, D.kvl[0], l - 1 - D.kvl[0], nullptr, false)) return rc;
        if (int rc = launch_chain(c, D, l - 1, 1, 1, gamma, c->d_Q())) return rc;
        D.kvl[0] = l + gamma - 1;
    }
    for (int j = 0; j < gamma && !chained; ++j) {
        float* Qj = c->d_Q() + (size_t)j * V;
        int rc;
        if (j == 0 && D.stream) {
            // switched in: the sinks it has not seen, then the last stream_window committed tokens; a longer backlog is skipped
            const int S = std::min(c->cfg.stream_sink, l);
            int have = D.kvl[0];
            rc = 0;
            if (have < S) { rc = forward(c, D, have, S - have, S == l ? Qj : nullptr, false); have = S; }
            const int start = std::max(have, l - c->cfg.stream_window);
            if (start > have) D.tail = start;
            if (!rc && start < l) rc = forward(c, D, start, l - start, Qj, false);
        } else if (j == 0) rc = forward(c, D, D.kvl[0], l - D.kvl[0], Qj, false);   // catch-up, ends with the last committed token
        else {
            c->head_est = D.head;                      // a drafter head goes on from its own estimate of the last feature
            c->embedded = true;                        // the draw of the token left its row
            rc = forward(c, D, l + j - 1, 1, Qj, false);
            c->embedded = false;
            c->head_est = false;
        }
        if (rc) return rc;
        NextRow next{};
        if (j + 1 < gamma) next = NextRow{D.w[0], D.d.dtype == METASD_BF16, D.d.d_model, l + j, D.hd, D.d.rope_theta, c->d_h(), c->d_rope()};
        if (launch_sample(c->stream, Qj, 1, V, T, c->cfg.seed, (uint32_t)c->sq[0].round, (uint32_t)j, 0u, c->d_hist() + l + j, 1,
                          c->d_draft() + j, next))
            return c->fail(METASD_E_HIP, "launch sample_rows failed");
    }
    c->sq[0].cur_k = k[0];
    c->cur_gamma = gamma;
    c->phase = PH_DRAFTED;
    return METASD_OK;
}

int32_t metasd_verify(metasd_ctx* c, int32_t gamma) {
    if (!c) return fail_global(METASD_E_INVALID, "NULL ctx");
    if (c->phase != PH_DRAFTED) return c->fail(METASD_E_ORDER, "verify: draft has not been run for this round");
    if (gamma != c->cur_gamma) return c->fail(METASD_E_INVALID, "verify: gamma %d differs from the drafted %d", gamma, c->cur_gamma);
    if (c->cfg.batch > 1) { if (int rc = verify_batch(c, gamma)) return rc; }
    else if (int rc = forward(c, c->target, c->sq[0].l - 1, gamma + 1, c->d_P(), true)) return rc;
    c->phase = PH_VERIFIED;
    return METASD_OK;
}

int32_t metasd_accept(metasd_ctx* c, int32_t gamma, int32_t* n_acc_out, int32_t* token_out, uint32_t* mask_out, double* bd_out) {
    if (!c) return fail_global(METASD_E_INVALID, "NULL ctx");
    if (c->phase != PH_VERIFIED) return c->fail(METASD_E_ORDER, "accept: verify has not been run for this round");
    if (gamma != c->cur_gamma) return c->fail(METASD_E_INVALID, "accept: gamma %d differs from the drafted %d", gamma, c->cur_gamma);
    if (c->cfg.batch > 1) return accept_batch(c, gamma, n_acc_out, token_out, mask_out, bd_out);
    const int V = c->target.d.vocab, l = c->sq[0].l;
    int32_t* res = c->d_res();
    metasd_ctx::ProfRec* pr = c->prof_take(METASD_PROF_ACCEPT, (double)(2 * gamma + 1) * V * 4);
    if (launch_accept(c->stream, c->d_P(), c->d_Q(), c->d_hist() + l, 1, gamma, V, c->cfg.temperature, c->cfg.seed,
                      one_round((uint32_t)c->sq[0].round), 0u, c->d_cand(), c->d_bd(), res, res + 1, (uint32_t*)(res + 2), c->d_hist(), l,
                      c->d_xchg(), pr ? pr->a : nullptr, pr ? pr->b : nullptr))
        return c->fail(METASD_E_HIP, "launch accept kernels failed");
    if (int rc = c->fetch_results()) return rc;
    const int32_t* hres = c->mirror<int32_t>(c->lay.res);     // n_acc, token, mask
    if (hres[1] == -2 && !c->mirror<GridBar>(c->lay.bar)->abort) {
        // the four workgroups of some position did not meet within their bounded wait: nothing was committed, the
        // logits are untouched - take the step again with one workgroup per position (no meeting between workgroups)
        if (launch_accept(c->stream, c->d_P(), c->d_Q(), c->d_hist() + l, 1, gamma, V, c->cfg.temperature, c->cfg.seed,
                          one_round((uint32_t)c->sq[0].round), 0u, c->d_cand(), c->d_bd(), res, res + 1, (uint32_t*)(res + 2), c->d_hist(), l, nullptr))
            return c->fail(METASD_E_HIP, "launch accept kernels failed");
        if (int rc = c->fetch_results()) return rc;
        c->accept_fallbacks += 1;
    }
    const int32_t* hd = c->mirror<int32_t>(c->lay.draft);
    const double* hbd = c->mirror<double>(c->lay.bd);
    if (c->mirror<GridBar>(c->lay.bar)->abort) {
        (void)hipMemsetAsync(c->d_bar(), 0, sizeof(GridBar), c->stream);
        c->phase = PH_NONE;
        return c->fail(METASD_E_HIP, "a bounded device-side wait between workgroups timed out (split-K reduction or device-wide barrier); call metasd_set_context to start over");
    }
    const int n = hres[0], token = hres[1];
    if (token == -2) { c->phase = PH_NONE; return c->fail(METASD_E_HIP, "accept: the workgroups of a position did not meet (exchange timed out); call metasd_set_context to start over"); }
    if (n < 0 || n > gamma || token < 0 || token >= V) return c->fail(METASD_E_HIP, "accept: device returned n_acc %d token %d", n, token);
    for (int j = 0; j < n; ++j) c->sq[0].hist[l + j] = hd[j];
    c->sq[0].hist[l + n] = token;
    // commit: rows 0..n of the verification block stay in the target's cache; the drafter keeps
    // the committed prefix it has processed (it never saw d_gamma)
    c->sq[0].l = l + n + 1;
    c->target.kvl[0] = l + n;
    c->drafters[c->sq[0].cur_k].kvl[0] = std::min(l + n, l + gamma - 1);
    // a drafter head keeps nothing it computed from estimated features: it will re-read the committed tokens of this round with
    // the target's own features (which the verification pass has just left in the feature table)
    if (c->drafters[c->sq[0].cur_k].head) c->drafters[c->sq[0].cur_k].kvl[0] = l;
    c->sq[0].round += 1;
    sync_shared_kv(c);
    c->phase = PH_READY;
    if (n_acc_out) *n_acc_out = n;
    if (token_out) *token_out = token;
    if (mask_out) *mask_out = (uint32_t)hres[2];
    if (bd_out) {
        double s = 0.0;
        for (int j = 0; j < gamma; ++j) s += hbd[j];
        *bd_out = s / (double)gamma;
    }
    return METASD_OK;
}

// ---- token trees (greedy): draft a tree of candidates, verify it in one pass with tree attention, accept the longest
// path that the target's own greedy choices follow

int32_t metasd_draft_tree(metasd_ctx* c, int32_t k, const metasd_tree* tree) {
    if (!c) return fail_global(METASD_E_INVALID, "NULL ctx");
    if (c->cfg.batch != 1) return c->fail(METASD_E_INVALID, "draft_tree: contexts with one sequence only");
    if (k < 0 || k >= c->cfg.K || !tree) return c->fail(METASD_E_INVALID, "draft_tree: bad drafter index or NULL tree");
    if (c->drafters[k].stream) return c->fail(METASD_E_INVALID, "draft_tree: drafters with a streaming cache draft chains only");
    if (c->phase != PH_READY) return c->fail(METASD_E_ORDER, "draft_tree: call set_context first / finish the previous round");
    const int n = tree->n;
    if (n < 2 || n > TREE_MAX || n > c->cfg.gamma_max + 1) return c->fail(METASD_E_INVALID, "draft_tree: tree of %d nodes; 2 .. min(%d, gamma_max + 1) supported", n, TREE_MAX);
    TreeShape ts{};
    ts.n = n;
    ts.parent[0] = -1;
    c->tdepth[0] = 0;
    c->tanc[0] = 1;
    for (int i = 1; i < n; ++i) {
        const int p = tree->parent[i], r = tree->rank[i];
        if (p < 0 || p >= i || r < 0 || r >= TREE_RANKS) return c->fail(METASD_E_INVALID, "draft_tree: node %d: parent must be an earlier node, rank 0..%d", i, TREE_RANKS - 1);
        c->tdepth[i] = c->tdepth[p] + 1;
        if (c->tdepth[i] < c->tdepth[i - 1]) return c->fail(METASD_E_INVALID, "draft_tree: nodes must come in breadth-first order (depth never decreases)");
        for (int j = 1; j < i; ++j)
            if (tree->parent[j] == p && tree->rank[j] == r) return c->fail(METASD_E_INVALID, "draft_tree: nodes %d and %d are the same child of node %d", j, i, p);
        ts.parent[i] = (int8_t)p;
        ts.rank[i] = (int8_t)r;
        c->tanc[i] = (uint16_t)(c->tanc[p] | (1u << i));
    }
    c->tmaxdepth = c->tdepth[n - 1];
    for (int d = 0, i = 0; d <= c->tmaxdepth + 1; ++d) {
        while (i < n && c->tdepth[i] < d) ++i;
        c->tlevel[d] = i;
    }
    if (c->tlevel[c->tmaxdepth] > c->cfg.gamma_max) return c->fail(METASD_E_INVALID, "draft_tree: %d nodes above the deepest level exceed gamma_max %d", c->tlevel[c->tmaxdepth], c->cfg.gamma_max);
    const int l = c->sq[0].l, base = l - 1;
    if (l + n + 1 > c->cfg.max_ctx) return c->fail(METASD_E_OVERFLOW, "draft_tree: l + nodes + 1 = %d exceeds max_ctx %d", l + n + 1, c->cfg.max_ctx);
    sync_shared_kv(c);
    Model& D = c->drafters[k];
    const int V = D.d.vocab;
    TreeBlk tb{};
    tb.on = 1; tb.base = base;
    for (int i = 0; i < n; ++i) { tb.anc[i] = c->tanc[i]; tb.depth[i] = (uint8_t)c->tdepth[i]; }
    for (int d = 0; d < c->tmaxdepth; ++d) {
        const int i0 = c->tlevel[d], m = c->tlevel[d + 1] - i0;
        float* Qd = c->d_Q() + (size_t)i0 * V;
        int rc;
        if (d == 0) rc = forward(c, D, D.kvl[0], l - D.kvl[0], Qd, false);      // the committed backlog, ending with the root
        else {
            tb.i0 = i0;
            c->tree = &tb;
            if (D.head) {                                // a head's node takes the head's estimate at its parent
                c->head_est = true;
                for (int r = 0; r < m; ++r) c->fsrc.idx[r] = (uint8_t)ts.parent[i0 + r];
            }
            rc = forward(c, D, base + i0, m, Qd, true);
            c->head_est = false;
            c->fsrc = FeatSrc{};
            c->tree = nullptr;
        }
        if (rc) return rc;
        if (c->cfg.temperature > 0.f)
            hipLaunchKernelGGL(tree_children_sample_kernel, dim3(m), dim3(AK_NT), 0, c->stream, (const float*)Qd, V, c->cfg.temperature, c->cfg.seed,
                               0u, (uint32_t)c->sq[0].round, ts, i0, c->d_hist() + base, c->d_draft());
        else
            hipLaunchKernelGGL(tree_children_kernel, dim3(m), dim3(AK_NT), 0, c->stream, (const float*)Qd, V, ts, i0, c->d_hist() + base, c->d_draft());
        LAUNCH_CHECK(c, "tree_children");
    }
    c->tshape = ts;
    c->sq[0].cur_k = k;
    c->phase = PH_TREE_DRAFTED;
    return METASD_OK;
}

int32_t metasd_verify_tree(metasd_ctx* c) {
    if (!c) return fail_global(METASD_E_INVALID, "NULL ctx");
    if (c->phase != PH_TREE_DRAFTED) return c->fail(METASD_E_ORDER, "verify_tree: draft_tree has not been run for this round");
    const int n = c->tshape.n, base = c->sq[0].l - 1;
    TreeBlk tb{};
    tb.on = 1; tb.base = base; tb.i0 = 0;
    for (int i = 0; i < n; ++i) { tb.anc[i] = c->tanc[i]; tb.depth[i] = (uint8_t)c->tdepth[i]; }
    c->tree = &tb;
    const int rc = forward(c, c->target, base, n, c->d_P(), true);
    c->tree = nullptr;
    if (rc) return rc;
    c->phase = PH_TREE_VERIFIED;
    return METASD_OK;
}

int32_t metasd_accept_tree(metasd_ctx* c, int32_t* n_acc_out, int32_t* token_out, int32_t* path_out) {
    if (!c) return fail_global(METASD_E_INVALID, "NULL ctx");
    if (c->phase != PH_TREE_VERIFIED) return c->fail(METASD_E_ORDER, "accept_tree: verify_tree has not been run for this round");
    const int n = c->tshape.n, V = c->target.d.vocab, l = c->sq[0].l, base = l - 1;
    if (c->cfg.temperature > 0.f) {
        hipLaunchKernelGGL(accept_tree_node_kernel, dim3(n), dim3(AK_NT), 0, c->stream, (const float*)c->d_P(), (const float*)c->d_Q(),
                           (const int32_t*)c->d_draft(), V, c->cfg.temperature, c->cfg.seed, 0u, (uint32_t)c->sq[0].round, c->tshape, c->d_tstep());
        LAUNCH_CHECK(c, "accept_tree (nodes)");
        hipLaunchKernelGGL(accept_tree_walk_kernel, dim3(1), dim3(64), 0, c->stream, (const int2*)c->d_tstep(), (const int32_t*)c->d_draft(),
                           c->tshape, c->d_res(), c->d_hist() + base);
    } else {
        int32_t* amax = reinterpret_cast<int32_t*>(c->d_tstep());   // (not among the tagged words of the chains: a token could be read as a tag)
        if (launch_sample(c->stream, c->d_P(), n, V, 0.f, c->cfg.seed, 0u, 0u, 0u, amax, 1, nullptr)) return c->fail(METASD_E_HIP, "launch argmax failed");
        hipLaunchKernelGGL(accept_tree_kernel, dim3(1), dim3(64), 0, c->stream, (const int32_t*)amax, (const int32_t*)c->d_draft(), c->tshape, c->d_res(),
                           c->d_hist() + base);
    }
    LAUNCH_CHECK(c, "accept_tree");
    Model& D = c->drafters[c->sq[0].cur_k];
    int rc = c->target.d.dtype == METASD_BF16 ? compact_kv<bf16_t>(c, c->target, base, TREE_MAX) : compact_kv<float>(c, c->target, base, TREE_MAX);
    if (!rc && !D.shared_kv && !D.head)                  // a head keeps nothing of the round: no rows to move
        rc = D.d.dtype == METASD_BF16 ? compact_kv<bf16_t>(c, D, base, c->tmaxdepth - 1) : compact_kv<float>(c, D, base, c->tmaxdepth - 1);
    if (rc) return rc;
    if (c->cfg.feature_heads) {                          // the target's features of the accepted nodes, from their slots to their positions
        const int Dm = c->target.d.d_model;
        hipLaunchKernelGGL(kv_compact_kernel<float>, dim3((unsigned)((Dm + 255) / 256)), dim3(256), 0, c->stream, c->d_feat(), 1, c->cfg.max_ctx, Dm,
                           base, (const int32_t*)c->d_res(), TREE_MAX, c->tshape.n);
        LAUNCH_CHECK(c, "feature rows of the accepted nodes");
    }
    if ((rc = c->fetch_results())) return rc;
    if (c->mirror<GridBar>(c->lay.bar)->abort) {
        (void)hipMemsetAsync(c->d_bar(), 0, sizeof(GridBar), c->stream);
        c->phase = PH_NONE;
        return c->fail(METASD_E_HIP, "a bounded device-side wait between workgroups timed out (split-K reduction); call metasd_set_context to start over");
    }
    const int32_t* hres = c->mirror<int32_t>(c->lay.res);
    const int32_t* htok = c->mirror<int32_t>(c->lay.draft);
    const int na = hres[0], token = hres[1];
    if (na < 0 || na > c->tmaxdepth || token < 0 || token >= V) return c->fail(METASD_E_HIP, "accept_tree: device returned n_acc %d token %d", na, token);
    for (int j = 0; j < na; ++j) {
        const int node = hres[2 + j];
        if (node < 1 || node >= n) return c->fail(METASD_E_HIP, "accept_tree: device returned path node %d", node);
        c->sq[0].hist[l + j] = htok[node];
        if (path_out) path_out[j] = node;
    }
    c->sq[0].hist[l + na] = token;
    c->sq[0].l = l + na + 1;
    c->target.kvl[0] = l + na;
    D.kvl[0] = std::min(l + na, l + c->tmaxdepth - 1);
    if (D.head) D.kvl[0] = l;                            // what a head computed from estimated features is not kept
    c->sq[0].round += 1;
    sync_shared_kv(c);
    c->phase = PH_READY;
    if (n_acc_out) *n_acc_out = na;
    if (token_out) *token_out = token;
    return METASD_OK;
}

// ---- stand-alone kernels

int32_t metasd_accept_logits(const float* P, const float* Q, const int32_t* d, int32_t rows, int32_t gamma, int32_t V,
                             float temperature, uint64_t seed, uint32_t round, uint32_t seq0, int32_t* n_acc, int32_t* token,
                             uint32_t* mask, double* bd, void* scratch, void* hip_stream) {
    if (!P || !Q || !d || !n_acc || !token || !scratch) return fail_global(METASD_E_INVALID, "accept_logits: NULL pointer");
    if (rows < 1 || rows > 65535 || gamma < 1 || gamma > 31 || !valid_vocab(V) || !(temperature >= 0.f))
        return fail_global(METASD_E_INVALID, "accept_logits: rows 1..65535, gamma 1..31, V %% 4 == 0, V <= 32768, T >= 0");
    // scratch: [rows (gamma+1)] candidates of 16 bytes, then the exchange words of the split kernel
    unsigned long long* xchg = (unsigned long long*)((char*)scratch + (size_t)rows * (gamma + 1) * 16);
    if (launch_accept((hipStream_t)hip_stream, P, Q, d, rows, gamma, V, temperature, seed, one_round(round), seq0, (int2*)scratch, bd, n_acc,
                      token, mask, nullptr, 0, xchg))
        return fail_global(METASD_E_HIP, "accept_logits: launch failed");
    return METASD_OK;
}

// Device address of `scratch` on the current device (asked for once per device, with that device current).
static int noalloc_scratch(unsigned char** out) {
    constexpr int MAX_DEV = 64;
    static std::mutex mu;
    static unsigned char* ptr[MAX_DEV] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail_global(METASD_E_HIP, "accept_logits_noalloc: hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= MAX_DEV) return fail_global(METASD_E_INVALID, "accept_logits_noalloc: device index %d not supported", dev);
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return fail_global(METASD_E_HIP, "accept_logits_noalloc: hipGetSymbolAddress: %s", hipGetErrorString(e));
        ptr[dev] = static_cast<unsigned char*>(p);
    }
    *out = ptr[dev];
    return METASD_OK;
}

int32_t metasd_accept_logits_noalloc(const float* P, const float* Q, const int32_t* d, int32_t rows, int32_t gamma, int32_t V,
                                     float temperature, uint64_t seed, uint32_t round, uint32_t seq0, int32_t* n_acc,
                                     int32_t* token, uint32_t* mask, double* bd, void* hip_stream) {
    if (!P || !Q || !d || !n_acc || !token) return fail_global(METASD_E_INVALID, "accept_logits_noalloc: NULL pointer");
    if (rows < 1 || rows > 65535 || gamma < 1 || gamma > 31 || !valid_vocab(V) || !(temperature >= 0.f))
        return fail_global(METASD_E_INVALID, "accept_logits_noalloc: rows 1..65535, gamma 1..31, V %% 4 == 0, V <= 32768, T >= 0");
    const size_t items = (size_t)rows * (gamma + 1);
    if (items > METASD_ACCEPT_NOALLOC_MAX_ITEMS)
        return fail_global(METASD_E_INVALID, "accept_logits_noalloc: rows * (gamma + 1) = %zu exceeds the built-in scratch of %d items; use metasd_accept_logits with a scratch buffer of your own",
                           items, METASD_ACCEPT_NOALLOC_MAX_ITEMS);
    unsigned char* sp = nullptr;
    if (int rc = noalloc_scratch(&sp)) return rc;
    hipStream_t st = (hipStream_t)hip_stream;
    // The array keeps what the last call left.  The part this call uses is cleared by a kernel (not a memset: the call
    // may be recorded into a graph, and a replay repeats this call's launch tag, so the words of the replay before
    // must be gone).
    const unsigned n16 = (unsigned)(items * 336 / 16);
    hipLaunchKernelGGL(zero_fill_kernel, dim3((n16 + 255) / 256), dim3(256), 0, st, reinterpret_cast<uint4*>(sp), n16);
    if (hipGetLastError() != hipSuccess) return fail_global(METASD_E_HIP, "accept_logits_noalloc: launch failed");
    unsigned long long* xchg = reinterpret_cast<unsigned long long*>(sp + items * 16);
    if (launch_accept(st, P, Q, d, rows, gamma, V, temperature, seed, one_round(round), seq0, reinterpret_cast<int2*>(sp), bd, n_acc, token, mask,
                      nullptr, 0, xchg))
        return fail_global(METASD_E_HIP, "accept_logits_noalloc: launch failed");
    return METASD_OK;
}

int32_t metasd_sample_logits(const float* logits, int32_t rows, int32_t V, float temperature, uint64_t seed, uint32_t round,
                             uint32_t pos, uint32_t seq0, int32_t* tok, void* hip_stream) {
    if (!logits || !tok) return fail_global(METASD_E_INVALID, "sample_logits: NULL pointer");
    if (rows < 1 || !valid_vocab(V) || !(temperature >= 0.f)) return fail_global(METASD_E_INVALID, "sample_logits: rows >= 1, V %% 4 == 0, V <= 32768, T >= 0");
    if (launch_sample((hipStream_t)hip_stream, logits, rows, V, temperature, seed, round, pos, seq0, tok, 1, nullptr))
        return fail_global(METASD_E_HIP, "sample_logits: launch failed");
    return METASD_OK;
}

int32_t metasd_philox_words(uint64_t seed, uint32_t c0_start, int32_t n, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t* out,
                            void* hip_stream) {
    if (!out || n < 1) return fail_global(METASD_E_INVALID, "philox_words: bad argument");
    hipLaunchKernelGGL(philox_words_kernel, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)hip_stream, seed, c0_start, n, c1, c2,
                       c3, out);
    if (hipGetLastError() != hipSuccess) return fail_global(METASD_E_HIP, "philox_words: launch failed");
    return METASD_OK;
}

int32_t metasd_stream_read(const void* src, size_t bytes, uint32_t* sink, void* hip_stream) {
    if (!src || !sink || bytes < 1024 || ((uintptr_t)src & 15)) return fail_global(METASD_E_INVALID, "stream_read: bad argument");
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1)
        return fail_global(METASD_E_HIP, "stream_read: cannot query the device");
    const int grid = std::min(ncu * 4, METASD_STREAM_READ_SINK_WORDS / 4);
    hipLaunchKernelGGL(stream_read_kernel, dim3(grid), dim3(256), 0, (hipStream_t)hip_stream, (const u32x4*)src, bytes / 1024, sink);
    if (hipGetLastError() != hipSuccess) return fail_global(METASD_E_HIP, "stream_read: launch failed");
    return METASD_OK;
}

// ---- per-kernel timing

int32_t metasd_profile(metasd_ctx* c, int32_t max_records) {
    if (!c) return fail_global(METASD_E_INVALID, "NULL ctx");
    if (max_records < 0 || max_records > (1 << 20)) return c->fail(METASD_E_INVALID, "profile: max_records out of range");
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    while ((int)c->prof.size() < max_records) {
        metasd_ctx::ProfRec r{};
        HIP_TRY(c, hipEventCreate(&r.a));
        hipError_t e = hipEventCreate(&r.b);
        if (e != hipSuccess) { (void)hipEventDestroy(r.a); return c->fail(METASD_E_HIP, "hipEventCreate: %s", hipGetErrorString(e)); }
        c->prof.push_back(r);
    }
    c->prof_used = 0;
    c->prof_on = max_records > 0;
    return METASD_OK;
}

int32_t metasd_profile_read(metasd_ctx* c, int32_t kind, double* ms_total, int64_t* launches, double* bytes_total) {
    if (!c) return fail_global(METASD_E_INVALID, "NULL ctx");
    if (kind < 0 || kind > 2) return c->fail(METASD_E_INVALID, "profile_read: unknown kind %d", kind);
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    double ms = 0.0, by = 0.0;
    int64_t n = 0;
    for (size_t i = 0; i < c->prof_used; ++i) {
        if (c->prof[i].kind != kind) continue;
        float t = 0.f;
        HIP_TRY(c, hipEventElapsedTime(&t, c->prof[i].a, c->prof[i].b));
        ms += t; by += c->prof[i].bytes; ++n;
    }
    if (ms_total) *ms_total = ms;
    if (launches) *launches = n;
    if (bytes_total) *bytes_total = by;
    return METASD_OK;
}

int32_t metasd_profile_shapes(metasd_ctx* c, int32_t target_only, int32_t max_rows, int32_t* n_out, int32_t* k_out, int32_t* m_out,
                              double* ms_out, int64_t* launches_out, double* bytes_out, int32_t* rows_out) {
    if (!c) return fail_global(METASD_E_INVALID, "NULL ctx");
    if (max_rows < 1 || !n_out || !k_out || !m_out || !ms_out || !launches_out || !bytes_out || !rows_out)
        return c->fail(METASD_E_INVALID, "profile_shapes: bad argument");
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    int rows = 0;
    for (size_t i = 0; i < c->prof_used; ++i) {
        const metasd_ctx::ProfRec& r = c->prof[i];
        if (r.kind != METASD_PROF_GEMM || (target_only && r.model != -1)) continue;
        int at = 0;
        while (at < rows && !(n_out[at] == r.n && k_out[at] == r.k && m_out[at] == r.m)) ++at;
        if (at == rows) {
            if (rows == max_rows) continue;               // table full: further shapes are left out
            n_out[at] = r.n; k_out[at] = r.k; m_out[at] = r.m; ms_out[at] = 0.0; launches_out[at] = 0; bytes_out[at] = 0.0;
            ++rows;
        }
        float t = 0.f;
        HIP_TRY(c, hipEventElapsedTime(&t, r.a, r.b));
        ms_out[at] += t; launches_out[at] += 1; bytes_out[at] += r.bytes;
    }
    *rows_out = rows;
    return METASD_OK;
}

// ---- introspection

int32_t metasd_peek(metasd_ctx* c, int32_t what, void** dev_ptr_out, size_t* bytes_out) {
    if (!c) return fail_global(METASD_E_INVALID, "NULL ctx");
    if (!dev_ptr_out || !bytes_out) return c->fail(METASD_E_INVALID, "peek: NULL output");
    const size_t V = (size_t)c->target.d.vocab;
    switch (what) {
        case METASD_PEEK_P: *dev_ptr_out = c->d_P(); *bytes_out = (size_t)c->cfg.batch * (c->cfg.gamma_max + 1) * V * 4; break;
        case METASD_PEEK_Q: *dev_ptr_out = c->d_Q(); *bytes_out = (size_t)c->cfg.batch * c->cfg.gamma_max * V * 4; break;
        case METASD_PEEK_HIST: *dev_ptr_out = c->d_hist(); *bytes_out = (size_t)c->cfg.batch * c->cfg.max_ctx * 4; break;
        case METASD_PEEK_BD: *dev_ptr_out = c->d_bd(); *bytes_out = (size_t)c->cfg.batch * c->cfg.gamma_max * 8; break;
        case METASD_PEEK_FEAT:
            if (!c->cfg.feature_heads) return c->fail(METASD_E_INVALID, "peek: this context keeps no features (metasd_config.feature_heads)");
            *dev_ptr_out = c->d_feat(); *bytes_out = (size_t)c->cfg.max_ctx * c->target.d.d_model * 4; break;
        case METASD_PEEK_DRAFT: *dev_ptr_out = c->d_draft(); *bytes_out = (size_t)c->cfg.batch * (c->cfg.gamma_max + 1) * 4; break;
        default: return c->fail(METASD_E_INVALID, "peek: unknown buffer %d", what);
    }
    return METASD_OK;
}

int32_t metasd_state_seq(const metasd_ctx* c, int32_t seq, int32_t model, int32_t* l_out, int32_t* kv_len_out, int32_t* round_out) {
    if (!c || model < -1 || model >= c->cfg.K || seq < 0 || seq >= c->cfg.batch) return fail_global(METASD_E_INVALID, "state: bad argument");
    if (l_out) *l_out = c->sq[seq].l;
    if (kv_len_out) *kv_len_out = model < 0 ? c->target.kvl[seq] : c->drafters[model].kvl[seq];
    if (round_out) *round_out = c->sq[seq].round;
    return METASD_OK;
}

int32_t metasd_accept_fallbacks(const metasd_ctx* c, int64_t* count_out) {
    if (!c || !count_out) return fail_global(METASD_E_INVALID, "accept_fallbacks: bad argument");
    *count_out = c->accept_fallbacks;
    return METASD_OK;
}

int32_t metasd_state(const metasd_ctx* c, int32_t model, int32_t* l_out, int32_t* kv_len_out, int32_t* round_out) {
    return metasd_state_seq(c, 0, model, l_out, kv_len_out, round_out);
}

}  // extern "C"
