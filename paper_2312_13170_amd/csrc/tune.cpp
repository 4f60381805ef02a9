// Tile-shape tuning table.  Each kernel family has a fixed list of compiled
// tile shapes (tiles.h).  For every (family, size bucket) the table holds the
// candidate to use; unset entries fall back to a built-in heuristic.  A
// "forced" candidate overrides everything for one family: the search
// (autotune.py) forces each candidate in turn and times the ordinary entry
// points with HIP events, then writes the winners back with li_tune_set.
#include <math.h>
#include <stdio.h>

#include <atomic>

#include "li_internal.h"
#include "tiles.h"

namespace li {
namespace {

#define LI_ENTRY(IDX, BM, BN, BK, WM, WN, SK, PF) {BM, BN, BK, WM, WN, SK, PF},
const TileCfg kGemmF32[] = {LI_GEMM_F32_CANDIDATES(LI_ENTRY)};
const TileCfg kSyrkF32[] = {LI_SYRK_F32_CANDIDATES(LI_ENTRY)};
const TileCfg kGemmLp[] = {LI_GEMM_LP_CANDIDATES(LI_ENTRY)};
const TileCfg kSyrkRows[] = {LI_SYRK_ROWS_CANDIDATES(LI_ENTRY)};
#undef LI_ENTRY
#define LI_CLASS_ENTRY(C, GI, SI, BT, BK, WM, WN, PF) {BT, BT, BK, WM, WN, 1, PF},
const TileCfg kGrouped[] = {LI_GROUPED_CLASSES(LI_CLASS_ENTRY)};
#undef LI_CLASS_ENTRY

constexpr int kFamilies = 7;
constexpr int kBuckets = 64;

const TileCfg *family(int k, int *n)
{
    switch (k) {
    case LI_KERNEL_GEMM_F32:
        *n = (int)(sizeof(kGemmF32) / sizeof(kGemmF32[0]));
        return kGemmF32;
    case LI_KERNEL_SYRK_F32:
        *n = (int)(sizeof(kSyrkF32) / sizeof(kSyrkF32[0]));
        return kSyrkF32;
    case LI_KERNEL_GEMM_LP:
    case LI_KERNEL_GEMM_LP_SPLIT:
        *n = (int)(sizeof(kGemmLp) / sizeof(kGemmLp[0]));
        return kGemmLp;
    case LI_KERNEL_SYRK_ROWS:
        *n = (int)(sizeof(kSyrkRows) / sizeof(kSyrkRows[0]));
        return kSyrkRows;
    case LI_KERNEL_GROUPED_GEMM:
    case LI_KERNEL_GROUPED_COV:
        *n = (int)(sizeof(kGrouped) / sizeof(kGrouped[0]));
        return kGrouped;
    default:
        *n = 0;
        return nullptr;
    }
}

// Version of a saved table, in its first line (none: 1), and the candidates
// whose shape has another number since a version.
constexpr int kTableVersion = 2;
struct Renumbered {
    int version;  // the last one with the old number
    int kernel, old_idx, idx;
};
const Renumbered kRenumbered[] = {
    {1, LI_KERNEL_SYRK_F32, 10, 30},    {1, LI_KERNEL_SYRK_F32, 20, 31},    {1, LI_KERNEL_SYRK_F32, 21, 32},
    {1, LI_KERNEL_SYRK_ROWS, 9, 18},    {1, LI_KERNEL_SYRK_ROWS, 10, 16},   {1, LI_KERNEL_SYRK_ROWS, 14, 19},
    {1, LI_KERNEL_SYRK_ROWS, 15, 20},   {1, LI_KERNEL_GROUPED_GEMM, 0, 4},  {1, LI_KERNEL_GROUPED_GEMM, 1, 3},
    {1, LI_KERNEL_GROUPED_GEMM, 2, 5},  {1, LI_KERNEL_GROUPED_COV, 0, 4},   {1, LI_KERNEL_GROUPED_COV, 1, 3},
    {1, LI_KERNEL_GROUPED_COV, 2, 5},
};

int current_number(int version, int kernel, int idx)
{
    for (const Renumbered &r : kRenumbered)
        if (version <= r.version && kernel == r.kernel && idx == r.old_idx) return r.idx;
    return idx;
}

// Entries hold candidate index + 1; the static zero-initialisation therefore
// means "unset" without any start-up code.
std::atomic<int> g_table[kFamilies][kBuckets];
std::atomic<int> g_forced[kFamilies];

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// The FP32 products' split tiles (three bf16 parts, split_tile.h): the one
// with the least predicted time
//   t = launch + rounds * tile + K * max(alone, shared * rounds)   [us]
// where rounds = ceil(tiles / 256) is the most tiles a compute unit takes,
// `alone` what a K step of one tile costs by itself (latency) and `shared`
// what it costs of a busy compute unit (throughput; several tiles of the
// small shapes are resident at once).  The constants are a least-squares
// fit to 226 shapes with M, N, K log-uniform from 64 to 8192 (10% rms); the
// pick is 1.4% slower than the fastest of these tiles on average.
struct SplitCost {
    int idx;
    double launch, tile, alone, shared;
};
const SplitCost kSplitF32[] = {
    {51, 0.00, 9.54, 0.0101, 0.0303},  // 128 x 128
    {52, 3.90, 1.59, 0.0129, 0.0128},  // 64 x 64
    {53, 0.09, 6.10, 0.0029, 0.0198},  // 64 x 128
    {54, 3.03, 2.22, 0.0052, 0.0071},  // 32 x 32, K-tile 64
    {55, 5.02, 0.41, 0.0102, 0.0055},  // 32 x 32, K-tile 32
};

int split_pick(int64_t M, int64_t N, int64_t K, double *predicted = nullptr)
{
    int best = kSplitF32[0].idx;
    double tbest = HUGE_VAL;
    for (const SplitCost &c : kSplitF32) {
        const TileCfg &t = kGemmF32[c.idx];
        const double rounds = (double)ceil_div(ceil_div(M, t.bm) * ceil_div(N, t.bn), 256);
        const double alone = c.alone, shared = c.shared * rounds;
        const double us = c.launch + rounds * c.tile + (double)K * (alone > shared ? alone : shared);
        if (us < tbest) {
            tbest = us;
            best = c.idx;
        }
    }
    if (predicted) *predicted = tbest;
    return best;
}

// Shorter reductions stay on the FP32 cores: a split tile starts with two
// K-tiles on their way through its pipeline (7001 x 5458 x 94: 105 us against
// 123 on the best split tile, 1463 x 1664 x 64: 9.0 against 10.1; 1168 x 1600
// x 126: 10.6 against 9.4).  From K = 120 on the split tiles are ahead or
// within 3%, but for some large outputs up to K = 150, which they keep for
// their error (4096 x 4096 x 128: 58.5 us against 53.7 with beta, 42.2 and 44.2
// without; 8192 x 8192 x 128: 207 and 219, 181 and 167).
constexpr int64_t kSplitMinK = 120;

// Results of fewer products than this stay on the FP32 cores wherever the
// split tiles would be taken, for their smaller error: the part products that
// the split leaves out reach half a unit in the last place of a product, which
// the shorter chain of roundings makes up for from two products on in the rms
// and from three on at worst (order 700, U[-1, 1), error over the sum of
// magnitudes, FP32 cores and split, rms and worst: K = 1 2.53e-8 and 2.58e-8,
// 6.0e-8 and 9.0e-8; K = 2 2.53e-8 and 2.14e-8, 1.1e-7 and 1.2e-7; K = 3
// 2.50e-8 and 1.84e-8, 1.5e-7 and 1.1e-7).  Both take 7.3 us there, a batch of
// 64 products of K = 4 23 us.
constexpr int64_t kSplitMinSum = 4;

// Built-in choice for slots the table does not hold: for the FP32 products
// the split tiles, and with a short reduction one of the shapes the search
// picked for the FP32 cores; the symmetric contractions likewise.
int heuristic(int kernel, int64_t M, int64_t N, int64_t K)
{
    const int64_t cus = 256;  // compute units of an MI355X
    if (kernel == LI_KERNEL_GEMM_F32) {
        if (K >= kSplitMinK && K <= kSplitMaxLd && N <= kSplitMaxLd) return split_pick(M, N, K);
        // (short reductions, rows too long for the split tiles) by the bit
        // length of the output's side, as searched
        const int side = tune_key(kernel, M, N, K);
        return side <= 8 ? 2 : side <= 11 ? 20 : side == 12 ? 44 : 49;
    }
    if (kernel == LI_KERNEL_SYRK_F32) {
        // M features (the order of the result), K samples.  Measured over
        // 136 shapes with M log-uniform from 32 to 4096 and K from 64 to
        // 32768 (times with the statistics): the picks are within 2% of the
        // fastest candidate on average.  Few samples: FP32 cores (3776 x 128:
        // 38 us against 47 on the best split tile; 320 x 211 from 17.5 to 17.0).
        // A small result with a short reduction: one wave per 32 x 32 tile
        // (512 x 512: 20.6 us against 23.5 in 64 x 64 phases; 631 x 745 the
        // other way, 25.7 and 23.4).  Otherwise phases, of 128 x 128 tiles
        // where the work outweighs their longer pipeline (1024 x 2048, 2.1e9
        // products: 39.1 us against 41.4 in 64 x 64; 896 x 1216, 1e9: 34.9 and 31.7).
        if (K <= 200 || (M > 704 && K <= 256)) return 17;
        if (M <= 704 && K < 700) return 27;
        return (double)M * (double)M * (double)K >= 2e9 ? 20 : 21;
    }
    if (kernel == LI_KERNEL_SYRK_ROWS) {
        // M is the order of C, K the reduction length (the rank).  Over 156
        // shapes (both updates, M from 128 to 4096, K from 64 to 8192): a
        // large result of a short rank on the FP32 cores (4096 x 128: syrk
        // 38.8 us against 43.1), a small one in 32 x 32 tiles (1000 x 400:
        // syr2k 20.0 us against 23.4 in 64 x 64 tiles split in four, 192 x 379
        // 14.8 and 18.2 in phases), with a longer rank split in four (500 x
        // 550: 11.5 us against 12.4 in 32 x 32, 15.1 in phases; 300 x 2000 the
        // other way, 15.6 and 13.2).
        // Otherwise phases, of 128 x 128 tiles where the work outweighs
        // their pipeline (2048 x 2048: 62.7 us against 67.1 in 64 x 64, syr2k
        // 108 and 126; 1024 x 1024 21.5 and 20.7; 4096 x 512 101 and 81), or
        // without cut tiles, which need no scratch, where eight rounds of them
        // hide the last one (8192 x 1024: 0.518 ms against 0.508; 6500 x 1500
        // 0.437 and 0.408; not with a shorter rank: 10000 x 161 0.42 ms whole,
        // 0.29 in 64 x 64 phases).
        if (K > kSplitMaxLd) return long_rank_pick(M);
        // Very short ranks on the FP32 cores as well, which have no pipeline
        // of K-tiles to fill (kernels alone, us, FP32 cores' 64 x 64 tile and
        // the split pick: syrk 1300 x 16 7.6 and 8.8, 1800 x 32 9.6 and 10.4, 1000
        // x 16 7.0 and 7.8; 1000 x 48 8.1 and 8.4, 1500 x 64 10.1 and 9.2).
        if (K < kSplitMinSum || (M > 512 && K < (M > 1152 ? 64 : 40) && M < 2048)) return 1;
        if (M >= 2048 && K < 160) return 16;
        // Small orders are split in four from rank 200 on for the error: uncut,
        // a 32 x 32 tile's depends on the rank alone (rms 8.8e-8 at 231, 9.4e-8
        // at 300, 1.03e-7 at 379), the FP32 cores' tile that it replaces was
        // cut in four and its error falls with the order (231 / 300 / 379:
        // order 100 0.99 / 1.15 / 1.10e-7, 80 0.97 / 1.11 / 1.02, 48 0.90 /
        // 1.02 / 0.93, 16 0.80 / 0.88 / 0.82; here cut 4.7 to 5.3e-8).
        if (M <= 640 && K >= (M <= 96 ? 200 : 400) && K < 1000) return 9;
        if (M <= 1152 && K < 700) return 17;
        if (M >= 8192 && K >= 640 && 4 * K < 3 * M) return 10;
        return K >= 640 && (double)M * (double)M * (double)K >= 2.5e9 ? 15 : 14;
    }
    if (kernel == LI_KERNEL_GROUPED_GEMM || kernel == LI_KERNEL_GROUPED_COV) {
        // Class 1 (64 x 64) for all but large problems: one class makes two
        // contraction kernels, and each further one adds two that share the
        // compute units with them badly (33 + 33 problems with sizes from 32
        // to 1024: 74 us in class 1 alone, 130 with the class of least
        // predicted work for each problem).  Class 0 (128 x 128)
        // where its padding is small (24 + 24 problems from 700 to 2500:
        // 1.49 ms, all in class 1 1.72; from 500 to 1200 0.371 and 0.382).
        if (K < kSplitMinSum) return 3;
        return M >= 768 && N >= 768 && K >= 256 ? 0 : 1;
    }
    if (kernel == LI_KERNEL_GEMM_LP || kernel == LI_KERNEL_GEMM_LP_SPLIT) {
        if (ceil_div(M, 256) * ceil_div(N, 256) >= cus) return kernel == LI_KERNEL_GEMM_LP ? 23 : 12;
        if (ceil_div(M, 128) * ceil_div(N, 128) >= cus / 2) return 9;
        return 4;
    }
    return 0;
}

}  // namespace

// Rank updates whose rows are too long for the split tiles: stream-K on the
// FP32 cores, in 64 x 64 tiles where these leave enough of the 128 x 128
// tiles' padding out to make up for their cost of 1.3 times per element (rank
// 2097157, syrk, 64 x 64 and 128 x 128: order 33 0.33 and 0.61 ms, 100 0.66
// and 0.66, 200 1.84 and 1.74, 300 2.87 and 3.30, 600 10.5 and 8.6).
int long_rank_pick(int64_t n)
{
    const int64_t t64 = ceil_div(n, 64), t128 = ceil_div(n, 128);
    return 1.3 * (double)(t64 * (t64 + 1)) < 4.0 * (double)(t128 * (t128 + 1)) ? 19 : 20;
}

double split_gemm_us(int64_t M, int64_t N, int64_t K)
{
    double us = 0.0;
    split_pick(M, N, K, &us);
    return us;
}

int tune_num(int kernel)
{
    int n;
    family(kernel, &n);
    return n;
}

const TileCfg &tune_cfg(int kernel, int idx)
{
    int n;
    return family(kernel, &n)[idx];
}

// Table slot of a call.  The GEMM families key their entry by the
// output's area: the reduction length changes the work
// per tile, not how many tiles fill the GPU (a 2048 x 2048 product with
// K = 4096 needs the tile of 2048^3, not that of 4096^3, which leaves half
// the compute units idle; an 8192 x 256 output needs the tile of the
// square of the same area).  Their entries are searched on square
// problems, for which the two rules agree.  The symmetric contractions key
// by two sizes: the order of the result M (bit length, at most 15), which
// sets how many output tiles there are, and a class of the reduction
// length K against M, which sets how long each tile's reduction is; split
// and stream-K candidates trade the two off.  Covariance (K = samples)
// classes: K < 1.5 M, < 3 M, < 6 M, beyond; the row-form updates, whose
// rank is often below the order: K < 0.75 M, < 3 M, < 12 M, beyond.
// The grouped families key by max(M, N, K).
int tune_key(int kernel, int64_t M, int64_t N, int64_t K)
{
    if (kernel == LI_KERNEL_GEMM_F32 || kernel == LI_KERNEL_GEMM_LP || kernel == LI_KERNEL_GEMM_LP_SPLIT) {
        // side of the square with the output's area (exact where M N fits
        // in 62 bits, the nearest double's root beyond)
        int64_t s = (int64_t)sqrt((double)M * (double)N);
        if (M < ((int64_t)1 << 31) && N < ((int64_t)1 << 31)) {
            const int64_t area = M * N;
            while (s > 0 && s * s > area) --s;
            while ((s + 1) * (s + 1) <= area) ++s;
        }
        return li_tune_bucket(s, s, 0);
    }
    if (kernel == LI_KERNEL_SYRK_F32 || kernel == LI_KERNEL_SYRK_ROWS) {
        int order = li_tune_bucket(M, 0, 0);
        if (order > 15) order = 15;
        // called as (M, M, K): the order of the result twice, then the
        // reduction length (the sample count for covariance)
        const double r = M > 0 ? (double)K / (double)M : 1e30;
        int cls;
        if (kernel == LI_KERNEL_SYRK_F32)
            cls = r < 1.5 ? 0 : r < 3.0 ? 1 : r < 6.0 ? 2 : 3;
        else
            cls = r < 0.75 ? 0 : r < 3.0 ? 1 : r < 12.0 ? 2 : 3;
        return order + 16 * cls;
    }
    return li_tune_bucket(M, N, K);
}

// Wave quantisation.  The GEMM tables are searched on square powers of
// two, whose tile counts divide evenly among the 256 compute units; other
// sizes of the same slot can leave most of the last round of tiles empty
// (3072^2 in 128 x 128 tiles: 576 tiles, three rounds for 2.25 rounds of
// work).  A round of one-work-group-per-CU tiles costs its tile area times
// the shape's relative cost per element, so the predicted time of a shape
// is ceil(tiles / 256) * area * cost.  When the table's choice is
// predicted more than 5% slower than the best of a family's steady
// shapes, that one runs instead.  Below a family's minimum output size the
// launch and the pipeline fill dominate and the table stands.
struct QuantCand {
    int idx;      // candidate of the family's list (tile shape from there)
    double cost;  // relative time per output element
    bool choosable;
};
// FP32: costs measured at 8192^3, where every shape's tiles divide evenly
const QuantCand kQuantF32[] = {
    {49, 1.000, true},   // 128 x 256, direct loads, two-stage ring
    {44, 1.015, true},   // 128 x 128, 16 waves, direct loads
    {25, 1.030, true},   // 64 x 128, direct loads, three-stage ring
    {19, 1.089, true},   // 64 x 64, direct loads, three-stage ring
    {18, 1.013, false},  // other table choices, costed only
    {15, 1.065, false},
    {24, 1.072, false},
    {20, 1.151, false},
};
// bf16 / fp16: costs measured from 2048 to 3840, where the 128 x 128 shape
// runs two rounds and the 256 x 256 one a single round
const QuantCand kQuantLp[] = {
    {19, 1.00, true},   // 256 x 256, loads between the matrix instructions
    {9, 1.88, true},    // 128 x 128, direct loads
    {23, 1.00, false},  // 256 x 256, four / five stage rings
    {24, 1.00, false},
};

// split-bf16 (both parts of each operand staged; the four-stage layouts
// do not apply): costs measured from 2048 to 3072
const QuantCand kQuantLpSplit[] = {
    {16, 1.00, true},   // 256 x 256, K-tile 64, direct loads
    {9, 1.60, true},    // 128 x 128, direct loads
    {12, 1.00, false},  // other 256 x 256 table choices, costed only
    {15, 1.00, false},
};

double quant_time(const TileCfg &c, double cost, int64_t M, int64_t N)
{
    const int64_t tiles = ceil_div(M, c.bm) * ceil_div(N, c.bn);
    return (double)ceil_div(tiles, 256) * (double)(c.bm * c.bn) * cost;
}

template <int NQ>
int refine(const QuantCand (&list)[NQ], const TileCfg *fam, double min_side, int t, int64_t M, int64_t N)
{
    if ((double)M * (double)N < min_side * min_side) return t;
    const QuantCand *cur = nullptr;
    for (const QuantCand &q : list)
        if (q.idx == t) cur = &q;
    if (!cur) return t;
    const QuantCand *best = nullptr;
    double tbest = 0;
    for (const QuantCand &q : list) {
        if (!q.choosable) continue;
        const double tq = quant_time(fam[q.idx], q.cost, M, N);
        if (!best || tq < tbest) {
            best = &q;
            tbest = tq;
        }
    }
    return quant_time(fam[cur->idx], cur->cost, M, N) > 1.05 * tbest ? best->idx : t;
}

// Only a table's entry gets here: the rules above name no tile split in a
// fixed number.  Split reductions of the covariance contraction launch
// (upper-triangle tiles) x (chunks) work-groups, each writing a partial tile.
// Split choices are searched where that count fits in one round of the
// 256 compute units; at the top of the same slot (orders up to twice as
// large) it spills into a second or later round, and with short chunks
// the partial tiles' traffic weighs as much as the products: there the
// phases of the split tile of the same size are faster (times with the
// statistics, FP32 cores in seven / split tile in seven / phases: 1500 features
// x 3000 samples 121 / 93 / 71 us, 1900 x 5000 234 / 174 / 142, 1800 x 3600
// 181 / 138 / 108; FP32 stream-K 96, 196, 148).  Chunks of 4096 and more
// amortise their partial tile.  The row-form updates keep their table
// entries.
int refine_cov_split(int t, int64_t M, int64_t K)
{
    const TileCfg &c = kSyrkF32[t];
    if (c.split_k <= 1) return t;
    const int64_t tt = ceil_div(M, c.bm), up = tt * (tt + 1) / 2;
    if (up * c.split_k <= 256 || K / c.split_k >= 4096) return t;
    return c.bm == 128 ? 20 : 21;  // phases
}

int tune_pick(int kernel, int64_t M, int64_t N, int64_t K)
{
    const int f = g_forced[kernel].load(std::memory_order_relaxed) - 1;
    if (f >= 0) return f;
    int t = g_table[kernel][tune_key(kernel, M, N, K)].load(std::memory_order_relaxed) - 1;
    if (t < 0) t = heuristic(kernel, M, N, K);
    if (kernel == LI_KERNEL_GEMM_F32) t = refine(kQuantF32, kGemmF32, 1536.0, t, M, N);
    if (kernel == LI_KERNEL_GEMM_LP) t = refine(kQuantLp, kGemmLp, 2048.0, t, M, N);
    if (kernel == LI_KERNEL_GEMM_LP_SPLIT) t = refine(kQuantLpSplit, kGemmLp, 2048.0, t, M, N);
    if (kernel == LI_KERNEL_SYRK_F32) t = refine_cov_split(t, M, K);
    return t;
}

}  // namespace li

extern "C" {

int32_t li_tune_num_candidates(int32_t kernel) { return li::tune_num(kernel); }

li_status li_tune_candidate(int32_t kernel, int32_t index, li_tile_config *out)
{
    int n;
    const li::TileCfg *f = li::family(kernel, &n);
    if (!f) return li::fail(LI_ERR_BAD_ENUM, "unknown kernel family %d", kernel);
    if (index < 0 || index >= n)
        return li::fail(LI_ERR_NOT_FOUND, "candidate %d out of range [0, %d)", index, n);
    if (!out) return li::fail(LI_ERR_NULL_POINTER, "out is NULL");
    out->bm = f[index].bm;
    out->bn = f[index].bn;
    out->bk = f[index].bk;
    out->waves_m = f[index].wm;
    out->waves_n = f[index].wn;
    out->split_k = f[index].split_k;
    out->prefetch = f[index].prefetch;
    return LI_OK;
}

int32_t li_tune_bucket(int64_t M, int64_t N, int64_t K)
{
    int64_t m = M;
    if (N > m) m = N;
    if (K > m) m = K;
    int b = 0;
    while (m > 0 && b < 63) {
        m >>= 1;
        ++b;
    }
    return b;
}

li_status li_tune_set(int32_t kernel, int32_t bucket, int32_t index)
{
    int n;
    if (!li::family(kernel, &n)) return li::fail(LI_ERR_BAD_ENUM, "unknown kernel family %d", kernel);
    if (bucket < 0 || bucket >= li::kBuckets)
        return li::fail(LI_ERR_INVALID_SIZE, "bucket %d out of range", bucket);
    if (index < -1 || index >= n)
        return li::fail(LI_ERR_NOT_FOUND, "candidate %d out of range [-1, %d)", index, n);
    li::g_table[kernel][bucket].store(index + 1);
    return LI_OK;
}

int32_t li_tune_get(int32_t kernel, int32_t bucket)
{
    int n;
    if (!li::family(kernel, &n) || bucket < 0 || bucket >= li::kBuckets) return -1;
    return li::g_table[kernel][bucket].load() - 1;
}

int32_t li_tune_key(int32_t kernel, int64_t M, int64_t N, int64_t K)
{
    int n;
    if (!li::family(kernel, &n) || M < 0 || N < 0 || K < 0) return -1;
    return li::tune_key(kernel, M, N, K);
}

int32_t li_tune_pick(int32_t kernel, int64_t M, int64_t N, int64_t K)
{
    int n;
    if (!li::family(kernel, &n) || M < 0 || N < 0 || K < 0) return -1;
    return li::tune_pick(kernel, M, N, K);
}

li_status li_tune_force(int32_t kernel, int32_t index)
{
    int n;
    if (!li::family(kernel, &n)) return li::fail(LI_ERR_BAD_ENUM, "unknown kernel family %d", kernel);
    if (index < -1 || index >= n)
        return li::fail(LI_ERR_NOT_FOUND, "candidate %d out of range [-1, %d)", index, n);
    li::g_forced[kernel].store(index + 1);
    return LI_OK;
}

li_status li_tune_save(const char *path)
{
    if (!path) return li::fail(LI_ERR_NULL_POINTER, "path is NULL");
    FILE *f = fopen(path, "w");
    if (!f) return li::fail(LI_ERR_NOT_FOUND, "cannot write %s", path);
    fprintf(f, "# li tuning table (gfx950) version %d: kernel slot candidate\n", li::kTableVersion);
    for (int k = 0; k < li::kFamilies; ++k)
        for (int b = 0; b < li::kBuckets; ++b) {
            const int v = li::g_table[k][b].load() - 1;
            if (v >= 0) fprintf(f, "%d %d %d\n", k, b, v);
        }
    const bool ok = fclose(f) == 0;
    return ok ? LI_OK : li::fail(LI_ERR_NOT_FOUND, "writing %s failed", path);
}

li_status li_tune_load(const char *path)
{
    if (!path) return li::fail(LI_ERR_NULL_POINTER, "path is NULL");
    FILE *f = fopen(path, "r");
    if (!f) return li::fail(LI_ERR_NOT_FOUND, "cannot open %s", path);
    struct Entry {
        int k, b, v;
    };
    Entry entries[li::kFamilies * li::kBuckets];
    int n = 0, line_no = 0, version = 1;
    char line[256];
    li_status st = LI_OK;
    while (st == LI_OK && fgets(line, sizeof(line), f)) {
        ++line_no;
        char *p = line;
        while (*p == ' ' || *p == '\t') ++p;
        if (n == 0 && sscanf(p, "# li tuning table (gfx950) version %d", &version) == 1 &&
            (version < 1 || version > li::kTableVersion)) {
            st = li::fail(LI_ERR_INVALID_SIZE, "%s:%d: table version %d, this library knows 1 to %d", path, line_no,
                          version, li::kTableVersion);
            break;
        }
        if (*p == '#' || *p == '\n' || *p == '\r' || *p == 0) continue;
        int k, b, v, cnt;
        if (sscanf(p, "%d %d %d %n", &k, &b, &v, &cnt) != 3 || (p[cnt] != 0 && p[cnt] != '#')) {
            st = li::fail(LI_ERR_INVALID_SIZE, "%s:%d: expected 'kernel slot candidate'", path, line_no);
            break;
        }
        int nc;
        if (!li::family(k, &nc) || b < 0 || b >= li::kBuckets || v < 0 || v >= nc) {
            st = li::fail(LI_ERR_INVALID_SIZE, "%s:%d: entry out of range", path, line_no);
            break;
        }
        if (n < li::kFamilies * li::kBuckets) entries[n++] = {k, b, li::current_number(version, k, v)};
    }
    fclose(f);
    if (st != LI_OK) return st;
    for (int i = 0; i < n; ++i) li::g_table[entries[i].k][entries[i].b].store(entries[i].v + 1);
    return LI_OK;
}

}  // extern "C"
