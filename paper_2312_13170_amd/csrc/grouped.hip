// Grouped execution: hundreds of independent, uneven GEMM and covariance
// problems in two launches captured in one HIP graph.
//
//  node 1  grouped_stats:    one work-group per (covariance problem, 64
//                            columns), eight threads per column: FP64
//                            column means (same chunking and merge order as
//                            the single-problem kernels, so the results are
//                            bitwise the same) and the centred data.
//  node 2  grouped_contract: per shape class and problem kind one launch
//                            over a table of every output tile of its
//                            problems (GEMM tiles and upper-triangle
//                            covariance tiles), dealt to the XCDs problem by
//                            problem (deal_tiles).  Each tile runs the same
//                            main loop and epilogue as the single-problem
//                            kernels with the tile shape chosen for its
//                            problem: the split tiles of split_tile.h, or
//                            the FP32 cores' for rows too long for them and
//                            for results of few products.
//
// 512 products and 512 covariances, sizes log-uniform from 32 to 1024: 868 us
// on the FP32 cores, 720 on the split tiles.  The three kernels each fill the
// compute units, so their times add (statistics 135, products 330,
// covariances 330 us): the statistics are near the copy rate (0.6 GB); a
// product's 64 x 64 tile takes 14 us for 9 K-tiles on average, half of it
// before its first and after its last, and is bound by the vector
// instructions that split its operands and by latency together (a third
// work-group per compute unit, at 80 registers and a few spills, is slower:
// 876 us against 810 in the same back-to-back loop).
// The covariance launches depend on node 1 (their tiles read the centred
// data); the GEMM launches are independent of it.
#include <hip/hip_runtime.h>

#include <stdlib.h>

#include <algorithm>
#include <new>
#include <vector>

#include "li_internal.h"
#include "split_tile.h"
#include "stats_dev.h"
#include "symm_kernels.h"
#include "tiles.h"

namespace li {
namespace {

struct GProb {
    int32_t kind, cfg, vec4, pad0;
    int64_t M, N, K;
    float alpha, beta, scale, pad1;
    const float *A;
    const float *B;
    float *C;
    float *Y;
    double *mean;
    int64_t rows_per_split, nsplit;
};

struct GTile {
    int32_t prob, tm, tn, pad;
};

struct GStatBlock {
    int32_t prob, col0;
};

template <int BT, int BK, int WM, int WN, bool KMAJOR, int PF>
using Tile = CandidateTile<BT, BT, BK, WM, WN, PF, KMAJOR, false, 0, kLoadScalar, PF>;

// Statistics of one covariance problem's block of kGStatCols columns: the
// kMergeGroups thread rows each merge one group of chunk partials (chunk
// moments and merge order as in the single-problem kernels, so the results
// are bitwise the same), one thread row merges the group results in order,
// then every thread row centres a share of the rows.
constexpr int kGStatCols = 64;
constexpr int kGStatThreads = kGStatCols * kMergeGroups;

__global__ __launch_bounds__(kGStatThreads) void grouped_stats(const GProb *__restrict__ probs,
                                                               const GStatBlock *__restrict__ blocks)
{
    __shared__ double sn[kMergeGroups][kGStatCols], sm[kMergeGroups][kGStatCols],
        sq[kMergeGroups][kGStatCols];
    __shared__ double smean[kGStatCols];
    const GStatBlock b = blocks[blockIdx.x];
    const GProb &p = probs[b.prob];
    const int64_t M = p.M, N = p.N;
    const int c = threadIdx.x % kGStatCols, g = threadIdx.x / kGStatCols;
    const int64_t j = (int64_t)b.col0 + c;
    const bool live = j < M;
    const float *col = p.A + j;
    const int64_t rps = p.rows_per_split, nsplit = p.nsplit;
    const int64_t cpg = chunks_per_group(nsplit);
    const int64_t s0 = g * cpg, s1 = s0 + cpg < nsplit ? s0 + cpg : nsplit;
    double gn = 0.0, gm = 0.0, gq = 0.0;
    if (live && s0 < s1) {
        int64_t r0, r1;
        chunk_rows(s0, rps, N, r0, r1);
        gn = (double)(r1 - r0);
        chunk_moments(col, M, r0, r1, gm, gq);
        for (int64_t s = s0 + 1; s < s1; ++s) {
            chunk_rows(s, rps, N, r0, r1);
            double mb, m2b;
            chunk_moments(col, M, r0, r1, mb, m2b);
            chan_merge(gn, gm, gq, (double)(r1 - r0), mb, m2b);
        }
    }
    sn[g][c] = gn;
    sm[g][c] = gm;
    sq[g][c] = gq;
    __syncthreads();
    if (g == 0) {
        // group 0 always holds chunk 0; empty groups (gn == 0) are skipped
        double n = sn[0][c], ma = sm[0][c], m2a = sq[0][c];
        for (int h = 1; h < kMergeGroups; ++h)
            if (sn[h][c] > 0.0) chan_merge(n, ma, m2a, sn[h][c], sm[h][c], sq[h][c]);
        if (live) p.mean[j] = ma;
        smean[c] = ma;
    }
    __syncthreads();
    if (!live) return;
    const double ma = smean[c];
    float *ycol = p.Y + j;
    // eight of this thread's rows in flight per step (data_out may be the
    // data itself: every element is still read before it is written, by
    // the same thread)
    constexpr int64_t RS = kMergeGroups;  // row stride of a thread
    int64_t r = g;
    for (; r + 7 * RS < N; r += 8 * RS) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = col[(r + u * RS) * M];
#pragma unroll
        for (int u = 0; u < 8; ++u) ycol[(r + u * RS) * M] = centre_value(x[u], ma, 0.0, false);
    }
    for (; r < N; r += RS) ycol[r * M] = centre_value(col[r * M], ma, 0.0, false);
}

template <class T>
__device__ __forceinline__ void gemm_tile(float *lds, const GProb &p, const GTile &td)
{
    const int64_t m0 = (int64_t)td.tm * T::BM, n0 = (int64_t)td.tn * T::BN;
    f32x16 acc[T::TM][T::TN];
    T::zero(acc);
    if constexpr (T::SPLIT) {
        const auto warm = T::warm_c(p.C, p.N, p.M, p.N, m0, n0, p.beta);
        if (p.alpha != 0.f) T::mainloop(lds, p.A, p.K, p.B, p.N, p.M, p.N, 0, p.K, m0, n0, acc);
        warm.touch();
        T::store_c(lds, acc, p.C, p.N, p.M, p.N, m0, n0, p.alpha, p.beta);
        return;
    }
    if (p.alpha != 0.f) T::mainloop(lds, p.A, p.K, p.B, p.N, p.M, p.N, 0, p.K, m0, n0, acc);
    if (p.beta != 0.f) {
        // the tile's C loads issued together, then one wait
        float cv[T::TM][T::TN][16];
        T::load_c(cv, p.C, p.N, p.M, p.N, m0, n0);
        T::epilogue_gemm_loaded(acc, cv, p.C, p.N, p.M, p.N, m0, n0, p.alpha, p.beta);
    } else {
        T::epilogue_gemm(acc, p.C, p.N, p.M, p.N, m0, n0, p.alpha, 0.f);
    }
}

template <class T>
__device__ __forceinline__ void syrk_tile(float *lds, const GProb &p, const GTile &td)
{
    const int64_t m0 = (int64_t)td.tm * T::BM, n0 = (int64_t)td.tn * T::BN;
    const SymArgs a{p.Y, nullptr, p.M, p.M, p.N, p.C, 0, p.scale, 0.f, 1, nullptr, nullptr};
    f32x16 acc[T::TM][T::TN];
    T::zero(acc);
    sym_reduce<T, kSymCols>(lds, a, 0, p.N, m0, n0, acc);
    finish_sym<T>(lds, acc, a, m0, n0);
}

constexpr int kXcds = 8;
// entry of work-group b: the XCDs' lists lie one after the other
__device__ __forceinline__ int table_entry(int b, int n) { return b % kXcds * (n / kXcds) + b / kXcds; }

// Contraction kernel of one shape class over the class's tile table (see
// deal_tiles).  PERSIST: a resident grid, work-group b takes tiles b,
// b + gridDim.x, ...; otherwise one work-group per tile, handed out by the
// hardware dispatcher in table order as compute units free up.
template <int BT, int BK, int WM, int WN, int PF, int KIND, bool PERSIST>
__global__ __launch_bounds__((Tile<BT, BK, WM, WN, false, PF>::NT)) void grouped_contract(const GProb *__restrict__ probs,
                                                                 const GTile *__restrict__ tiles,
                                                                 int ntiles)
{
    // one main loop per kernel; its loads take rows of any alignment
    using G = Tile<BT, BK, WM, WN, false, PF>;
    using S = Tile<BT, BK, WM, WN, true, PF>;
    constexpr int L1 = KIND == LI_PROBLEM_GEMM ? G::LDS_FLOATS : S::LDS_FLOATS;
    __shared__ __attribute__((aligned(16))) float lds[L1];
    if (PERSIST) {
        for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
            const GTile td = tiles[table_entry(t, ntiles)];
            if (td.prob < 0) continue;
            const GProb &p = probs[td.prob];
            if (KIND == LI_PROBLEM_GEMM)
                gemm_tile<G>(lds, p, td);
            else
                syrk_tile<S>(lds, p, td);
            __syncthreads();
        }
    } else {
        const GTile td = tiles[table_entry((int)blockIdx.x, ntiles)];
        if (td.prob < 0) return;
        const GProb &p = probs[td.prob];
        if (KIND == LI_PROBLEM_GEMM)
            gemm_tile<G>(lds, p, td);
        else
            syrk_tile<S>(lds, p, td);
    }
}

struct ShapeClass {
    int cls, gemm_idx, syrk_idx, bt, bk, wm, wn, pf, threads;
    const void *kernel[2];   // [LI_PROBLEM_GEMM], [LI_PROBLEM_COVARIANCE]: one work-group per tile
    const void *persist[2];  // the same on a resident grid
};

#define LI_CLASS(C, GI, SI, BT, BK, WM, WN, PF)                                                     \
    {C, GI, SI, BT, BK, WM, WN, PF, Tile<BT, BK, WM, WN, false, PF>::NT,                            \
     {(const void *)grouped_contract<BT, BK, WM, WN, PF, LI_PROBLEM_GEMM, false>,                   \
      (const void *)grouped_contract<BT, BK, WM, WN, PF, LI_PROBLEM_COVARIANCE, false>},            \
     {(const void *)grouped_contract<BT, BK, WM, WN, PF, LI_PROBLEM_GEMM, true>,                    \
      (const void *)grouped_contract<BT, BK, WM, WN, PF, LI_PROBLEM_COVARIANCE, true>}},
const ShapeClass kClasses[] = {LI_GROUPED_CLASSES(LI_CLASS)};
#undef LI_CLASS
constexpr int kNumClasses = (int)(sizeof(kClasses) / sizeof(kClasses[0]));
// one tile table and one persistent launch per (class, kind)
constexpr int kSlots = 2 * kNumClasses;

// The classes must use the same compiled candidates as the single-problem
// kernels (same index, same shape), so a problem gives bitwise the same
// result grouped or alone.
bool shapes_consistent()
{
    for (const ShapeClass &c : kClasses) {
        const TileCfg &g = tune_cfg(LI_KERNEL_GEMM_F32, c.gemm_idx);
        const TileCfg &s = tune_cfg(LI_KERNEL_SYRK_F32, c.syrk_idx);
        if (g.bm != c.bt || g.bn != c.bt || g.bk != c.bk || g.wm != c.wm || g.wn != c.wn ||
            g.prefetch != c.pf || g.split_k != 1)
            return false;
        if (s.bm != c.bt || s.bn != c.bt || s.bk != c.bk || s.wm != c.wm || s.wn != c.wn ||
            s.prefetch != c.pf || s.split_k != 1)
            return false;
    }
    return true;
}

// Class of a problem: the tuning table's entry for the grouped family of its
// kind (forced > table > built-in heuristic); rows of `ld` elements that the
// split tiles' offsets cannot span take the FP32 cores' class.
constexpr int kFp32Class = 3;
static_assert(kNumClasses > kFp32Class, "the class of the FP32 cores is in the list");
int pick_class(int kernel, int64_t M, int64_t N, int64_t K, int64_t ld)
{
    if (ld > kSplitMaxLd) return kFp32Class;
    const int c = tune_pick(kernel, M, N, K);
    return c >= 0 && c < kNumClasses ? c : 0;
}

inline bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

// The tiles of one problem in a shape class, each of the same cost.
struct Bundle {
    double cost;  // of one tile
    std::vector<GTile> tiles;
};

// The table of a class: work-group b runs on XCD b mod 8 and takes tile b / 8
// of that XCD's list (neighbouring entries share a line of its L2).  A problem's tiles go to one XCD (cut into parts
// where one would outweigh a 32nd of the work), whose L2 then reads its
// operands from memory once; the XCDs' loads are balanced greedily, largest
// part first, and each XCD takes its heaviest tiles first.  Shorter lists end
// in entries without a problem.  512 + 512 problems, sizes
// log-uniform from 32 to 1024: 0.53 GB of L2 misses in the products, the batch 828
// us; with tiles dealt in runs of eight regardless of problem 1.2 GB, 849 us.
std::vector<GTile> deal_tiles(std::vector<Bundle> &all)
{
    constexpr int X = kXcds;
    double total = 0;
    for (const Bundle &b : all) total += b.cost * (double)b.tiles.size();
    std::vector<Bundle> parts;
    for (const Bundle &b : all) {
        const size_t most = std::max<size_t>(1, (size_t)(total / 32 / b.cost));
        for (size_t k = 0; k < b.tiles.size(); k += most)
            parts.push_back({b.cost, std::vector<GTile>(b.tiles.begin() + k,
                                                        b.tiles.begin() + std::min(k + most, b.tiles.size()))});
    }
    std::stable_sort(parts.begin(), parts.end(), [](const Bundle &x, const Bundle &y) {
        return x.cost * (double)x.tiles.size() > y.cost * (double)y.tiles.size();
    });
    std::vector<const Bundle *> list[X];
    double load[X] = {};
    for (const Bundle &b : parts) {
        const int x = (int)(std::min_element(load, load + X) - load);
        load[x] += b.cost * (double)b.tiles.size();
        list[x].push_back(&b);
    }
    size_t longest = 0;
    std::vector<GTile> of[X];
    for (int x = 0; x < X; ++x) {
        std::stable_sort(list[x].begin(), list[x].end(),
                         [](const Bundle *p, const Bundle *q) { return p->cost > q->cost; });
        for (const Bundle *b : list[x]) of[x].insert(of[x].end(), b->tiles.begin(), b->tiles.end());
        longest = std::max(longest, of[x].size());
    }
    std::vector<GTile> table;
    for (int x = 0; x < X; ++x) {
        of[x].resize(longest, GTile{-1, 0, 0, 0});
        table.insert(table.end(), of[x].begin(), of[x].end());
    }
    return table;
}

struct SpanRec {
    uintptr_t lo, hi;
    int prob;
    bool out;
};

}  // namespace
}  // namespace li

struct li_group_plan {
    std::vector<li_problem> problems;
    std::vector<int> cfg, vec4;
    li::GProb *d_probs = nullptr;
    li::GStatBlock *d_stat = nullptr;
    li::GTile *d_tiles[li::kSlots] = {};
    int ntiles[li::kSlots] = {};
    int grid[li::kSlots] = {};
    int nstat = 0, device = 0;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    void *loop_ws = nullptr;
    double flops = 0.0;
};

namespace {

void plan_free(li_group_plan *p)
{
    if (!p) return;
    if (p->exec) (void)hipGraphExecDestroy(p->exec);
    if (p->graph) (void)hipGraphDestroy(p->graph);
    if (p->d_probs) (void)hipFree(p->d_probs);
    for (int c = 0; c < li::kSlots; ++c)
        if (p->d_tiles[c]) (void)hipFree(p->d_tiles[c]);
    if (p->d_stat) (void)hipFree(p->d_stat);
    if (p->loop_ws) (void)hipFree(p->loop_ws);
    delete p;
}

li_status validate_problem(const li_problem &q, int i, std::vector<li::SpanRec> &spans)
{
    using li::fail;
    if (q.kind != LI_PROBLEM_GEMM && q.kind != LI_PROBLEM_COVARIANCE)
        return fail(LI_ERR_BAD_ENUM, "problem %d: unknown kind %d", i, q.kind);
    if (q.M < 0 || q.N < 0 || q.K < 0) return fail(LI_ERR_INVALID_SIZE, "problem %d: negative size", i);
    uint64_t a, b, c;
    auto add = [&](const void *ptr, uint64_t bytes, bool out) {
        if (ptr && bytes) spans.push_back({(uintptr_t)ptr, (uintptr_t)ptr + bytes, i, out});
    };
    if (q.kind == LI_PROBLEM_GEMM) {
        if (!li::matrix_bytes(q.M, q.K, 4, &a) || !li::matrix_bytes(q.K, q.N, 4, &b) ||
            !li::matrix_bytes(q.M, q.N, 4, &c))
            return fail(LI_ERR_INVALID_SIZE, "problem %d: extent too large", i);
        const bool out_any = q.M > 0 && q.N > 0;
        const bool reads = out_any && q.K > 0 && q.alpha != 0.f;
        if (!reads) a = b = 0;
        if (!out_any) c = 0;
        if ((a && !q.A) || (b && !q.B) || (c && !q.C))
            return fail(LI_ERR_NULL_POINTER, "problem %d: NULL operand", i);
        add(q.A, a, false);
        add(q.B, b, false);
        add(q.C, c, true);
    } else {
        if (q.M > 0 && q.N < 2) return fail(LI_ERR_INVALID_SIZE, "problem %d: covariance needs N >= 2", i);
        uint64_t m8 = (uint64_t)q.M * 8;
        if (!li::matrix_bytes(q.N, q.M, 4, &a) || !li::matrix_bytes(q.M, q.M, 4, &c))
            return fail(LI_ERR_INVALID_SIZE, "problem %d: extent too large", i);
        if (q.M == 0) a = c = m8 = 0;
        if ((a && (!q.A || !q.data_out)) || (c && !q.C) || (m8 && !q.mean))
            return fail(LI_ERR_NULL_POINTER, "problem %d: NULL operand", i);
        if (q.data_out != q.A && li::overlaps({q.A, a}, {q.data_out, a}))
            return fail(LI_ERR_OVERLAP, "problem %d: data_out partially overlaps data", i);
        if (q.data_out == q.A) {
            add(q.A, a, true);
        } else {
            add(q.A, a, false);
            add(q.data_out, a, true);
        }
        add(q.C, c, true);
        add(q.mean, m8, true);
    }
    return LI_OK;
}

// No output may overlap any other buffer of the plan (inputs may be shared
// read-only between problems).  Sort by start and sweep.
li_status check_plan_overlaps(std::vector<li::SpanRec> &spans)
{
    std::sort(spans.begin(), spans.end(), [](const li::SpanRec &x, const li::SpanRec &y) {
        return x.lo < y.lo || (x.lo == y.lo && x.hi < y.hi);
    });
    // track the open span reaching furthest, and the furthest-reaching output
    size_t far_any = (size_t)-1, far_out = (size_t)-1;
    for (size_t k = 0; k < spans.size(); ++k) {
        const li::SpanRec &s = spans[k];
        if (far_out != (size_t)-1 && spans[far_out].hi > s.lo)
            return li::fail(LI_ERR_OVERLAP, "problem %d: an output overlaps a buffer of problem %d",
                            spans[far_out].prob, s.prob);
        if (s.out && far_any != (size_t)-1 && spans[far_any].hi > s.lo)
            return li::fail(LI_ERR_OVERLAP, "problem %d: an output overlaps a buffer of problem %d",
                            s.prob, spans[far_any].prob);
        if (far_any == (size_t)-1 || s.hi > spans[far_any].hi) far_any = k;
        if (s.out && (far_out == (size_t)-1 || s.hi > spans[far_out].hi)) far_out = k;
    }
    return LI_OK;
}

}  // namespace

extern "C" {

li_status li_group_plan_create(const li_problem *problems, int32_t count, li_group_plan **plan)
{
    using namespace li;
    if (!plan) return fail(LI_ERR_NULL_POINTER, "plan is NULL");
    *plan = nullptr;
    if (count < 0) return fail(LI_ERR_INVALID_SIZE, "count must be >= 0");
    if (count > 0 && !problems) return fail(LI_ERR_NULL_POINTER, "problems is NULL");
    std::vector<SpanRec> spans;
    for (int i = 0; i < count; ++i) {
        li_status s = validate_problem(problems[i], i, spans);
        if (s) return s;
    }
    if (li_status s = check_plan_overlaps(spans)) return s;
    if (li_status s = ensure_device()) return s;
    if (!shapes_consistent()) return fail(LI_ERR_HIP, "grouped tile shapes do not match the compiled candidates");

    const char *pe = getenv("LI_GROUPED_PERSIST");
    const bool persist = pe && pe[0] == '1';
    li_group_plan *p = new (std::nothrow) li_group_plan();
    if (!p) return fail(LI_ERR_HIP, "out of host memory");
    (void)hipGetDevice(&p->device);
    p->problems.assign(problems, problems + count);
    std::vector<GProb> hp(count);
    std::vector<Bundle> work[kSlots];
    // a tile's pipeline fill and epilogue take about as long as 128 k
    auto tile_cost = [](int bt, double k) { return (double)bt * bt * (k + 128.0); };
    std::vector<GStatBlock> stat;
    size_t loop_ws = 0;
    for (int i = 0; i < count; ++i) {
        const li_problem &q = problems[i];
        GProb g{};
        g.kind = q.kind;
        g.M = q.M;
        g.N = q.N;
        g.K = q.K;
        g.alpha = q.alpha;
        g.beta = q.beta;
        g.A = q.A;
        g.B = q.B;
        g.C = q.C;
        g.Y = q.data_out;
        g.mean = q.mean;
        int cls;
        if (q.kind == LI_PROBLEM_GEMM) {
            // (no reduction without alpha)
            cls = pick_class(LI_KERNEL_GROUPED_GEMM, q.M, q.N, q.alpha != 0.f ? q.K : 0, std::max(q.K, q.N));
            const int bt = kClasses[cls].bt;
            g.cfg = kClasses[cls].gemm_idx;
            g.vec4 = (q.alpha == 0.f || (q.K % 4 == 0 && q.N % 4 == 0 && aligned16(q.A) && aligned16(q.B))) ? 1 : 0;
            const int tm = (int)((q.M + bt - 1) / bt), tn = (int)((q.N + bt - 1) / bt);
            Bundle w{tile_cost(bt, q.alpha != 0.f ? (double)q.K : 0.0), {}};
            for (int a = 0; a < tm; ++a)
                for (int b = 0; b < tn; ++b) w.tiles.push_back({i, a, b, 0});
            work[2 * cls + LI_PROBLEM_GEMM].push_back(std::move(w));
            p->flops += 2.0 * q.M * q.N * q.K + 3.0 * q.M * q.N;
        } else {
            cls = pick_class(LI_KERNEL_GROUPED_COV, q.M, q.M, q.N, q.M);
            const int bt = kClasses[cls].bt;
            g.cfg = kClasses[cls].syrk_idx;
            g.vec4 = (q.M % 4 == 0 && aligned16(q.data_out)) ? 1 : 0;
            g.scale = q.N > 1 ? (float)(1.0 / (double)(q.N - 1)) : 0.f;
            if (q.M > 0) {
                const StatsPlan sp = stats_plan(q.M, q.N);
                g.rows_per_split = sp.rows_per_split;
                g.nsplit = sp.nsplit;
                for (int64_t c0 = 0; c0 < q.M; c0 += kGStatCols) stat.push_back({i, (int32_t)c0});
                loop_ws = std::max(loop_ws, stats_workspace_bytes(q.M, q.N));
                const int tm = (int)((q.M + bt - 1) / bt);
                Bundle w{tile_cost(bt, (double)q.N), {}};
                for (int a = 0; a < tm; ++a)
                    for (int b = a; b < tm; ++b) w.tiles.push_back({i, a, b, 0});
                work[2 * cls + LI_PROBLEM_COVARIANCE].push_back(std::move(w));
            }
            p->flops += (double)q.N * q.M * (q.M + 1);
        }
        p->cfg.push_back(g.cfg);
        p->vec4.push_back(g.vec4);
        hp[i] = g;
    }

    auto up = [&](void **dst, const void *src, size_t bytes) -> bool {
        if (bytes == 0) return true;
        if (hipMalloc(dst, bytes) != hipSuccess) return false;
        return hipMemcpy(*dst, src, bytes, hipMemcpyHostToDevice) == hipSuccess;
    };
    bool ok = up((void **)&p->d_probs, hp.data(), hp.size() * sizeof(GProb)) &&
              up((void **)&p->d_stat, stat.data(), stat.size() * sizeof(GStatBlock));
    for (int c = 0; c < kSlots && ok; ++c) {
        const std::vector<GTile> table = deal_tiles(work[c]);
        p->ntiles[c] = (int)table.size();
        const ShapeClass &sc = kClasses[c / 2];
        if (persist) {
            // as many work-groups as can be resident at once
            int per_cu = 1;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, sc.persist[c % 2], sc.threads,
                                                             0) != hipSuccess ||
                per_cu < 1) {
                (void)hipGetLastError();
                per_cu = 1;
            }
            p->grid[c] = std::min(p->ntiles[c], per_cu * device_cu_count() / kXcds * kXcds);
        } else {
            p->grid[c] = p->ntiles[c];
        }
        ok = up((void **)&p->d_tiles[c], table.data(), table.size() * sizeof(GTile));
    }
    p->nstat = (int)stat.size();
    if (ok && loop_ws) ok = hipMalloc(&p->loop_ws, loop_ws) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        plan_free(p);
        return fail(LI_ERR_HIP, "device allocation for the plan failed");
    }

    // graph: one persistent launch per (class, kind); only the covariance
    // launches depend on grouped_stats (they read the centred data), the
    // GEMM launches depend on nothing
    hipError_t e = hipGraphCreate(&p->graph, 0);
    hipGraphNode_t stat_node = nullptr;
    bool any = false;
    if (e == hipSuccess && p->nstat > 0) {
        void *args[] = {(void *)&p->d_probs, (void *)&p->d_stat};
        hipKernelNodeParams kp{};
        kp.func = (void *)grouped_stats;
        kp.gridDim = dim3((unsigned)p->nstat);
        kp.blockDim = dim3(kGStatThreads);
        kp.sharedMemBytes = 0;
        kp.kernelParams = args;
        kp.extra = nullptr;
        e = hipGraphAddKernelNode(&stat_node, p->graph, nullptr, 0, &kp);
        any = true;
    }
    for (int c = 0; c < kSlots && e == hipSuccess; ++c) {
        if (p->ntiles[c] == 0) continue;
        const ShapeClass &sc = kClasses[c / 2];
        void *args[] = {(void *)&p->d_probs, (void *)&p->d_tiles[c], (void *)&p->ntiles[c]};
        hipKernelNodeParams kp{};
        kp.func = const_cast<void *>(persist ? sc.persist[c % 2] : sc.kernel[c % 2]);
        kp.gridDim = dim3((unsigned)p->grid[c]);
        kp.blockDim = dim3((unsigned)sc.threads);
        kp.sharedMemBytes = 0;
        kp.kernelParams = args;
        kp.extra = nullptr;
        const bool after_stats = c % 2 == LI_PROBLEM_COVARIANCE && stat_node;
        hipGraphNode_t n = nullptr;
        e = hipGraphAddKernelNode(&n, p->graph, after_stats ? &stat_node : nullptr, after_stats ? 1 : 0,
                                  &kp);
        any = true;
    }
    if (e == hipSuccess && any) e = hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        plan_free(p);
        return fail(LI_ERR_HIP, "building the plan's graph failed: %s", hipGetErrorString(e));
    }
    *plan = p;
    return LI_OK;
}

li_status li_group_plan_launch(li_group_plan *plan, li_stream stream)
{
    if (!plan) return li::fail(LI_ERR_NULL_POINTER, "plan is NULL");
    int dev = -1;
    (void)hipGetDevice(&dev);
    if (dev != plan->device) return li::fail(LI_ERR_UNSUPPORTED_DEVICE, "plan belongs to device %d, current is %d", plan->device, dev);
    if (!plan->exec) return LI_OK;  // nothing to compute
    hipError_t e = hipGraphLaunch(plan->exec, (hipStream_t)stream);
    if (e != hipSuccess) return li::hip_fail((int)e, "hipGraphLaunch");
    return LI_OK;
}

li_status li_group_plan_launch_loop(li_group_plan *plan, li_stream stream)
{
    if (!plan) return li::fail(LI_ERR_NULL_POINTER, "plan is NULL");
    int dev = -1;
    (void)hipGetDevice(&dev);
    if (dev != plan->device) return li::fail(LI_ERR_UNSUPPORTED_DEVICE, "plan belongs to device %d, current is %d", plan->device, dev);
    for (size_t i = 0; i < plan->problems.size(); ++i) {
        const li_problem &q = plan->problems[i];
        int err = 0;
        if (q.kind == LI_PROBLEM_GEMM) {
            if (q.M == 0 || q.N == 0) continue;
            err = li::launch_gemm_f32(plan->cfg[i], q.M, q.N, q.K, q.alpha, q.A, q.K, q.B, q.N, q.beta,
                                      q.C, q.N, stream);
        } else {
            if (q.M == 0) continue;
            err = li::launch_stats(q.M, q.N, q.A, q.data_out, q.mean, nullptr, 0, 0.0, plan->loop_ws, stream);
            if (!err)
                err = li::launch_syrk_f32(plan->cfg[i], q.M, q.N, q.data_out, q.C, 0,
                                          (float)(1.0 / (double)(q.N - 1)), nullptr, stream);
        }
        if (err) return li::hip_fail(err, "per-instance launch");
    }
    return LI_OK;
}

double li_group_plan_flops(const li_group_plan *plan) { return plan ? plan->flops : 0.0; }

void li_group_plan_destroy(li_group_plan *plan) { plan_free(plan); }

}  // extern "C"
