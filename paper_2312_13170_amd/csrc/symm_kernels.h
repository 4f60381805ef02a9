// Symmetric contractions on the split tile (split_tile.h, bf16 matrix cores) and
// the FP32 matrix-core tile (f32_tile.h).
//
// Only block tiles with tile column >= tile row are computed; the epilogue
// writes each value to (r, c) and (c, r).  Three
// operand forms share the kernels:
//   kSymCols : S = Y^T Y, Y (kdim x n) row-major; both operands k-major
//              (covariance / correlation after centring; T has A_KMAJOR).
//              With T::XFORM the operand is the raw data and the centring
//              happens in the loads (the fused statistics kernels).
//   kSymRows : P = X X^T, X (n x kdim) row-major; both operands have k
//              contiguous (syrk; T has B_NMAJOR).
//   kSymRows2: P = X Z^T + Z X^T, X and Z (n x kdim) row-major (syr2k): the
//              four staged references X[i][k], Z[j][k], Z[i][k], X[j][k] are
//              two reductions into the same accumulators.
// Epilogue modes are those of epilogue_syrk.
#pragma once

#include <hip/hip_runtime.h>

#include "f32_tile.h"
#include "li_internal.h"
#include "split_tile.h"

namespace li {

enum { kSymCols = 0, kSymRows = 1, kSymRows2 = 2 };

struct SymArgs {
    const float *X;  // operand (Y for kSymCols)
    const float *Z;  // second operand of kSymRows2, else unused
    int64_t ld;      // leading dimension of X and Z
    int64_t n;       // order of the result
    int64_t kdim;    // reduction length
    float *S;        // n x n result
    int mode;
    float scale;     // mode 0: multiplier; mode 2: alpha
    float beta;      // mode 2 only
    int reads;       // 0: operands are not read (alpha == 0), result = beta*S
    const double *mean;    // tiles with XFORM: column means of the raw data X
    const double *factor;  // and, for XFORM 2, the normalisation factors
};

template <class T, int FORM>
__device__ __forceinline__ void sym_reduce(float *lds, const SymArgs &a, int64_t kbeg,
                                           int64_t kend, int64_t m0, int64_t n0,
                                           f32x16 (&acc)[T::TM][T::TN])
{
    if constexpr (T::SPLIT) {
        typename T::XRegs xr;
        T::load_xregs(xr, a.mean, a.factor, a.n, a.n, m0, n0);
        constexpr bool two = FORM == kSymRows2;
        T::contract(lds, a.X, two ? a.Z : a.X, two ? a.Z : nullptr, two ? a.X : nullptr, a.ld, a.ld, a.n, a.n, kbeg,
                    kend, m0, n0, acc, &xr);
        return;
    } else if constexpr (T::XFORM != 0) {
        typename T::XRegs xr;
        T::load_xregs(xr, a.mean, a.factor, a.n, a.n, m0, n0);
        T::mainloop(lds, a.X, a.ld, a.X, a.ld, a.n, a.n, kbeg, kend, m0, n0, acc, true, &xr);
        return;
    }
    if constexpr (!T::SPLIT) {
        T::mainloop(lds, a.X, a.ld, FORM == kSymRows2 ? a.Z : a.X, a.ld, a.n, a.n, kbeg, kend, m0, n0, acc);
        if (FORM == kSymRows2) T::mainloop(lds, a.Z, a.ld, a.X, a.ld, a.n, a.n, kbeg, kend, m0, n0, acc);
    }
}

// Fused centring (T::XFORM) subtracts the column mean rounded to FP32,
// m = mean + d, so every centred value of a column is off by the same -d
// (times the FP32 factor f for correlation).  The values centred with the
// FP64 mean sum to zero over a column (up to that mean's rounding), so the
// reduced products over the N samples gain N f_a f_b d_a d_b, which is
// removed here before the epilogue: each value is again the contraction of
// the FP64-centred data, up to the FP32 rounding of its products and sums.  The term is relative to the
// result about 2^-48 (|mean_a| / sd_a)(|mean_b| / sd_b): negligible for
// means within a few thousand standard deviations, larger than the FP32
// tolerance beyond about 1e5.
template <class T>
__device__ __forceinline__ void fused_shift_correct_block(f32x16 &acc, int i, int j, const SymArgs &a, int64_t m0,
                                                          int64_t n0, int vtid = -1)
{
    if constexpr (T::XFORM != 0) {
        const int tid = vtid >= 0 ? vtid : (int)threadIdx.x;
        const int lane = tid & 63, wave = tid >> 6;
        const int wm0 = (wave / T::WN) * (T::BM / T::WM), wn0 = (wave % T::WN) * (T::BN / T::WN);
        const double rn = sqrt((double)a.kdim);
        // sqrt(N) f d of column c (0 outside the matrix, whose values are
        // never stored)
        auto shift = [&](int64_t c) -> double {
            if (c >= a.n) return 0.0;
            const double mu = a.mean[c];
            const double d = (double)(float)mu - mu;
            const double f = T::XFORM == 2 ? (double)(float)a.factor[c] : 1.0;
            return rn * f * d;
        };
        const double cb = shift(n0 + T::acc_col(wn0, j, lane));
#pragma unroll
        for (int v = 0; v < 16; ++v)
            acc[v] = (float)((double)acc[v] - shift(m0 + T::acc_row(wm0, i, v, lane)) * cb);
    }
}

template <class T>
__device__ __forceinline__ void fused_shift_correct(f32x16 (&acc)[T::TM][T::TN], const SymArgs &a,
                                                    int64_t m0, int64_t n0, int vtid = -1)
{
#pragma unroll
    for (int i = 0; i < T::TM; ++i)
#pragma unroll
        for (int j = 0; j < T::TN; ++j) fused_shift_correct_block<T>(acc[i][j], i, j, a, m0, n0, vtid);
}

// sqrt(N) f d of column c of the raw data (see fused_shift_correct_block), 0
// outside the matrix
template <class T>
__device__ __forceinline__ double fused_shift(const SymArgs &a, int64_t c)
{
    if (c >= a.n) return 0.0;
    const double mu = a.mean[c], d = (double)(float)mu - mu;
    return sqrt((double)a.kdim) * (T::XFORM == 2 ? (double)(float)a.factor[c] : 1.0) * d;
}

// The symmetric epilogue (epilogue_syrk's modes) from LDS: the block of the
// result at (r0, c0) with c0 >= r0, ROWS x COLS in t (leading dimension LD),
// written to both triangles by NTH threads; a block below the diagonal is
// its mirror's, and on the diagonal the upper triangle's values go to both.
// The direct and the mirrored copy are 16-byte stores of whole lines, each
// from a short loop (SplitTile::store_c says why).  shift: with T::XFORM the
// rows' and then the columns' shifts.
template <class T, int ROWS, int COLS, int LD, int NTH>
__device__ __forceinline__ void write_sym(const float *t, const double *shift, int tid, const SymArgs &a, int64_t r0,
                                          int64_t c0)
{
    if (r0 > c0) return;
    const bool diag = r0 == c0, reads = a.mode == 2 && a.beta != 0.f;
    auto value = [&](int r, int c) {
        float x = t[r * LD + c];
        if constexpr (T::XFORM != 0) x = (float)((double)x - shift[r] * shift[ROWS + c]);
        return x;
    };
    auto put = [&](int64_t row, int64_t col, f32x4 y) {
        float *p = a.S + row * a.n + col;
        const bool full = col + 3 < a.n;
        f32x4 o = {};
        if (reads) {
            if (full)
                o = *reinterpret_cast<const f32x4u *>(p);
            else
                for (int e = 0; e < 4; ++e)
                    if (col + e < a.n) o[e] = p[e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (a.mode == 1)
                y[e] = row == col + e ? 1.0f : y[e];
            else
                y[e] = reads ? T::combine(a.scale, y[e], a.beta, o[e]) : y[e] * a.scale;
        }
        if (full)
            *reinterpret_cast<f32x4u *>(p) = y;
        else
            for (int e = 0; e < 4; ++e)
                if (col + e < a.n) p[e] = y[e];
    };
#pragma unroll 2
    for (int x = tid; x < ROWS * COLS / 4; x += NTH) {
        const int r = x / (COLS / 4), c = x % (COLS / 4) * 4;
        if (r0 + r >= a.n || c0 + c >= a.n) continue;
        f32x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = diag && r > c + e ? value(c + e, r) : value(r, c + e);
        put(r0 + r, c0 + c, y);
    }
    if (diag) return;
#pragma unroll 2
    for (int x = tid; x < ROWS * COLS / 4; x += NTH) {
        const int c = x / (ROWS / 4), r = x % (ROWS / 4) * 4;
        if (c0 + c >= a.n || r0 + r >= a.n) continue;
        f32x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = value(r + e, c);
        put(c0 + c, r0 + r, y);
    }
}

// The finished accumulators of the tile at (m0, n0) to the result; reached by
// every thread of the work-group.
template <class T>
__device__ __forceinline__ void finish_sym(float *lds, f32x16 (&acc)[T::TM][T::TN], const SymArgs &a, int64_t m0,
                                           int64_t n0)
{
    if constexpr (T::SPLIT) {
        double *shift = reinterpret_cast<double *>(lds + (T::BM * T::OLD + 1) / 2 * 2);
        if (T::active()) T::stage_acc(lds, acc);
        if constexpr (T::XFORM != 0)
            for (int x = threadIdx.x; x < T::BM + T::BN; x += T::NT)
                shift[x] = fused_shift<T>(a, x < T::BM ? m0 + x : n0 + x - T::BM);
        __syncthreads();
        write_sym<T, T::BM, T::BN, T::OLD, T::NT>(lds, shift, threadIdx.x, a, m0, n0);
        __syncthreads();  // (the next tile's stages reuse the LDS)
    } else {
        fused_shift_correct<T>(acc, a, m0, n0);
        epilogue_syrk<T>(acc, a.S, a.n, m0, n0, a.mode, a.scale, a.beta);
    }
}

// One 32 x 32 block per wave of a reduce kernel: the summed accumulators acc
// of block (i, j) of the tile at (m0, n0), tile thread vtid.
template <class T>
__device__ __forceinline__ void finish_sym_block(f32x16 &acc, int i, int j, int vtid, const SymArgs &a,
                                                 int64_t m0, int64_t n0)
{
    fused_shift_correct_block<T>(acc, i, j, a, m0, n0, vtid);
    const f32x16 block[1][1] = {{acc}};
    epilogue_syrk<T>(block, a.S, a.n, m0, n0, a.mode, a.scale, a.beta, vtid, i, j);
}

// Raw accumulators of one tile as a partial result: BM * BN floats, laid out
// chunk-major ([chunk][thread] float4s, chunk = 4 consecutive registers), so
// one store or load instruction of a wave touches 1 KiB contiguously.
template <class T>
__device__ __forceinline__ void store_partial(const f32x16 (&acc)[T::TM][T::TN], float *dst, int tid)
{
    f32x4 *d = reinterpret_cast<f32x4 *>(dst);
#pragma unroll
    for (int i = 0; i < T::TM; ++i)
#pragma unroll
        for (int j = 0; j < T::TN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                d[((i * T::TN + j) * 4 + q) * T::ET + tid] =
                    f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
}

// one 32 x 32 block of a partial result added to acc
template <class T>
__device__ __forceinline__ void add_partial_block(f32x16 &acc, int i, int j, const float *src, int tid)
{
    const f32x4 *p = reinterpret_cast<const f32x4 *>(src);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4 x = p[((i * T::TN + j) * 4 + q) * T::ET + tid];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[4 * q + e] += x[e];
    }
}

template <class T>
__device__ __forceinline__ void add_partial(f32x16 (&acc)[T::TM][T::TN], const float *src, int tid)
{
#pragma unroll
    for (int i = 0; i < T::TM; ++i)
#pragma unroll
        for (int j = 0; j < T::TN; ++j) add_partial_block<T>(acc[i][j], i, j, src, tid);
}

template <class T, int FORM>
__global__ __launch_bounds__(T::NT) void sym_kernel(SymArgs a, int tiles)
{
    static_assert(T::BM == T::BN, "symmetric contraction needs square tiles");
    __shared__ __attribute__((aligned(16))) float lds[T::LDS_FLOATS];
    const int nb = tiles * (tiles + 1) / 2;
    const int t = xcd_remap(blockIdx.x, nb);
    int tm, tn;
    upper_tile(t, tiles, tm, tn);
    const int64_t m0 = (int64_t)tm * T::BM, n0 = (int64_t)tn * T::BN;
    f32x16 acc[T::TM][T::TN];
    T::zero(acc);
    if (a.reads) sym_reduce<T, FORM>(lds, a, 0, a.kdim, m0, n0, acc);
    finish_sym<T>(lds, acc, a, m0, n0);
}

// Split reduction: work-group w computes the partial sum of tile (w mod
// tiles) over the w-th chunk of the reduction and stores its raw
// accumulators (each thread its own registers, contiguous); the reduce
// kernel adds the chunks of a tile in chunk order (deterministic) and runs
// the usual epilogue.  Consecutive work-groups take neighbouring tiles of
// one chunk, so an XCD's L2 holds the operand panels they share.
template <class T, int FORM>
__global__ __launch_bounds__(T::NT) void sym_split_kernel(SymArgs a, float *__restrict__ part,
                                                          int tiles, int splits, int64_t kchunk)
{
    __shared__ __attribute__((aligned(16))) float lds[T::LDS_FLOATS];
    const int nb = tiles * (tiles + 1) / 2;
    const int w = xcd_remap(blockIdx.x, nb * splits);
    const int t = w % nb, sidx = w / nb;
    int tm, tn;
    upper_tile(t, tiles, tm, tn);
    const int64_t m0 = (int64_t)tm * T::BM, n0 = (int64_t)tn * T::BN;
    const int64_t kbeg = (int64_t)sidx * kchunk;
    const int64_t kend = kbeg + kchunk < a.kdim ? kbeg + kchunk : a.kdim;
    f32x16 acc[T::TM][T::TN];
    T::zero(acc);
    sym_reduce<T, FORM>(lds, a, kbeg, kend, m0, n0, acc);
    if (!T::active()) return;
    store_partial<T>(acc, part + (int64_t)(sidx * nb + t) * T::BM * T::BN, threadIdx.x);
}

// Reduce kernels: 256-thread work-groups, kReduceSlices of them per tile,
// each taking one 32 x 32 block of the accumulators of 256 of the tile's
// threads (so a 128 x 128 tile is reduced by four work-groups whatever its
// waves, and the additions of a tile with many partials run side by side).
constexpr int kReduceThreads = 256;

template <class T>
constexpr int reduce_slices()
{
    return T::ET / kReduceThreads * T::TM * T::TN;
}

// the tile thread and the block of this work-group
template <class T>
__device__ __forceinline__ void reduce_slice(int &t, int &vtid, int &i, int &j)
{
    constexpr int S = reduce_slices<T>(), B = T::TM * T::TN;
    t = blockIdx.x / S;
    const int s = blockIdx.x % S;
    vtid = (s / B) * kReduceThreads + threadIdx.x;
    i = s % B / T::TN;
    j = s % B % T::TN;
}

template <class T>
__global__ __launch_bounds__(kReduceThreads) void sym_split_reduce_kernel(SymArgs a,
                                                                          const float *__restrict__ part,
                                                                          int tiles, int splits)
{
    static_assert(T::ET % kReduceThreads == 0, "tile threads must split into reduce slices");
    const int nb = tiles * (tiles + 1) / 2;
    int t, vtid, i, j, tm, tn;
    reduce_slice<T>(t, vtid, i, j);
    upper_tile(t, tiles, tm, tn);
    f32x16 acc = {};
    for (int s = 0; s < splits; ++s)
        add_partial_block<T>(acc, i, j, part + (int64_t)(s * nb + t) * T::BM * T::BN, vtid);
    const int64_t m0 = (int64_t)tm * T::BM, n0 = (int64_t)tn * T::BN;
    finish_sym_block<T>(acc, i, j, vtid, a, m0, n0);
}

// ------------------------------------------------------------ stream-K
// The nb upper tiles times kt K-tiles form one iteration space; work-group
// g of G takes iterations [g total / G, (g + 1) total / G), so every
// work-group does the same amount of reduction whatever nb is (the split
// above quantises nb * splits work-groups onto the compute units).  A range
// covers whole tiles (written directly) and at most two tile pieces: its
// first segment (partial slot 0) and its last (slot 1).  The fixup kernel
// adds the pieces of every shared tile in work-group order (deterministic)
// and runs the epilogue.
constexpr int kStreamMaxGroups = 512;

__host__ __device__ __forceinline__ int64_t sk_begin(int64_t g, int64_t total, int G)
{
    return g * total / G;
}

// the work-group whose range contains iteration i
__device__ __forceinline__ int sk_owner(int64_t i, int64_t total, int G)
{
    return (int)(((i + 1) * G + total - 1) / total - 1);
}

template <class T, int FORM>
__global__ __launch_bounds__(T::NT) void sym_streamk_kernel(SymArgs a, float *__restrict__ part,
                                                            int tiles, int kt)
{
    __shared__ __attribute__((aligned(16))) float lds[T::LDS_FLOATS];
    const int nb = tiles * (tiles + 1) / 2;
    // (neighbouring ranges, which share panels, on one XCD)
    const int G = gridDim.x;
    const int g = xcd_remap(blockIdx.x, G);
    const int64_t total = (int64_t)nb * kt;
    const int64_t beg = sk_begin(g, total, G), end = sk_begin(g + 1, total, G);
    for (int64_t it = beg; it < end;) {
        const int t = (int)(it / kt);
        const int64_t tile_end = (int64_t)(t + 1) * kt;
        const int64_t stop = end < tile_end ? end : tile_end;
        const bool first = it == beg;
        const int64_t k0 = it - (int64_t)t * kt, k1 = stop - (int64_t)t * kt;
        int tm, tn;
        upper_tile(t, tiles, tm, tn);
        const int64_t m0 = (int64_t)tm * T::BM, n0 = (int64_t)tn * T::BN;
        const int64_t kend = k1 * T::BK < a.kdim ? k1 * T::BK : a.kdim;
        f32x16 acc[T::TM][T::TN];
        T::zero(acc);
        sym_reduce<T, FORM>(lds, a, k0 * T::BK, kend, m0, n0, acc);
        it = stop;
        if (k0 == 0 && k1 == kt)
            finish_sym<T>(lds, acc, a, m0, n0);
        else
            store_partial<T>(acc, part + ((int64_t)g * 2 + (first ? 0 : 1)) * T::BM * T::BN, threadIdx.x);
    }
}

template <class T>
__global__ __launch_bounds__(kReduceThreads) void sym_streamk_fixup_kernel(SymArgs a,
                                                                           const float *__restrict__ part,
                                                                           int tiles, int kt, int G)
{
    const int nb = tiles * (tiles + 1) / 2;
    int t, vtid, i, j, tm, tn;
    reduce_slice<T>(t, vtid, i, j);
    const int64_t total = (int64_t)nb * kt;
    const int g0 = sk_owner((int64_t)t * kt, total, G), g1 = sk_owner((int64_t)(t + 1) * kt - 1, total, G);
    if (g0 == g1) return;  // one work-group reduced the whole tile
    upper_tile(t, tiles, tm, tn);
    f32x16 acc = {};
    // the tile is g0's second segment if g0 started in an earlier tile, and
    // every other group's first; four pieces in flight, added in group order
    const bool late = sk_begin(g0, total, G) < (int64_t)t * kt;
    add_partial_block<T>(acc, i, j, part + ((int64_t)g0 * 2 + (late ? 1 : 0)) * T::BM * T::BN, vtid);
#pragma unroll 4
    for (int g = g0 + 1; g <= g1; ++g) add_partial_block<T>(acc, i, j, part + (int64_t)g * 2 * T::BM * T::BN, vtid);
    const int64_t m0 = (int64_t)tm * T::BM, n0 = (int64_t)tn * T::BN;
    finish_sym_block<T>(acc, i, j, vtid, a, m0, n0);
}

// ------------------------------------------------------------ phases
// The schedule of the split tiles where one work-group per upper tile would
// leave compute units idle.  A phase cuts the reduction of `ntiles` tiles
// into `chunks` equal parts, one work-group each; a plan is up to three
// phases, launched as one grid in their order: whole tiles as long as they
// fill the W work-groups that run at one time, then p chunks of as many
// tiles as fit them, then the last tiles in more chunks.  136 tiles on 256
// compute units: 128 tiles in two chunks, 8 tiles in 32 chunks, 64 + 4 of 128
// K-tiles, the 68 of an even division.  Unlike stream-K's ranges, the units
// that run at one time are at the same k: units are numbered chunk by chunk,
// an XCD takes neighbouring ones, and so reads each operand panel's K-tile
// once into its L2 (covariance 2048 x 4096: stream-K 4.7 million L2 misses a
// call, 78% of the requests; phases 1.7 million, the kernel 106 us).  A work-group is one unit: a grid of W
// that loops over its units kept their addresses in registers across the
// loop and spilled (125 us).  Pieces (partial tiles) lie unit by unit; the
// reduce kernel adds a tile's in a fixed order (deterministic).
struct SymPhase {
    int tile0, ntiles, chunks, piece0;  // piece0: number of the phase's first piece
};
struct SymPlan {
    SymPhase ph[3];
    int n, units, split0, pieces;  // split0: first tile that is cut
};

// 32 x 32 blocks of a tile
template <class T>
constexpr int phase_blocks()
{
    return T::BM / 32 * (T::BN / 32);
}

template <class T, int FORM>
__global__ __launch_bounds__(T::NT) void sym_phase_kernel(SymArgs a, float *__restrict__ part, int tiles, int kt,
                                                          SymPlan plan)
{
    __shared__ __attribute__((aligned(16))) float lds[T::LDS_FLOATS];
    int b = blockIdx.x, f = 0;
    while (b >= plan.ph[f].ntiles * plan.ph[f].chunks) {
        b -= plan.ph[f].ntiles * plan.ph[f].chunks;
        ++f;
    }
    const SymPhase ph = plan.ph[f];
    const int u = xcd_remap(b, ph.ntiles * ph.chunks);
    const int c = u / ph.ntiles, t = ph.tile0 + u % ph.ntiles;
    int tm, tn;
    upper_tile(t, tiles, tm, tn);
    const int64_t m0 = (int64_t)tm * T::BM, n0 = (int64_t)tn * T::BN;
    const int64_t k0 = (int64_t)kt * c / ph.chunks * T::BK, k1 = (int64_t)kt * (c + 1) / ph.chunks * T::BK;
    f32x16 acc[T::TM][T::TN];
    T::zero(acc);
    sym_reduce<T, FORM>(lds, a, k0, k1 < a.kdim ? k1 : a.kdim, m0, n0, acc);
    if (ph.chunks == 1) {
        finish_sym<T>(lds, acc, a, m0, n0);
    } else if (T::active()) {
        store_partial<T>(acc, part + (int64_t)(ph.piece0 + u) * T::BM * T::BN, threadIdx.x);
    }
}

// The sum of the pieces of cut tile t over one of its 32 x 32 blocks, in LDS
// (sum[0], [32][33]), by a work-group of kReduceThreads: each wave sums every
// fourth chunk, the four sums meet in LDS (a fixed order).  Bound by reading
// the pieces; with one wave per block, all its chunks in turn, too few loads
// were in flight (correlation 501 x 20011, 25 chunks of 10 tiles: 17.9 us,
// now 6.2; covariance 2048 x 4096: 13.0, now 10.9).
constexpr int kPhaseLd = 33;
template <class T>
__device__ __forceinline__ void phase_sum(float (&sum)[kReduceThreads / 64][32 * kPhaseLd],
                                          const float *__restrict__ part, const SymPlan &plan, int t, int s)
{
    constexpr int B = T::TM * T::TN, W = kReduceThreads / 64;
    const int w = s / B, i = s % B / T::TN, j = s % T::TN;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm0 = (w / T::WN) * (T::BM / T::WM), wn0 = (w % T::WN) * (T::BN / T::WN);
    SymPhase ph = plan.ph[plan.n - 1];
    if (t < ph.tile0) ph = plan.ph[plan.n - 2];
    f32x16 acc = {};
    const float *p = part + (int64_t)(ph.piece0 + t - ph.tile0) * T::BM * T::BN;
#pragma unroll 4
    for (int c = wave; c < ph.chunks; c += W)
        add_partial_block<T>(acc, i, j, p + (int64_t)c * ph.ntiles * T::BM * T::BN, w * 64 + lane);
#pragma unroll
    for (int v = 0; v < 16; ++v)
        sum[wave][(T::acc_row(wm0, i, v, lane) - wm0 - 32 * i) * kPhaseLd + T::acc_col(wn0, j, lane) - wn0 - 32 * j] =
            acc[v];
    __syncthreads();
    for (int x = threadIdx.x; x < 32 * kPhaseLd; x += kReduceThreads) {
        float y = sum[0][x];
#pragma unroll
        for (int q = 1; q < W; ++q) y += sum[q][x];
        sum[0][x] = y;
    }
    __syncthreads();
}

// first row and column of block s of a tile of type T
template <class T>
__device__ __forceinline__ void phase_block(int s, int &br, int &bc)
{
    constexpr int B = T::TM * T::TN;
    const int w = s / B;
    br = (w / T::WN) * (T::BM / T::WM) + s % B / T::TN * 32;
    bc = (w % T::WN) * (T::BN / T::WN) + s % T::TN * 32;
}

template <class T>
__global__ __launch_bounds__(kReduceThreads) void sym_phase_reduce_kernel(SymArgs a, const float *__restrict__ part,
                                                                          int tiles, SymPlan plan)
{
    constexpr int S = phase_blocks<T>();
    __shared__ __attribute__((aligned(16))) float sum[kReduceThreads / 64][32 * kPhaseLd];
    __shared__ double shift[64];
    const int t = plan.split0 + blockIdx.x / S, s = blockIdx.x % S;
    int tm, tn, br, bc;
    upper_tile(t, tiles, tm, tn);
    phase_block<T>(s, br, bc);
    const int64_t r0 = (int64_t)tm * T::BM + br, c0 = (int64_t)tn * T::BN + bc;
    if (r0 > c0 || c0 >= a.n) return;  // (below the diagonal: the mirrored block's)
    if constexpr (T::XFORM != 0) {
        const int l = threadIdx.x;
        if (l < 64) shift[l] = fused_shift<T>(a, l < 32 ? r0 + l : c0 + l - 32);
    }
    phase_sum<T>(sum, part, plan, t, s);
    write_sym<T, 32, 32, kPhaseLd, kReduceThreads>(sum[0], shift, threadIdx.x, a, r0, c0);
}

// The plan for nb tiles of kt K-tiles on W work-groups.  Predicted time: a
// K-tile of a busy compute unit takes `us`, every cut phase another `fill`
// (its pipeline's start and its pieces' stores), the reduce kernel 4 us and
// `piece` per piece.  Chunks are at least eight K-tiles long: shorter ones
// only add pieces (one 64 x 64 tile, 11776 samples: 256 chunks 0.21 ms, 46
// chunks 0.035 ms).
inline SymPlan sym_plan(int64_t nb, int64_t kt, int64_t W, double us, double fill, double piece,
                        double *predicted = nullptr)
{
    SymPlan best{};
    double tbest = 0;
    const int64_t whole = nb / W * W, rest = nb - whole, most = kt / 8 > 1 ? kt / 8 : 1;
    for (int64_t q = 0; q < 4; ++q) {
        // q == 0: the rest whole as well; else W / rest + q - 1 chunks
        int64_t p = q == 0 ? 1 : W / (rest > 0 ? rest : 1) + q - 1;
        if (q > 0 && (rest == 0 || p < 2)) continue;
        if (p > most) p = most;
        const int64_t na = p * rest <= W ? rest : W / p, nl = rest - na;
        int64_t pl = nl > 0 ? W / nl : 0;
        if (pl > most) pl = most;
        SymPlan s{};
        double t = (double)(whole / W) * kt * us;
        auto add = [&](int64_t tile0, int64_t ntiles, int64_t chunks) {
            if (ntiles == 0) return;
            const bool cut = chunks > 1;
            s.ph[s.n++] = SymPhase{(int)tile0, (int)ntiles, (int)chunks, s.pieces};
            if (cut) s.pieces += (int)(ntiles * chunks);
            t += (double)((kt + chunks - 1) / chunks) * us + (cut ? fill : 0.0);
        };
        if (whole > 0) {
            s.ph[s.n++] = SymPhase{0, (int)whole, 1, 0};
        }
        if (p == 1) {
            add(whole, rest, 1);
            s.split0 = (int)nb;
        } else {
            add(whole, na, p);
            if (nl > 0 && pl < 2) continue;
            add(whole + na, nl, pl);
            s.split0 = (int)whole;
        }
        if (s.pieces > 0) t += 4.0 + s.pieces * piece;
        if (best.n == 0 || t < tbest) {
            best = s;
            tbest = t;
        }
    }
    for (int f = 0; f < best.n; ++f) best.units += best.ph[f].ntiles * best.ph[f].chunks;
    if (predicted) *predicted = tbest;
    return best;
}

// Work-groups of tile type T that run at one time (a plan has at most two
// pieces for each).  The 64 x 64 tile gains 13% from a second work-group on a
// compute unit where the chunks are long.
template <class T>
SymPlan sym_plan_for(int64_t nb, int64_t kt, int passes, double *predicted = nullptr)
{
    const int64_t cus = device_cu_count();
    const bool big = T::BM >= 128;
    const int64_t W = !big && nb * kt >= cus * 2 * 32 ? 2 * cus : cus;
    return sym_plan(nb, kt, W < kStreamMaxGroups ? W : kStreamMaxGroups, (big ? 1.05 : W > cus ? 0.84 : 0.45) * passes,
                    big ? 4.0 : 2.0, big ? 0.02 : 0.005, predicted);
}

// Bytes of split-K partials a candidate list may need for order n.
// (split_k == 0 marks stream-K and the phases: two pieces per work-group)
#define LI_SYM_SPLIT_BYTES(IDX, BM, BN, BK, WM, WN, SK, PF)                                        \
    if (SK > 1) {                                                                                \
        const int64_t t = (n + BM - 1) / BM;                                                     \
        const size_t b = (size_t)SK * (size_t)(t * (t + 1) / 2) * BM * BN * sizeof(float);       \
        if (b > best) best = b;                                                                  \
    } else if (SK == 0) {                                                                        \
        const size_t b = (size_t)2 * kStreamMaxGroups * BM * BN * sizeof(float);                 \
        if (b > best) best = b;                                                                  \
    }

// Enqueue one symmetric contraction with tile type T.  splits > 1 (split
// reduction) and splits == 0 (stream-K over `groups` work-groups) need the
// partial workspace `ws`.
template <class T, int FORM>
int run_sym(const SymArgs &a, int splits, float *ws, hipStream_t s)
{
    const int tiles = (int)((a.n + T::BM - 1) / T::BM);
    const int nb = tiles * (tiles + 1) / 2;
    const bool whole = splits == 1 || !a.reads || a.kdim == 0;
    if (whole || T::ET % kReduceThreads != 0) {
        // (work-groups smaller than one reduce slice: one kernel, no split)
        if (!whole) return (int)hipErrorInvalidValue;
        hipLaunchKernelGGL((sym_kernel<T, FORM>), dim3(nb), dim3(T::NT), 0, s, a, tiles);
        return (int)hipGetLastError();
    }
    const int kt = (int)((a.kdim + T::BK - 1) / T::BK);
    if constexpr (T::ET % kReduceThreads == 0 && T::SPLIT) {
        SymPlan plan{};
        if (splits == 0) {
            plan = sym_plan_for<T>(nb, kt, FORM == kSymRows2 ? 2 : 1);
        } else {
            plan.ph[0] = SymPhase{0, nb, splits, 0};
            plan.n = 1;
            plan.units = plan.pieces = nb * splits;
        }
        if (plan.pieces > 0 && !ws) return (int)hipErrorInvalidValue;
        hipLaunchKernelGGL((sym_phase_kernel<T, FORM>), dim3((unsigned)plan.units), dim3(T::NT), 0, s, a, ws, tiles,
                           kt, plan);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess || plan.pieces == 0) return (int)e;
        hipLaunchKernelGGL(sym_phase_reduce_kernel<T>, dim3((unsigned)((nb - plan.split0) * phase_blocks<T>())),
                           dim3(kReduceThreads), 0, s, a, (const float *)ws, tiles, plan);
        return (int)hipGetLastError();
    } else if constexpr (T::ET % kReduceThreads == 0) {
        if (!ws) return (int)hipErrorInvalidValue;
        if (splits == 0) {
            // stream-K work-groups: as many as are resident at once
            const int64_t total = (int64_t)nb * kt;
            const int groups = device_cu_count() * T::SK_PER_CU;
            int G = groups < kStreamMaxGroups ? groups : kStreamMaxGroups;
            if (G > total) G = (int)total;
            if (G < 1) G = 1;
            hipLaunchKernelGGL((sym_streamk_kernel<T, FORM>), dim3(G), dim3(T::NT), 0, s, a, ws, tiles, kt);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return (int)e;
            hipLaunchKernelGGL(sym_streamk_fixup_kernel<T>, dim3(nb * reduce_slices<T>()), dim3(kReduceThreads), 0, s,
                               a, (const float *)ws, tiles, kt, G);
            return (int)hipGetLastError();
        }
        int64_t kchunk = (a.kdim + splits - 1) / splits;
        kchunk = (kchunk + T::BK - 1) / T::BK * T::BK;
        hipLaunchKernelGGL((sym_split_kernel<T, FORM>), dim3(nb * splits), dim3(T::NT), 0, s, a, ws, tiles, splits,
                           kchunk);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return (int)e;
        hipLaunchKernelGGL(sym_split_reduce_kernel<T>, dim3(nb * reduce_slices<T>()), dim3(kReduceThreads), 0, s, a,
                           (const float *)ws, tiles, splits);
        return (int)hipGetLastError();
    }
}

// One candidate of the symmetric lists.  The direct-to-LDS loop (PF 4) needs
// 16-byte rows (v4) and, where its caller says so (whole), whole K-tiles;
// otherwise mode ALT of the register path takes vector loads, and mode 2 or
// ALT scalar ones.  Modes 9 to 11 are the split tiles, which take every shape
// with rows of up to kSplitMaxLd elements.
template <int BM, int BN, int BK, int WM, int WN, int PF, int ALT, bool COLS, int XF, int FORM>
int run_sym_candidate(const SymArgs &a, bool v4, bool whole, int splits, float *ws, hipStream_t s)
{
    if constexpr (PF >= 9) {
        if (a.ld > kSplitMaxLd) return (int)hipErrorInvalidValue;
        return run_sym<SplitTile<BM, BN, BK, WM, WN, split_waves(PF), true, COLS, !COLS, XF>, FORM>(a, splits, ws, s);
    } else {
        constexpr int SCALAR = ALT == 4 ? 2 : ALT;
        if (!v4) return run_sym<F32Tile<BM, BN, BK, WM, WN, COLS, kLoadScalar, SCALAR, !COLS, XF>, FORM>(a, splits, ws, s);
        return whole ? run_sym<F32Tile<BM, BN, BK, WM, WN, COLS, kLoadVec4, PF, !COLS, XF>, FORM>(a, splits, ws, s)
                     : run_sym<F32Tile<BM, BN, BK, WM, WN, COLS, kLoadVec4, ALT, !COLS, XF>, FORM>(a, splits, ws, s);
    }
}

}  // namespace li
