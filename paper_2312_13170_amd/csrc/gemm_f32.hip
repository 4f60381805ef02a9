// FP32 GEMM and the column-form symmetric contraction (matrix cores,
// loop-internalised reduction; see split_tile.h and f32_tile.h for the tiling
// and symm_kernels.h for the symmetric kernels and the phases).
#include <hip/hip_runtime.h>

#include "f32_tile.h"
#include "li_internal.h"
#include "split_tile.h"
#include "symm_kernels.h"
#include "tiles.h"

namespace li {
namespace {

// ---------------------------------------------------------------- GEMM
// C = alpha*A*B + beta*C, A M x K, B K x N, C M x N, row-major.
// tile rows of a band in which work-groups walk the tiles (grouped_tile)
constexpr int kGroupM = 8;

template <class T>
__global__ __launch_bounds__(T::NT) void gemm_f32_kernel(const float *__restrict__ A, int64_t lda,
                                                         const float *__restrict__ B, int64_t ldb,
                                                         float *__restrict__ C, int64_t ldc,
                                                         int64_t M, int64_t N, int64_t K,
                                                         float alpha, float beta, int tiles_m,
                                                         int tiles_n, int group_m)
{
    __shared__ __attribute__((aligned(16))) float lds[T::LDS_FLOATS];
    const int nb = tiles_m * tiles_n;
    const int t = xcd_remap(blockIdx.x, nb);
    int tm, tn;
    grouped_tile(t, tiles_m, tiles_n, group_m, tm, tn);
    const int64_t m0 = (int64_t)tm * T::BM, n0 = (int64_t)tn * T::BN;
    f32x16 acc[T::TM][T::TN];
    T::zero(acc);
    if constexpr (T::SPLIT) {
        const auto warm = T::warm_c(C, ldc, M, N, m0, n0, beta);
        if (alpha != 0.f) T::mainloop(lds, A, lda, B, ldb, M, N, 0, K, m0, n0, acc);
        warm.touch();
    } else {
        if (alpha != 0.f) T::mainloop(lds, A, lda, B, ldb, M, N, 0, K, m0, n0, acc);
    }
    T::store_c(lds, acc, C, ldc, M, N, m0, n0, alpha, beta);
}

template <class T>
int run_gemm(int64_t M, int64_t N, int64_t K, float alpha, const float *A, int64_t lda,
             const float *B, int64_t ldb, float beta, float *C, int64_t ldc, hipStream_t s)
{
    const int tiles_m = (int)((M + T::BM - 1) / T::BM);
    const int tiles_n = (int)((N + T::BN - 1) / T::BN);
    const int nb = tiles_m * tiles_n;
    hipLaunchKernelGGL(gemm_f32_kernel<T>, dim3(nb), dim3(T::NT), 0, s, A, lda, B, ldb, C, ldc, M,
                       N, K, alpha, beta, tiles_m, tiles_n, kGroupM);
    return (int)hipGetLastError();
}

// a candidate of the FP32 cores that takes every shape
constexpr int kGemmF32Plain = 18;

inline bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

// One candidate of the list.  Prefetch modes 5-7 are modes 1-3 with B
// transposed into LDS; the direct-to-LDS modes (4: three-stage ring, 8:
// two-stage ring) need 16-byte rows and fall back to mode 2 otherwise; mode 8
// runs as mode 4 (which takes a ragged last K-tile; mode 2 where three stages
// do not fit in LDS) when K is not a multiple of the K-tile.  Modes 9 to 11
// are the split tiles; rows too long for their 32-bit offsets take the FP32
// cores.
template <int BM, int BN, int BK, int WM, int WN, int PF>
int run_gemm_candidate(bool v4, int64_t M, int64_t N, int64_t K, float alpha, const float *A, int64_t lda,
                       const float *B, int64_t ldb, float beta, float *C, int64_t ldc, hipStream_t s)
{
#define LI_RUN(LOAD, MODE, TR) \
    run_gemm<F32Tile<BM, BN, BK, WM, WN, false, LOAD, MODE, false, 0, TR>>(M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, s)
    if constexpr (PF >= 9) {
        using T = SplitTile<BM, BN, BK, WM, WN, split_waves(PF), true, false, false>;
        if (lda > kSplitMaxLd || ldb > kSplitMaxLd)
            return launch_gemm_f32(kGemmF32Plain, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, s);
        return run_gemm<T>(M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, s);
    } else {
        constexpr bool TR = PF > 4 && PF < 8;
        constexpr int MODE = TR ? PF - 4 : PF;
        // the three-stage ring when it fits in LDS, else the register path
        constexpr int RAGGED = PF == 8 ? ((BM + BN) * BK * 4 * 3 <= 160 * 1024 ? 4 : 2) : MODE;
        if (!v4) return LI_RUN(kLoadScalar, (PF == 4 || PF == 8 ? 2 : MODE), TR);
        return PF != 8 || K % BK == 0 ? LI_RUN(kLoadVec4, MODE, TR) : LI_RUN(kLoadVec4, RAGGED, TR);
    }
#undef LI_RUN
}

// ------------------------------------------------------------ phased GEMM
// The split tiles in the phases of the symmetric contractions
// (symm_kernels.h): whole tiles as long as they fill the compute units, the
// rest cut along K into pieces that the reduce kernel adds.
template <class T>
__global__ __launch_bounds__(T::NT) void gemm_phase_kernel(const float *__restrict__ A, const float *__restrict__ B,
                                                           float *__restrict__ C, int64_t M, int64_t N, int64_t K,
                                                           float alpha, float beta, int tiles_m, int tiles_n, int kt,
                                                           SymPlan plan, float *__restrict__ part)
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
    grouped_tile(t, tiles_m, tiles_n, kGroupM, tm, tn);
    const int64_t m0 = (int64_t)tm * T::BM, n0 = (int64_t)tn * T::BN;
    const int64_t k0 = (int64_t)kt * c / ph.chunks * T::BK, k1 = (int64_t)kt * (c + 1) / ph.chunks * T::BK;
    f32x16 acc[T::TM][T::TN];
    T::zero(acc);
    T::mainloop(lds, A, K, B, N, M, N, k0, k1 < K ? k1 : K, m0, n0, acc);
    if (ph.chunks == 1) {
        T::store_c(lds, acc, C, N, M, N, m0, n0, alpha, beta);
    } else if (T::active()) {
        store_partial<T>(acc, part + (int64_t)(ph.piece0 + u) * T::BM * T::BN, threadIdx.x);
    }
}

template <class T>
__global__ __launch_bounds__(kReduceThreads) void gemm_phase_reduce_kernel(float *__restrict__ C, int64_t M, int64_t N,
                                                                           float alpha, float beta, int tiles_m,
                                                                           int tiles_n, SymPlan plan,
                                                                           const float *__restrict__ part)
{
    constexpr int S = phase_blocks<T>();
    __shared__ __attribute__((aligned(16))) float sum[kReduceThreads / 64][32 * kPhaseLd];
    const int t = plan.split0 + blockIdx.x / S, s = blockIdx.x % S;
    int tm, tn, br, bc;
    grouped_tile(t, tiles_m, tiles_n, kGroupM, tm, tn);
    phase_block<T>(s, br, bc);
    const int64_t r0 = (int64_t)tm * T::BM + br, c0 = (int64_t)tn * T::BN + bc;
    if (r0 >= M || c0 >= N) return;
    const int r = threadIdx.x / 8, c = threadIdx.x % 8 * 4;
    float *p = C + (r0 + r) * N + c0 + c;
    const int n = r0 + r >= M ? 0 : N - c0 - c < 4 ? (int)(N - c0 - c) : 4;  // elements of this thread
    float old[4] = {};
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (e < n && beta != 0.f) old[e] = p[e];
    phase_sum<T>(sum, part, plan, t, s);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float x = sum[0][r * kPhaseLd + c + e];
        if (e < n) p[e] = beta != 0.f ? T::combine(alpha, x, beta, old[e]) : alpha * x;
    }
}

template <class T>
SymPlan gemm_phase_plan(int64_t M, int64_t N, int64_t K, double *predicted = nullptr)
{
    return sym_plan_for<T>((M + T::BM - 1) / T::BM * ((N + T::BN - 1) / T::BN), (K + T::BK - 1) / T::BK, 1, predicted);
}

template <class T>
double phase_us(int64_t M, int64_t N, int64_t K)
{
    double us = 0.0;
    gemm_phase_plan<T>(M, N, K, &us);
    return us;
}

template <class T>
int run_gemm_phases(int64_t M, int64_t N, int64_t K, float alpha, const float *A, const float *B, float beta, float *C,
                    float *ws, hipStream_t s)
{
    const int tiles_m = (int)((M + T::BM - 1) / T::BM), tiles_n = (int)((N + T::BN - 1) / T::BN);
    const int nb = tiles_m * tiles_n, kt = (int)((K + T::BK - 1) / T::BK);
    const SymPlan plan = gemm_phase_plan<T>(M, N, K);
    hipLaunchKernelGGL(gemm_phase_kernel<T>, dim3((unsigned)plan.units), dim3(T::NT), 0, s, A, B, C, M, N, K, alpha,
                       beta, tiles_m, tiles_n, kt, plan, ws);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || plan.pieces == 0) return (int)e;
    hipLaunchKernelGGL(gemm_phase_reduce_kernel<T>, dim3((unsigned)((nb - plan.split0) * phase_blocks<T>())),
                       dim3(kReduceThreads), 0, s, C, M, N, alpha, beta, tiles_m, tiles_n, plan, (const float *)ws);
    return (int)hipGetLastError();
}

using PhaseTile128 = SplitTile<128, 128, 32, 2, 2, 4, true, false, false>;
using PhaseTile64 = SplitTile<64, 64, 32, 2, 2, 4, true, false, false>;

// ---------------------------------------------------------- stream-K GEMM
// (for rows too long for the split tiles' offsets, on the FP32 cores)
// The nb output tiles times kt K-tiles form one iteration space split
// evenly over the G work-groups (the schedule of the symmetric
// contractions, symm_kernels.h): a range covers whole tiles, stored with
// alpha and beta at once, and at most two tile pieces, stored raw in the
// workspace; the fixup adds the pieces of every shared tile in work-group
// order (deterministic) and applies alpha and beta.  The work per
// work-group is the same whatever the tile count, so shapes whose tiles
// leave compute units idle (few tiles and a long K, or a last wave of tiles
// that fills few of them) keep every unit busy.
template <class T>
__global__ __launch_bounds__(T::NT) void gemm_streamk_kernel(const float *__restrict__ A, int64_t lda,
                                                             const float *__restrict__ B, int64_t ldb,
                                                             float *__restrict__ C, int64_t ldc,
                                                             int64_t M, int64_t N, int64_t K, float alpha,
                                                             float beta, int tiles_n, int nb, int kt,
                                                             float *__restrict__ part)
{
    __shared__ __attribute__((aligned(16))) float lds[T::LDS_FLOATS];
    const int G = gridDim.x, g = blockIdx.x;
    const int64_t total = (int64_t)nb * kt;
    const int64_t beg = sk_begin(g, total, G), end = sk_begin(g + 1, total, G);
    for (int64_t it = beg; it < end;) {
        const int t = (int)(it / kt);
        const int64_t tile_end = (int64_t)(t + 1) * kt;
        const int64_t stop = end < tile_end ? end : tile_end;
        const int64_t k0 = it - (int64_t)t * kt, k1 = stop - (int64_t)t * kt;
        const int64_t m0 = (int64_t)(t / tiles_n) * T::BM, n0 = (int64_t)(t % tiles_n) * T::BN;
        const int64_t kend = k1 * T::BK < K ? k1 * T::BK : K;
        f32x16 acc[T::TM][T::TN];
        T::zero(acc);
        T::mainloop(lds, A, lda, B, ldb, M, N, k0 * T::BK, kend, m0, n0, acc);
        if (k0 == 0 && k1 == kt) {
            if (beta != 0.f) {
                float cv[T::TM][T::TN][16];
                T::load_c(cv, C, ldc, M, N, m0, n0);
                T::epilogue_gemm_loaded(acc, cv, C, ldc, M, N, m0, n0, alpha, beta);
            } else {
                T::epilogue_gemm(acc, C, ldc, M, N, m0, n0, alpha, 0.f);
            }
        } else {
            store_partial<T>(acc, part + ((int64_t)g * 2 + (it == beg ? 0 : 1)) * T::BM * T::BN,
                             threadIdx.x);
        }
        it = stop;
    }
}

// One work-group of the tile's shape per tile; tiles one work-group
// reduced whole were stored already.
template <class T>
__global__ __launch_bounds__(T::NT) void gemm_streamk_fixup_kernel(const float *__restrict__ part,
                                                                   float *__restrict__ C, int64_t ldc,
                                                                   int64_t M, int64_t N, float alpha,
                                                                   float beta, int tiles_n, int nb,
                                                                   int kt, int G)
{
    const int t = blockIdx.x;
    const int64_t total = (int64_t)nb * kt;
    const int g0 = sk_owner((int64_t)t * kt, total, G), g1 = sk_owner((int64_t)(t + 1) * kt - 1, total, G);
    if (g0 == g1) return;
    f32x16 acc[T::TM][T::TN];
    T::zero(acc);
    for (int g = g0; g <= g1; ++g) {
        // the tile is g's first segment unless g started in an earlier tile
        const int slot = sk_begin(g, total, G) / kt == t ? 0 : 1;
        add_partial<T>(acc, part + ((int64_t)g * 2 + slot) * T::BM * T::BN, threadIdx.x);
    }
    const int64_t m0 = (int64_t)(t / tiles_n) * T::BM, n0 = (int64_t)(t % tiles_n) * T::BN;
    if (beta != 0.f) {
        float cv[T::TM][T::TN][16];
        T::load_c(cv, C, ldc, M, N, m0, n0);
        T::epilogue_gemm_loaded(acc, cv, C, ldc, M, N, m0, n0, alpha, beta);
    } else {
        T::epilogue_gemm(acc, C, ldc, M, N, m0, n0, alpha, 0.f);
    }
}

// The stream-K tile: 128 x 128 x 32 on 16 waves, the three-stage
// direct-to-LDS ring (which takes ragged ranges); the register path when
// rows are not 16-byte aligned.
using SkTileVec = F32Tile<128, 128, 32, 4, 4, false, kLoadVec4, 4>;
using SkTileScalar = F32Tile<128, 128, 32, 4, 4, false, kLoadScalar, 2>;

struct SkPlan {
    int tiles_n, nb, kt, G;
};

// Whether and how the stream-K schedule (or its place in phases) runs M x N x
// K: with at least 32 K-tiles per output tile, when the tiles number fewer than the compute
// units or their last wave fills at most 60% of them (and there are fewer
// than four waves, beyond which that tail matters little).
bool gemm_streamk_plan(int64_t M, int64_t N, int64_t K, SkPlan &p)
{
    constexpr int64_t BM = 128, BN = 128, BK = 32;
    const int64_t cus = device_cu_count();
    const int64_t tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN, kt = (K + BK - 1) / BK;
    const int64_t nb = tm * tn;
    if (M <= 0 || N <= 0 || kt < 32 || cus <= 0) return false;
    const int64_t rem = nb % cus;
    const bool underfilled = nb < cus;
    const bool short_tail = nb < 4 * cus && rem != 0 && rem * 10 <= cus * 6;
    if (!underfilled && !short_tail) return false;
    if (nb > (int64_t)1 << 30 || kt > (int64_t)1 << 30) return false;
    int64_t G = cus < kStreamMaxGroups ? cus : kStreamMaxGroups;
    if (G > nb * kt) G = nb * kt;
    p.tiles_n = (int)tn;
    p.nb = (int)nb;
    p.kt = (int)kt;
    p.G = (int)G;
    return true;
}

template <class T>
int run_gemm_streamk(const SkPlan &p, int64_t M, int64_t N, int64_t K, float alpha, const float *A,
                     const float *B, float beta, float *C, float *ws, hipStream_t s)
{
    hipLaunchKernelGGL(gemm_streamk_kernel<T>, dim3(p.G), dim3(T::NT), 0, s, A, K, B, N, C, N, M, N, K,
                       alpha, beta, p.tiles_n, p.nb, p.kt, ws);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
    hipLaunchKernelGGL(gemm_streamk_fixup_kernel<T>, dim3(p.nb), dim3(T::NT), 0, s, (const float *)ws, C,
                       N, M, N, alpha, beta, p.tiles_n, p.nb, p.kt, p.G);
    return (int)hipGetLastError();
}

}  // namespace

int launch_gemm_f32(int cfg, int64_t M, int64_t N, int64_t K, float alpha, const float *A,
                    int64_t lda, const float *B, int64_t ldb, float beta, float *C, int64_t ldc,
                    void *stream)
{
    hipStream_t s = (hipStream_t)stream;
    const bool v4 = (alpha == 0.f || (K % 4 == 0 && N % 4 == 0 && lda % 4 == 0 && ldb % 4 == 0 &&
                                      aligned16(A) && aligned16(B)));
    switch (cfg) {
#define LI_CASE(IDX, BM, BN, BK, WM, WN, SK, PF) \
    case IDX:                                    \
        return run_gemm_candidate<BM, BN, BK, WM, WN, PF>(v4, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, s);
        LI_GEMM_F32_CANDIDATES(LI_CASE)
#undef LI_CASE
    default:
        return (int)hipErrorInvalidValue;
    }
}

size_t gemm_streamk_bytes(int64_t M, int64_t N, int64_t K)
{
    SkPlan p;
    if (!gemm_streamk_plan(M, N, K, p)) return 0;
    return (size_t)2 * p.G * 128 * 128 * sizeof(float);
}

int launch_gemm_f32_streamk(int64_t M, int64_t N, int64_t K, float alpha, const float *A,
                            const float *B, float beta, float *C, float *ws, void *stream)
{
    SkPlan p;
    if (!gemm_streamk_plan(M, N, K, p) || !ws) return (int)hipErrorInvalidValue;
    hipStream_t s = (hipStream_t)stream;
    if (K <= kSplitMaxLd && N <= kSplitMaxLd) {
        // The least predicted time of the plain schedule and of phases of 128
        // x 128 and of 64 x 64 tiles, whose plans' own prediction is scaled to
        // these kernels (measured, us, plain / 128 / 64: 1024 x 1024 x 4096
        // 70.6 / 57.1 / 72.3; 300 x 200 x 4100 33.2 / 21.0 / 15.3; 512 x 512 x
        // 65536 480 / 170 / 235; 1000 x 1500 x 3000 69.8 / 73.2 / 83.2; 3000^3
        // 345 / 293 / 373.  Stream-K on the FP32 cores: 87.5, 47.1, 274, 94.5,
        // 466).
        const double plain = split_gemm_us(M, N, K);
        const double t128 = 1.18 * phase_us<PhaseTile128>(M, N, K) + 5.0;
        const double t64 = 1.02 * phase_us<PhaseTile64>(M, N, K) + 6.0;
        // Few tiles: always cut, for the error.  Stream-K on the FP32 cores,
        // which took these calls before, cuts each of the fewer tiles into
        // more ranges (rms at K = 1024 / 2000 / 4096: 1 tile 1.5e-7 / 1.8 / 2.3,
        // 16 1.6 / 2.2 / 3.0, 24 1.9 / 2.5 / 3.5, 40 2.3 / 3.2 / 4.5); uncut
        // split tiles have 1.7 / 2.5 / 3.7 whatever their number, cut ones 0.9 /
        // 1.0 / 1.0 with 1 and 1.2 / 1.7 / 1.2 with 24.  Only calls of 12 to 16
        // tiles and K below 1200 would be faster uncut (512 x 512 x 1024: 11.2 us
        // against 13.2).
        const bool few = p.nb < 32;
        if ((few || t128 < plain) && t128 <= t64)
            return run_gemm_phases<PhaseTile128>(M, N, K, alpha, A, B, beta, C, ws, s);
        if (few || t64 < plain) return run_gemm_phases<PhaseTile64>(M, N, K, alpha, A, B, beta, C, ws, s);
        return launch_gemm_f32(tune_pick(LI_KERNEL_GEMM_F32, M, N, K), M, N, K, alpha, A, K, B, N, beta, C, N, stream);
    }
    const bool v4 = K % 4 == 0 && N % 4 == 0 && aligned16(A) && aligned16(B);
    return v4 ? run_gemm_streamk<SkTileVec>(p, M, N, K, alpha, A, B, beta, C, ws, s)
              : run_gemm_streamk<SkTileScalar>(p, M, N, K, alpha, A, B, beta, C, ws, s);
}

size_t syrk_split_bytes(int64_t n)
{
    size_t best = 0;
    LI_SYRK_F32_CANDIDATES(LI_SYM_SPLIT_BYTES)
    return best;
}

size_t syrk_split_bytes_cfg(int cfg, int64_t n)
{
    // what run_sym touches for this candidate: split partials of every
    // upper tile, or two stream-K pieces per work-group of its grid
    switch (cfg) {
#define LI_CASE(IDX, BM, BN, BK, WM, WN, SK, PF)                                                   \
    case IDX: {                                                                                \
        const int64_t t = (n + BM - 1) / BM;                                                   \
        if (SK > 1) return (size_t)SK * (size_t)(t * (t + 1) / 2) * BM * BN * sizeof(float);   \
        if (SK == 0) {                                                                         \
            int g = device_cu_count() * CandidateTile<BM, BN, BK, WM, WN, PF, true, false, 0, kLoadVec4, PF>::SK_PER_CU; \
            if (g > kStreamMaxGroups) g = kStreamMaxGroups;                                    \
            return (size_t)2 * g * BM * BN * sizeof(float);                                    \
        }                                                                                      \
        return 0;                                                                              \
    }
        LI_SYRK_F32_CANDIDATES(LI_CASE)
#undef LI_CASE
    default:
        return syrk_split_bytes(n);
    }
}

int launch_syrk_f32(int cfg, int64_t M, int64_t N, const float *Y, float *S, int mode, float scale,
                    float *split_ws, void *stream)
{
    hipStream_t s = (hipStream_t)stream;
    const bool v4 = (M % 4 == 0 && aligned16(Y));
    const SymArgs a{Y, nullptr, M, M, N, S, mode, scale, 0.f, 1, nullptr, nullptr};
    switch (cfg) {
#define LI_CASE(IDX, BM, BN, BK, WM, WN, SK, PF)                                                        \
    case IDX:                                                                                           \
        return run_sym_candidate<BM, BN, BK, WM, WN, PF, PF, true, 0, kSymCols>(a, v4, true, SK, split_ws, s);
        LI_SYRK_F32_CANDIDATES(LI_CASE)
#undef LI_CASE
    default:
        return (int)hipErrorInvalidValue;
    }
}

}  // namespace li
