// FP32 block tile on the bf16 matrix cores: every operand element is split
// exactly into three bf16 parts and six of the nine part products are summed.
//
//   x = x0 + x1 + x2,  x0 = x cut to bf16, x1 = bf16(x - x0), x2 = x - x0 - x1
//
// Both subtractions are exact, and 3 x 8 significant bits hold the 24 of an
// FP32 value, so the parts are the value; only the middle one is rounded (to
// nearest even), which leaves a third part of either sign.  The products
// x2*y1, x1*y2 and x2*y2, together below 3 * 2^-25 of x*y and of either sign,
// are left out; the other six are exact in the matrix cores' FP32 sums.  The
// leading products x0*y0 go to one accumulator and the other five to a
// second one, whose sums are 2^-7 of the first's, so that the roundings that
// count are those of the leading sum alone.  The FP32 cores round every
// product and every two-wide sum; against 64 bits the split is 3 times
// closer (rms relative to the result's, U[-1, 1), K = 256 / 2048 / 8192:
// 9.1e-8 / 2.5e-7 / 5.5e-7, FP32 cores 2.9e-7 / 8.1e-7 / 1.6e-6; one
// accumulator for all six products 2.5e-7 / 7.0e-7 / 1.45e-6).
//
// Why: six bf16 products still run 2.6 times as fast as one on the FP32
// cores (2.5 PFLOP/s / 6 against 157 TFLOP/s).  Measured (li_gemm, beta != 0,
// FP32 cores before): 2048^3 0.130 -> 0.089 ms, 8192^3 7.8 -> 5.4 ms,
// 1531 x 1027 x 777 38.5 -> 25.0 us, 512^3 12.8 -> 8.1 us.  At 8192^3 the
// bf16 cores then execute 1.2 PFLOP/s, 0.9 of what a large bf16 product of
// the vendor library reaches on this card (power-limited clock).
//
// Elements that the three parts cannot hold are noticed: a third part with
// bits below bf16's (magnitudes of about 2^-110 and less) while splitting,
// infinities and NaN, and sums that left the finite range, by the NaN or
// infinity they leave in the block tile.  The block tile is then reduced
// again on the FP32 cores, so every input gives what they give.
//
// Work split.  Splitting is paid once per element and block tile: PW
// splitting waves load the next K-tiles from memory, split them and store
// the parts to one of two LDS stages, while WM x WN matrix waves read the
// other stage and do nothing but LDS reads and matrix instructions (one
// barrier per K-tile).  Done by the same waves, the two did not overlap (the
// compiler keeps the splitting's 240 vector instructions apart from the
// matrix instructions: 2048^3 0.116 ms).  A K-tile of 128 x 128 x 32 takes
// the four matrix waves 1536 cycles; splitting takes 26 vector cycles per
// element, about 850 per SIMD, in the issue slots the matrix instructions
// leave free.  Two accumulators of 64 x 64 per wave, their operands twice
// (the next step's are read during this one's products) and the splitting
// waves' two K-tiles in flight fit the 256 registers that two waves per SIMD
// leave each.
//
// LDS.  A stage holds, per operand, part and 16-wide k step, [row][16] with
// the row's two 16-byte chunks swapped in every other group of eight rows:
// the 16-byte reads of a wave then run at 256 bytes per cycle (128 without
// the swap).  A step's region is skewed by 128 bytes so that the two steps
// that a wave's stores touch do not share banks.
//
// Loads use buffer descriptors: a uniform base per K-tile, one 32-bit offset
// per piece and lane and a uniform row offset, so no vector instruction
// forms an address (20 64-bit additions per K-tile before; 8192^3 5.75 ->
// 5.4 ms).  They are plain dword loads (k-major operands: consecutive lanes,
// consecutive columns) and 16-byte loads at 4-byte alignment (k-contiguous
// ones), so one kernel serves all shapes and alignments.
#pragma once

#include "f32_tile.h"

namespace li {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

// Two values to their three bf16 parts, packed.  `lost` collects the bits of
// the third parts that bf16 cannot hold (non-zero low halves).
__device__ __forceinline__ void split_pair(float x, float y, uint32_t &p0, uint32_t &p1, uint32_t &p2,
                                           uint32_t &lost)
{
    constexpr uint32_t kHigh = 0xffff0000u, kPack = 0x07060302u;  // high halves of two words
    uint32_t u = __builtin_bit_cast(uint32_t, x), v = __builtin_bit_cast(uint32_t, y);
    p0 = __builtin_amdgcn_perm(v, u, kPack);
    x -= __builtin_bit_cast(float, u & kHigh);
    y -= __builtin_bit_cast(float, v & kHigh);
    p1 = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2_t));
    u = __builtin_bit_cast(uint32_t, x - __builtin_bit_cast(float, p1 << 16));
    v = __builtin_bit_cast(uint32_t, y - __builtin_bit_cast(float, p1 & kHigh));
    p2 = __builtin_amdgcn_perm(v, u, kPack);
    lost |= u | v;
}

// Longest rows (elements) of an operand: offsets inside a block tile are 32-bit
// byte offsets (256 rows, or 64 k values, of this many elements).
constexpr int64_t kSplitMaxLd = (int64_t)1 << 21;

// Splitting waves of the main-loop modes 9 to 11 of the candidate lists.
constexpr int split_waves(int mode) { return mode == 10 ? 2 : mode == 11 ? 8 : 4; }

// Loads of one operand's K-tile of R rows (the other index: m or n) and BK k
// values into registers, and their split stores into a stage.
// KMAJOR: element (row, k) at P[k ld + row], else P[row ld + k].
template <int R, int BK, int NT, bool KMAJOR, int XFORM>
struct SplitLoader {
    static constexpr int KS = BK / 16;
    static constexpr int STEP = R * 16 + 64;  // bf16 elements of one k step, with the skew
    static constexpr int PART = KS * STEP;
    // k-contiguous: pieces of 4 k of one row; k-major: 8 k of one row
    static constexpr int PK = KMAJOR ? 8 : 4;
    static constexpr int PIECES = R * BK / PK;
    static_assert(PIECES % NT == 0, "pieces must divide evenly among threads");
    static constexpr int PER = PIECES / NT;

    float v[PER][PK];

    __device__ __forceinline__ static int piece_row(int c) { return KMAJOR ? c % R : c / (BK / 4); }
    __device__ __forceinline__ static int piece_k(int c) { return KMAJOR ? (c / R) * 8 : (c % (BK / 4)) * 4; }

    // byte offsets of this thread's pieces from the tile's first element;
    // rows past the matrix repeat its last one (their products are never
    // stored).  ld is at most kSplitMaxLd.
    __device__ __forceinline__ static void offsets(uint32_t (&off)[PER], int64_t ld, int64_t rows, int64_t r0, int tid)
    {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = tid + i * NT;
            const int64_t last = rows - 1 - r0;
            const int r = piece_row(c) < last ? piece_row(c) : (int)last;
            const uint32_t l = (uint32_t)ld;
            off[i] = 4u * (KMAJOR ? (uint32_t)piece_k(c) * l + (uint32_t)r : (uint32_t)r * l + (uint32_t)piece_k(c));
        }
    }

    // base: the tile's first element at this K-tile; left: k values that
    // remain from there (values past them are 0, or `fill`, which the
    // transform maps to 0)
    template <bool FULL>
    __device__ __forceinline__ void load(const float *__restrict__ base, const uint32_t (&off)[PER], int64_t ld,
                                         int64_t left, const float (&fill)[PER], int tid)
    {
        // buffer loads: a uniform descriptor of this K-tile, the lane's 32-bit
        // offset and a uniform row offset, so no vector instruction forms an
        // address
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, 0xffffffff, 0x00027000);
        const int ld4 = (int)ld * 4;
        if constexpr (FULL) {
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                if constexpr (KMAJOR) {
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        v[i][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, off[i], j * ld4, 0));
                } else {
                    const auto raw = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off[i], 0, 0);
                    static_assert(sizeof(raw) == 16, "16-byte loads");
                    const f32x4 x = __builtin_bit_cast(f32x4, raw);
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[i][j] = x[j];
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < PER; ++i)
#pragma unroll
                for (int j = 0; j < PK; ++j) {
                    v[i][j] = XFORM ? fill[i] : 0.f;
                    if (piece_k(tid + i * NT) + j < left)
                        v[i][j] = __builtin_bit_cast(
                            float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, off[i] + (KMAJOR ? 0 : 4 * j), KMAJOR ? j * ld4 : 0, 0));
                }
        }
    }

    __device__ __forceinline__ void store(uint16_t *lds, uint32_t &lost, const float (&m)[PER], const float (&f)[PER], int tid) const
    {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = tid + i * NT;
            const int r = piece_row(c), k = piece_k(c);
            uint32_t p[3][PK / 2];
#pragma unroll
            for (int j = 0; j < PK; j += 2) {
                float x = v[i][j], y = v[i][j + 1];
                if (XFORM != 0) {
                    x -= m[i];
                    y -= m[i];
                }
                if (XFORM == 2) {
                    x *= f[i];
                    y *= f[i];
                }
                split_pair(x, y, p[0][j / 2], p[1][j / 2], p[2][j / 2], lost);
            }
            uint16_t *d = lds + (k / 16) * STEP + r * 16 + ((((k >> 3) & 1) ^ ((r >> 3) & 1)) << 3) + (k & 4);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                if constexpr (KMAJOR)
                    *reinterpret_cast<u32x4_t *>(d + q * PART) = u32x4_t{p[q][0], p[q][1], p[q][2], p[q][3]};
                else
                    *reinterpret_cast<u32x2_t *>(d + q * PART) = u32x2_t{p[q][0], p[q][1]};
            }
        }
    }

    // matrix-core operand: 8 k of row `row` at k step `s`, half h
    __device__ __forceinline__ static bf16x8_t frag(const uint16_t *lds, int part, int s, int row, int h)
    {
        return *reinterpret_cast<const bf16x8_t *>(lds + part * PART + s * STEP + row * 16 + ((h ^ ((row >> 3) & 1)) << 3));
    }
};

template <int BM_, int BN_, int BK_, int WM_, int WN_, int PW_, bool DUAL, bool A_KMAJOR, bool B_NMAJOR, int XFORM_ = 0>
struct SplitTile : F32Tile<BM_, BN_, 32, WM_, WN_, A_KMAJOR, kLoadScalar, 1, B_NMAJOR, 0> {
    // the FP32 tile of the same accumulator layout: epilogues, and (Safe, with
    // the transform) the reduction of block tiles that the split cannot hold
    using Base = F32Tile<BM_, BN_, 32, WM_, WN_, A_KMAJOR, kLoadScalar, 1, B_NMAJOR, 0>;
    using Safe = F32Tile<BM_, BN_, 32, WM_, WN_, A_KMAJOR, kLoadScalar, 1, B_NMAJOR, XFORM_>;
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, PW = PW_;
    static constexpr int TM = Base::TM, TN = Base::TN;
    static constexpr int XFORM = XFORM_;
    static constexpr int ET = 64 * WM * WN;  // threads of the matrix waves, which hold the result
    static constexpr int PT = 64 * PW;       // threads of the splitting waves
    static constexpr int NT = ET + PT;
    static constexpr int BK = BK_, KS = BK / 16;
    static_assert(BK % 32 == 0, "an even number of k steps keeps the operand sets' parity");
    static constexpr int NS = 2;  // K-tiles in flight from memory (register sets)
    using LA = SplitLoader<BM, BK, PT, A_KMAJOR, XFORM>;
    using LB = SplitLoader<BN, BK, PT, !B_NMAJOR, XFORM>;
    static constexpr int STAGE = 3 * (LA::PART + LB::PART);  // bf16 elements
    static constexpr int SPLIT_FLOATS = STAGE;               // two stages of 2-byte elements
    static constexpr int SAFE_FLOATS = Safe::LDS_FLOATS;
    static constexpr int LDS_FLOATS = SPLIT_FLOATS > SAFE_FLOATS ? SPLIT_FLOATS : SAFE_FLOATS;
    static_assert(LDS_FLOATS * 4 <= 160 * 1024, "stages must fit in LDS");

    static constexpr bool SPLIT = true;
    static constexpr int SK_PER_CU = LDS_FLOATS * 8 <= 160 * 1024 ? 2 : 1;

    // only the matrix waves hold the result after the main loop
    __device__ __forceinline__ static bool active() { return threadIdx.x < ET; }

    struct XRegs {
        const double *mean, *factor;
    };
    __device__ __forceinline__ static void load_xregs(XRegs &x, const double *mean, const double *factor, int64_t,
                                                      int64_t, int64_t, int64_t)
    {
        x.mean = mean;
        x.factor = factor;
    }

    template <class L>
    __device__ __forceinline__ static void columns(const XRegs *x, int64_t n, int64_t r0, int tid, float (&m)[L::PER],
                                                   float (&f)[L::PER])
    {
#pragma unroll
        for (int i = 0; i < L::PER; ++i) {
            m[i] = f[i] = 0.f;
            if constexpr (XFORM != 0) {
                const int64_t c = r0 + L::piece_row(tid + i * PT);
                if (c < n) m[i] = (float)x->mean[c];
                if (XFORM == 2 && c < n) f[i] = (float)x->factor[c];
            }
        }
    }

    // LDS writes and reads of the work-group ordered by a barrier that does
    // not wait for the global loads in flight
    __device__ __forceinline__ static void lds_barrier()
    {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    }

    // Operands of one 16-wide k step, and its matrix instructions.
    struct Frag {
        bf16x8_t a[3][TM], b[3][TN];
    };

    __device__ __forceinline__ static void read_frag(Frag &f, const uint16_t *st, int s, int wm0, int wn0, int lane)
    {
        const int l32 = lane & 31, h = lane >> 5;
#pragma unroll
        for (int p = 0; p < 3; ++p) {
#pragma unroll
            for (int i = 0; i < TM; ++i) f.a[p][i] = LA::frag(st, p, s, wm0 + 32 * i + l32, h);
#pragma unroll
            for (int j = 0; j < TN; ++j) f.b[p][j] = LB::frag(st + 3 * LA::PART, p, s, wn0 + 32 * j + l32, h);
        }
    }

    static constexpr int N_MFMA = 6 * TM * TN, N_READ = 3 * (TM + TN);

    // Interleaves the next step's operand reads with the first matrix
    // instructions of this one.
    template <int m = 0>
    __device__ __forceinline__ static void interleave()
    {
        if constexpr (m < N_MFMA) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            if constexpr (m < N_READ) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            interleave<m + 1>();
        }
    }

    __device__ __forceinline__ static void mma(const Frag &f, f32x16 (&hi)[TM][TN], f32x16 (&lo)[TM][TN])
    {
        constexpr int PA[6] = {0, 0, 1, 1, 0, 2}, PB[6] = {0, 1, 0, 1, 2, 0};
#pragma unroll
        for (int t = 0; t < 6; ++t)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    f32x16 &c = t == 0 || !DUAL ? hi[i][j] : lo[i][j];
                    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[PA[t]][i], f.b[PB[t]][j], c, 0, 0, 0);
                }
    }

    // Matrix waves: hi, lo += the products of nk K-tiles.
    __device__ __forceinline__ static void multiply(const uint16_t *lds, int nk, f32x16 (&hi)[TM][TN],
                                                    f32x16 (&lo)[TM][TN])
    {
        const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        const int wm0 = (w / WN) * (BM / WM), wn0 = (w % WN) * (BN / WN);
        const uint16_t *cur = lds, *nxt = lds + STAGE;
        Frag f, g;
        __builtin_amdgcn_s_setprio(1);
        lds_barrier();  // K-tile 0 is stored
        read_frag(f, cur, 0, wm0, wn0, lane);
        __builtin_amdgcn_sched_barrier(0);
        for (int t = 0; t + 1 < nk; ++t) {
#pragma unroll
            for (int s = 0; s < KS; s += 2) {
                read_frag(g, cur, s + 1, wm0, wn0, lane);
                mma(f, hi, lo);
                interleave();
                __builtin_amdgcn_sched_barrier(0);
                if (s + 2 == KS) lds_barrier();  // K-tile t + 1 is stored, K-tile t is read
                __builtin_amdgcn_sched_barrier(0);
                read_frag(f, s + 2 == KS ? nxt : cur, s + 2 == KS ? 0 : s + 2, wm0, wn0, lane);
                mma(g, hi, lo);
                interleave();
                __builtin_amdgcn_sched_barrier(0);
            }
            const uint16_t *x = cur;
            cur = nxt;
            nxt = x;
        }
#pragma unroll
        for (int s = 0; s < KS; s += 2) {
            read_frag(g, cur, s + 1, wm0, wn0, lane);
            mma(f, hi, lo);
            if (s + 2 < KS) read_frag(f, cur, s + 2, wm0, wn0, lane);
            mma(g, hi, lo);
        }
        lds_barrier();
        __builtin_amdgcn_s_setprio(0);
    }

    // Splitting waves: nk K-tiles into the two stages in turn, loaded NS
    // K-tiles ahead of their split.
    __device__ __forceinline__ static void produce(uint16_t *lds, const float *A, int64_t lda, const float *B,
                                                   int64_t ldb, int64_t M, int64_t N, int64_t kbeg, int64_t kend,
                                                   int64_t m0, int64_t n0, int nk, uint32_t &lost, const XRegs *xr)
    {
        const int tid = (int)threadIdx.x - ET;
        float ma[LA::PER], fa[LA::PER], mb[LB::PER], fb[LB::PER];
        columns<LA>(xr, M, m0, tid, ma, fa);
        columns<LB>(xr, N, n0, tid, mb, fb);
        LA la[NS];
        LB lb[NS];
        uint32_t oa[LA::PER], ob[LB::PER];
        LA::offsets(oa, lda, M, m0, tid);
        LB::offsets(ob, ldb, N, n0, tid);
        const int64_t adv_a = A_KMAJOR ? BK * lda : BK, adv_b = B_NMAJOR ? BK : BK * ldb;
        const float *pa = A_KMAJOR ? A + kbeg * lda + m0 : A + m0 * lda + kbeg;
        const float *pb = B_NMAJOR ? B + n0 * ldb + kbeg : B + kbeg * ldb + n0;
        int64_t left = kend - kbeg;
        auto load = [&](auto full, int set) {
            if (decltype(full)::value || left >= BK) {
                la[set].template load<true>(pa, oa, lda, left, ma, tid);
                lb[set].template load<true>(pb, ob, ldb, left, mb, tid);
            } else {
                la[set].template load<false>(pa, oa, lda, left, ma, tid);
                lb[set].template load<false>(pb, ob, ldb, left, mb, tid);
            }
            pa += adv_a;
            pb += adv_b;
            left -= BK;
        };
        auto store = [&](int set) {
            uint16_t *st = lds + (set & 1) * STAGE;
            la[set].store(st, lost, ma, fa, tid);
            lb[set].store(st + 3 * LA::PART, lost, mb, fb, tid);
        };
        constexpr std::true_type full{};
        constexpr std::false_type any{};
        // Whole K-tiles run a loop without branches around its loads, so the
        // waits count them exactly; the last tiles take the checked loads.
        int t = 0;
        if (left >= 2 * NS * BK) {
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                load(full, i);
                __builtin_amdgcn_sched_barrier(0);
            }
            for (; left >= NS * BK; t += NS)
#pragma unroll
                for (int i = 0; i < NS; ++i) {
                    store(i);
                    load(full, i);
                    __builtin_amdgcn_sched_barrier(0);
                    lds_barrier();  // K-tile t + i is stored, the one before is read
                }
        } else {
#pragma unroll
            for (int i = 0; i < NS; ++i)
                if (left > 0) load(any, i);
        }
        for (; t < nk; t += NS)
#pragma unroll
            for (int i = 0; i < NS; ++i)
                if (t + i < nk) {
                    store(i);
                    if (left > 0) load(any, i);
                    lds_barrier();
                }
        lds_barrier();
    }

    // hi, lo += A B over k in [kbeg, kend)
    __device__ __forceinline__ static void reduce(uint16_t *lds, const float *A, int64_t lda, const float *B,
                                                  int64_t ldb, int64_t M, int64_t N, int64_t kbeg, int64_t kend,
                                                  int64_t m0, int64_t n0, f32x16 (&hi)[TM][TN],
                                                  f32x16 (&lo)[TM][TN], uint32_t &lost, const XRegs *xr)
    {
        const int nk = (int)((kend - kbeg + BK - 1) / BK);
        // nk + 1 barriers on both sides
        if (active())
            multiply(lds, nk, hi, lo);
        else
            produce(lds, A, lda, B, ldb, M, N, kbeg, kend, m0, n0, nk, lost, xr);
    }

    // acc += A B on the FP32 matrix cores: the matrix waves run the FP32
    // tile's loop, the others meet its barriers (one per K-tile and one).
    __device__ __forceinline__ static void reduce_safe(float *lds, const float *A, int64_t lda, const float *B,
                                                       int64_t ldb, int64_t M, int64_t N, int64_t kbeg,
                                                       int64_t kend, int64_t m0, int64_t n0,
                                                       f32x16 (&acc)[TM][TN], const XRegs *xr)
    {
        if (active()) {
            typename Safe::XRegs sx;
            if constexpr (XFORM != 0) Safe::load_xregs(sx, xr->mean, xr->factor, M, N, m0, n0);
            Safe::mainloop(lds, A, lda, B, ldb, M, N, kbeg, kend, m0, n0, acc, false, XFORM ? &sx : nullptr);
        } else {
            const int64_t nk = (kend - kbeg + Safe::BK - 1) / Safe::BK;
            for (int64_t t = 0; t < nk + 1; ++t) __syncthreads();
        }
    }

    // acc = A B (+ A1 B1 when A1 is given) over k in [kbeg, kend); acc holds
    // the result in the matrix waves.
    __device__ __forceinline__ static void contract(float *lds, const float *A, const float *B, const float *A1,
                                                    const float *B1, int64_t lda, int64_t ldb, int64_t M,
                                                    int64_t N, int64_t kbeg, int64_t kend, int64_t m0, int64_t n0,
                                                    f32x16 (&acc)[TM][TN], const XRegs *xr)
    {
        uint32_t lost = 0;
        if (kend > kbeg) {
            f32x16 lo[TM][TN];
            Base::zero(acc);
            Base::zero(lo);
            uint16_t *l16 = reinterpret_cast<uint16_t *>(lds);
            for (int pass = 0; pass < (A1 ? 2 : 1); ++pass)
                reduce(l16, pass ? A1 : A, lda, pass ? B1 : B, ldb, M, N, kbeg, kend, m0, n0, acc, lo, lost, xr);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    if (DUAL) acc[i][j] += lo[i][j];
            bool bad = (lost & 0xffffu) != 0;
            // an infinity or NaN among the sums (0 * x is 0 for finite x)
            if (active()) {
                float s = 0.f;
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int v = 0; v < 16; ++v) s = __builtin_fmaf(acc[i][j][v], 0.f, s);
                bad |= !(s == 0.f);
            }
            if (__syncthreads_or(bad)) {
                Base::zero(acc);
                reduce_safe(lds, A, lda, B, ldb, M, N, kbeg, kend, m0, n0, acc, xr);
                if (A1) reduce_safe(lds, A1, lda, B1, ldb, M, N, kbeg, kend, m0, n0, acc, xr);
            }
        }
    }

    // C = alpha acc + beta C over the in-range part of the tile (beta == 0: C
    // is not read).  Every row of the wave's blocks is a uniform address plus
    // one 32-bit lane offset: the code of a block tile is short, which counts
    // where a work-group runs it once (instruction fetch).
    template <bool FULL>
    __device__ __forceinline__ static void write_c(const f32x16 (&acc)[TM][TN], float *C, int64_t ldc, int rows,
                                                   int cols, float alpha, float beta)
    {
        const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        const int wm0 = (w / WN) * (BM / WM), wn0 = (w % WN) * (BN / WN);
        const int r0 = 4 * (lane >> 5), c0 = lane & 31;
        const uint32_t voff = 4u * ((uint32_t)r0 * (uint32_t)ldc + (uint32_t)c0);
        char *base = reinterpret_cast<char *>(C + (int64_t)wm0 * ldc + wn0);
        auto at = [&](int i, int j, int v) {
            const int64_t row = 32 * i + 8 * (v >> 2) + (v & 3);
            return reinterpret_cast<float *>(base + row * ldc * 4 + 128 * j + voff);
        };
        auto ok = [&](int i, int j, int v) {
            return FULL || (wm0 + 32 * i + 8 * (v >> 2) + (v & 3) + r0 < rows && wn0 + 32 * j + c0 < cols);
        };
        float old[TM][TN][16];
        if (beta != 0.f) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v)
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        old[i][j][v] = 0.f;
                        if (ok(i, j, v)) old[i][j][v] = *at(i, j, v);
                    }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        if (ok(i, j, v)) *at(i, j, v) = Base::combine(alpha, acc[i][j][v], beta, old[i][j][v]);
        } else {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        if (ok(i, j, v)) *at(i, j, v) = alpha * acc[i][j][v];
        }
    }

    __device__ __forceinline__ static void store_c(const f32x16 (&acc)[TM][TN], float *C, int64_t ldc, int64_t M,
                                                   int64_t N, int64_t m0, int64_t n0, float alpha, float beta)
    {
        float *c = C + m0 * ldc + n0;
        const int rows = M - m0 < BM ? (int)(M - m0) : BM, cols = N - n0 < BN ? (int)(N - n0) : BN;
        if (rows == BM && cols == BN)
            write_c<true>(acc, c, ldc, rows, cols, alpha, beta);
        else
            write_c<false>(acc, c, ldc, rows, cols, alpha, beta);
    }

    __device__ __forceinline__ static void mainloop(float *lds, const float *A, int64_t lda, const float *B,
                                                    int64_t ldb, int64_t M, int64_t N, int64_t kbeg, int64_t kend,
                                                    int64_t m0, int64_t n0, f32x16 (&acc)[TM][TN], bool = true,
                                                    const XRegs *xr = nullptr)
    {
        contract(lds, A, B, nullptr, nullptr, lda, ldb, M, N, kbeg, kend, m0, n0, acc, xr);
    }
};

}  // namespace li
