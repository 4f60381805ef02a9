// FP32 block tile on the bf16 matrix cores: every operand element is split
// exactly into three bf16 parts and six of the nine part products are summed.
//
//   x = x0 + x1 + x2,  x0 = bf16(x), x1 = bf16(x - x0), x2 = x - x0 - x1
//
// (to nearest even; Henry, Tang and Heinecke, "Leveraging the bfloat16
// Artificial Intelligence Datatype For Higher-Precision Computations", 2019).
// Both subtractions are exact, and 3 x 8 significant bits hold the 24 of an
// FP32 value, so the parts are the value.  A rounded first part leaves at
// most 2^-8 of x's power of two to the second and 2^-17 to the third, so the
// products x2*y1, x1*y2 and x2*y2, which are left out, are together below
// (2 + 2^-8) * 2^-25 of x*y, of either sign (rms 0.18 * 2^-25; with the first
// part cut instead up to 7.9 * 2^-25, rms 0.71); the other six are exact in
// the matrix cores' FP32 sums.  A result of a single product is then off by
// up to one unit in the last place, half of it the omission's (rms 2.6e-8 of
// it, 2.5e-8 where the product is rounded alone).  The leading products
// x0*y0 go to one accumulator and the other five to a second one, whose sums
// are 2^-7 of the first's, so that the roundings that count are those of the
// leading sum alone.  The FP32 cores round every product and every two-wide
// sum; against 64 bits the split is 3 times closer (rms relative to the
// result's, U[-1, 1), K = 256 / 2048 / 8192: 9.1e-8 / 2.5e-7 / 5.5e-7, FP32
// cores 2.9e-7 / 8.1e-7 / 1.6e-6; one accumulator for all six products
// 2.5e-7 / 7.0e-7 / 1.45e-6).
//
// Why: six bf16 products still run 2.6 times as fast as one on the FP32
// cores (2.5 PFLOP/s / 6 against 157 TFLOP/s).  Measured (li_gemm, beta != 0,
// FP32 cores before): 2048^3 0.130 -> 0.088 ms, 8192^3 7.8 -> 5.2 to 5.4 ms,
// 1531 x 1027 x 777 38.5 -> 23.2 us, 512^3 12.8 -> 7.8 us.  At 8192^3 the
// bf16 cores then execute 1.25 PFLOP/s, near what a large bf16 product of the
// vendor library reaches on this card (power-limited clock).
//
// Range.  An infinity or NaN of an operand is one in its first part, so the
// leading sum alone is then what the FP32 cores give (x0*y0 has the sign of
// x*y, and is NaN where x*y is), and the second accumulator, which mixes in
// products of infinity and zero parts, is left out of such results.  Three
// things need the FP32 cores: values that round to infinity as bf16, sums
// that leave the finite range, and third parts with bits below bf16's last
// one, 2^-133, which magnitudes of about 2^-110 and less may have (noticed
// while splitting).  A block tile that holds a result that is not finite, or
// that lost bits, reads its operands once more: it is reduced again on the
// FP32 cores where a finite operand of 2^62 / sqrt(k) or more may be why the
// result is not finite, or where the lost bits, at most 2^-133 of each
// element, may count in a result (reduce_again).  So every input gives what
// the FP32 cores give.  2048^3, 90 us: 126 us with a NaN in every row, 134
// with a hundredth of A below 1e-36, 248 where every tile is reduced again
// (results of 1e-35); the FP32 cores take 130.  (A scale of 2^16 on both operands, which brings
// every small value into the parts' range, is one product per element: 1.5%
// at 8192^3, 4% where the splitting bounds the tile, syrk 768 x 704.)
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
// 5.4 ms).  All are 16-byte loads at 4-byte alignment, so one kernel serves
// all shapes and alignments.  Half of the splitting waves load one operand
// and half the other, which keeps their loop free of branches: a merge of
// paths makes the compiler wait for every load in flight.
//
// What a work-group runs once is fetched from memory at about 15 ns per
// instruction, so prologue and epilogue are short loops (store_c).
#pragma once

#include "f32_tile.h"
#include "li_internal.h"

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
    // (fused with a product that made x, the remainder would have more bits
    // than x)
#pragma clang fp contract(off)
    constexpr uint32_t kHigh = 0xffff0000u, kPack = 0x07060302u;  // high halves of two words
    p0 = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2_t));
    x -= __builtin_bit_cast(float, p0 << 16);
    y -= __builtin_bit_cast(float, p0 & kHigh);
    p1 = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2_t));
    const uint32_t u = __builtin_bit_cast(uint32_t, x - __builtin_bit_cast(float, p1 << 16));
    const uint32_t v = __builtin_bit_cast(uint32_t, y - __builtin_bit_cast(float, p1 & kHigh));
    p2 = __builtin_amdgcn_perm(v, u, kPack);
    lost |= u | v;
}

// Splitting waves of the main-loop modes 9 to 11 of the candidate lists.
constexpr int split_waves(int mode) { return mode == 10 ? 2 : mode == 11 ? 8 : 4; }

// Loads of one operand's K-tile of R rows (the other index: m or n) and BK k
// values into registers, and their split stores into a stage.
// KMAJOR: element (row, k) at P[k ld + row], else P[row ld + k].
//
// A piece is four k of one row (k-contiguous operands: one 16-byte load) or
// of CW = 4 neighbouring rows (k-major: four 16-byte loads, one per k; eight
// lanes take eight pieces of four k, the next lanes the next rows, so a load
// instruction of a wave reads whole 128-byte lines of eight k rows; dword
// loads of one row per lane took four times the load instructions: 8192^3
// 5.47 -> 5.13 ms, 2048 x 2048 x 4096 0.168 -> 0.162 ms).
// Each row's four k go to the stage with one 8-byte store per part.  The rows
// of a k-major operand stand permuted inside their group of 32 (slot), so
// that the CW stores of a wave each fall on distinct banks; the accumulators'
// row or column index is permuted the same way (SplitTile::acc_row, acc_col).
template <int R, int BK, int NT, bool KMAJOR, int XFORM>
struct SplitLoader {
    static constexpr int THREADS = NT;
    static constexpr int KS = BK / 16;
    static constexpr int STEP = R * 16 + 64;  // bf16 elements of one k step, with the skew
    static constexpr int PART = KS * STEP;
    static constexpr int CW = KMAJOR ? 4 : 1;
    static constexpr int PIECES = R * BK / 4 / CW;
    static_assert(PIECES % NT == 0, "pieces must divide evenly among threads");
    static constexpr int PER = PIECES / NT;
    static constexpr int LOADS = KMAJOR ? 4 * PER : PER;

    // as loaded: for k-contiguous operands four k of a row, for k-major ones four
    // rows of each k.  Elements are taken out of the vectors only where they are
    // stored (piece): shuffles of loop-carried values, placed by the compiler at
    // the end of the loop body, waited there for the loads just issued (8192^3:
    // 5.66 ms, 5.12 without).
    f32x4 v[PER][CW];  // CW is 4 or 1

    __device__ __forceinline__ float element(int i, int e, int j) const { return KMAJOR ? v[i][KMAJOR ? j : 0][e] : v[i][0][j]; }

    // place of row r in a stage, and the row at place p
    __device__ __forceinline__ static int slot(int r) { return KMAJOR ? (r & ~31) + 8 * (r & 3) + ((r & 31) >> 2) : r; }
    __device__ __forceinline__ static int row_at(int p) { return KMAJOR ? (p & ~31) + 4 * (p & 7) + ((p & 31) >> 3) : p; }

    __device__ __forceinline__ static int piece_row(int c)
    {
        return KMAJOR ? (c >> 3) % (R / CW) * CW : c / (BK / 4);
    }
    __device__ __forceinline__ static int piece_k(int c)
    {
        return KMAJOR ? ((c >> 3) / (R / CW) * 8 + (c & 7)) * 4 : c % (BK / 4) * 4;
    }

    // This thread's pieces of the tile at row r0: byte offsets from the first
    // element of the K-tile's row r0 (k-contiguous) or row 0 (k-major), and
    // places in a stage.  Pieces past the matrix load its last rows again
    // (products never stored, but finite where the matrix is); a k-major
    // piece that is partly outside loads the last CW rows and stores those
    // that the piece before it holds in the places past the matrix, so every
    // place of a stage is written once.  ld is at most kSplitMaxLd.
    __device__ __forceinline__ static void places(uint32_t (&off)[PER], int (&at)[PER][CW], int64_t ld, int64_t rows,
                                                  int64_t r0, int tid)
    {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = tid + i * NT;
            const int k = piece_k(c), r = piece_row(c);
            const uint32_t l = (uint32_t)ld;
            int shift = 0;  // rows of a partly outside piece that lie before it
            if (KMAJOR) {
                int64_t g = r0 + r;
                if (g > rows - CW) {
                    if (g < rows && rows >= CW) shift = (int)(g - (rows - CW));
                    g = rows - CW;
                }
                if (g < 0) g = 0;  // (fewer than CW rows: checked loads)
                off[i] = 4u * ((uint32_t)k * l + (uint32_t)g);
            } else {
                const int64_t last = rows - 1 - r0;
                off[i] = 4u * ((uint32_t)(r < last ? r : (int)last) * l + (uint32_t)k);
            }
#pragma unroll
            for (int e = 0; e < CW; ++e) {
                const int p = slot(r + (e >= shift ? e - shift : CW - shift + e));
                at[i][e] = (k / 16) * STEP + p * 16 + ((((k >> 3) & 1) ^ ((p >> 3) & 1)) << 3) + (k & 4);
            }
        }
    }

    // A whole K-tile, base its first element (see places).  Buffer loads: a
    // uniform descriptor of this K-tile, the lane's 32-bit offset and a uniform
    // row offset, so no vector instruction forms an address.
    __device__ __forceinline__ void load(const float *__restrict__ base, const uint32_t (&off)[PER], int64_t ld)
    {
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, 0xffffffff, 0x00027000);
        const int ld4 = (int)ld * 4;
#pragma unroll
        for (int i = 0; i < PER; ++i)
#pragma unroll
            for (int j = 0; j < CW; ++j) {
                const auto raw = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off[i], j * ld4, 0);
                v[i][j] = __builtin_bit_cast(f32x4, raw);
            }
    }

    // The same, element by element: `left` k values remain from base (those
    // past them are 0, or `fill`, which the transform maps to 0), of a k-major
    // operand of fewer than CW rows.
    __device__ __forceinline__ void load_checked(const float *__restrict__ base, const uint32_t (&off)[PER], int64_t ld,
                                                 int64_t left, int64_t rows, const float (&fill)[PER][CW], int tid)
    {
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, 0xffffffff, 0x00027000);
        const int ld4 = (int)ld * 4;
#pragma unroll
        for (int i = 0; i < PER; ++i)
#pragma unroll
            for (int j = 0; j < CW; ++j)
#pragma unroll
                for (int e = 0; e < CW; ++e) {
                    float x = XFORM ? fill[i][e] : 0.f;
                    if (piece_k(tid + i * NT) + j < left && e < rows)
                        x = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, off[i] + 4 * e, j * ld4, 0));
                    v[i][j][e] = x;
                }
    }

    // A partial K-tile: `left` k values from base on, the matrix ending at
    // `bytes` from there.  16-byte loads as in a whole K-tile; a piece past
    // `left` gets an offset out of the descriptor's range, where loads return 0,
    // as they do for the elements of the last row's last piece past the end.
    __device__ __forceinline__ void load_part(const float *__restrict__ base, const uint32_t (&off)[PER], int64_t ld,
                                              int left, int64_t bytes, int tid)
    {
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0,
                                                            (int)(bytes < 0x7fffffff ? bytes : 0x7fffffff), 0x00027000);
#pragma unroll
        for (int i = 0; i < PER; ++i)
#pragma unroll
            for (int j = 0; j < CW; ++j) {
                const uint32_t o = off[i] + (KMAJOR ? (uint32_t)j * (uint32_t)ld * 4u : 0u);
                const auto raw = __builtin_amdgcn_raw_buffer_load_b128(
                    rsrc, piece_k(tid + i * NT) + (KMAJOR ? j : 0) < left ? o : 0xfffffff0u, 0, 0);
                v[i][j] = __builtin_bit_cast(f32x4, raw);
            }
    }

    // (values past `left` become 0, or `fill`, which the transform maps to 0)
    __device__ __forceinline__ void mask(int left, const float (&fill)[PER][CW], int tid)
    {
#pragma unroll
        for (int i = 0; i < PER; ++i)
#pragma unroll
            for (int j = 0; j < CW; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (piece_k(tid + i * NT) + (KMAJOR ? j : e) >= left)
                        v[i][j][e] = XFORM ? fill[i][KMAJOR ? e : 0] : 0.f;
    }

    __device__ __forceinline__ void store(uint16_t *lds, const int (&at)[PER][CW], uint32_t &lost,
                                          const float (&m)[PER][CW], const float (&f)[PER][CW])
    {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
#pragma unroll
            for (int j = 0; j < CW; ++j) asm volatile("" : "+v"(v[i][j]));
#pragma unroll
            for (int e = 0; e < CW; ++e) {
                uint32_t p[3][2];
#pragma unroll
                for (int j = 0; j < 4; j += 2) {
                    float x = element(i, e, j), y = element(i, e, j + 1);
                    if (XFORM != 0) {
                        x -= m[i][e];
                        y -= m[i][e];
                    }
                    if (XFORM == 2) {
                        x *= f[i][e];
                        y *= f[i][e];
                    }
                    split_pair(x, y, p[0][j / 2], p[1][j / 2], p[2][j / 2], lost);
                }
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    *reinterpret_cast<u32x2_t *>(lds + q * PART + at[i][e]) = u32x2_t{p[q][0], p[q][1]};
            }
        }
    }

    // matrix-core operand: 8 k of place p at k step s, half h
    __device__ __forceinline__ static bf16x8_t frag(const uint16_t *lds, int part, int s, int p, int h)
    {
        return *reinterpret_cast<const bf16x8_t *>(lds + part * PART + s * STEP + p * 16 + ((h ^ ((p >> 3) & 1)) << 3));
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
    // splitting waves of each operand
    static constexpr int PWA = PW / 2, PWB = PW - PWA;
    static constexpr int NT = ET + 64 * PW;
    static constexpr int BK = BK_, KS = BK / 16;
    static_assert(BK % 32 == 0, "an even number of k steps keeps the operand sets' parity");
    using LA = SplitLoader<BM, BK, 64 * PWA, A_KMAJOR, XFORM>;
    using LB = SplitLoader<BN, BK, 64 * PWB, !B_NMAJOR, XFORM>;
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

    // the transform of this thread's rows (those its pieces read, see places)
    template <class L>
    __device__ __forceinline__ static void columns(const XRegs *x, int64_t n, int64_t r0, int tid,
                                                   float (&m)[L::PER][L::CW], float (&f)[L::PER][L::CW])
    {
#pragma unroll
        for (int i = 0; i < L::PER; ++i)
#pragma unroll
            for (int e = 0; e < L::CW; ++e) {
                m[i][e] = f[i][e] = 0.f;
                if constexpr (XFORM != 0) {
                    int64_t g = r0 + L::piece_row(tid + i * L::THREADS);
                    if (g > n - L::CW) g = n - L::CW;
                    if (g < 0) g = 0;
                    if (g + e < n) m[i][e] = (float)x->mean[g + e];
                    if (XFORM == 2 && g + e < n) f[i][e] = (float)x->factor[g + e];
                }
            }
    }

    // Row / column of accumulator element v of block (tm, tn) in the tile: a
    // k-major operand's rows stand permuted (SplitLoader::row_at).
    __device__ __forceinline__ static int acc_row(int wm0, int tm, int v, int lane)
    {
        return A_KMAJOR ? wm0 + 32 * tm + 16 * (lane >> 5) + 4 * (v & 3) + (v >> 2) : Base::acc_row(wm0, tm, v, lane);
    }
    __device__ __forceinline__ static int acc_col(int wn0, int tn, int lane)
    {
        return wn0 + 32 * tn + LB::row_at(lane & 31);
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

    // Matrix waves: hi, lo += the products of nk K-tiles, the first in stage s0.
    __device__ __forceinline__ static void multiply(const uint16_t *lds, int nk, int s0, f32x16 (&hi)[TM][TN],
                                                    f32x16 (&lo)[TM][TN])
    {
        const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        const int wm0 = (w / WN) * (BM / WM), wn0 = (w % WN) * (BN / WN);
        const uint16_t *cur = lds + s0 * STAGE, *nxt = lds + (1 - s0) * STAGE;
        Frag f, g;
        __builtin_amdgcn_s_setprio(1);
        lds_barrier();  // K-tile 0 is stored
        read_frag(f, cur, 0, wm0, wn0, lane);
        __builtin_amdgcn_sched_barrier(0);
        // (the last K-tile reads operands past it, which nothing uses)
        for (int t = 0; t < nk; ++t) {
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
        __builtin_amdgcn_s_setprio(0);
    }

    // Splitting waves of one operand (L; tile at row r0 of `rows`): nk K-tiles
    // into its part of the two stages in turn, loaded two K-tiles ahead of
    // their split.  P1: the operand of a second product over the same k, or
    // NULL (k-contiguous operands only).  The partial K-tiles (np, one of each
    // product) come first, into the stages that leave the whole ones starting
    // at stage 0; their loads are in flight with those of the first whole ones.
    template <class L, bool KMAJOR>
    __device__ __forceinline__ static void produce(uint16_t *lds, const float *P, const float *P1, int64_t ld,
                                                   int64_t rows, int64_t kbeg, int64_t kend, int64_t r0, int nk,
                                                   int np, int tid, uint32_t &lost, const XRegs *xr)
    {
        float m[L::PER][L::CW], f[L::PER][L::CW];
        columns<L>(xr, rows, r0, tid, m, f);
        L l[2];
        uint32_t off[L::PER];
        int at[L::PER][L::CW];
        L::places(off, at, ld, rows, r0, tid);
        const int64_t adv = KMAJOR ? BK * ld : BK, first = KMAJOR ? kbeg * ld : r0 * ld + kbeg;
        // Whole K-tiles run a loop without branches around its loads, so the
        // waits count them exactly; loads past the last whole K-tile repeat
        // it.  Code that runs once per block tile is kept short: its
        // instructions come from memory.
        const int n1 = (int)((kend - kbeg) / BK), left = (int)((kend - kbeg) % BK);
        auto store = [&](int set, int stage) { l[set].store(lds + (stage & 1) * STAGE, at, lost, m, f); };
        if (KMAJOR && rows < L::CW) {
            // too few rows for 16-byte loads
            for (int t = 0; t < nk; ++t) {
                const int64_t kt = t < np ? n1 : t - np;
                l[0].load_checked(P + first + kt * adv, off, ld, kend - kbeg - kt * BK, rows, m, tid);
                store(0, t + np);
                lds_barrier();
            }
            lds_barrier();
            return;
        }
        const int nfast = nk - np;
        const float *p = P + first;
        int loaded = 0;
        auto load = [&](int set) {
            l[set].load(p, off, ld);
            ++loaded;
            p += loaded < nfast ? adv : 0;
            if (!KMAJOR && P1 && loaded == n1) p = P1 + first;
            __builtin_amdgcn_sched_barrier(0);
        };
        auto load_part = [&](const float *q) {
            const int64_t last = KMAJOR ? (kend - 1) * ld + rows : (rows - 1) * ld + kend;
            l[0].load_part(q + first + n1 * adv, off, ld, left, (last - first - n1 * adv) * 4, tid);
            __builtin_amdgcn_sched_barrier(0);
        };
        if (np > 0) load_part(P);
        if (nfast > 0) load(1);
#pragma unroll 1
        for (int t = 0; t < np; ++t) {
            if (!KMAJOR && t > 0) load_part(P1);
            l[0].mask(left, m, tid);
            store(0, t + np);
            lds_barrier();
        }
        if (nfast > 0) {
            load(0);
            int t = 0;
            for (; t + 2 <= nfast; t += 2) {
                store(1, 0);
                load(1);
                lds_barrier();  // K-tile t is stored, the one before is read
                store(0, 1);
                load(0);
                lds_barrier();
            }
            if (t < nfast) {
                store(1, 0);
                lds_barrier();
            }
        }
        lds_barrier();
    }

    // hi, lo += A B (+ A1 B1 where given, k-contiguous operands) over k in
    // [kbeg, kend)
    __device__ __forceinline__ static void reduce(uint16_t *lds, const float *A, const float *A1, int64_t lda,
                                                  const float *B, const float *B1, int64_t ldb, int64_t M, int64_t N,
                                                  int64_t kbeg, int64_t kend, int64_t m0, int64_t n0,
                                                  f32x16 (&hi)[TM][TN], f32x16 (&lo)[TM][TN], uint32_t &lost,
                                                  const XRegs *xr)
    {
        const int two = A1 ? 2 : 1, nk = (int)((kend - kbeg + BK - 1) / BK) * two;
        const int np = (kend - kbeg) % BK ? two : 0;
        // nk + 1 barriers on every side
        const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) - WM * WN;
        if (w < 0)
            multiply(lds, nk, np & 1, hi, lo);
        else if (w < PWA)
            produce<LA, A_KMAJOR>(lds, A, A1, lda, M, kbeg, kend, m0, nk, np, (int)threadIdx.x - ET, lost, xr);
        else
            produce<LB, !B_NMAJOR>(lds + 3 * LA::PART, B, B1, ldb, N, kbeg, kend, n0, nk, np,
                                   (int)threadIdx.x - ET - 64 * PWA, lost, xr);
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

    // This thread's share of an operand's R rows (those of the matrix) and of k
    // in [kbeg, kend): whether a finite (transformed) value reaches `limit`.
    template <bool KMAJOR, int R>
    __device__ __forceinline__ static bool reaches(const float *P, int64_t ld, int64_t rows, int64_t kbeg,
                                                   int64_t kend, int64_t r0, float limit, const XRegs *xr)
    {
        constexpr int KL = KMAJOR ? NT / R : 32, RL = KMAJOR ? R : NT / 32;  // threads over k and over rows
        static_assert(KL >= 1 && RL >= 1, "threads must cover the rows");
        const int kt = KMAJOR ? threadIdx.x / RL : threadIdx.x % KL;
        float most = 0.f;
        for (int r = KMAJOR ? threadIdx.x % RL : threadIdx.x / KL; r < R && r0 + r < rows && kt < KL; r += RL) {
            float m = 0.f, f = 1.f;
            if constexpr (XFORM != 0) m = (float)xr->mean[r0 + r];
            if constexpr (XFORM == 2) f = (float)xr->factor[r0 + r];
            const float *p = KMAJOR ? P + r0 + r : P + (r0 + r) * ld;
#pragma unroll 8
            for (int64_t k = kbeg + kt; k < kend; k += KL) {
                const float x = p[KMAJOR ? k * ld : k], y = __builtin_fabsf(XFORM ? (x - m) * f : x);
                most = __builtin_fmaxf(most, y < __builtin_inff() ? y : 0.f);
            }
        }
        return most >= limit;
    }

    // Of a tile with results that are not finite (odd) or third parts that
    // lost bits (lost): whether it has to be reduced on the FP32 cores.  acc:
    // its results, from the leading sums alone where those are not finite.
    // Reached by every thread.
    __device__ __forceinline__ static bool reduce_again(const f32x16 (&acc)[TM][TN], bool odd, bool lost,
                                                        const float *A, const float *B, const float *A1,
                                                        const float *B1, int64_t lda, int64_t ldb, int64_t M,
                                                        int64_t N, int64_t kbeg, int64_t kend, int64_t m0,
                                                        int64_t n0, const XRegs *xr)
    {
        odd = __syncthreads_or(odd);
        lost = __syncthreads_or(lost);
        if (odd && lost) return true;
        const int bits = 64 - __builtin_clzll((uint64_t)(kend - kbeg));
        // operands below 2^62 / sqrt(k) keep every sum in the finite range;
        // where bits were lost, operands below 2^32 lose less than k 2^-100 of
        // a result: nothing of one that is 2^30 times as large
        const float limit = odd ? __builtin_ldexpf(1.f, 62 - bits / 2) : 0x1p32f;
        bool again = false;
        if (lost && active()) {
            float least = __builtin_inff();
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) least = __builtin_fminf(least, __builtin_fabsf(acc[i][j][v]));
            again = least < __builtin_ldexpf(1.f, bits - 70);
        }
        if (__syncthreads_or(again)) return true;
        for (int pass = 0; pass < (A1 ? 2 : 1); ++pass)
            again = again || reaches<A_KMAJOR, BM>(pass ? A1 : A, lda, M, kbeg, kend, m0, limit, xr) ||
                    reaches<!B_NMAJOR, BN>(pass ? B1 : B, ldb, N, kbeg, kend, n0, limit, xr);
        return __syncthreads_or(again);
    }

    // acc = A B (+ A1 B1 when A1 is given) over k in [kbeg, kend); acc holds
    // the result in the matrix waves.
    __device__ __forceinline__ static void contract(float *lds, const float *A, const float *B, const float *A1,
                                                    const float *B1, int64_t lda, int64_t ldb, int64_t M,
                                                    int64_t N, int64_t kbeg, int64_t kend, int64_t m0, int64_t n0,
                                                    f32x16 (&acc)[TM][TN], const XRegs *xr)
    {
        if (kend <= kbeg) return;
        uint32_t bits = 0;
        f32x16 lo[TM][TN];
        Base::zero(acc);
        Base::zero(lo);
        uint16_t *l16 = reinterpret_cast<uint16_t *>(lds);
        reduce(l16, A, A1, lda, B, B1, ldb, M, N, kbeg, kend, m0, n0, acc, lo, bits, xr);
        const bool lost = (bits & 0xffffu) != 0;
        float x = 0.f;  // (0 * x is 0 for finite x)
        if (active()) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    lo[i][j] += acc[i][j];
#pragma unroll
                    for (int v = 0; v < 16; ++v) x = __builtin_fmaf(lo[i][j][v], 0.f, x);
                }
        }
        const bool odd = !(x == 0.f);
        // (what is rare stands behind the rest: a jump is a wait for instructions)
        if (__builtin_expect(!__syncthreads_or(odd || lost), 1)) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = lo[i][j];
        } else {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v)
                        acc[i][j][v] = __builtin_isfinite(acc[i][j][v]) ? lo[i][j][v] : acc[i][j][v];
            if (reduce_again(acc, odd, lost, A, B, A1, B1, lda, ldb, M, N, kbeg, kend, m0, n0, xr)) {
                Base::zero(acc);
                reduce_safe(lds, A, lda, B, ldb, M, N, kbeg, kend, m0, n0, acc, xr);
                if (A1) reduce_safe(lds, A1, lda, B1, ldb, M, N, kbeg, kend, m0, n0, acc, xr);
                if (active()) permute_acc(acc);
            }
        }
    }

    // The FP32 tile's accumulators (rows and columns in order) to those of
    // this tile (acc_row, acc_col).
    __device__ __forceinline__ static void permute_acc(f32x16 (&acc)[TM][TN])
    {
        const int lane = threadIdx.x & 63, l32 = lane & 31, h = lane >> 5;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const f32x16 x = acc[i][j];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int col = LB::row_at(l32);
                    if constexpr (A_KMAJOR) {
                        // row 16 h + 4 (v % 4) + v / 4 is in lane half v % 2,
                        // register 8 h + lo
                        const int lo = 4 * ((v >> 1) & 1) + (v >> 2);
                        const float a = __shfl(x[lo], col + 32 * (v & 1), 64), b = __shfl(x[lo + 8], col + 32 * (v & 1), 64);
                        acc[i][j][v] = h ? b : a;
                    } else {
                        acc[i][j][v] = __shfl(x[v], col + 32 * h, 64);
                    }
                }
            }
    }

    // The accumulators to LDS, [BM][OLD] in the tile's order.
    static constexpr int OLD = BN + 1;
    static_assert(BM * OLD + 2 * (BM + BN) <= LDS_FLOATS, "the tile and its columns' shifts must fit");
    __device__ __forceinline__ static void stage_acc(float *lds, const f32x16 (&acc)[TM][TN])
    {
        const int lane = threadIdx.x & 63, w = (int)(threadIdx.x >> 6);
        const int wm0 = (w / WN) * (BM / WM), wn0 = (w % WN) * (BN / WN);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    lds[acc_row(wm0, i, v, lane) * OLD + acc_col(wn0, j, lane)] = acc[i][j][v];
    }

    // One element of each line of the tile of C, for store_c to find them in
    // the L2: read by the matrix waves before the main loop, used (touched)
    // after it, which otherwise would wait for memory once more at its end.
    static constexpr int WARM = (BM * (BN / 32) + ET - 1) / ET;
    struct WarmC {
        float x[WARM];
        __device__ __forceinline__ void touch() const
        {
#pragma unroll
            for (int i = 0; i < WARM; ++i) asm volatile("" ::"v"(x[i]));
        }
    };
    __device__ __forceinline__ static WarmC warm_c(const float *C, int64_t ldc, int64_t M, int64_t N, int64_t m0,
                                                   int64_t n0, float beta)
    {
        WarmC w;
#pragma unroll
        for (int i = 0; i < WARM; ++i) {
            const int line = (int)threadIdx.x + i * ET;
            const int64_t row = m0 + line / (BN / 32), col = n0 + line % (BN / 32) * 32;
            w.x[i] = 0.f;
            if (beta != 0.f && active() && line < BM * (BN / 32) && row < M && col < N) w.x[i] = C[row * ldc + col];
        }
        return w;
    }

    // C = alpha acc + beta C over the in-range part of the tile (beta == 0: C
    // is not read), by all waves.  The tile goes through LDS so that every
    // access to C is a 16-byte one of whole lines and the code is a short
    // loop: a work-group runs it once, and unrolled over the accumulators it
    // was bound by its instruction fetch (covariance 2048 x 32, all 136 tiles
    // at once: 45 us).
    __device__ __forceinline__ static void store_c(float *lds, const f32x16 (&acc)[TM][TN], float *C, int64_t ldc,
                                                   int64_t M, int64_t N, int64_t m0, int64_t n0, float alpha,
                                                   float beta)
    {
        if (active()) stage_acc(lds, acc);
        __syncthreads();
        constexpr int QC = BN / 4;
#pragma unroll 4
        for (int x = threadIdx.x; x < BM * QC; x += NT) {
            const int r = x / QC, c = x % QC * 4;
            const int64_t row = m0 + r, col = n0 + c;
            if (row >= M || col >= N) continue;
            float *p = C + row * ldc + col;
            const float *t = lds + r * OLD + c;
            f32x4 y{t[0], t[1], t[2], t[3]};
            if (col + 3 < N) {
                if (beta != 0.f) {
                    const f32x4 o = *reinterpret_cast<const f32x4u *>(p);
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] = Base::combine(alpha, y[e], beta, o[e]);
                } else {
                    y *= alpha;
                }
                *reinterpret_cast<f32x4u *>(p) = y;
            } else {
                for (int e = 0; e < 4 && col + e < N; ++e)
                    p[e] = beta != 0.f ? Base::combine(alpha, t[e], beta, p[e]) : alpha * t[e];
            }
        }
    }

    __device__ __forceinline__ static void mainloop(float *lds, const float *A, int64_t lda, const float *B,
                                                    int64_t ldb, int64_t M, int64_t N, int64_t kbeg, int64_t kend,
                                                    int64_t m0, int64_t n0, f32x16 (&acc)[TM][TN], bool = true,
                                                    const XRegs *xr = nullptr)
    {
        contract(lds, A, B, nullptr, nullptr, lda, ldb, M, N, kbeg, kend, m0, n0, acc, xr);
    }
};

// The tile type of a candidate: the split tile for modes 9 to 11, else the
// FP32 cores' (LOAD and MODE are its load mode and main-loop mode).
template <int BM, int BN, int BK, int WM, int WN, int PF, bool A_KMAJOR, bool B_NMAJOR, int XFORM, int LOAD, int MODE>
using CandidateTile = typename std::conditional<
    (PF >= 9), SplitTile<BM, BN, BK, WM, WN, split_waves(PF), true, A_KMAJOR, B_NMAJOR, XFORM>,
    F32Tile<BM, BN, BK, WM, WN, A_KMAJOR, LOAD, (PF >= 9 ? 1 : MODE), B_NMAJOR, XFORM>>::type;

}  // namespace li
