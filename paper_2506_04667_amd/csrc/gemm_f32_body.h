// Tile body of the grouped GEMM in fp32 storage, on the 16-bit matrix cores without giving up fp32 precision.
//
// v_mfma_f32_32x32x2_f32 multiplies at a sixteenth of the bf16 rate, and an fp32 GEMM on it is bound by nothing else
// (a 256 x 256 x 32 K-tile takes 8.6 us, its operands arrive in 2).  The method is the published one of splitting an fp32
// value into three bf16 ones (Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For
// Higher-Precision Computations", ARITH 2019): a1 = a rounded to bf16 (8 significant bits), a2 = a - a1 rounded, a3 = what is
// left, at most 7 bits, so that a = a1 + a2 + a3 (|a| >= 2^-110; below that a3 is cut off at 2^-133, and f32_check_sums sees to
// the sums for which that counts).  Then
//   a b = a1 b1 + (a1 b2 + a2 b1) + (a1 b3 + a2 b2 + a3 b1) + (a2 b3 + a3 b2 + a3 b3)
// and the last bracket, of either sign, is below 2^-24 |a b| (rms 2^-27 |a b|): an fp32 product's own rounding at worst.  (A
// sum of one product alone is good to 3 x 2^-24, rms 0.58 x 2^-24, because the instruction keeps one guard bit where it lines
// up its terms; a rounded fp32 product: 1 and 0.42.)  Six bf16 MFMAs with fp32
// accumulation per step replace sixteen fp32 ones' time, and an accumulator is rounded 6 times per 32 terms instead of 16
// times, so sums come out more accurate than on the fp32 instruction (relative error of 2048-term sums against float64:
// 5.3e-7 for normal operands and 2.7e-7 for positive ones, 6.1e-7 and 4.0e-7 on the fp32 instruction).
// a1 and a2 have to be rounded to nearest: with a1 cut off, a2 has the sign of a, what is left out and what is
// rounded no longer cancel, and sums of positive products came out with 4.7e-7.  Values that round to an infinity
// (above 2^128 - 2^119) give NaN sums and go the way of the infinities, f32_check_sums.
// Measured, per GEMM of 275 GFLOP (64 experts of about 500 rows, K = N = 2048): 2.17 ms on the fp32 instruction (127
// TFLOP/s), 1.28 ms here (215 TFLOP/s, i.e. 1.29 PFLOP/s of bf16 products; an 8192^3 bf16 matrix product reaches 1.25 to 1.4 on
// this chip).  Counters of such a launch (1.32 ms in that run): matrix cores busy 59 % of the cycles, VALU issue 26 %, LDS 42 % (19 of
// them bank conflicts), so no unit is full: what is left are the waits at the two barriers of a K-tile and the reloads of spilled
// registers among them (the 256 x 256 bodies use all 256 and spill 4 to 7; the equal-span kernel 44 around its calls).  The
// 128 x 128 and 64 x 64 bodies convert more per product: matrix cores 36 and 28 %, VALU 33 and 44 %.
//
// Data path, per workgroup of WM x WN wavefronts and K-tile of 32:
//   * A (activations; through the gather table when there is one) comes to registers a K-tile ahead, is split there
//     once per workgroup and stored to LDS as three planes in MFMA operand order;
//   * B (weights; [k][n] as stored, or [n][k] for NT) goes to LDS raw by direct copies and is split by the wavefronts
//     as they read their operands: a wavefront's columns are only needed by the WM wavefronts of its column, and raw B
//     takes two thirds of the LDS that planes would: 2 x (48 + 32) KB for a 256 x 256 tile, all of a CU's 160 KB;
//   * a K-tile is 2 TM blocks: the first TM multiply the left half of the wavefront's columns, the others the right
//     half.  The pieces of the half that is not being multiplied are made meanwhile (the right half's of this K-tile
//     during the left half's products, the left half's of the next one during the right half's), so conversions ride
//     in the shadow of the MFMAs: 350 VALU operations per wavefront, 264 of them splits, against 192 MFMAs of four issue slots each.
// Operand order: the weight piece is the first MFMA operand, so a lane holds, for one row, four consecutive columns.
#pragma once
#include "common.h"
#include "kernels.h"
#include "lds_copy.h"

#include <type_traits>

namespace moe {
namespace {

template <bool NT, int WM_, int WN_, int TM_, int TN_>
struct F32Cfg {
    static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_;        // wavefronts; 16 x 16 MFMA tiles per wavefront
    static constexpr int BM = WM * TM * 16, BN = WN * TN * 16, BK = 32;
    static constexpr int WAVES = WM * WN, THREADS = WAVES * 64;
    static constexpr int A_PLANE = BM * 64;             // bf16 [BM][32] in operand order
    static constexpr int A_BYTES = 3 * A_PLANE;
    static constexpr int B_BYTES = BN * 128;            // fp32 [32][BN] or [BN][32]
    static constexpr int STAGE = A_BYTES + B_BYTES;
    static constexpr int LDS = 2 * STAGE;
    static constexpr int A_ITEMS = BM * 4 / THREADS;    // runs of 8 k of one row per thread
    static constexpr int B_COPIES = B_BYTES / 1024 / WAVES;
    static_assert(TM % 2 == 0 && TN % 2 == 0 && BM * 4 % THREADS == 0 && B_BYTES % (1024 * WAVES) == 0, "tile / threads mismatch");
    static_assert(LDS <= 160 * 1024, "LDS budget of a gfx950 CU");
};

typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

// two values into their three pieces each, as packed pairs
__device__ __forceinline__ void split2(float v0, float v1, uint32_t& p0, uint32_t& p1, uint32_t& p2) {
    p0 = pack2<BF16>(v0, v1);
    const float r0 = v0 - __builtin_bit_cast(float, p0 << 16), r1 = v1 - __builtin_bit_cast(float, p0 & 0xffff0000u);
    p1 = pack2<BF16>(r0, r1);
    const float s0 = r0 - __builtin_bit_cast(float, p1 << 16), s1 = r1 - __builtin_bit_cast(float, p1 & 0xffff0000u);
    p2 = __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, s1), __builtin_bit_cast(uint32_t, s0), 0x07060302u);   // the two upper halves
}

struct Pieces { u32x4 p[3]; };                          // 8 consecutive k as three bf16 MFMA operands (exact sum)

__device__ __forceinline__ Pieces split8(const float (&v)[8]) {
    Pieces o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        uint32_t a, b, c;
        split2(v[2 * j], v[2 * j + 1], a, b, c);
        o.p[0][j] = a; o.p[1][j] = b; o.p[2][j] = c;
    }
    return o;
}

__device__ __forceinline__ f32x4 mma_bf16(const u32x4& w, const u32x4& x, const f32x4& c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, x), c, 0, 0, 0);
}

// Sums that the split products do not get right are made again, on the fp32 instruction: NaN and those below 2^-80 (but not 0).
//  * The pieces of an infinity are an infinity and NaNs, so every sum it enters comes out NaN, where fp32 products give an
//    infinity (or a NaN); an overflowing product's smaller terms can meet its infinity with the other sign too.
//  * Below 2^-110 a value's last piece has bits that bf16 has no room for, up to 2^-133: more than 2^-24 of a sum of at least
//    2^-80 only where the other factor is above 2^29.  (Values below 2^-134 count as zero, and a sum of nothing else is 0.)
// A wavefront decides for its own part of the tile once its sums are there (two operations per sum), and reads the operands
// from memory itself: no other wavefront takes part.  A layer with nothing but such sums (T = 4096, H = I = 2048, E = 16, x
// times 2^-100, or a NaN in every sum) takes 3.1 ms, 0.97 ms with ordinary ones; with one scalar sum after the other it was
// 74 ms.
constexpr uint32_t kSmallSum = 0x17800000u;             // 2^-80
template <bool NT, int WM, int TM, int TN>
__device__ __forceinline__ void f32_check_sums(const GemmArgs& a, f32x4 (&acc)[TM][TN], int grp, int row0, int n0, int rows, int wm, int wn,
                                               int live, int r16, int kq, int k_begin, int k_end) {
    uint32_t least = 0xffffffffu;                       // least magnitude, doubled and less one: zero is the largest
    bool nan = false;
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const f32x4 v = acc[t][tn];
#pragma unroll
            for (int q = 0; q < 4; ++q) least = min(least, (__builtin_bit_cast(uint32_t, (float)v[q]) << 1) - 1u);
            nan |= __builtin_isunordered(v[0], v[1]) | __builtin_isunordered(v[2], v[3]);
        }
    if (!__any(nan || least < 2 * kSmallSum - 1u)) return;
    auto tile_row = [&](int t) __attribute__((always_inline)) { return ((t >> 1) * WM + wm) * 32 + (t & 1) * 16; };
    const float* const A = (const float*)a.A + (a.a_row_index ? (size_t)0 : (size_t)grp * a.a_group_stride);
    const float* const B = (const float*)a.B + (size_t)grp * a.b_group_stride;
    const float* x[TM];                                 // rows and columns beyond the last repeat it, as above
    const float* w[TN];
#pragma unroll
    for (int t = 0; t < TM; ++t) {
        const int r = min(row0 + tile_row(t) + r16, rows - 1);
        x[t] = A + (size_t)(a.a_row_index ? a.a_row_index[(size_t)grp * a.a_index_stride + r] : r) * a.lda;
    }
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        const int n = min(n0 + (wn * TN + tn) * 16 + r16, a.N - 1);
        w[tn] = B + (NT ? (size_t)n * a.ldb : (size_t)n);
    }
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) acc[t][tn] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    for (int k0 = k_begin; k0 < k_end; k0 += 16) {      // lane group kq: k0 + 4 kq .. + 3, one of them per instruction
        const int k = k0 + kq * 4;
        const bool ok = k < k_end;                      // k_end is a multiple of 8
        f32x4 xv[TM], wv[TN];
#pragma unroll
        for (int t = 0; t < TM; ++t) xv[t] = ok && t < live ? *(const f32x4*)(x[t] + k) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            if constexpr (NT) {
                wv[tn] = ok ? *(const f32x4*)(w[tn] + k) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) wv[tn][j] = ok ? w[tn][(size_t)(k + j) * a.ldb] : 0.0f;
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int t = 0; t < TM; ++t)
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) acc[t][tn] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[tn][j], xv[t][j], acc[t][tn], 0, 0, 0);
    }
}

// Bias, activation and store of a wavefront's sums: four consecutive columns of one row per lane and MFMA tile.  With
// `partial` the raw sums of the row tiles with live rows go there instead; with ADD they are added to what C holds (no bias,
// no activation).
template <bool NT, int WM, int TM, int TN, int BN, bool ADD = false>
__device__ __forceinline__ void f32_epilogue(const GemmArgs& a, f32x4 (&acc)[TM][TN], int grp, int row0, int n0, int rows, int wm, int wn,
                                             int live, int r16, int kq, float* __restrict__ partial) {
    auto tile_row = [&](int t) __attribute__((always_inline)) { return ((t >> 1) * WM + wm) * 32 + (t & 1) * 16; };
    if (partial) {
#pragma unroll
        for (int t = 0; t < TM; ++t) {
            if (t >= live) break;
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
                *(f32x4*)(partial + (size_t)(tile_row(t) + r16) * BN + (wn * TN + tn) * 16 + kq * 4) = acc[t][tn];
        }
        return;
    }
    const int N = a.N, act = a.act, ldc = a.ldc;
    float* const c_base = (float*)a.C + (size_t)grp * a.c_group_stride;
    const bool vec = (N & 3) == 0 && (ldc & 3) == 0;    // whole 16-byte stores (the group stride is a multiple of 4 too)
    const float* const bias = a.bias ? (const float*)a.bias + (size_t)grp * a.bias_group_stride : nullptr;
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        const int col = n0 + (wn * TN + tn) * 16 + kq * 4;
        if (col >= N) continue;
        float bv[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (bias) {
#pragma unroll
            for (int q = 0; q < 4; ++q) bv[q] = bias[min(col + q, N - 1)];
        }
#pragma unroll
        for (int t = 0; t < TM; ++t) {
            const int row = row0 + tile_row(t) + r16;
            if (row >= rows) continue;
            f32x4 v;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = ADD ? acc[t][tn][q] : apply_act(acc[t][tn][q] + bv[q], act);
            float* const c = c_base + (size_t)row * ldc + col;
            if (vec) {
                if constexpr (ADD) v += *(const f32x4*)c;
                *(f32x4*)c = v;
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (col + q < N) c[q] = ADD ? v[q] + c[q] : v[q];
            }
        }
    }
}

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// K-tiles [kt0, kt1) (kt0 < kt1) of the BM x BN tile at (row0, n0) of group grp, whose live rows are `rows`.
// partial == nullptr: bias, activation and the store to C.  Otherwise the raw sums go to partial[BM][BN] (row-major)
// for a later pass to add up, or with ADD they are added to C.  Ends with a workgroup barrier after the last LDS access, so the caller may start another
// tile at once.  K must be a multiple of 8; lda, ldb and the group strides multiples of 4; operands 16-byte aligned.
template <bool NT, int WM, int WN, int TM, int TN, bool ADD = false>
__device__ __forceinline__ void f32_tile(const GemmArgs& a, unsigned char* smem, int grp, int row0, int n0, int rows, int kt0, int kt1,
                                         float* __restrict__ partial) {
    using C = F32Cfg<NT, WM, WN, TM, TN>;
    constexpr int BM = C::BM, BN = C::BN, BK = C::BK, THREADS = C::THREADS, STAGE = C::STAGE, A_PLANE = C::A_PLANE;
    constexpr int A_ITEMS = C::A_ITEMS, B_COPIES = C::B_COPIES, HN = TN / 2, NB = 2 * TM;

    // operands in device memory, said explicitly: a caller that is not a kernel passes the arguments through memory
    typedef const __attribute__((address_space(1))) float* gfloat;
    typedef const __attribute__((address_space(1))) f32x4* gvec;
    const int K = uniform(a.K), N = uniform(a.N), lda = uniform(a.lda), ldb = uniform(a.ldb);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uniform(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int r16 = lane & 15, kq = lane >> 4;
    const uint32_t lds_base = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;

    // ---- A: global -> registers -> three planes.  Item i of a thread: 8 consecutive k of one row.  Rows at or beyond
    // the live ones repeat the last live row (their sums are never stored); k beyond K are zeros. ----
    const gfloat a_base = (gfloat)uniform((const unsigned char*)((const float*)a.A + (a.a_row_index ? (size_t)0 : (size_t)grp * a.a_group_stride)));
    int a_row[A_ITEMS];                                 // row numbers, not pointers: half the registers
    const int koct = tid & 3;
    // item i's place in a plane is (THREADS / 4) rows, i.e. that many / 16 KB, after item 0's
    const int a_st = (tid >> 6) * 1024 + koct * 256 + ((((tid >> 2) & 15) + 4 * koct) & 15) * 16;   // rotated: conflict-free both ways
#pragma unroll
    for (int i = 0; i < A_ITEMS; ++i) {
        const int r = (tid + i * THREADS) >> 2;
        const int rr = min(row0 + r, rows - 1);
        a_row[i] = a.a_row_index ? a.a_row_index[(size_t)grp * a.a_index_stride + rr] : rr;
    }
    // the large tile has registers for one item in flight only: its second item is loaded when the first has been stored
    constexpr bool ONE = TM == 8;
    f32x4 ra[ONE ? 1 : A_ITEMS][2];
    auto load_a = [&](int kt, int i) __attribute__((always_inline)) {
        const int k0 = kt * BK;
        f32x4 (&r)[2] = ra[ONE ? 0 : i];
        int row = a_row[i];
        asm volatile("" : "+v"(row));                   // so that the address is made here
        const gfloat p = a_base + (size_t)(uint32_t)row * (uint32_t)lda + koct * 8 + k0;
        if (k0 + BK <= K) {
            r[0] = *(gvec)p;
            r[1] = *(gvec)(p + 4);
        } else {
            const bool ok = k0 + koct * 8 < K;
            r[0] = ok ? *(gvec)p : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            r[1] = ok ? *(gvec)(p + 4) : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    };
    auto store_a = [&](int i, int stage_off) __attribute__((always_inline)) {
        unsigned char* const at = smem + stage_off + a_st + i * (THREADS / 64) * 1024;
#pragma unroll
        for (int h = 0; h < 2; ++h) {                   // four k at a time: half the registers on the way
            uint32_t o[3][2];
#pragma unroll
            for (int q = 0; q < 2; ++q) split2(ra[ONE ? 0 : i][h][2 * q], ra[ONE ? 0 : i][h][2 * q + 1], o[0][q], o[1][q], o[2][q]);
#pragma unroll
            for (int p = 0; p < 3; ++p) *(u32x2*)(at + p * A_PLANE + h * 8) = u32x2{o[p][0], o[p][1]};
            if (ONE && !NT) asm volatile("" ::: "memory");     // (not merged into one 16-byte store that needs all of them at once)
        }
    };

    // ---- B: direct copies, 1 KB per wavefront and copy.  [k][n]: chunk c (16 bytes) of row k lives at
    // c ^ (((k >> 3) & 3) << 2), so the four k-octets that a wavefront reads together lie in different banks;
    // [n][k]: chunk c of row n lives at c ^ ((n >> 1) & 7).  Columns beyond N (rows beyond K) repeat valid ones: the
    // sums are never stored (the A values they meet are zero). ----
    const unsigned char* const b_grp = uniform((const unsigned char*)((const float*)a.B + (size_t)grp * a.b_group_stride + (NT ? (size_t)n0 * ldb : (size_t)0)));
    // offset of copy j's lanes from the K-tile's base: copy j is RPC rows after copy 0, with the same columns but for NT's
    // chunk 4 places on in odd copies, so one or two lane offsets and a scalar step serve all copies
    constexpr int RPC = NT ? 8 : 256 / BN;              // rows of one copy
    auto b_lane_off = [&](int j, int k_left, int lane) __attribute__((always_inline)) -> uint32_t {
        if constexpr (NT) {
            const int r = (wave * B_COPIES + j) * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
            return (uint32_t)(min(n0 + r, N - 1) - n0) * (uint32_t)(ldb * 4) + (uint32_t)min(c * 4, k_left - 4) * 4;
        } else {
            const int k = (wave * B_COPIES + j) * RPC + lane / (BN / 4), c = (lane % (BN / 4)) ^ (((k >> 3) & 3) << 2);
            return (uint32_t)min(k, k_left - 1) * (uint32_t)(ldb * 4) + (uint32_t)min(n0 + c * 4, ldb - 4) * 4;
        }
    };
    static_assert(NT || B_COPIES * RPC <= 8, "a wavefront's rows of B lie in one k-octet: one swizzle for all its copies");
    uint32_t b_off[NT ? 2 : 1];
#pragma unroll
    for (int j = 0; j < (NT ? 2 : 1); ++j) b_off[j] = b_lane_off(j, BK, lane) - (uint32_t)(j * RPC) * (uint32_t)(ldb * 4);
    auto issue_b = [&](int kt, int stage_off, int first, int last) __attribute__((always_inline)) {
        const int k0 = kt * BK;
        const unsigned char* base = b_grp + (NT ? (size_t)k0 * 4 : (size_t)k0 * ldb * 4);
        const uint32_t d = lds_base + stage_off + C::A_BYTES + wave * (B_COPIES * 1024);
        if (k0 + BK <= K && (!NT || n0 + BN <= N)) {
#pragma unroll
            for (int j = first; j < last; ++j) copy_to_lds_stream(base + (size_t)(j * RPC) * ldb * 4, b_off[NT ? j & 1 : 0], d + j * 1024);
        } else {
            int lane_t = lane;                          // opaque to the compiler: the tail's offsets are computed here, not kept in registers
            asm volatile("" : "+v"(lane_t));
#pragma unroll
            for (int j = first; j < last; ++j) copy_to_lds_stream(base, b_lane_off(j, K - k0, lane_t), d + j * 1024);
        }
    };

    // ---- operand reads ----
    // 32-row blocks of the tile are dealt to the wavefront rows in turn, so that few live rows spread over all of them:
    // the wavefront's row tile t covers rows ((t >> 1) * WM + wm) * 32 + (t & 1) * 16 + 0..15
    auto tile_row = [&](int t) __attribute__((always_inline)) { return ((t >> 1) * WM + wm) * 32 + (t & 1) * 16; };
    const int x_rd = wm * 2048 + kq * 256 + ((r16 + 4 * kq) & 15) * 16;
    auto read_x = [&](int t, int stage_off, int p) __attribute__((always_inline)) {
        return *(const u32x4*)(smem + stage_off + x_rd + ((t >> 1) * WM * 2 + (t & 1)) * 1024 + p * A_PLANE);
    };
    const int bn = wn * TN * 16 + r16;                  // column of tile 0 of this lane
    const int w_rd = C::A_BYTES + (NT ? bn * 128 : kq * 8 * BN * 4 + ((((bn >> 2) ^ (kq << 2)) << 4) | ((bn & 3) << 2)));
    const int w_sw = NT ? (bn >> 1) & 7 : 0;            // the same for every column tile of the lane
    auto read_w = [&](int tn, int stage_off, float (&v)[8]) __attribute__((always_inline)) {
        if constexpr (NT) {
            const unsigned char* p = smem + stage_off + w_rd + tn * 16 * 128;
            const f32x4 lo = *(const f32x4*)(p + (((2 * kq) ^ w_sw) << 4)), hi = *(const f32x4*)(p + (((2 * kq + 1) ^ w_sw) << 4));
#pragma unroll
            for (int q = 0; q < 4; ++q) { v[q] = lo[q]; v[4 + q] = hi[q]; }
        } else {
            // chunk (column / 4) ^ (kq << 2): the swizzle moves the 16-column tile, so a tile's address is one XOR away
            int at = (stage_off + w_rd) ^ (tn << 6);
            asm volatile("" : "+v"(at));                // one address per tile, the rows in the instructions' offsets
            const unsigned char* p = smem + at;
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = *(const float*)(p + q * BN * 4);
        }
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    Pieces wf[TN], xf;
    float rw[8];                                        // raw weights on their way to the next wf

    // row tiles of this wavefront with live rows (uniform over the wavefront)
    const int live = min(2 * (max((rows - row0 + 31) / 32 - wm + WM - 1, 0) / WM), TM);

    // ---- schedule of a K-tile: block q multiplies row tile q % TM with the left (q < TM) or right half of the columns.
    // Around the products: the right half's pieces are made early in the K-tile, the next K-tile's A planes are stored in
    // the middle and the left half's next pieces are made at the end.  Barrier Y: every wavefront has finished the
    // previous K-tile, so the other stage's A planes may be overwritten.  Barrier X: the next K-tile's A planes are
    // written, its B copies have landed, and everybody has read this K-tile's raw B, so the copies after next may start. ----
    struct At { int read, convert; };
    constexpr At kRight[2] = {{0, 1}, {TM == 8 ? 2 : 1, TM == 8 ? 3 : 2}};
    constexpr int kY = TM == 8 ? 4 : TM == 4 ? 3 : 1;
    constexpr int kA = TM == 1 ? 0 : TM == 2 ? 1 : 4, kA2 = 9;          // blocks that store the items (large tile: item 0, item 1)
    constexpr int kX = TM == 8 ? 10 : TM == 4 ? 5 : 2;
    constexpr At kLeft[2] = {{TM == 8 ? 11 : kX, TM == 8 ? 12 : kX + 1}, {TM == 8 ? 13 : kX + 1, TM == 8 ? 14 : kX + 2}};
    static_assert(TM == 8 || TM == 4 || (TM == 2 && HN == 1), "the schedule is laid out for these");
    static_assert(!ONE || A_ITEMS == 2, "the large tile's schedule has two items");
    const int nk = kt1 - kt0;

    auto block = [&](auto q_tag, auto live_tag, int u, int s_off) __attribute__((always_inline)) {
        constexpr int q = decltype(q_tag)::value, LIVE = decltype(live_tag)::value;
        const int n_off = STAGE - s_off;                // the next K-tile's stage
        if constexpr (q == kY) asm volatile("s_barrier" ::: "memory");
        if constexpr (q == kX) {
            wait_copies_and_barrier<0>();
            if (u + 2 < nk) {
#pragma unroll
                for (int i = 0; i < (ONE ? 1 : A_ITEMS); ++i) load_a(kt0 + u + 2, i);
            }
            if (ONE) __builtin_amdgcn_sched_barrier(0);
        }
        // The large tile's copies of B go out over the blocks that are left: together behind the barrier, 32 copies of 16 address cycles hold the
        // wavefronts up (T = 16384, H = I = 2048, E = 64 2797 -> 2689 us per layer, matrix cores busy 55 -> 59 % of the cycles; the smaller tiles lose
        // up to 4 % by it, and the equal-span kernel neither gains nor loses on average: E = 24 of 4096 tokens 0.99, E = 8 1.04 times)
        constexpr int OVER = ONE ? NB - kX : 1;
        if constexpr (q >= kX && q < kX + OVER) {
            constexpr int c0 = (q - kX) * B_COPIES / OVER, c1 = (q - kX + 1) * B_COPIES / OVER;
            if constexpr (c1 > c0) {
                if (u + 2 < nk) issue_b(kt0 + u + 2, s_off, c0, c1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (LIVE > 0) {
#pragma unroll
            for (int j = 0; j < HN; ++j) {
                // (the empty asm keeps the compiler from moving a conversion down to the first product that needs it)
                auto convert = [&](Pieces& w) __attribute__((always_inline)) {
                    w = split8(rw);
                    asm volatile("" : "+v"(w.p[0]), "+v"(w.p[1]), "+v"(w.p[2]));
                };
                if (q == kRight[j].convert) convert(wf[HN + j]);
                if (q == kLeft[j].convert) convert(wf[j]);
            }
#pragma unroll
            for (int j = 0; j < HN; ++j) {
                if (q == kRight[j].read) read_w(HN + j, s_off, rw);
                if (q == kLeft[j].read) read_w(j, n_off, rw);
            }
        }
        if constexpr (q == kA) {
#pragma unroll
            for (int i = 0; i < (ONE ? 1 : A_ITEMS); ++i) store_a(i, n_off);
        }
        if constexpr (ONE && q == kA2) store_a(1, n_off);
        // the rows of the next block with products; after the last one they are the next K-tile's, whose planes are only
        // written once barrier X is passed: a wavefront that is done with its products before reads them there
        constexpr int next = q % TM + 1 < LIVE ? q + 1 : q < TM ? TM : NB;
        constexpr bool late = LIVE > 0 && TM + LIVE - 1 < kX;
        if constexpr (late && q == kX) {
#pragma unroll
            for (int px = 0; px < 3; ++px) xf.p[px] = read_x(0, n_off, px);
        }
        if constexpr (q % TM < LIVE) {
            // each piece of the rows is read for the next block once this one is done with it: ordered like this, every
            // read has at least half a block to arrive and no second set of registers is needed
            constexpr int t = q % TM, h = q / TM;
            auto mma = [&](int pw, int px) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < HN; ++j) acc[t][h * HN + j] = mma_bf16(wf[h * HN + j].p[pw], xf.p[px], acc[t][h * HN + j]);
            };
            auto fetch = [&](int px) __attribute__((always_inline)) {
                if constexpr (next < NB || !late) xf.p[px] = read_x(next % TM, next < NB ? s_off : n_off, px);
            };
            static_assert(next < NB || late || q >= kX, "the next K-tile's planes are read after barrier X");
            mma(0, 2);
            fetch(2);
            mma(1, 1);
            mma(0, 1);
            fetch(1);
            mma(2, 0);
            mma(1, 0);
            mma(0, 0);
            fetch(0);
#pragma unroll
            for (int i = 0; i < 6; ++i) {
#pragma unroll
                for (int j = 0; j < HN; ++j) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA,
                    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);  // then up to four VALU operations
                }
                if (i == 0 || i == 2 || i == 5) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // the LDS read of the freed piece
                if (i == 3) __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);                      // and those of the raw weights
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (ONE && q == kA) {
            load_a(min(kt0 + u + 1, kt1 - 1), 1);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // one copy of the loop per count of live row tiles: products with rows that nobody stores are left out
    auto main_loop = [&](auto live_tag) __attribute__((always_inline)) {
        int s_off = 0;
        for (int u = 0; u < nk; ++u) {
            static_for<0, NB>([&](auto q_tag) __attribute__((always_inline)) { block(q_tag, live_tag, u, s_off); });
            s_off = STAGE - s_off;
        }
    };

    issue_b(kt0, 0, 0, B_COPIES);
    if (!ONE) {
#pragma unroll
        for (int i = 0; i < A_ITEMS; ++i) load_a(kt0, i);
    }
#pragma unroll
    for (int i = 0; i < A_ITEMS; ++i) {
        if (ONE) load_a(kt0, i);
        store_a(i, 0);
    }
    wait_copies_and_barrier<0>();
    if (nk > 1) {
        issue_b(kt0 + 1, STAGE, 0, B_COPIES);
#pragma unroll
        for (int i = 0; i < (ONE ? 1 : A_ITEMS); ++i) load_a(kt0 + 1, i);
    }
#pragma unroll
    for (int j = 0; j < HN; ++j) {
        read_w(j, 0, rw);
        wf[j] = split8(rw);
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) xf.p[p] = read_x(0, 0, p);
    if (live == TM) main_loop(std::integral_constant<int, TM>{});
    else if (live == 0) main_loop(std::integral_constant<int, 0>{});
    else if (TM >= 4 && live == 2) main_loop(std::integral_constant<int, (TM >= 4 ? 2 : TM)>{});
    else if (TM >= 8 && live == 4) main_loop(std::integral_constant<int, (TM >= 8 ? 4 : TM)>{});
    else if (TM >= 8) main_loop(std::integral_constant<int, (TM >= 8 ? 6 : TM)>{});
    wait_copies_and_barrier<0>();

    f32_check_sums<NT, WM, TM, TN>(a, acc, grp, row0, n0, rows, wm, wn, live, r16, kq, kt0 * BK, min(kt1 * BK, K));
    f32_epilogue<NT, WM, TM, TN, BN, ADD>(a, acc, grp, row0, n0, rows, wm, wn, live, r16, kq, partial);
}

// The same tile body for at most 64 rows (a decode step's experts, the last rows of a larger group): 64 x 256, 8 wavefronts
// side by side with 64 x 32 each, so every weight is split by the one wavefront that needs it.  With few rows the matrix
// cores have a quarter of the large tile's products and the weights' way from HBM is what counts (2.4 us per K-tile at 64 rows
// with all CUs streaming, 6.3 us for 256 rows): both operands come by
// direct copies through a ring of three K-tiles, requested two K-tiles ahead, and a K-tile has one barrier.  During the
// products of K-tile u the next one's rows go from the ring to the planes (4 k per thread) and its weights from the ring to
// registers.
struct F32Low {
    static constexpr int BM = 64, BN = 256, BK = 32, TM = 4, TN = 2, WAVES = 8, THREADS = 512, RING = 3;
    static constexpr int A_RAW = BM * 128, B_RAW = BN * 128, A_PLANE = BM * 64;
    static constexpr int A_AT = RING * B_RAW, PLANES_AT = A_AT + RING * A_RAW;
    static constexpr int LDS = PLANES_AT + 2 * 3 * A_PLANE;
    static constexpr int COPIES = 1 + B_RAW / 1024 / WAVES;             // per wavefront and K-tile
};
static_assert(F32Low::LDS <= 160 * 1024, "LDS budget of a gfx950 CU");

template <bool NT>
__device__ __forceinline__ void f32_tile_low(const GemmArgs& a, unsigned char* smem, int grp, int row0, int n0, int rows, int kt0, int kt1,
                                             float* __restrict__ partial) {
    using C = F32Low;
    constexpr int BN = C::BN, BK = C::BK, TM = C::TM, TN = C::TN, A_PLANE = C::A_PLANE;
    const int K = uniform(a.K), N = uniform(a.N), lda = uniform(a.lda), ldb = uniform(a.ldb);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uniform(tid >> 6);
    const int r16 = lane & 15, kq = lane >> 4;
    const uint32_t lds_base = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;

    // ---- copies: one of 8 rows x 128 bytes of A (chunk c of row r at c ^ ((r >> 1) & 7)), four of B as in f32_tile ----
    const unsigned char* const b_grp = uniform((const unsigned char*)((const float*)a.B + (size_t)grp * a.b_group_stride + (NT ? (size_t)n0 * ldb : (size_t)0)));
    const unsigned char* const a_grp = uniform((const unsigned char*)((const float*)a.A + (a.a_row_index ? (size_t)0 : (size_t)grp * a.a_group_stride)));
    const unsigned char* a_lane;                        // this lane's row and chunk, without the K-tile
    int a_chunk;
    {
        const int r = wave * 8 + (lane >> 3);
        const int rr = min(row0 + r, rows - 1);
        const int row = a.a_row_index ? a.a_row_index[(size_t)grp * a.a_index_stride + rr] : rr;
        a_chunk = (lane & 7) ^ ((r >> 1) & 7);
        a_lane = a_grp + (size_t)row * lda * 4;
    }
    auto b_lane_off = [&](int j, int k_left) __attribute__((always_inline)) -> uint32_t {
        if constexpr (NT) {
            const int r = (wave * 4 + j) * 8 + (lane >> 3), c = (lane & 7) ^ ((r >> 1) & 7);
            return (uint32_t)(min(n0 + r, N - 1) - n0) * (uint32_t)(ldb * 4) + (uint32_t)min(c * 4, k_left - 4) * 4;
        } else {
            const int k = wave * 4 + j, c = lane ^ (((k >> 3) & 3) << 2);
            return (uint32_t)min(k, k_left - 1) * (uint32_t)(ldb * 4) + (uint32_t)min(n0 + c * 4, ldb - 4) * 4;
        }
    };
    uint32_t b_off[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) b_off[j] = b_lane_off(j, BK);
    const int nk = kt1 - kt0;
    int slot = 0;                                       // ring slot of the next request
    auto issue = [&](int kt) __attribute__((always_inline)) {
        const int k0 = kt * BK, left = K - k0;
        copy_to_lds_lane(a_lane + (size_t)k0 * 4 + min(a_chunk * 4, left - 4) * 4, lds_base + C::A_AT + slot * C::A_RAW + wave * 1024);
        const unsigned char* base = b_grp + (NT ? (size_t)k0 * 4 : (size_t)k0 * ldb * 4);
        const uint32_t d = lds_base + slot * C::B_RAW + wave * 4096;
#pragma unroll
        for (int j = 0; j < 4; ++j) copy_to_lds_stream(base, left >= BK ? b_off[j] : b_lane_off(j, left), d + j * 1024);
        slot = slot == C::RING - 1 ? 0 : slot + 1;
    };

    // ---- this thread's share of the A split: chunk sc of row sr ----
    const int sr = tid >> 3, sc = tid & 7;
    const int s_rd = C::A_AT + sr * 128 + ((sc ^ ((sr >> 1) & 7)) << 4);
    const int s_wr = C::PLANES_AT + (sr >> 4) * 1024 + (sc >> 1) * 256 + ((((sr & 15) + 4 * (sc >> 1)) & 15) << 4) + (sc & 1) * 8;
    const int x_rd = C::PLANES_AT + kq * 256 + ((r16 + 4 * kq) & 15) * 16;
    const int bn = wave * 32 + r16;
    const int w_rd = NT ? bn * 128 : kq * 8 * BN * 4 + ((((bn >> 2) ^ (kq << 2)) << 4) | ((bn & 3) << 2));
    const int w_sw = NT ? (bn >> 1) & 7 : 0;

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int live = min(2 * ((rows - row0 + 31) / 32), TM);

    // K-tile kt (in ring slot `from`): its rows to planes `to`, its weights to `w`
    auto take = [&](int kt, int from, int to, Pieces (&w)[TN]) __attribute__((always_inline)) {
        f32x4 v = *(const f32x4*)(smem + s_rd + from * C::A_RAW);
        if (kt * BK + sc * 4 >= K) v = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        float rw[TN][8];
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            if constexpr (NT) {
                const unsigned char* p = smem + from * C::B_RAW + w_rd + tn * 16 * 128;
                const f32x4 lo = *(const f32x4*)(p + (((2 * kq) ^ w_sw) << 4)), hi = *(const f32x4*)(p + (((2 * kq + 1) ^ w_sw) << 4));
#pragma unroll
                for (int q = 0; q < 4; ++q) { rw[tn][q] = lo[q]; rw[tn][4 + q] = hi[q]; }
            } else {
                int at = (from * C::B_RAW + w_rd) ^ (tn << 6);
                asm volatile("" : "+v"(at));            // one address per tile, the rows in the instructions' offsets
#pragma unroll
                for (int q = 0; q < 8; ++q) rw[tn][q] = *(const float*)(smem + at + q * BN * 4);
            }
        }
        uint32_t o[3][2];
        split2(v[0], v[1], o[0][0], o[1][0], o[2][0]);
        split2(v[2], v[3], o[0][1], o[1][1], o[2][1]);
#pragma unroll
        for (int p = 0; p < 3; ++p) *(u32x2*)(smem + s_wr + to * 3 * A_PLANE + p * A_PLANE) = u32x2{o[p][0], o[p][1]};
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            w[tn] = split8(rw[tn]);
            asm volatile("" : "+v"(w[tn].p[0]), "+v"(w[tn].p[1]), "+v"(w[tn].p[2]));   // made here, not where first needed
        }
    };
    auto multiply = [&](int planes, auto live_tag, const Pieces (&w)[TN]) __attribute__((always_inline)) {
        constexpr int LIVE = decltype(live_tag)::value;
#pragma unroll
        for (int t = 0; t < LIVE; ++t) {
            Pieces x;
#pragma unroll
            for (int p = 0; p < 3; ++p) x.p[p] = *(const u32x4*)(smem + x_rd + planes * 3 * A_PLANE + t * 1024 + p * A_PLANE);
            constexpr int PW[6] = {0, 1, 0, 2, 1, 0}, PX[6] = {2, 1, 1, 0, 0, 0};
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) acc[t][tn] = mma_bf16(w[tn].p[PW[q]], x.p[PX[q]], acc[t][tn]);
        }
    };

    issue(kt0);
    if (nk > 1) issue(kt0 + 1);
    if (nk > 2) issue(kt0 + 2);
    if (nk > 2) wait_copies_and_barrier<2 * C::COPIES>();
    else wait_copies_and_barrier<0>();
    Pieces w0[TN], w1[TN];
    take(kt0, 0, 0, w0);
    auto main_loop = [&](auto live_tag) __attribute__((always_inline)) {
        int next = 1;                                   // ring slot of K-tile u + 1
        // even K-tiles use w0 and planes 0, odd ones w1 and planes 1
        auto step = [&](int u, int par, const Pieces (&w)[TN], Pieces (&wn)[TN]) __attribute__((always_inline)) {
            // K-tile u + 1 has landed and everybody has taken K-tile u out of the ring: its slot is free again
            if (u + 2 < nk) wait_copies_and_barrier<C::COPIES>();
            else wait_copies_and_barrier<0>();
            if (u + 3 < nk) issue(kt0 + u + 3);
            take(kt0 + u + 1, next, par ^ 1, wn);       // (after the last K-tile: old data that nobody uses)
            multiply(par, live_tag, w);
#pragma unroll
            for (int i = 0; i < 12 * decltype(live_tag)::value; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // one MFMA,
                __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);      // then up to four VALU operations
            }
            __builtin_amdgcn_sched_barrier(0);
            next = next == C::RING - 1 ? 0 : next + 1;
        };
        for (int u = 0; u < nk; u += 2) {
            step(u, 0, w0, w1);
            if (u + 1 < nk) step(u + 1, 1, w1, w0);
        }
    };
    if (live == TM) main_loop(std::integral_constant<int, TM>{});
    else main_loop(std::integral_constant<int, 2>{});
    wait_copies_and_barrier<0>();
    f32_check_sums<NT, 1, TM, TN>(a, acc, grp, row0, n0, rows, 0, wave, live, r16, kq, kt0 * BK, min(kt1 * BK, K));
    f32_epilogue<NT, 1, TM, TN, BN>(a, acc, grp, row0, n0, rows, 0, wave, live, r16, kq, partial);
}

}  // namespace
}  // namespace moe
