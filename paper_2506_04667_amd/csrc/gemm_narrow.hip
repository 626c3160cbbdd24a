// Expert FFN products in 16-bit storage of launches with too few tasks for the weight-streaming kernel (gemm_stream_body.h), and of layers
// too narrow for it: C[g] = act(A[g] B[g] + bias[g]) over the live rows, in tiles of 128 x 128, one workgroup each.
//
// What bounds such a launch is how many CUs have a task and how the last round of tasks fills up, and for one task the latency of
// its chain: lists, addresses, first K-tile, K loop, epilogue.  A quarter of the streaming kernel's tile has four times the tasks,
// a quarter of the epilogue and, with 80 KB of LDS, a second workgroup on its CU whose products and copies run under the other's
// latencies; workgroups are dealt by the hardware as others end.  The price is that operands cross L2 twice as often per product.
//
// Copies are direct (global_load_lds_dwordx4) through a ring of five K-tiles of 32 k, requested four K-tiles ahead.  Activations and
// [n][k] weights lie in LDS as 128 rows of 64 bytes, 16-byte chunk c of row r at c ^ ((r >> 2) & 3); [k][n] weights as 32 k-rows of 256
// bytes, chunk c of row k at c ^ swz_b(k), read back in MFMA operand order with ds_read_b64_tr_b16.  A K-tile that ends beyond K
// is filled up with zeros in both operands, so any K that is a multiple of 8 will do.
#include "gemm_stream_body.h"

#include <algorithm>

namespace moe {
namespace {

constexpr int R_BM = 128, R_BN = 128, R_BK = 32, R_THREADS = 256, R_T = 4;     // tile; 16-wide MFMA tiles of a wavefront, each way
constexpr int R_ROW = R_BK * 2, R_KROW = R_BN * 2;                             // bytes of a row of 32 k, of a k-row of 128 columns
constexpr int R_HALF = R_BM * R_ROW, R_STAGE = 2 * R_HALF, R_STAGES = 5, R_LDS = R_STAGES * R_STAGE;
constexpr int R_COPIES = R_STAGE / 1024 / (R_THREADS / 64);                    // 1 KB copies per wavefront and K-tile
static_assert(R_STAGES == 5 && 2 * R_LDS <= 160 * 1024, "two workgroups per CU, and the waits count four K-tiles ahead");
static_assert(2 * R_BM == kUnitRowsLarge && R_BM == kUnitRowsSmall, "the unit lists are cut in halves and wholes of the tile");

__device__ __forceinline__ int swz_r(int r) { return (r >> 2) & 3; }

// blocks of the live units of 256 and of 128 rows: an XCD takes every 8th unit, all its tiles together
__host__ __device__ inline int narrow_unit_slots(int units) { return (units + kXcds - 1) / kXcds * kXcds; }

template <class S, int ACT, bool NK, bool F32OUT>
__global__ __launch_bounds__(R_THREADS, 2) void ffn_gemm_narrow_kernel(StreamArgs a) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    typedef uint16_t elem;
    const StreamPhase& P = a.ph[0];
    const int ncol = (P.N + R_BN - 1) / R_BN;
    const int nrow_l = ffn_units_nrow_large(a.max_rows), nrow_s = ffn_units_nrow_small(a.max_rows);
    const int32_t* const list_l = a.lists + 1;
    const int32_t* const list_s = a.lists + ffn_units_small_offset(a.groups, a.max_rows) + 1;
    const int n_l = nrow_l ? uniform(list_l[0]) : 0, n_s = uniform(list_s[0]);
    int id = blockIdx.x, grp, row0, n0;
    const int blocks_l = narrow_unit_slots(n_l) * 2 * ncol;
    if (id < blocks_l) {
        const int s = id / kXcds, u = s / (2 * ncol) * kXcds + id % kXcds, t = s % (2 * ncol);
        if (u >= n_l) return;
        const int unit = uniform(list_l[1 + u]);
        grp = unit / nrow_l;
        row0 = unit % nrow_l * kUnitRowsLarge + (t & 1) * R_BM;
        n0 = (t >> 1) * R_BN;
    } else {
        id -= blocks_l;
        const int s = id / kXcds, u = s / ncol * kXcds + id % kXcds;
        if (u >= n_s) return;
        const int unit = uniform(list_s[1 + u]);
        grp = unit / nrow_s;
        row0 = unit % nrow_s * kUnitRowsSmall;
        n0 = s % ncol * R_BN;
    }
    const int rows = uniform(min(a.rows_dev[grp], a.rows_cap));        // > row0
    const int nk = (P.K + R_BK - 1) / R_BK;

    const int lane = threadIdx.x & 63, wave = uniform((int)threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1, r16 = lane & 15, kq = lane >> 4;
    const size_t a_group = P.a_row_index ? (size_t)0 : (size_t)grp * P.a_group_stride;
    const unsigned char* a_base = uniform((const unsigned char*)((const elem*)P.A + a_group));
    const unsigned char* b_base = uniform((const unsigned char*)((const elem*)P.B + (size_t)grp * P.b_group_stride));
    const uint32_t lda2 = (uint32_t)P.lda * 2, ldb2 = (uint32_t)P.ldb * 2;
    // copy j of a wavefront: 16 rows of 4 chunks, or 4 k-rows of 16; rows and columns beyond the last repeat it
    uint32_t a_off[2], b_off[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int r = (wave * 2 + j) * 16 + (lane >> 2), c = (lane & 3) ^ swz_r(r);
        int grow = min(row0 + r, rows - 1);
        if (P.a_row_index) grow = P.a_row_index[(size_t)grp * P.a_index_stride + grow];
        a_off[j] = (uint32_t)grow * lda2 + c * 16;
        if constexpr (NK) {
            b_off[j] = (uint32_t)min(n0 + r, P.N - 1) * ldb2 + c * 16;
        } else {
            const int k = (wave * 2 + j) * 4 + kq;
            b_off[j] = (uint32_t)k * ldb2 + min(n0 + (r16 ^ swz_b(k)) * 8, P.N - 8) * 2;
        }
    }
    const uint32_t lds_wave = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)smem + wave * 2048;
    const size_t b_step = NK ? (size_t)R_ROW : (size_t)R_BK * ldb2;
    int to = 0;                                         // stage of the next request
    auto issue = [&](int u) __attribute__((always_inline)) {
        const uint32_t d = lds_wave + to * R_STAGE;
        const int left = P.K - u * R_BK;
        if (left >= R_BK) {
#pragma unroll
            for (int j = 0; j < 2; ++j) copy_to_lds_stream(b_base, b_off[j], d + R_HALF + j * 1024);
#pragma unroll
            for (int j = 0; j < 2; ++j) copy_to_lds(a_base, a_off[j], d + j * 1024);
        } else {                                        // a chunk of 8 k is inside K or beyond it
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int r = (wave * 2 + j) * 16 + (lane >> 2);
                const bool in = ((lane & 3) ^ swz_r(r)) * 8 < left, b_in = NK ? in : (wave * 2 + j) * 4 + kq < left;
                copy_to_lds_lane(b_in ? b_base + b_off[j] : (const unsigned char*)&stream_zeros, d + R_HALF + j * 1024);
                copy_to_lds_lane(in ? a_base + a_off[j] : (const unsigned char*)&stream_zeros, d + j * 1024);
            }
        }
        a_base += R_ROW;
        b_base += b_step;
        to = to + 1 == R_STAGES ? 0 : to + 1;
    };

    f32x4 acc[R_T][R_T];
#pragma unroll
    for (int i = 0; i < R_T; ++i)
#pragma unroll
        for (int j = 0; j < R_T; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // row tiles of this wavefront with a live row
    const int live = uniform(min(max((rows - row0 - wm * (R_T * 16) + 15) / 16, 0), R_T));
    const int a_rd = (wm * R_T * 16 + r16) * R_ROW + ((kq ^ swz_r(r16)) << 4);           // row tile i: + i * 16 rows
    const int bk = kq * 8 + (r16 >> 2);                 // k of the first transpose read; the second is k + 4
    const int b_rd = R_HALF + (NK ? (wn * R_T * 16 + r16) * R_ROW + ((kq ^ swz_r(r16)) << 4)
                                  : bk * R_KROW + (((wn * R_T * 2 + ((r16 & 3) >> 1)) ^ swz_b(bk)) << 4) + (r16 & 1) * 8);
    for (int u = 0; u < R_STAGES - 1 && u < nk; ++u) issue(u);
    int at = 0;                                         // stage of K-tile u
    for (int u = 0; u < nk; ++u) {
        // K-tile u has landed, and everybody is done with K-tile u - 1, whose stage the next request fills
        if (u + 3 < nk) wait_copies_and_barrier<3 * R_COPIES>();
        else if (u + 2 < nk) wait_copies_and_barrier<2 * R_COPIES>();
        else if (u + 1 < nk) wait_copies_and_barrier<R_COPIES>();
        else wait_copies_and_barrier<0>();
        if (u + R_STAGES - 1 < nk) issue(u + R_STAGES - 1);
        const unsigned char* const st = smem + at * R_STAGE;
        at = at + 1 == R_STAGES ? 0 : at + 1;
        s16x8 w[R_T], x[R_T];
#pragma unroll
        for (int j = 0; j < R_T; ++j) {
            if constexpr (NK) {
                w[j] = *(const s16x8*)(st + b_rd + j * 16 * R_ROW);
            } else {
                const unsigned char* const p = st + (b_rd ^ (j << 5));
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * R_KROW));
                w[j] = s16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            }
        }
        if (live == R_T) {
#pragma unroll
            for (int i = 0; i < R_T; ++i) x[i] = *(const s16x8*)(st + a_rd + i * 16 * R_ROW);
#pragma unroll
            for (int i = 0; i < R_T; ++i)
#pragma unroll
                for (int j = 0; j < R_T; ++j) acc[i][j] = Mma16<S>::run(w[j], x[i], acc[i][j]);
        } else {
#pragma unroll
            for (int i = 0; i < R_T - 1; ++i) {
                if (i >= live) continue;
                x[i] = *(const s16x8*)(st + a_rd + i * 16 * R_ROW);
#pragma unroll
                for (int j = 0; j < R_T; ++j) acc[i][j] = Mma16<S>::run(w[j], x[i], acc[i][j]);
            }
        }
    }

    // a lane's four sums of a tile are four consecutive columns of row r16
    const int col_w = n0 + wn * (R_T * 16);
    const size_t c_base = (size_t)grp * P.c_group_stride;
    float bias[R_T][4];
#pragma unroll
    for (int j = 0; j < R_T; ++j) {
        u32x2 bits = {0u, 0u};
        if (!NK && P.bias)
            bits = *(const u32x2*)((const elem*)P.bias + (size_t)grp * P.bias_group_stride + min(col_w + j * 16 + kq * 4, P.N - 4));
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const uint32_t word = bits[b >> 1];
            bias[j][b] = bits16_to_float<S>((uint16_t)((b & 1) ? (word >> 16) : (word & 0xffffu)));
        }
    }
#pragma unroll
    for (int i = 0; i < R_T; ++i) {
        if (i >= live) continue;
        const int tile_row = row0 + wm * (R_T * 16) + i * 16;
#pragma unroll
        for (int j = 0; j < R_T; j += 2) {
            if constexpr (F32OUT) {                     // lanes 8 rows apart swap halves of two tiles: a store writes whole lines
                const bool low = r16 < 8;
                f32x4 v[2] = {acc[i][j], acc[i][j + 1]};
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const float got = swap_8_lanes(low ? v[1][b] : v[0][b]);
                    v[0][b] = low ? v[0][b] : got;
                    v[1][b] = low ? got : v[1][b];
                }
                const int row = tile_row + (r16 & 7), col = col_w + (j + (low ? 0 : 1)) * 16 + kq * 4;
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    if (row + 8 * h < rows && col < P.N)
                        __builtin_nontemporal_store(v[h], (f32x4*)((float*)P.C + c_base + (size_t)(row + 8 * h) * P.ldc + col));
            } else {                                    // lanes 16 apart swap halves of two tiles and store 8 columns each
                u32x4 v;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    uint32_t t[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        t[h] = pack2<S>(apply_act16_t<ACT>(acc[i][j + h][2 * q] + bias[j + h][2 * q]),
                                        apply_act16_t<ACT>(acc[i][j + h][2 * q + 1] + bias[j + h][2 * q + 1]));
                    const auto sw = __builtin_amdgcn_permlane16_swap(t[0], t[1], false, false);
                    v[q] = sw[0]; v[2 + q] = sw[1];
                }
                const int row = tile_row + r16, col = col_w + (j + (kq & 1)) * 16 + (kq >> 1) * 8;
                if (row < rows && col < P.N) *(u32x4*)((elem*)P.C + c_base + (size_t)row * P.ldc + col) = v;
            }
        }
    }
}

template <class S, int ACT, bool NK, bool F32OUT>
hipError_t prepare_narrow_t() {
    static DeviceFlags limit_raised = {};
    return raise_lds_limit(reinterpret_cast<const void*>(ffn_gemm_narrow_kernel<S, ACT, NK, F32OUT>), R_LDS, limit_raised);
}

template <class S, int ACT, bool NK = false, bool F32OUT = false>
hipError_t launch_narrow_t(const GemmArgs& g, hipStream_t stream) {
    if (hipError_t e = prepare_narrow_t<S, ACT, NK, F32OUT>(); e != hipSuccess) return e;
    // a group has at most max_rows / 128 row tiles, whichever list they are in; each list's units are dealt in eights
    const long long units = (long long)g.groups * ffn_units_nrow_small(g.max_rows) + 3 * kXcds;
    const long long blocks = (units + kXcds - 1) / kXcds * kXcds * ((g.N + R_BN - 1) / R_BN);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    StreamArgs a{};
    a.ph[0] = to_phase(g);
    a.rows_dev = g.rows_dev; a.rows_cap = g.rows_cap; a.max_rows = g.max_rows;
    a.lists = g.units;
    a.groups = g.groups;
    hipLaunchKernelGGL((ffn_gemm_narrow_kernel<S, ACT, NK, F32OUT>), dim3((unsigned)blocks), dim3(R_THREADS), R_LDS, stream, a);
    return hipGetLastError();
}

template <class S>
hipError_t launch_narrow_s(const GemmArgs& g, hipStream_t stream) {
    if (g.b_is_nk) return g.c_f32 ? launch_narrow_t<S, 3, true, true>(g, stream) : launch_narrow_t<S, 3, true>(g, stream);
    switch (g.act) {
        case 0: return launch_narrow_t<S, 0>(g, stream);
        case 1: return launch_narrow_t<S, 1>(g, stream);
        case 2:
            // The clamped polynomial is the streaming kernel's, for its own shapes.  The others always had the closer form: relative error
            // of y in fp16 (E = 8 of 190 rows, H = 328, I = 840) 2.952e-4 with the polynomial, 2.948e-4 so, and in the tail, below
            // v = -3, h itself is off by up to 5e-5 where it should be 1e-4 and less.
            return stream_gemm_shape_ok(g.dtype, g.N, g.K, g.lda, g.ldb, g.ldc, g.a_rows_total) ? launch_narrow_t<S, 2>(g, stream)
                                                                                                : launch_narrow_t<S, kActGeluErf>(g, stream);
        default: return launch_narrow_t<S, 3>(g, stream);
    }
}

template <class S>
hipError_t prepare_narrow_s() {
    hipError_t e = prepare_narrow_t<S, 0, false, false>();
    if (e == hipSuccess) e = prepare_narrow_t<S, 1, false, false>();
    if (e == hipSuccess) e = prepare_narrow_t<S, 2, false, false>();
    if (e == hipSuccess) e = prepare_narrow_t<S, 3, false, false>();
    if (e == hipSuccess) e = prepare_narrow_t<S, kActGeluErf, false, false>();
    if (e == hipSuccess) e = prepare_narrow_t<S, 3, true, false>();
    if (e == hipSuccess) e = prepare_narrow_t<S, 3, true, true>();
    return e;
}

}  // namespace

hipError_t prepare_gemm_narrow() {
    const hipError_t e = prepare_narrow_s<BF16>();
    return e != hipSuccess ? e : prepare_narrow_s<F16>();
}

bool narrow_gemm_eligible(const GemmArgs& a) {
    if (a.dtype == 0 || a.a_is_km || a.rows_dev == nullptr || a.units == nullptr) return false;
    if (a.b_is_nk ? a.act != 3 || a.bias != nullptr : a.c_f32) return false;
    return a.K % 8 == 0 && a.K >= 8 && a.N % 8 == 0 && a.N >= 8 && a.lda % 8 == 0 && a.ldb % 8 == 0 && a.ldc % 8 == 0 &&
           // copies address an operand as a 64-bit base plus 32-bit byte offsets
           a.a_rows_total * a.lda * 2 < (1ll << 32) && (long long)(a.b_is_nk ? a.N : R_BK) * a.ldb * 2 < (1ll << 32);
}

// Both GEMMs of expert FFNs of bf16, us, streaming kernel / this one.  At most one tile of this kernel per CU: E = 8 of 190 rows, H = 328,
// I = 840 48 / 28; E = 4 of 64, H = I = 512 44 / 23; E = 16 of 64 and 128, H = I = 2048 70 / 62 and 76 / 72; E = 32 of 8 and 128, H = I =
// 1024 44 / 40 and 48 / 44.  With somewhat more a few CUs have two and the rest wait for them, with many the operands' way from L2
// decides: E = 24 of 128, H = I = 1536 (288 tiles) 71 / 103; E = 64 of 128, H = I = 1024 (512) 73 / 81; E = 16 of 512, H = I = 2048 127 /
// 232.  Few rows have next to no activations to bring in, and finer tasks even out the last round of the weights' stream.  Whole forward
// calls timed in turn, capacities of 1 to 8 rows, top-2: H = I = 1024, E = 96, T = 384 101 / 94, T = 48 69.8 / 67.3; H = I = 1536, E = 64, T =
// 256 136 / 127; H = I = 2880, E = 48, T = 100 312 / 298; H = 4096, I = 1536, E = 64, T = 64 274 / 264; H = I = 2048, E = 128, T = 64
// 253 / 248 on one card and 259 / 259 on another, T = 512 355 / 355, T = 16 106.4 / 107.2; top-8, H = 7168, I = 2048, E = 32, T = 32
// 341 / 343.  16 rows, E = 128 (both GEMMs) 344 / 352.  [n][k] weights in half lines do not gain from that.
bool narrow_gemm_worth(const GemmArgs& a, int cus) {
    const long long all = (long long)a.groups * ((a.max_rows + R_BM - 1) / R_BM), ncol = (a.N + R_BN - 1) / R_BN;
    const long long likely = a.rows_likely > 0 ? std::min(all, a.groups + a.rows_likely / R_BM) : all;
    return likely * ncol <= cus || (!a.b_is_nk && a.max_rows <= 8 && likely * ncol * 2 >= 3 * cus);
}

hipError_t launch_gemm_narrow(const GemmArgs& a, hipStream_t stream) {
    return a.dtype == 1 ? launch_narrow_s<BF16>(a, stream) : launch_narrow_s<F16>(a, stream);
}

}  // namespace moe
