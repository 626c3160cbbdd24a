// Weight gradients of the backward pass in 16-bit storage: C[g][m][n] = sum over k of A[g][k][m] B[g][k][n] in fp32, where k
// runs over an expert's live slots (dW1 = xe^T da, dW2 = h^T ge) or over the tokens (dWg = x^T dL).  Both operands are read as
// they are stored, k outermost, and one launch takes all the products.  (Large layers with full slots make dW1 and dW2 on the
// weight-streaming kernel: api.hip has the line.)
//
// An output element is often a sum of few products and the output is larger than the operands: with 64 slots per expert (H = I =
// 2048, E = 128) stores bound it, at 6.1 TB/s; at 256 slots it is the time of its loads, 0.72 ms, and that of its stores, 0.69, which
// share a CU's path to L2 and add up in every form that was tried.  A tile is 128 x 256 with four wavefronts and 72 KB of
// LDS, two workgroups to a CU, so that one's products and latencies lie under the other's; a workgroup makes one tile, and nobody waits for
// its stores.  (256 x 256: 3 % faster there, 11 % slower at 64 to 100 slots; 128 x 128: 17 % slower.)  Sums stop at the last live slot,
// where the GEMMs that this kernel took over ran to the padded capacity, and long sums of few tiles are cut into slices.
//
// Copies are direct (global_load_lds_dwordx4) through a ring of three K-tiles of 32 k, requested two K-tiles ahead; LDS rows are
// k-rows, 16-byte chunk c of row k at c ^ swz_b(k), read back in MFMA operand order with ds_read_b64_tr_b16 as in the
// weight-streaming kernel.  Rows from an expert's last live one to the next multiple of 32 hold zeros in both operands.
#include "gemm_stream_body.h"

namespace moe {
namespace {

constexpr int W_BM = 128, W_BN = 256, W_BK = 32, W_THREADS = 256, W_TM = 8, W_TN = 4;
constexpr int W_A_ROW = W_BM * 2, W_B_ROW = W_BN * 2;                   // bytes of a k-row
constexpr int W_A_STAGE = W_BK * W_A_ROW, W_STAGE = W_A_STAGE + W_BK * W_B_ROW, W_STAGES = 3;
constexpr int W_LDS = W_STAGES * W_STAGE;
constexpr int W_COPIES = W_STAGE / 1024 / (W_THREADS / 64);             // per wavefront and K-tile: 2 of A, 4 of B
static_assert(2 * W_LDS <= 160 * 1024, "two workgroups per CU");

struct WgradArgs {
    WgradProblem p[kWgradProblems];
    int end[kWgradProblems];                            // workgroups of the problems up to and including this one
};

// All tiles of one sum on one XCD: they share the operands' panels through its L2.  With few sums, and not a multiple of 8, some
// XCDs would have twice the work of others or none: then the tiles are dealt in order.
__host__ __device__ inline bool wgrad_by_xcd(int parts) { return parts % kXcds == 0 || parts >= 8 * kXcds; }

__device__ __forceinline__ s16x8 read_transposed(const unsigned char* p, int row_bytes) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * row_bytes));
    return s16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
}

template <class S>
__global__ __launch_bounds__(W_THREADS, 2) void wgrad_kernel(WgradArgs a) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    int id = blockIdx.x, which = 0;
    while (which < kWgradProblems - 1 && id >= a.end[which]) ++which;
    if (which) id -= a.end[which - 1];
    const WgradProblem& P = a.p[which];
    const int ncol = (P.N + W_BN - 1) / W_BN, nrow = (P.M + W_BM - 1) / W_BM, per_group = ncol * nrow;
    const int parts = P.groups * P.slices;              // part = slice * groups + group
    const bool by_xcd = wgrad_by_xcd(parts);
    const int s = by_xcd ? id / kXcds : id;
    const int part = by_xcd ? (s / per_group) * kXcds + id % kXcds : s / per_group;
    if (part >= parts) return;
    const int slice = part / P.groups, grp = part % P.groups;
    const int m0 = s % per_group / ncol * W_BM, n0 = s % per_group % ncol * W_BN;
    const int k_live = P.rows_dev ? min(P.rows_dev[grp], P.rows_cap) : P.rows_cap;
    const int tiles = (k_live + W_BK - 1) / W_BK;
    const int kt0 = (int)((long long)tiles * slice / P.slices), nk = (int)((long long)tiles * (slice + 1) / P.slices) - kt0;

    const int lane = threadIdx.x & 63, wave = uniform((int)threadIdx.x >> 6);
    const int r16 = lane & 15, kq = lane >> 4;
    f32x4 acc[W_TM][W_TN];
#pragma unroll
    for (int i = 0; i < W_TM; ++i)
#pragma unroll
        for (int j = 0; j < W_TN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    if (nk > 0) {
        const size_t lda2 = (size_t)P.lda * 2, ldb2 = (size_t)P.ldb * 2;
        const unsigned char* const a_base = uniform((const unsigned char*)P.A + (size_t)grp * P.a_group_stride * 2);
        const unsigned char* const b_base = uniform((const unsigned char*)P.B + (size_t)grp * P.b_group_stride * 2);
        const uint32_t lds_base = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
        // a copy of A is 4 k-rows of 16 chunks, one of B 2 k-rows of 32; columns beyond the last repeat it; rows of A beyond a_rows are
        // zeros, as their B is (a row of A in their place could hold an infinity)
        const int ra = lane >> 4, rb = lane >> 5;
        uint32_t a_col[2], b_col[4];
#pragma unroll
        for (int j = 0; j < 2; ++j) a_col[j] = (uint32_t)min(m0 + ((lane & 15) ^ swz_b((wave * 2 + j) * 4 + ra)) * 8, P.lda - 8) * 2;
#pragma unroll
        for (int j = 0; j < 4; ++j) b_col[j] = (uint32_t)min(n0 + ((lane & 31) ^ swz_b((wave * 4 + j) * 2 + rb)) * 8, P.ldb - 8) * 2;
        const uint32_t a_lane = (uint32_t)ra * (uint32_t)lda2, b_lane = (uint32_t)rb * (uint32_t)ldb2;
        const int a_rows = P.a_rows;
        auto issue = [&](int u) __attribute__((always_inline)) {
            const uint32_t d = lds_base + u % W_STAGES * W_STAGE;
            const int k0 = (kt0 + u) * W_BK;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int k = k0 + (wave * 2 + j) * 4;
                const unsigned char* const row = a_base + (size_t)k * lda2;
                const uint32_t off = a_lane + a_col[j], to = d + (wave * 2 + j) * 1024;
                if (k + 4 <= a_rows) copy_to_lds(row, off, to);
                else copy_to_lds_lane(k + ra < a_rows ? row + off : (const unsigned char*)&stream_zeros, to);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                copy_to_lds(b_base + (size_t)(k0 + (wave * 4 + j) * 2) * ldb2, b_lane + b_col[j], d + W_A_STAGE + (wave * 4 + j) * 1024);
        };
        const int bk = kq * 8 + (r16 >> 2), sw = swz_b(bk);             // k of the first transpose read; the second is k + 4
        const int a_rd = bk * W_A_ROW + ((((r16 & 3) >> 1) ^ sw) << 4) + (r16 & 1) * 8;     // row tile i: ^ (i << 5)
        const int b_rd = W_A_STAGE + bk * W_B_ROW + (((wave * W_TN * 2 + ((r16 & 3) >> 1)) ^ sw) << 4) + (r16 & 1) * 8;
        issue(0);
        if (nk > 1) issue(1);
        for (int u = 0; u < nk; ++u) {
            // K-tile u has landed, and everybody is done with K-tile u - 1, whose stage the next request fills
            if (u + 1 < nk) wait_copies_and_barrier<W_COPIES>();
            else wait_copies_and_barrier<0>();
            if (u + 2 < nk) issue(u + 2);
            const unsigned char* const st = smem + u % W_STAGES * W_STAGE;
            s16x8 w[W_TN];
#pragma unroll
            for (int j = 0; j < W_TN; ++j) w[j] = read_transposed(st + (b_rd ^ (j << 5)), W_B_ROW);
#pragma unroll
            for (int i = 0; i < W_TM; ++i) {
                const s16x8 x = read_transposed(st + (a_rd ^ (i << 5)), W_A_ROW);
#pragma unroll
                for (int j = 0; j < W_TN; ++j) acc[i][j] = Mma16<S>::run(w[j], x, acc[i][j]);
            }
        }
    }

    // a lane's four sums of a tile are four consecutive columns of one row, a tile's row half a line: lanes 8 rows apart swap
    // halves of two neighbouring tiles, so that a store writes whole lines
    float* const C = P.C + (size_t)part * P.c_group_stride;
    const bool low = r16 < 8, vec = (P.ldc & 3) == 0;   // (the group stride is a multiple of 4 with ldc)
    const int N = P.N, M = P.M;
#pragma unroll
    for (int i = 0; i < W_TM; ++i) {
        const int row = m0 + i * 16 + (r16 & 7);
#pragma unroll
        for (int j = 0; j < W_TN; j += 2) {
            f32x4 v[2] = {acc[i][j], acc[i][j + 1]};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float got = swap_8_lanes(low ? v[1][q] : v[0][q]);
                v[0][q] = low ? v[0][q] : got;
                v[1][q] = low ? got : v[1][q];
            }
            const int col = n0 + wave * (W_TN * 16) + (j + (low ? 0 : 1)) * 16 + kq * 4;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (row + 8 * h >= M || col >= N) continue;
                float* const c = C + (size_t)(row + 8 * h) * P.ldc + col;
                if (vec) {
                    __builtin_nontemporal_store(v[h], (f32x4*)c);
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (col + q < N) c[q] = v[h][q];
                }
            }
        }
    }
}

template <class S>
hipError_t prepare_wgrad_t() {
    static DeviceFlags limit_raised = {};
    return raise_lds_limit(reinterpret_cast<const void*>(wgrad_kernel<S>), W_LDS, limit_raised);
}

template <class S>
hipError_t launch_wgrad_t(const WgradArgs& a, hipStream_t stream) {
    if (hipError_t e = prepare_wgrad_t<S>(); e != hipSuccess) return e;
    hipLaunchKernelGGL(wgrad_kernel<S>, dim3((unsigned)a.end[kWgradProblems - 1]), dim3(W_THREADS), W_LDS, stream, a);
    return hipGetLastError();
}

}  // namespace

hipError_t prepare_wgrad() {
    const hipError_t e = prepare_wgrad_t<BF16>();
    return e != hipSuccess ? e : prepare_wgrad_t<F16>();
}

long long wgrad_tiles(int groups, int M, int N) { return (long long)groups * ((M + W_BM - 1) / W_BM) * ((N + W_BN - 1) / W_BN); }

hipError_t launch_wgrad(const WgradProblem (&p)[kWgradProblems], int dtype, hipStream_t stream) {
    WgradArgs a{};
    long long end = 0;
    for (int i = 0; i < kWgradProblems; ++i) {
        a.p[i] = p[i];
        const long long parts = (long long)p[i].groups * p[i].slices;
        if (parts > 0x7ffffff8LL) return hipErrorInvalidValue;
        end += wgrad_tiles(1, p[i].M, p[i].N) * (wgrad_by_xcd((int)parts) ? (parts + kXcds - 1) / kXcds * kXcds : parts);
        if (end > 0x7fffffffLL) return hipErrorInvalidValue;
        a.end[i] = (int)end;
    }
    return dtype == 1 ? launch_wgrad_t<BF16>(a, stream) : launch_wgrad_t<F16>(a, stream);
}

}  // namespace moe
