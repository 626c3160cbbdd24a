// Expert FFN tasks in fp32 storage (Sec. 3.1 task abstraction; Eq. ffn): a persistent kernel over the live work only.
//
// As six bf16 products per fp32 one (gemm_f32_body.h) these GEMMs are slow next to their bytes with a 256 x 256
// tile, and what a launch of whole tiles loses is balance: a layer with few experts has about as many
// tiles as the chip has CUs (or far fewer), an expert's last row tile may hold a handful of live rows, and tiles
// beyond an expert's live rows are launched only to exit.  Here the work is cut the other way round.  The live
// (expert, 256-row tile) units come from a list built on the device once routing is known, each with its weight:
// the time of one of its iterations, from its live 32-row MFMA tiles (the tile body leaves out the MFMAs of the others).  unit x column tile (256 wide) x
// K-tile (32 deep) is one iteration, numbered unit by unit, K innermost; workgroup w of G (one per CU) starts at
// the iteration where the running weight reaches w / G of the total: about equal matrix-core work for every
// workgroup whatever the routing.  A workgroup's range covers the end of one tile, some whole tiles and the
// beginning of another.  Whole tiles get their epilogue at once; the sums of a partly covered tile go to one of the
// workgroup's two fp32 tiles in the caller's workspace, and a second small launch adds the pieces of each cut tile
// in the order of the workgroups that made them (a fixed order: results are the same run to run) and applies bias
// and activation.  No workgroup ever waits for another.
#include "ffn_units.h"
#include "gemm_f32_body.h"

namespace moe {
namespace {

// 256 x 256 tile: 8 wavefronts (2 x 4), each 128 x 64; one workgroup per CU
constexpr int F_WM = 2, F_WN = 4, F_TM = 8, F_TN = 4;
using FCfg = F32Cfg<false, F_WM, F_WN, F_TM, F_TN>;
constexpr int F_BM = FCfg::BM, F_BN = FCfg::BN, F_BK = FCfg::BK, F_THREADS = FCfg::THREADS;
constexpr int F_LDS = FCfg::LDS > F32Low::LDS ? FCfg::LDS : F32Low::LDS;
static_assert(F32Low::BN == F_BN && F32Low::BK == F_BK && F32Low::THREADS == F_THREADS, "both bodies compute pieces of the same tiles");

// upper bound of the workgroups worth launching: the iterations at full capacity, at most kF32MaxWorkgroups
long long f32_workgroups_bound(int groups, int max_rows, int N, int K) {
    const long long t = (long long)groups * f32_units_nrow(max_rows) * ((N + F_BN - 1) / F_BN) * ((K + F_BK - 1) / F_BK);
    return t < kF32MaxWorkgroups ? (t > 0 ? t : 1) : kF32MaxWorkgroups;
}
static_assert(F_BM == kF32UnitRows && F_BN == kF32TileCols && F_BK == kF32TileK, "the unit list and the dealing are cut in the tile's sizes");
constexpr int kFixupSplit = 16, kFixupThreads = 256;    // workgroups that share the fix-up of one cut tile, by rows
static_assert(F_BN % 4 == 0 && F_BM * F_BN / 4 % (kFixupThreads * kFixupSplit) == 0 && F_BM % kFixupSplit == 0, "fix-up thread mapping");

struct F32StreamArgs {
    GemmArgs g;
    const int32_t* list;                                // { n_units, ids[cap], cum[cap + 1] }, cap = groups * nrow
    float* partials;                                    // [G][2][F_BM][F_BN]
    int nrow;                                           // row tiles per group the ids are numbered with
};

__device__ __forceinline__ F32Work work_of(const F32StreamArgs& a) {
    const int32_t* ids = a.list + 1;
    return F32Work(ids, ids + (long long)a.g.groups * a.nrow, a.list[0], (a.g.N + F_BN - 1) / F_BN, (a.g.K + F_BK - 1) / F_BK);
}

// One piece of a tile.  Not inlined: inside the loop over a workgroup's pieces the compiler would keep the tile
// body's per-thread addresses alive across iterations and run out of registers.  The LDS array is named here, not
// passed in, so that the body's accesses stay LDS instructions.
__device__ __noinline__ void f32_tile_piece(const GemmArgs& g, int grp, int row0, int n0, int rows, int kt0, int kt1, float* partial) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    f32_tile<false, F_WM, F_WN, F_TM, F_TN>(g, smem, uniform(grp), uniform(row0), uniform(n0), uniform(rows), uniform(kt0), uniform(kt1), partial);
}
__device__ __noinline__ void f32_low_piece(const GemmArgs& g, int grp, int row0, int n0, int rows, int kt0, int kt1, float* partial) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    f32_tile_low<false>(g, smem, uniform(grp), uniform(row0), uniform(n0), uniform(rows), uniform(kt0), uniform(kt1), partial);
}


__global__ __launch_bounds__(F_THREADS) void ffn_f32_stream_kernel(F32StreamArgs a) {
    const int w = blockIdx.x, G = gridDim.x;
    const F32Work k = work_of(a);
    const long long begin = k.boundary(w, G), end = k.boundary(w + 1, G);
    bool first = true;
    for (long long it = begin; it < end;) {
        const long long tile = it / k.nk;
        const int kt0 = (int)(it - tile * k.nk);
        const int kt1 = (int)min((long long)k.nk, kt0 + (end - it));
        const int id = k.ids[tile / k.ncol], ct = (int)(tile % k.ncol);
        const int grp = id / a.nrow, rt = id % a.nrow;
        const int rows = min(a.g.rows_dev[grp], a.g.rows_cap);
        const bool whole = kt0 == 0 && kt1 == k.nk;
        float* partial = whole ? nullptr : a.partials + ((size_t)w * 2 + (first ? 0 : 1)) * (F_BM * F_BN);
        // (2.4 us per iteration at 64 rows against 3.2 in the large body with the same rows live, all CUs streaming weights)
        if (rows - rt * F_BM <= F32Low::BM) f32_low_piece(a.g, grp, rt * F_BM, ct * F_BN, rows, kt0, kt1, partial);
        else f32_tile_piece(a.g, grp, rt * F_BM, ct * F_BN, rows, kt0, kt1, partial);
        it += kt1 - kt0;
        first = false;
    }
}

// Workgroups (w, 0 .. kFixupSplit - 1) add up the tile that range w begins but does not finish: its own piece, then those of the
// workgroups after it, in order, until the tile's last K-tile; then bias, activation and the store.
// Latency bounds it: a range's boundary is a search through the unit list, and the pieces come from HBM or the last cache.  So the
// lanes search 64 boundaries at once, the pieces are requested four at a time, and 16 workgroups share a tile (T = 2048, H = 1024, I =
// 4096, E = 16: 36.6 -> 33.6 us for about two pieces a tile, 118 MB read and 67 MB written, and 43.1 -> 30.8 for about four, 77 and 17 MB).
__global__ __launch_bounds__(kFixupThreads) void ffn_f32_fixup_kernel(F32StreamArgs a, int G) {
    const int w = blockIdx.x, lane = threadIdx.x & 63;
    const F32Work k = work_of(a);
    int first = w;                                      // the range whose first iteration lane 0 holds
    long long bound = k.boundary(min(w + lane, G), G);
    auto start_of = [&](int v) __attribute__((always_inline)) {        // v uniform, ascending from call to call
        if (v >= first + 64) {
            first = v;
            bound = k.boundary(min(v + lane, G), G);
        }
        const uint32_t lo = __builtin_amdgcn_readlane((int)bound, v - first), hi = __builtin_amdgcn_readlane((int)(bound >> 32), v - first);
        return (long long)((uint64_t)hi << 32 | lo);
    };
    const long long begin = start_of(w), end = start_of(w + 1);
    const long long tile = k.tile_to_fix(begin, end);
    if (tile < 0) return;                               // nothing cut here, or the cut tile was begun by an earlier workgroup
    const long long tb = tile * k.nk, te = tb + k.nk;
    const int id = k.ids[tile / k.ncol], ct = (int)(tile % k.ncol);
    const int grp = id / a.nrow, rt = id % a.nrow;
    const int rows = min(a.g.rows_dev[grp], a.g.rows_cap);
    const int row0 = rt * F_BM, n0 = ct * F_BN;
    constexpr int V = F_BM * F_BN / 4 / kFixupThreads / kFixupSplit, AT_ONCE = 4;   // float4s per thread and piece; pieces in flight
    const int part = blockIdx.y * V * kFixupThreads;    // this workgroup's share of the tile: F_BM / kFixupSplit rows
    if (row0 + part / (F_BN / 4) >= rows) return;
    f32x4 sum[V], t[AT_ONCE][V];
    auto load = [&](int v, int which, f32x4 (&to)[V]) __attribute__((always_inline)) {
        const f32x4* p = (const f32x4*)(a.partials + ((size_t)v * 2 + which) * (F_BM * F_BN));
#pragma unroll
        for (int i = 0; i < V; ++i)
            if (row0 + (part + i * kFixupThreads) / (F_BN / 4) < rows) to[i] = p[part + i * kFixupThreads + threadIdx.x];
    };
    load(w, begin == tb ? 0 : 1, sum);
    int v = w + 1;
    long long vb = end;                                 // range v begins here; ranges may be empty
    while (v < G && vb < te) {
        int n = 0;
#pragma unroll
        for (int q = 0; q < AT_ONCE; ++q) {
            long long ve = vb;
            while (v < G && vb < te && (ve = start_of(v + 1)) == vb) ++v;
            if (v >= G || vb >= te) break;
            load(v, 0, t[q]);                           // the tile is v's first piece
            n = q + 1;
            vb = ve;
            ++v;
        }
#pragma unroll
        for (int q = 0; q < AT_ONCE; ++q) {
            if (q >= n) break;
#pragma unroll
            for (int i = 0; i < V; ++i) {
                if (row0 + (part + i * kFixupThreads) / (F_BN / 4) >= rows) continue;
                sum[i][0] += t[q][i][0]; sum[i][1] += t[q][i][1]; sum[i][2] += t[q][i][2]; sum[i][3] += t[q][i][3];
            }
        }
    }
    const size_t c_base = (size_t)grp * a.g.c_group_stride;
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const int idx = part + i * kFixupThreads + threadIdx.x;
        const int row = row0 + idx / (F_BN / 4), col = n0 + (idx % (F_BN / 4)) * 4;
        if (row >= rows || col >= a.g.N) continue;      // N is a multiple of 4
        f32x4 o;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float bias = a.g.bias ? ((const float*)a.g.bias)[(size_t)grp * a.g.bias_group_stride + col + j] : 0.0f;
            o[j] = apply_act(sum[i][j] + bias, a.g.act);
        }
        *(f32x4*)((float*)a.g.C + c_base + (size_t)row * a.g.ldc + col) = o;
    }
}

__global__ __launch_bounds__(1024) void f32_units_kernel(const int32_t* __restrict__ rows_dev, int rows_cap, int groups, int max_rows,
                                                         int32_t* __restrict__ out) {
    __shared__ int wave_total[32];
    build_row_units(rows_dev, rows_cap, groups, max_rows, out, wave_total, 1024);
}

// one workgroup per CU, but never more than the iterations there can be (a workgroup with no work still costs two
// partial tiles of workspace)
int f32_grid(int groups, int max_rows, int N, int K) {
    const long long bound = f32_workgroups_bound(groups, max_rows, N, K);
    const long long g = device_cu_count();
    return (int)(g < bound ? g : bound);
}

// One workgroup per (group, row tile, column tile); tiles beyond a group's live rows exit at once.  All tiles of a group
// run on one XCD when there are enough groups, as in the 16-bit kernel (gemm.hip).
// SPANS: the K-tiles in spans of a.k_span k, each span's sums added to those of the spans before it in C.
template <bool NT, int WM, int WN, int TM, int TN, bool SPANS>
__global__ __launch_bounds__(WM * WN * 64, 2) void f32_gemm_kernel(GemmArgs a) {
    using C = F32Cfg<NT, WM, WN, TM, TN>;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int ncol = (a.N + C::BN - 1) / C::BN, nrow = (a.max_rows + C::BM - 1) / C::BM;
    const int per_group = nrow * ncol;
    int id = blockIdx.x, grp;
    if (a.groups >= kXcds) {
        const int s = id / kXcds;
        grp = (s / per_group) * kXcds + id % kXcds;
        id = s % per_group;
    } else {
        grp = id / per_group;
        id %= per_group;
    }
    if (grp >= a.groups) return;
    const int row0 = id / ncol * C::BM, n0 = id % ncol * C::BN;
    const int rows = a.rows_dev ? min(a.rows_dev[grp], a.rows_cap) : a.rows_fixed;
    if (row0 >= rows) return;
    const int nk = ((a.k_dev ? max(min(a.k_dev[grp], a.k_cap), 1) : a.K) + C::BK - 1) / C::BK;
    if constexpr (SPANS) {
        const int span = a.k_span / C::BK;
        f32_tile<NT, WM, WN, TM, TN>(a, smem, grp, row0, n0, rows, 0, min(span, nk), nullptr);
        for (int kt = span; kt < nk; kt += span)
            f32_tile<NT, WM, WN, TM, TN, true>(a, smem, grp, row0, n0, rows, kt, min(kt + span, nk), nullptr);
    } else {
        f32_tile<NT, WM, WN, TM, TN>(a, smem, grp, row0, n0, rows, 0, nk, nullptr);
    }
}

// the same for groups of at most 64 rows
template <bool NT>
__global__ __launch_bounds__(F32Low::THREADS, 2) void f32_gemm_low_kernel(GemmArgs a) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int ncol = (a.N + F32Low::BN - 1) / F32Low::BN;
    const int grp = blockIdx.x / ncol, n0 = blockIdx.x % ncol * F32Low::BN;
    const int rows = a.rows_dev ? min(a.rows_dev[grp], a.rows_cap) : a.rows_fixed;
    if (rows <= 0) return;
    const int K = a.k_dev ? max(min(a.k_dev[grp], a.k_cap), 1) : a.K;
    f32_tile_low<NT>(a, smem, grp, 0, n0, rows, 0, (K + F32Low::BK - 1) / F32Low::BK, nullptr);
}

template <bool NT>
hipError_t prepare_f32_low() {
    static DeviceFlags limit_raised = {};
    return raise_lds_limit(reinterpret_cast<const void*>(f32_gemm_low_kernel<NT>), F32Low::LDS, limit_raised);
}

template <bool NT>
hipError_t launch_f32_low(const GemmArgs& a, hipStream_t stream) {
    if (hipError_t e = prepare_f32_low<NT>(); e != hipSuccess) return e;
    const long long blocks = (long long)a.groups * ((a.N + F32Low::BN - 1) / F32Low::BN);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(f32_gemm_low_kernel<NT>, dim3((unsigned)blocks), dim3(F32Low::THREADS), F32Low::LDS, stream, a);
    return hipGetLastError();
}

template <bool NT, int WM, int WN, int TM, int TN, bool SPANS = false>
hipError_t prepare_f32_cfg() {
    static DeviceFlags limit_raised = {};
    return raise_lds_limit(reinterpret_cast<const void*>(f32_gemm_kernel<NT, WM, WN, TM, TN, SPANS>), F32Cfg<NT, WM, WN, TM, TN>::LDS, limit_raised);
}

template <bool NT, int WM, int WN, int TM, int TN, bool SPANS = false>
hipError_t launch_f32_cfg(const GemmArgs& a, hipStream_t stream) {
    using C = F32Cfg<NT, WM, WN, TM, TN>;
    if (hipError_t e = prepare_f32_cfg<NT, WM, WN, TM, TN, SPANS>(); e != hipSuccess) return e;
    const long long ncol = (a.N + C::BN - 1) / C::BN, nrow = (a.max_rows + C::BM - 1) / C::BM;
    const long long groups = a.groups >= kXcds ? (long long)(a.groups + kXcds - 1) / kXcds * kXcds : a.groups;
    const long long blocks = groups * nrow * ncol;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((f32_gemm_kernel<NT, WM, WN, TM, TN, SPANS>), dim3((unsigned)blocks), dim3(C::THREADS), C::LDS, stream, a);
    return hipGetLastError();
}

template <bool NT>
hipError_t launch_f32_t(const GemmArgs& a, hipStream_t stream) {
    const int body = f32_tile_body(a.groups, a.max_rows, a.N, device_cu_count());
    if constexpr (!NT) {
        if (a.k_span > 0 && a.K > a.k_span) {
            if (a.act != 3 || a.bias || a.k_span % 32 != 0) return hipErrorInvalidValue;
            switch (body) {
                case kF32Body256: return launch_f32_cfg<NT, 2, 4, 8, 4, true>(a, stream);
                case kF32Body128: return launch_f32_cfg<NT, 2, 2, 4, 4, true>(a, stream);
                default: return launch_f32_cfg<NT, 2, 2, 2, 2, true>(a, stream);
            }
        }
    }
    switch (body) {
        case kF32Body64x256: return launch_f32_low<NT>(a, stream);
        case kF32Body256: return launch_f32_cfg<NT, 2, 4, 8, 4>(a, stream);
        case kF32Body128: return launch_f32_cfg<NT, 2, 2, 4, 4>(a, stream);
        default: return launch_f32_cfg<NT, 2, 2, 2, 2>(a, stream);
    }
}

}  // namespace

// Tile choice from the row bound alone (live counts are only known on the device): a launch takes about
// ceil(tiles / CUs) x tile area / efficiency.  256 x 256 fills a CU by itself; two 128 x 128 or four 64 x 64 tiles share
// one and read each operand from LDS two and four times as often per product.  The efficiencies are the matrix cores' busy
// shares at K of 1024 and more, roughly: 53 % (256 x 256, T = 16384, H = I = 2048, E = 64; 59 % since its copies are spread over the
// K-tile, the line is still the one laid before), 36 % (128 x 128) and 28 % (64 x 64, both T = 2048, H = 1024, I = 4096, E = 16, whose
// last round is not full); that of the 64 x 256 tile is an estimate.
int f32_tile_body(int groups, int max_rows, int N, int cus_) {
    const long long cus = cus_;
    auto cost = [&](int b, double eff) {
        const long long tiles = (long long)groups * ((max_rows + b - 1) / b) * ((N + b - 1) / b);
        return (double)((tiles + cus - 1) / cus) * (double)(b * b) / eff;
    };
    const double c256 = cost(256, 1.0), c128 = cost(128, 0.85), c64 = cost(64, 0.55);
    // groups of at most 64 rows: the 64 x 256 tile reads each weight from LDS once, but needs four times fewer workgroups
    const double low = (double)((groups * ((N + 255ll) / 256) + cus - 1) / cus) * (64 * 256) / 0.7;
    if (max_rows <= F32Low::BM && low <= c64) return kF32Body64x256;
    if (c64 < c128 && c64 < c256) return kF32Body64;
    return c128 < c256 ? kF32Body128 : kF32Body256;
}

// (the copies of B reach a K-tile of [k][n] or 256 rows of [n][k] weights with 32-bit offsets: beyond that the products run
// on the fp32 instruction, gemm.hip)
bool f32_gemm_eligible(const GemmArgs& a) {
    return a.dtype == 0 && !a.fp32_mfma && a.K % 8 == 0 && a.K >= 8 && a.lda % 4 == 0 && a.ldb % 4 == 0 && a.a_group_stride % 4 == 0 &&
           a.b_group_stride % 4 == 0 && a.c_group_stride % 4 == 0 && (long long)a.ldb * 4 * (a.b_is_nk ? 256 : 32) < (1ll << 32);
}

hipError_t launch_gemm_f32(const GemmArgs& a, hipStream_t stream) {
    return a.b_is_nk ? launch_f32_t<true>(a, stream) : launch_f32_t<false>(a, stream);
}

size_t f32_units_ints(int groups, int max_rows) { return (size_t)f32_units_total_ints(groups, max_rows); }
size_t f32_partials_bytes(int groups, int max_rows, int H, int I) {
    const long long g1 = f32_workgroups_bound(groups, max_rows, I, H), g2 = f32_workgroups_bound(groups, max_rows, H, I);
    return (size_t)(g1 > g2 ? g1 : g2) * 2 * F_BM * F_BN * sizeof(float);
}

hipError_t launch_f32_units(const int32_t* rows_dev, int rows_cap, int groups, int max_rows, int32_t* units, hipStream_t stream) {
    hipLaunchKernelGGL(f32_units_kernel, dim3(1), dim3(1024), 0, stream, rows_dev, rows_cap, groups, max_rows, units);
    return hipGetLastError();
}

static hipError_t prepare_f32_stream() {
    static DeviceFlags limit_raised = {};
    return raise_lds_limit(reinterpret_cast<const void*>(ffn_f32_stream_kernel), F_LDS, limit_raised);
}

hipError_t prepare_gemm_f32() {
    hipError_t e = prepare_f32_stream();
    if (e == hipSuccess) e = prepare_f32_cfg<false, 2, 4, 8, 4>();
    if (e == hipSuccess) e = prepare_f32_cfg<false, 2, 2, 4, 4>();
    if (e == hipSuccess) e = prepare_f32_cfg<false, 2, 2, 2, 2>();
    if (e == hipSuccess) e = prepare_f32_cfg<false, 2, 4, 8, 4, true>();
    if (e == hipSuccess) e = prepare_f32_cfg<false, 2, 2, 4, 4, true>();
    if (e == hipSuccess) e = prepare_f32_cfg<false, 2, 2, 2, 2, true>();
    if (e == hipSuccess) e = prepare_f32_cfg<true, 2, 4, 8, 4>();
    if (e == hipSuccess) e = prepare_f32_cfg<true, 2, 2, 4, 4>();
    if (e == hipSuccess) e = prepare_f32_cfg<true, 2, 2, 2, 2>();
    if (e == hipSuccess) e = prepare_f32_low<false>();
    if (e == hipSuccess) e = prepare_f32_low<true>();
    return e;
}

// Meant for launches whose whole tiles would not fill the chip evenly: fewer than four rounds of 256 x 256 tiles over the CUs
// at full capacity, but enough work that the second launch does not show (eight iterations per CU).  The line was laid
// when both ways ran on the fp32 instruction.  With the split products and three sizes of whole tiles it is right for skewed
// loads and light last tiles (T = 2048, H = 1024, I = 4096, E = 16: Zipf 1.2 0.44 ms against 0.58 in whole tiles; balanced 0.65
// either way) and above it (T = 16384, H = I = 2048, E = 64: 2.90 ms in whole tiles, 3.16 here), but too wide for balanced loads
// of full tiles: T = 4096, H = I = 2048, E = 8, 0.89 ms against 0.71; T = 12288, E = 24, 2.42 against 2.04; T = 512, E = 32, 0.28
// against 0.24.
bool f32_spans_worth(int groups, int max_rows, int N, int K, int cus_) {
    const long long units = (long long)groups * f32_units_nrow(max_rows), ncol = (N + F_BN - 1) / F_BN, cus = cus_;
    if (units > 0x7fffffffLL / ncol) return false;
    const long long tiles = units * ncol;
    return tiles < 4 * cus && tiles * ((K + F_BK - 1) / F_BK) >= 8 * cus;
}

bool f32_stream_eligible(const GemmArgs& a) {
    if (!f32_gemm_eligible(a) || a.b_is_nk || a.c_f32 || !a.units || !a.partials || !a.rows_dev) return false;
    if (a.N % 4 != 0 || a.ldc % 4 != 0) return false;
    return f32_spans_worth(a.groups, a.max_rows, a.N, a.K, device_cu_count());
}

hipError_t launch_gemm_f32_stream(const GemmArgs& g, hipStream_t stream) {
    if (hipError_t e = prepare_f32_stream(); e != hipSuccess) return e;
    F32StreamArgs a{};
    a.g = g;
    a.list = g.units;
    a.partials = g.partials;
    a.nrow = f32_units_nrow(g.max_rows);
    const int G = f32_grid(g.groups, g.max_rows, g.N, g.K);
    hipLaunchKernelGGL(ffn_f32_stream_kernel, dim3(G), dim3(F_THREADS), F_LDS, stream, a);
    if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    hipLaunchKernelGGL(ffn_f32_fixup_kernel, dim3(G, kFixupSplit), dim3(kFixupThreads), 0, stream, a, G);
    return hipGetLastError();
}

}  // namespace moe
