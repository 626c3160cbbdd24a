// Launchers of the fused gate kernels ("FusedGate" of Alg. 1); the kernel bodies are in gate_fused_body.h.
#include "gate_fused_body.h"

namespace moe {
namespace {

struct GateArgs {
    const unsigned char *x, *Wg;
    const float* gate_bias;
    int T, H, E, k;
    float* logits;
    int32_t* topk_expert;
    float* topk_weight;
    int32_t* route_counts;
    int slices;
    float* partial;                                     // [slices][T][E]
};

template <class S, int BN, bool LIN>
__global__ __launch_bounds__(G_THREADS) void gate_fused_kernel(GateArgs a) {
    gate_fused_tile<S, BN, LIN>(a.x, a.Wg, a.gate_bias, a.T, a.H, a.E, a.k, 1, a.logits, a.topk_expert, a.topk_weight, a.route_counts,
                                (int)blockIdx.x);
}

// The K-tiles in slices, each by a workgroup of its own: a tile of 64 tokens keeps one CU busy for H / 64 (fp32: H / 32) K-tiles one
// after the other, about 0.5 us (0.7) each, however few tiles there are.
template <class S, int BN, bool LIN>
__global__ __launch_bounds__(G_THREADS) void gate_slice_kernel(GateArgs a) {
    constexpr int LP = BN + 4;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tile = blockIdx.x / a.slices, slice = blockIdx.x % a.slices;
    gate_logits_tile<S, BN, LIN>(a.x, a.Wg, nullptr, a.T, a.H, a.E, tile, slice, slice + 1, a.slices);
    const int row0 = tile * G_BM, quads = a.E / 4;
    float* const out = a.partial + ((size_t)slice * a.T + row0) * a.E;
    for (int i = threadIdx.x; i < G_BM * quads; i += G_THREADS) {
        const int r = i / quads, e = i % quads * 4;
        if (row0 + r < a.T) *(f32x4*)(out + (size_t)r * a.E + e) = *(const f32x4*)((const float*)smem + r * LP + e);
    }
    // the next launch adds its workgroups' shares of the chunk's counts up
    if (a.route_counts && slice == 0)
        for (int e = threadIdx.x; e < a.E; e += G_THREADS) a.route_counts[(size_t)tile * a.E + e] = 0;
}

// The slices' sums added up in order, and the rest of the gate, 16 tokens to a workgroup: one CU brings in about 60 KB/us, and 64 tokens are
// 512 KB of sums (E = 128, 16 slices).  T = 64 8.4 -> 5.0 us; T = 4096, E = 32 15.0 -> 9.2.
constexpr int F_ROWS = 16, F_WGTHREADS = 256;
template <int BN>
__global__ __launch_bounds__(F_WGTHREADS) void gate_finish_kernel(GateArgs a) {
    constexpr int LP = BN + 4, TOK = F_ROWS / (F_WGTHREADS / 64);
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    float* const lg = (float*)smem;
    const int tile = blockIdx.x, row0 = tile * F_ROWS, quads = a.E / 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t step = (size_t)a.T * a.E;
    // the rows of this wavefront's tokens: two quads of experts and eight slices in flight per lane
    for (int i0 = lane; i0 < TOK * quads; i0 += 128) {
        f32x4 sum[2];
        const float* p[2];
        int cell[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int i = min(i0 + u * 64, TOK * quads - 1), r = wave * TOK + i / quads, e = i % quads * 4;
            p[u] = a.partial + (size_t)min(row0 + r, a.T - 1) * a.E + e;       // (beyond the last token: not used)
            cell[u] = r * LP + e;
            sum[u] = *(const f32x4*)p[u];
        }
        constexpr int kTrip = 8;
        for (int s0 = 1; s0 < a.slices; s0 += kTrip) {
            f32x4 v[2][kTrip];
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int q = 0; q < kTrip; ++q) v[u][q] = *(const f32x4*)(p[u] + (size_t)min(s0 + q, a.slices - 1) * step);
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int q = 0; q < kTrip; ++q)
                    if (s0 + q < a.slices) sum[u] += v[u][q];
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (a.gate_bias) sum[u] += *(const f32x4*)(a.gate_bias + cell[u] % LP);
            *(f32x4*)(lg + cell[u]) = sum[u];
        }
    }
    __syncthreads();
    gate_select_tile<BN, F_ROWS, F_WGTHREADS>(a.T, a.E, a.k, a.logits, a.topk_expert, a.topk_weight, a.route_counts, tile);
}

template <int BN> constexpr int finish_lds() { return (F_ROWS * (BN + 4 + BN) + BN) * 4; }
static_assert(finish_lds<256>() <= 64 * 1024, "no limit to raise");

// the kernels' LDS limits on the current device (once per device)
template <class S, int BN, bool LIN>
hipError_t prepare_gate_fused_t() {
    static DeviceFlags whole = {}, slice = {};
    hipError_t e = raise_lds_limit(reinterpret_cast<const void*>(gate_fused_kernel<S, BN, LIN>), GateCfg<S, BN>::LDS_BYTES, whole);
    if (e == hipSuccess) e = raise_lds_limit(reinterpret_cast<const void*>(gate_slice_kernel<S, BN, LIN>), GateCfg<S, BN>::LDS_BYTES, slice);
    return e;
}

template <class S, int BN, bool LIN>
hipError_t launch_gate_fused_t(const GateArgs& a, hipStream_t stream) {
    if (hipError_t e = prepare_gate_fused_t<S, BN, LIN>(); e != hipSuccess) return e;
    constexpr int lds_bytes = GateCfg<S, BN>::LDS_BYTES;
    const unsigned tiles = (unsigned)((a.T + G_BM - 1) / G_BM);
    if (a.slices > 1) {
        hipLaunchKernelGGL((gate_slice_kernel<S, BN, LIN>), dim3(tiles * (unsigned)a.slices), dim3(G_THREADS), lds_bytes, stream, a);
        hipLaunchKernelGGL(gate_finish_kernel<BN>, dim3((unsigned)((a.T + F_ROWS - 1) / F_ROWS)), dim3(F_WGTHREADS), finish_lds<BN>(), stream, a);
    } else {
        hipLaunchKernelGGL((gate_fused_kernel<S, BN, LIN>), dim3(tiles), dim3(G_THREADS), lds_bytes, stream, a);
    }
    return hipGetLastError();
}

template <class S>
hipError_t launch_gate_fused_s(const GateArgs& a, hipStream_t stream) {
    if constexpr (S::kBytes == 4) {
        if (a.E <= 64) return launch_gate_fused_t<F32, 64, false>(a, stream);
    } else {
        if (a.E % 8 != 0) return a.E <= 128 ? launch_gate_fused_t<S, 128, true>(a, stream) : launch_gate_fused_t<S, 256, true>(a, stream);
    }
    return a.E <= 128 ? launch_gate_fused_t<S, 128, false>(a, stream) : launch_gate_fused_t<S, 256, false>(a, stream);
}

template <class S>
hipError_t prepare_gate_fused_16() {
    hipError_t e = prepare_gate_fused_t<S, 128, false>();
    if (e == hipSuccess) e = prepare_gate_fused_t<S, 256, false>();
    if (e == hipSuccess) e = prepare_gate_fused_t<S, 128, true>();
    if (e == hipSuccess) e = prepare_gate_fused_t<S, 256, true>();
    return e;
}

}  // namespace

hipError_t prepare_gate_fused() {
    hipError_t e = prepare_gate_fused_t<F32, 64, false>();
    if (e == hipSuccess) e = prepare_gate_fused_t<F32, 128, false>();
    if (e == hipSuccess) e = prepare_gate_fused_t<F32, 256, false>();
    if (e == hipSuccess) e = prepare_gate_fused_16<BF16>();
    if (e == hipSuccess) e = prepare_gate_fused_16<F16>();
    return e;
}

// (rows of Wg are read 16 bytes at a time in fp32 and, where E is a multiple of 8, in 16-bit storage; 8 bytes where it is one of 4)
bool gate_fused_eligible(int T, int H, int E, int k, int dtype) {
    const int el = dtype == 0 ? 4 : 2, kt = 128 / el;
    return E % 4 == 0 && E >= 4 && E <= 256 && H % 8 == 0 && H >= 8 && k >= 1 && k <= E &&
           (long long)G_BM * H * el < (1ll << 31) && (long long)kt * E * el < (1ll << 31);
}

// Slices of at least four K-tiles, at most a workgroup per CU and kGateSlices slices; worth a second launch (about 5 us) where each
// tile's chain of K-tiles gets shorter by more than that.
int gate_slices(int T, int H, int dtype, int cus, size_t partial_bytes, int E) {
    const int nk = gate_k_tiles(H, dtype == 0 ? 4 : 2), tiles = (T + G_BM - 1) / G_BM;
    constexpr int kGateSlices = 16;
    long long s = nk / 4 < kGateSlices ? nk / 4 : kGateSlices;
    if (s > cus / tiles) s = cus / tiles;
    const long long room = (long long)(partial_bytes / ((size_t)T * E * sizeof(float)));
    if (s > room) s = room;
    if (s < 2 || nk - nk / s < (dtype == 0 ? 12 : 18)) return 1;
    return (int)s;
}

hipError_t launch_gate_fused(const void* x, const void* Wg, const float* gate_bias, int T, int H, int E, int k,
                             int dtype, float* logits, int32_t* topk_expert, float* topk_weight,
                             int32_t* route_counts, int slices, float* partial, hipStream_t stream) {
    static_assert(G_BM == 64, "a workgroup's tokens are one chunk of the routing scan");
    const GateArgs a{(const unsigned char*)x, (const unsigned char*)Wg, gate_bias, T, H, E, k, logits, topk_expert, topk_weight,
                     route_counts, slices, partial};
    switch (dtype) {
        case 0: return launch_gate_fused_s<F32>(a, stream);
        case 1: return launch_gate_fused_s<BF16>(a, stream);
        default: return launch_gate_fused_s<F16>(a, stream);
    }
}

}  // namespace moe
