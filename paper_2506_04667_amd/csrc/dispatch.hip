// Dispatch on one GPU (Alg. 1 "Dispatch"): builds the routing table
// T_phi(e, c) = (token, combine weight) with token-order slot assignment and
// drops beyond the capacity C, then packs the kept token rows into the per-expert
// buffer xe[E, C_pad, H] (the one-GPU residue of the symmetric layout's (C, H)
// cells, capacity aligned to the row tile as in Sec. 3.2.1).
//
// Slot assignment is integer work and fully deterministic: the (token, choice)
// pairs, in token-major order, are cut into chunks of 64 tokens (64 k pairs); a
// pair's slot is the number of pairs before it that name the same expert.
//   count: one workgroup per chunk histograms its pairs by expert (LDS integer atomics).
//          The fused gate kernel, whose workgroups own the same 64 tokens, writes these
//          counts itself (the routing table as a by-product of the gate, Alg. 1), and the
//          launch is skipped, as it is when there are few pairs (below);
//   route: one workgroup per chunk adds up the counts of the chunks before it (or, with few
//          pairs, counts those pairs again itself) and hands out its pairs' slots; further workgroups
//          add up all counts: the experts' demand, the empty ends of the routing table, and the
//          FFN kernels' list of live (expert, row tile) units.
// Many chunks or experts (launch_route has the line): one wavefront per expert scans the counts in a launch of its own.
#include "route_body.h"

namespace moe {
namespace {

constexpr int kChunkTokens = 64;                        // tokens per chunk = tokens per fused-gate workgroup

// One workgroup per chunk: per-expert counts in an LDS histogram (integer atomics, so the result does not
// depend on their order).
__global__ __launch_bounds__(256) void route_count_kernel(const int32_t* __restrict__ topk_expert, long long P,
                                                          int chunk_pairs, int T, int k, bool choice_major, int E,
                                                          int32_t* __restrict__ counts) {
    extern __shared__ int32_t hist[];                // [E]
    for (int e = threadIdx.x; e < E; e += 256) hist[e] = 0;
    __syncthreads();
    const long long p0 = (long long)blockIdx.x * chunk_pairs;
    const long long p1 = p0 + chunk_pairs < P ? p0 + chunk_pairs : P;
    for (long long p = p0 + threadIdx.x; p < p1; p += 256) {
        const int e = topk_expert[pair_index(p, T, k, choice_major)];
        if (e >= 0 && e < E) atomicAdd(&hist[e], 1);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += 256) counts[(size_t)blockIdx.x * E + e] = hist[e];
}

// One wavefront per expert: exclusive scan of its per-chunk counts.  The launch also empties the routing table
// (slot_token = -1, slot_weight = 0).
__global__ __launch_bounds__(256) void route_scan_kernel(int32_t* __restrict__ counts, int n_chunks, int E,
                                                         int32_t* __restrict__ expert_demand,
                                                         int32_t* __restrict__ slot_token,
                                                         float* __restrict__ slot_weight, long long EC) {
    route_clear_tables(slot_token, slot_weight, EC, blockIdx.x * (long long)blockDim.x + threadIdx.x, (long long)gridDim.x * blockDim.x);
    const int e = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (e < E) route_scan_expert(counts, n_chunks, E, e, expert_demand);
}

// Pairs that a workgroup of route_kernel counts again itself rather than have them counted in a launch of their own.
constexpr int kRouteRecountPairs = 8192;

// Where a workgroup of route_kernel finds how many pairs before its own name each expert.
enum RouteBase { kRouteRecount, kRouteCounts, kRouteScanned };

struct RouteArgs {
    const int32_t* topk_expert; const float* topk_weight;
    long long P; int chunk_pairs, n_chunks, T, E, k, C; bool choice_major;
    const int32_t* counts;                           // kRouteCounts: [chunk][E] counts; kRouteScanned: their exclusive scan
    int32_t *slot, *expert_demand, *slot_token; float* slot_weight;
    int32_t* ffn_units; bool f32_units;
    int waves;                                       // wavefronts that hand out a chunk's slots
    int total_wgs;                                   // workgroups before the chunks': demand, empty slots, unit list
};

// The first total_wgs workgroups: what depends on the whole count.  Then one workgroup per chunk: its pairs' slots.
// Slots that a kept pair fills and slots that stay empty are disjoint, so nothing has to be cleared before.
// Latency bounds it: 1024 threads have up to eight rows of counts each in flight, and the pairs of a chunk are ranked by up
// to 16 wavefronts at once.  In the layer, against the scan and the scatter (one wavefront per chunk) as launches of their own:
// 9.4 us for 10.9 at T = 16384, E = 128, top-2; 6.8 for 15.1 at T = 4096, E = 32, top-8; 7.0 for 10.3 at 64 tokens, E = 128; and
// 7.0 for 14.5, the count's launch among them, where the pairs are counted again (T = 4096, E = 16, top-2).
template <RouteBase BASE>
__global__ __launch_bounds__(1024) void route_kernel(RouteArgs a) {
    extern __shared__ int32_t pre[];                 // [E] pairs before this workgroup's that name the expert; then cnt[waves][E]
    __shared__ int wave_total[32];
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid % kWave, wave = tid / kWave, E = a.E;
    const int chunk = (int)blockIdx.x - a.total_wgs;
    const bool total = chunk < 0;
    const int limit = total ? a.n_chunks : chunk;    // chunks to add up
    const int nbits = route_expert_bits(E);
    // 64 pairs per wavefront at a time; the first ones are fetched while the pairs before are counted
    const long long p_begin = (long long)chunk * a.chunk_pairs, p_end = min(p_begin + a.chunk_pairs, a.P);
    auto fetch = [&](long long p, long long& m, int& e, float& w) {
        const bool mine = !total && wave < a.waves && p < p_end;
        m = mine ? pair_index(p, a.T, a.k, a.choice_major) : -1;
        e = mine ? a.topk_expert[m] : -1;
        w = mine ? a.topk_weight[m] : 0.0f;
    };
    long long m;
    int e;
    float w;
    fetch(p_begin + wave * kWave + lane, m, e, w);
    if constexpr (BASE == kRouteScanned) {
        for (int e = tid; e < E; e += nt) pre[e] = total ? a.expert_demand[e] : a.counts[(size_t)chunk * E + e];
    } else {
        for (int e = tid; e < E; e += nt) pre[e] = 0;
        __syncthreads();
        if constexpr (BASE == kRouteCounts) {
            const int vec = E % 4 == 0 ? 4 : 1, cols = E / vec;         // cols <= 1024
            const int group = tid / cols, groups = nt / cols, e0 = tid % cols * vec;
            if (group < groups) {
                int sum[4] = {0, 0, 0, 0};
                constexpr int kTrip = 8;             // loads in flight; those beyond the last chunk are left out
                for (int c0 = group; c0 < limit; c0 += kTrip * groups) {
                    u32x4 v[kTrip];
#pragma unroll
                    for (int i = 0; i < kTrip; ++i) {
                        const int c = c0 + i * groups;
                        v[i] = u32x4{0u, 0u, 0u, 0u};
                        if (c < limit) {
                            const int32_t* const p = a.counts + (size_t)c * E + e0;
                            if (vec == 4) v[i] = *(const u32x4*)p;
                            else v[i][0] = (uint32_t)*p;
                        }
                    }
#pragma unroll
                    for (int i = 0; i < kTrip; ++i)
#pragma unroll
                        for (int q = 0; q < 4; ++q) sum[q] += (int)v[i][q];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (sum[q]) atomicAdd(&pre[e0 + q], sum[q]);
            }
        } else {
            const int n = (int)min((long long)limit * a.chunk_pairs, a.P);
            constexpr int kTrip = kRouteRecountPairs / 1024;
            int e[kTrip];
#pragma unroll
            for (int i = 0; i < kTrip; ++i) {
                const int q = i * 1024 + tid;
                e[i] = q < n ? a.topk_expert[pair_index32(q, a.T, a.k, a.choice_major)] : -1;
            }
#pragma unroll
            for (int i = 0; i < kTrip; ++i) {
                if (i * 1024 + wave * kWave >= n) break;
                const bool valid = e[i] >= 0 && e[i] < E;
                int rank, group;
                route_match(valid ? e[i] : 0, valid, nbits, rank, group);
                if (valid && rank == 0) atomicAdd(&pre[e[i]], group);
            }
        }
    }
    __syncthreads();
    if (total) {
        const int j = blockIdx.x;
        if (BASE != kRouteScanned) {
            if (j == 0)
                for (int e = tid; e < E; e += nt) a.expert_demand[e] = pre[e];
            for (int e = j * (nt / kWave) + wave; e < E; e += a.total_wgs * (nt / kWave))
                for (int s = min(pre[e], a.C) + lane; s < a.C; s += kWave) {
                    a.slot_token[(size_t)e * a.C + s] = -1;
                    a.slot_weight[(size_t)e * a.C + s] = 0.0f;
                }
        }
        if (j == a.total_wgs - 1 && a.ffn_units) {
            if (a.f32_units) build_row_units(pre, a.C, E, a.C, a.ffn_units, wave_total, nt);
            else build_ffn_units(pre, a.C, E, a.C, a.ffn_units, wave_total, nt);
        }
        return;
    }
    if (a.waves == 0) {                              // no room in LDS for counts per wavefront
        if (wave == 0)
            route_scatter_chunk(a.topk_expert, a.topk_weight, a.P, a.chunk_pairs, a.T, a.choice_major, E, a.k, a.C, a.slot, a.slot_token,
                                a.slot_weight, chunk, pre);
        return;
    }
    // counts per wavefront and expert, their running sum over the wavefronts, then the slots
    int32_t* const cnt = pre + E + wave * E;         // this wavefront's row (the first a.waves wavefronts have one)
    for (long long p0 = p_begin; p0 < p_end; p0 += a.waves * kWave) {
        if (p0 != p_begin) fetch(p0 + wave * kWave + lane, m, e, w);
        const bool valid = e >= 0 && e < E;
        if (!valid) e = 0;
        int rank = 0, group = 0;
        if (wave < a.waves) {
            for (int i = lane; i < E; i += kWave) cnt[i] = 0;
            route_match(e, valid, nbits, rank, group);
            wave_lds_sync();
            if (valid && rank == 0) cnt[e] = group;
        }
        __syncthreads();
        for (int i = tid; i < E; i += nt) {
            int run = pre[i];
            for (int v = 0; v < a.waves; ++v) {
                const int n = pre[E + v * E + i];
                pre[E + v * E + i] = run;
                run += n;
            }
            pre[i] = run;
        }
        __syncthreads();
        if (m >= 0) {
            const int s = valid ? cnt[e] + rank : 0;
            const bool kept = valid && s < a.C;
            a.slot[m] = kept ? s : -1;
            if (kept) {
                a.slot_token[(size_t)e * a.C + s] = (int32_t)(m / a.k);
                a.slot_weight[(size_t)e * a.C + s] = w;
            }
        }
        if (wave < a.waves) wave_lds_sync();         // the row is read before it is cleared again
    }
}

// One workgroup per token: the row is read once and written to each kept slot.
__global__ __launch_bounds__(256) void pack_kernel(const u32x4* __restrict__ x, const int32_t* __restrict__ topk_expert,
                                                   const int32_t* __restrict__ slot, int row_chunks, int k, int E,
                                                   int C, int C_pad, u32x4* __restrict__ xe) {
    const int t = blockIdx.x;
    for (int c = threadIdx.x; c < row_chunks; c += blockDim.x) {
        const u32x4 v = x[(size_t)t * row_chunks + c];
        for (int j = 0; j < k; ++j) {
            const int s = slot[(size_t)t * k + j];
            if (s < 0 || s >= C) continue;
            const int e = topk_expert[(size_t)t * k + j];
            if (e < 0 || e >= E) continue;
            xe[((size_t)e * C_pad + s) * row_chunks + c] = v;
        }
    }
}

}  // namespace

int route_chunk_tokens() { return kChunkTokens; }
int route_chunks(int T) { return (T + kChunkTokens - 1) / kChunkTokens; }

// One launch reads every count once per chunk, so its traffic grows with the square of the chunks: up to
// kRouteOneLaunchChunks chunks and kRouteOneLaunchCounts counts it is the faster form, beyond that the scan in a launch of its own.
constexpr int kRouteOneLaunchChunks = 1024, kRouteOneLaunchCounts = 65536;

hipError_t launch_route(const int32_t* topk_expert, const float* topk_weight, int T, int E, int k, int C,
                        bool choice_major, int32_t* counts, bool counts_ready, int32_t* slot, int32_t* expert_demand,
                        int32_t* slot_token, float* slot_weight, int32_t* ffn_units, bool f32_units, hipStream_t stream) {
    const int n_chunks = route_chunks(T);
    const long long EC = (long long)E * C;
    RouteArgs a{};
    a.topk_expert = topk_expert; a.topk_weight = topk_weight;
    a.P = (long long)T * k; a.chunk_pairs = kChunkTokens * k; a.n_chunks = n_chunks;
    a.T = T; a.E = E; a.k = k; a.C = C; a.choice_major = choice_major;
    a.counts = counts; a.slot = slot; a.expert_demand = expert_demand; a.slot_token = slot_token; a.slot_weight = slot_weight;
    a.ffn_units = ffn_units; a.f32_units = f32_units;
    const bool one_launch = E <= 1024 && n_chunks <= kRouteOneLaunchChunks && (long long)n_chunks * E <= kRouteOneLaunchCounts;
    const bool recount = one_launch && !counts_ready && a.P <= kRouteRecountPairs;
    // wavefronts per chunk: 64 k pairs, 32 KB of counts
    a.waves = k < 16 ? k : 16;
    if (a.waves * E > 8192) a.waves = E <= 4096 ? 8192 / E : 0;
    const size_t lds = (size_t)E * sizeof(int32_t) * (1 + a.waves);
    if (!counts_ready && !recount)
        hipLaunchKernelGGL(route_count_kernel, dim3(n_chunks), dim3(256), (size_t)E * sizeof(int32_t), stream,
                           topk_expert, a.P, a.chunk_pairs, T, k, choice_major, E, counts);
    if (one_launch) {
        const long long wgs = (EC + 16383) / 16384;
        a.total_wgs = wgs > 64 ? 64 : (int)wgs;
        const dim3 grid(n_chunks + a.total_wgs), block(1024);
        if (recount) hipLaunchKernelGGL(route_kernel<kRouteRecount>, grid, block, lds, stream, a);
        else hipLaunchKernelGGL(route_kernel<kRouteCounts>, grid, block, lds, stream, a);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(route_scan_kernel, dim3((E + 3) / 4), dim3(256), 0, stream, counts, n_chunks, E,
                       expert_demand, slot_token, slot_weight, EC);
    a.total_wgs = ffn_units ? 1 : 0;
    hipLaunchKernelGGL(route_kernel<kRouteScanned>, dim3(n_chunks + a.total_wgs), dim3(a.waves > 4 ? a.waves * kWave : 256), lds, stream, a);
    return hipGetLastError();
}

hipError_t launch_pack(const void* x, const int32_t* topk_expert, const int32_t* slot, int T, int H, int k,
                       int E, int C, int C_pad, int dtype, void* xe, hipStream_t stream) {
    const int bytes = dtype == 0 ? 4 : 2;
    const int row_chunks = H * bytes / 16;
    hipLaunchKernelGGL(pack_kernel, dim3(T), dim3(256), 0, stream, (const u32x4*)x, topk_expert, slot,
                       row_chunks, k, E, C, C_pad, (u32x4*)xe);
    return hipGetLastError();
}

}  // namespace moe
