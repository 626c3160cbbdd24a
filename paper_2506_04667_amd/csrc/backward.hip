// Helper kernels of the layer's backward pass (gradients under a fixed routing; the paper leaves training to
// future work, so this follows the chain rule of Eq. "ffn" and Eqs. "combine 1/2" as stated in include/moe.h).
// The dense contractions of the backward pass run on the grouped GEMM kernels; what is here is the data movement
// and elementwise work between them: gathering rows through the routing table, the activation and its
// derivative, the softmax Jacobian of the gate, transposes that turn weight-gradient products into row-major
// GEMMs, column sums for the bias gradients, and the final gather of dx.  Every reduction has a fixed order, so
// gradients are bit-identical from run to run.
#include "common.h"
#include "kernels.h"

#include <type_traits>

namespace moe {
namespace {

// derivative of phi_1 at the pre-activation v (act codes of moe_act)
__device__ __forceinline__ float act_grad(float v, int act) {
    switch (act) {
        case 0: return v > 0.0f ? 1.0f : 0.0f;
        case 1: {
            const float c = 0.7978845608028654f;
            const float t = tanh_fast(c * (v + 0.044715f * v * v * v));
            return 0.5f * (1.0f + t) + 0.5f * v * (1.0f - t * t) * c * (1.0f + 3.0f * 0.044715f * v * v);
        }
        case 2: return 0.5f * (1.0f + erf_as(v * 0.7071067811865476f)) + v * __expf(-0.5f * v * v) * 0.3989422804014327f;
        default: return 1.0f;
    }
}

// 16 bytes that this kernel reads once: the non-temporal hint (on this chip reads of data that is not in any cache run at
// half the rate without it)
__device__ __forceinline__ u32x4 load_once(const void* base, size_t chunk) { return __builtin_nontemporal_load((const u32x4*)base + chunk); }

// a 16-byte chunk of storage <-> its S::kVec values as floats
template <class S>
__device__ __forceinline__ void chunk_to_floats(const u32x4& v, float (&f)[S::kVec]) {
    if constexpr (S::kBytes == 4) {
#pragma unroll
        for (int q = 0; q < 4; ++q) { const uint32_t u = v[q]; f[q] = __builtin_bit_cast(float, u); }
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t u = v[q];
            f[2 * q] = bits16_to_float<S>((uint16_t)(u & 0xffffu));
            f[2 * q + 1] = bits16_to_float<S>((uint16_t)(u >> 16));
        }
    }
}
template <class S>
__device__ __forceinline__ u32x4 floats_to_chunk(const float (&f)[S::kVec]) {
    u32x4 v;
    if constexpr (S::kBytes == 4) {
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = __builtin_bit_cast(uint32_t, f[q]);
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = (uint32_t)float_to_bits16<S>(f[2 * q]) | ((uint32_t)float_to_bits16<S>(f[2 * q + 1]) << 16);
    }
    return v;
}

// Rows of an expert's buffers with `live` live ones that are written: those, and zeros up to the end of the K-tile in which the
// weight gradients' sums over the rows end (their products read no further; row_step is its depth).
__device__ __forceinline__ int written_rows(int live, int row_step) { return (max(live, 1) + row_step - 1) / row_step * row_step; }

// One workgroup per slot row (e, s), s < C_pad: xe[e, s, :] = x[token, :] and ge[e, s, :] = dout[token, :]
// for a live slot, zeros for an empty one that the weight gradients read.  16 bytes per lane.
// ge and the slot's combine weight change their sign together for about half of the tokens.  Everything made of them is a
// product of the two and comes out as without, except the rounding of dh = ge W2^T: the matrix instructions line up their terms
// by cutting them off towards minus infinity, every dh is low by a little, and db1, a sum over an expert's rows, would add that
// up (4096 rows, H = 2048, fp32: relative error 4.5e-6 against 8.4e-7).  The sign is the token's, not the slot's, so that a
// token's choices stay low or high together, which the softmax's Jacobian takes out again.
// In fp16 a power of two goes the other way from the weight to ge as well: h = w phi(a) is stored in fp16, whose numbers end at
// 2^-24, and a weight of 2^-20 left it 4 bits (dW2 of such rows: off by 2.6 %, 0.03 % like this).  Half of what the weight is smaller than the
// row of dout puts both at the same distance from that end; it leaves weight and row alone where the row is the smaller one.
__device__ __forceinline__ bool negated(int token) { return ((uint32_t)token * 0x9e3779b1u >> 31) != 0; }

// The workgroups after the rows' transpose Wg for bwd_finish_kernel, a 32 x 32 tile each: WgT[e][h] = Wg[h][e].
template <class elem>
__device__ __forceinline__ void transpose_gate_weights(const elem* __restrict__ Wg, elem* __restrict__ WgT, int H, int E, int tile_id) {
    __shared__ elem tile[32][33];
    const int nh = (H + 31) / 32, h0 = tile_id % nh * 32, e0 = tile_id / nh * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;             // 32 x 8
    for (int r = ty; r < 32; r += 8)
        if (h0 + r < H && e0 + tx < E) tile[r][tx] = Wg[(size_t)(h0 + r) * E + e0 + tx];
    __syncthreads();
    for (int r = ty; r < 32; r += 8)
        if (e0 + r < E && h0 + tx < H) WgT[(size_t)(e0 + r) * H + h0 + tx] = tile[tx][r];
}

template <class S>
__global__ __launch_bounds__(256) void bwd_gather_kernel(const void* __restrict__ x, const void* __restrict__ dout,
                                                         const int32_t* __restrict__ slot_token, float* __restrict__ slot_weight,
                                                         const int32_t* __restrict__ expert_demand, int H, int C, int C_pad, int row_step,
                                                         void* __restrict__ xe, void* __restrict__ ge, int rows,
                                                         const void* __restrict__ Wg, void* __restrict__ WgT, int E) {
    if ((int)blockIdx.x >= rows) {
        typedef typename S::store_t elem;
        return transpose_gate_weights((const elem*)Wg, (elem*)WgT, H, E, (int)blockIdx.x - rows);
    }
    const size_t row = blockIdx.x;
    const int e = (int)(row / C_pad), s = (int)(row % C_pad);
    if (s >= written_rows(min(expert_demand[e], C), row_step)) return;
    const int tok = s < C ? slot_token[(size_t)e * C + s] : -1;
    const int row_chunks = H / S::kVec;
    const bool neg = tok >= 0 && negated(tok);
    const uint32_t sign = !neg ? 0u : S::kBytes == 4 ? 0x80000000u : 0x80008000u;
    int shift = 0;                                      // ge is divided by 2^shift
    if constexpr (std::is_same<S, F16>::value) {
        if (tok >= 0) {                                 // the same for the whole workgroup
            __shared__ uint32_t part[4];
            uint32_t most = 0;                          // largest magnitude of the row, as bits
            for (int c = threadIdx.x; c < row_chunks; c += 256) {
                const u32x4 v = ((const u32x4*)dout)[(size_t)tok * row_chunks + c];
#pragma unroll
                for (int q = 0; q < 4; ++q) most = max(most, max(v[q] & 0x7fffu, v[q] >> 16 & 0x7fffu));
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, off));
            if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = most;
            __syncthreads();
            most = max(max(part[0], part[1]), max(part[2], part[3]));
            const float w = slot_weight[(size_t)e * C + s];
            const int w_exp = (int)(__builtin_bit_cast(uint32_t, w) >> 23) - 127, row_exp = (int)(most >> 10) - 15;
            shift = min(max((row_exp - w_exp) / 2, 0), min(max(-w_exp, 0), 24));
            __syncthreads();                            // every thread has read the weight
        }
    }
    if (tok >= 0 && (neg || shift) && threadIdx.x == 0) {
        const float w = slot_weight[(size_t)e * C + s];
        slot_weight[(size_t)e * C + s] = ldexpf(neg ? -w : w, shift);
    }
    for (int c = threadIdx.x; c < row_chunks; c += 256) {
        u32x4 xv = {0u, 0u, 0u, 0u}, gv = {0u, 0u, 0u, 0u};
        if (tok >= 0) {
            xv = load_once(x, (size_t)tok * row_chunks + c);
            gv = load_once(dout, (size_t)tok * row_chunks + c) ^ sign;
            if constexpr (std::is_same<S, F16>::value) {
                if (shift) {
                    float f[S::kVec];
                    chunk_to_floats<S>(gv, f);
#pragma unroll
                    for (int q = 0; q < S::kVec; ++q) f[q] = ldexpf(f[q], -shift);
                    gv = floats_to_chunk<S>(f);
                }
            }
        }
        ((u32x4*)xe)[row * row_chunks + c] = xv;
        ((u32x4*)ge)[row * row_chunks + c] = gv;
    }
}

// the value that lane j (uniform) holds, whether or not that lane takes part in the current pass: a shuffle reads 0 from
// lanes that are switched off, as most are in the last pass over a row whose length is not a multiple of 64 chunks
__device__ __forceinline__ int lane_value(int v, int j) { return __builtin_amdgcn_readlane(v, j); }
__device__ __forceinline__ float lane_value(float v, int j) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), j)); }
__device__ __forceinline__ long long lane_value(long long v, int j) {
    const uint32_t lo = __builtin_amdgcn_readlane((int)v, j), hi = __builtin_amdgcn_readlane((int)(v >> 32), j);
    return (long long)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// One workgroup per slot row (e, s), s < C_pad: with w the row's combine weight and dh = dout W2^T (fp32; dout and w both
// with the sign that bwd_gather_kernel gave them),
//   h = w phi(a) (may be in the place of a),  da = w dh phi'(a)  (fp32 storage: may be in the place of dh),
//   p[e, s] = w (<phi(a), dh> + <dout, b2>)  =  w <dout, phi(a) W2 + b2>,
// the weight times the gradient with respect to it.  dh is there anyway, so the gate's Jacobian needs neither
// y = phi(a) W2 + b2 nor another pass over dout (a sixth of the backward pass's matrix work: at T = 16384, H = I = 2048,
// E = 128, bf16 that product, the dot products with its rows and a separate pass for h were 0.36 of 3.2 ms; at T = 2048,
// H = 1024, I = 4096, E = 16, fp32 0.43 of 2.02 ms).  The weight goes to h and da in fp32, so dout itself is the other operand
// of dW2 and is not rounded again.  Empty rows that the weight gradients read give h = da = 0 (p is not written).  The row's sum is
// added in a fixed order.
template <class S>
__global__ __launch_bounds__(256) void bwd_act_kernel(const void* a, const float* dh, const void* __restrict__ ge,
                                                      const void* __restrict__ b2, const int32_t* __restrict__ expert_demand,
                                                      const float* __restrict__ slot_weight, int C, int C_pad, int row_step, int H, int I, int act,
                                                      void* h, void* da, float* __restrict__ p) {
    constexpr int VEC = S::kVec;
    __shared__ float part[4];
    const size_t row = blockIdx.x;
    const int e = (int)(row / C_pad), s = (int)(row % C_pad);
    const int n = min(expert_demand[e], C);
    if (s >= written_rows(n, row_step)) return;
    const bool live = s < n;
    const float w = live ? slot_weight[(size_t)e * C + s] : 0.0f;
    const int row_chunks = I / VEC;
    float sum = 0.0f;
    for (int c = threadIdx.x; c < row_chunks; c += 256) {
        u32x4 o = {0u, 0u, 0u, 0u}, d = {0u, 0u, 0u, 0u};
        if (live) {
            float av[VEC], gf[VEC], hv[VEC];
            chunk_to_floats<S>(load_once(a, row * row_chunks + c), av);
#pragma unroll
            for (int q = 0; q < VEC; q += 4) {
                const f32x4 g4 = __builtin_nontemporal_load((const f32x4*)(dh + row * I + (size_t)c * VEC + q));
                gf[q] = g4[0]; gf[q + 1] = g4[1]; gf[q + 2] = g4[2]; gf[q + 3] = g4[3];
            }
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                const float v = apply_act(av[q], act);
                sum = fmaf(v, gf[q], sum);
                hv[q] = w * v;
                gf[q] *= w * act_grad(av[q], act);
            }
            o = floats_to_chunk<S>(hv);
            d = floats_to_chunk<S>(gf);
        }
        ((u32x4*)h)[row * row_chunks + c] = o;
        ((u32x4*)da)[row * row_chunks + c] = d;
    }
    if (!live) return;                                  // the same for the whole workgroup
    if (b2) {
        const int out_chunks = H / VEC;
        for (int c = threadIdx.x; c < out_chunks; c += 256) {
            float gf[VEC], bv[VEC];
            chunk_to_floats<S>(load_once(ge, row * out_chunks + c), gf);
            chunk_to_floats<S>(((const u32x4*)b2)[(size_t)e * out_chunks + c], bv);
#pragma unroll
            for (int q = 0; q < VEC; ++q) sum = fmaf(gf[q], bv[q], sum);
        }
    }
    sum = wave_sum(sum);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) p[row] = w * (part[0] + part[1] + part[2] + part[3]);
}

// One wavefront per token (k <= 64): p_ij = w_ij dL/dw_ij of kept pairs (0 for dropped ones), then the Jacobian of the
// softmax over the k selected logits: dl_ij = w_ij (dL/dw_ij - sum_j' w_ij' dL/dw_ij') = p_ij - w_ij sum_j' p_ij'.
// Writes dl[T, k] (fp32) and the dense matrix dL[T, ld] (storage type, zero where the token did not select the
// expert), which turns dWg = x^T dL into a GEMM.
template <class S>
__global__ __launch_bounds__(256) void bwd_gate_kernel(const float* __restrict__ p, const int32_t* __restrict__ topk_expert,
                                                       const float* __restrict__ topk_weight, const int32_t* __restrict__ slot,
                                                       int T, int T_pad, int k, int E, int C, int C_pad, int ld,
                                                       float* __restrict__ dl, void* __restrict__ dL) {
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (t >= T) {                                       // rows T .. T_pad - 1 of dL exist for the GEMM's sake: zeros
        if (t < T_pad)
            for (int c = lane; c < ld; c += 64) store_from_float<S>(dL, (size_t)t * ld + c, 0.0f);
        return;
    }
    int e_l = -1;
    float w_l = 0.0f, p_l = 0.0f;
    if (lane < k) {
        e_l = topk_expert[(size_t)t * k + lane];
        w_l = topk_weight[(size_t)t * k + lane];
        const int s = slot[(size_t)t * k + lane];
        if (s >= 0 && s < C && e_l >= 0 && e_l < E) p_l = p[(size_t)e_l * C_pad + s];
    }
    const float dl_l = p_l - w_l * wave_sum(p_l);
    if (lane < k) dl[(size_t)t * k + lane] = dl_l;
    for (int c = lane; c < ld; c += 64) {
        float v = 0.0f;
        for (int j = 0; j < k; ++j) {
            const int e = lane_value(e_l, j);
            const float d = lane_value(dl_l, j);
            if (e == c) v = d;
        }
        store_from_float<S>(dL, (size_t)t * ld + c, v);
    }
}

// out[g][c][r] = in[g][r][c] for r < R, c < Cc in fp32; out rows have ld_out >= R entries, those at and beyond R are zero.  With
// expert_demand, only up to the end of the K-tile of 32 rows in which the weight gradients' sums end: nothing beyond is read, and in
// holds zeros from the last live row to there.
// Bound by memory: 64 x 64 tiles through LDS (a pitch of 65 words, so that neither side meets a bank twice), 16 bytes per lane on both
// sides (Cc and ld_out are multiples of 4).  With 4 bytes per lane and all of ld_out, h^T, xe^T and x^T of T = 2048, H = 1024, I = 4096, E = 16
// (320 slots each, 256 live) took 52, 17 and 12 us; 23.6, 9.6 and 5.5 now.
__global__ __launch_bounds__(256) void bwd_transpose_kernel(const float* __restrict__ in, float* __restrict__ out, int R, int Cc, int ld_out,
                                                            const int32_t* __restrict__ expert_demand, int C) {
    constexpr int TS = 64, QUADS = TS / 4, TRIPS = TS * QUADS / 256;
    __shared__ float tile[TS][TS + 1];
    const size_t g = blockIdx.z;
    const int r0 = blockIdx.x * TS, c0 = blockIdx.y * TS;
    const int end = expert_demand ? min(written_rows(min(expert_demand[g], C), 32), ld_out) : ld_out;   // entries of an output row
    if (r0 >= end) return;
    const int last = min(R, end), q = threadIdx.x % QUADS * 4, i0 = threadIdx.x / QUADS;
    f32x4 v[TRIPS];
#pragma unroll
    for (int t = 0; t < TRIPS; ++t) {
        const int r = r0 + i0 + t * (256 / QUADS), c = c0 + q;
        v[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (r < last && c < Cc) v[t] = __builtin_nontemporal_load((const f32x4*)(in + (g * R + r) * Cc + c));
    }
#pragma unroll
    for (int t = 0; t < TRIPS; ++t)
#pragma unroll
        for (int b = 0; b < 4; ++b) tile[i0 + t * (256 / QUADS)][q + b] = v[t][b];
    __syncthreads();
#pragma unroll
    for (int t = 0; t < TRIPS; ++t) {
        const int i = i0 + t * (256 / QUADS), c = c0 + i, r = r0 + q;
        if (c < Cc && r < end) *(f32x4*)(out + (g * Cc + c) * ld_out + r) = f32x4{tile[q][i], tile[q + 1][i], tile[q + 2][i], tile[q + 3][i]};
    }
}

// out[e][c] = sum over the live rows r of weight[e][r] in[e][r][c] (fp32; WEIGHTED false: of in[e][r][c]).  A workgroup of four wavefronts owns 64 chunks of 16
// bytes of the columns of one expert; wavefront w adds the rows w, w + 4, ... in ascending order, four loads in flight
// per lane, and the four partial sums are added in wavefront order: a fixed order, the same from run to run.
template <class S, bool WEIGHTED>
__device__ __forceinline__ void bwd_colsum(const void* __restrict__ in, const float* __restrict__ weight,
                                           const int32_t* __restrict__ expert_demand, int C, int C_pad, int cols, float* __restrict__ out,
                                           int e, int block, float* __restrict__ lds) {
    constexpr int VEC = S::kVec;
    float (*part)[64][VEC] = (float (*)[64][VEC])lds;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row_chunks = cols / VEC, c = block * 64 + lane;
    const int n = min(expert_demand[e], C);
    float acc[VEC];
#pragma unroll
    for (int q = 0; q < VEC; ++q) acc[q] = 0.0f;
    if (c < row_chunks) {
        const u32x4* p = (const u32x4*)in + (size_t)e * C_pad * row_chunks + c;
        const float* const wrow = WEIGHTED ? weight + (size_t)e * C : nullptr;
        auto add = [&](const u32x4& v, int r) {
            float f[VEC];
            chunk_to_floats<S>(v, f);
            const float w = WEIGHTED ? wrow[r] : 1.0f;
#pragma unroll
            for (int q = 0; q < VEC; ++q) acc[q] = WEIGHTED ? fmaf(w, f[q], acc[q]) : acc[q] + f[q];
        };
        int r = wave;
        for (; r + 12 < n; r += 16) {
            u32x4 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = __builtin_nontemporal_load(p + (size_t)(r + 4 * i) * row_chunks);
#pragma unroll
            for (int i = 0; i < 4; ++i) add(v[i], r + 4 * i);
        }
        for (; r < n; r += 4) add(__builtin_nontemporal_load(p + (size_t)r * row_chunks), r);
    }
    if (wave > 0) {
#pragma unroll
        for (int q = 0; q < VEC; ++q) part[wave - 1][lane][q] = acc[q];
    }
    __syncthreads();
    if (wave == 0 && c < row_chunks) {
#pragma unroll
        for (int w = 0; w < 3; ++w)
#pragma unroll
            for (int q = 0; q < VEC; ++q) acc[q] += part[w][lane][q];
#pragma unroll
        for (int q = 0; q < VEC; ++q) out[(size_t)e * cols + c * VEC + q] = acc[q];
    }
}

// dgate_bias[e] = sum of dl over the pairs that selected e: one workgroup per expert, fixed reduction tree.
__device__ __forceinline__ void bwd_gate_bias(const int32_t* __restrict__ topk_expert, const float* __restrict__ dl, long long P,
                                              float* __restrict__ dgate_bias, int e, float* __restrict__ part) {
    float acc = 0.0f;
    const long long P4 = P / 4;                         // four pairs per thread and load (both tables are 16-byte aligned)
    constexpr int kTrip = 4;                            // loads of either table in flight
    for (long long p0 = threadIdx.x; p0 < P4; p0 += 256 * kTrip) {
        u32x4 ev[kTrip];
        f32x4 dv[kTrip];
#pragma unroll
        for (int i = 0; i < kTrip; ++i) {
            const long long p = min(p0 + i * 256, P4 - 1);
            ev[i] = ((const u32x4*)topk_expert)[p];
            dv[i] = ((const f32x4*)dl)[p];
        }
#pragma unroll
        for (int i = 0; i < kTrip; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (p0 + i * 256 < P4 && (int)ev[i][q] == e) acc += dv[i][q];
    }
    for (long long p = P4 * 4 + threadIdx.x; p < P; p += 256)
        if (topk_expert[p] == e) acc += dl[p];
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s >= 1; s >>= 1) {
        if ((int)threadIdx.x < s) part[threadIdx.x] += part[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) dgate_bias[e] = part[0];
}

// out[i] = part[0][i] + part[1][i] + ... in that order, i < n4
__device__ __forceinline__ void bwd_sum_slices(const f32x4* __restrict__ part, int slices, long long n4, f32x4* __restrict__ out, long long i) {
    if (i >= n4) return;
    f32x4 acc = part[i];
    for (int g = 1; g < slices; ++g) {
        const f32x4 v = part[(size_t)g * n4 + i];
        acc[0] += v[0]; acc[1] += v[1]; acc[2] += v[2]; acc[3] += v[3];
    }
    out[i] = acc;
}

// One wavefront per token: dx_i = sum over kept choices of dxe[e_ij, slot_ij, :] (ascending j), then
// + sum over all k choices of dl_ij * Wg[:, e_ij] (rows of WgT), in fp32.  Lane j holds the routing entries of choice j
// (k <= 64); a lane owns 16-byte chunks lane, lane + 64, ... of the row.
template <class S>
__device__ __forceinline__ void bwd_dx(const void* __restrict__ dxe, const void* __restrict__ WgT, const int32_t* __restrict__ topk_expert,
                                       const int32_t* __restrict__ slot, const float* __restrict__ dl, int T, int H, int k, int E, int C,
                                       int C_pad, float* __restrict__ dx, int block) {
    constexpr int VEC = S::kVec;
    const int t = block * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (t >= T) return;
    long long row_lane = -1;
    int e_lane = -1;
    float dl_lane = 0.0f;
    if (lane < k) {
        const int s = slot[(size_t)t * k + lane], e = topk_expert[(size_t)t * k + lane];
        if (e >= 0 && e < E) {
            e_lane = e;
            dl_lane = dl[(size_t)t * k + lane];
            if (s >= 0 && s < C) row_lane = (long long)e * C_pad + s;
        }
    }
    const int row_chunks = H / VEC;
    const u32x4* const dv = (const u32x4*)dxe;
    const u32x4* const wv = (const u32x4*)WgT;
    auto fma_chunk = [&](float (&acc)[VEC], float w, const u32x4& v) {
        if constexpr (S::kBytes == 4) {
#pragma unroll
            for (int q = 0; q < 4; ++q) { const uint32_t u = v[q]; acc[q] = fmaf(w, __builtin_bit_cast(float, u), acc[q]); }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t u = v[q];
                acc[2 * q] = fmaf(w, bits16_to_float<S>((uint16_t)(u & 0xffffu)), acc[2 * q]);
                acc[2 * q + 1] = fmaf(w, bits16_to_float<S>((uint16_t)(u >> 16)), acc[2 * q + 1]);
            }
        }
    };
    for (int c = lane; c < row_chunks; c += 64) {
        float acc[VEC];
#pragma unroll
        for (int q = 0; q < VEC; ++q) acc[q] = 0.0f;
        for (int j = 0; j < k; ++j) {
            const long long row = lane_value(row_lane, j);
            if (row >= 0) fma_chunk(acc, 1.0f, __builtin_nontemporal_load(dv + (size_t)row * row_chunks + c));
        }
        for (int j = 0; j < k; ++j) {
            const int e = lane_value(e_lane, j);
            const float d = lane_value(dl_lane, j);
            if (e >= 0) fma_chunk(acc, d, wv[(size_t)e * row_chunks + c]);
        }
#pragma unroll
        for (int q = 0; q < VEC; q += 4)
            *(f32x4*)(dx + (size_t)t * H + (size_t)c * VEC + q) = f32x4{acc[q], acc[q + 1], acc[q + 2], acc[q + 3]};
    }
}

// What is left once the weight gradients' products are made, in one launch: each of these is a few microseconds in a small layer,
// where a launch costs as much.  Workgroups in the order of the fields' ends; dx, the longest, comes last.
template <class S>
__global__ __launch_bounds__(256) void bwd_finish_kernel(BwdFinish a) {
    __shared__ __attribute__((aligned(16))) float lds[3 * 64 * S::kVec];
    static_assert(3 * 64 * S::kVec >= 256, "the gate bias's reduction");
    const int b = blockIdx.x;
    if (b < a.E) return bwd_gate_bias(a.topk_expert, a.dl, (long long)a.T * a.k, a.dgate_bias, b, lds);
    if (b < a.end_db2) {
        const int i = b - a.E, per = (a.end_db2 - a.E) / a.E;
        return bwd_colsum<S, true>(a.ge, a.slot_weight, a.expert_demand, a.C, a.C_pad, a.H, a.db2, i / per, i % per, lds);
    }
    if (b < a.end_db1) {
        const int i = b - a.end_db2, per = (a.end_db1 - a.end_db2) / a.E;
        return bwd_colsum<S, false>(a.da, nullptr, a.expert_demand, a.C, a.C_pad, a.I, a.db1, i / per, i % per, lds);
    }
    int start = a.end_db1;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        if (b < a.end_sum[q]) {
            const BwdSlices& m = a.sum[q];
            return bwd_sum_slices((const f32x4*)m.part, m.slices, m.n / 4, (f32x4*)m.out, (long long)(b - start) * 256 + threadIdx.x);
        }
        start = a.end_sum[q];
    }
    bwd_dx<S>(a.dxe, a.WgT, a.topk_expert, a.slot, a.dl, a.T, a.H, a.k, a.E, a.C, a.C_pad, a.dx, b - start);
}

}  // namespace

__global__ __launch_bounds__(256) void bwd_fill_rows_kernel(int32_t* __restrict__ rows, int E, int first, int second) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < 2 * E) rows[i] = i < E ? first : second;
}

hipError_t launch_bwd_fill_rows(int32_t* rows, int E, int first, int second, hipStream_t s) {
    hipLaunchKernelGGL(bwd_fill_rows_kernel, dim3((2 * E + 255) / 256), dim3(256), 0, s, rows, E, first, second);
    return hipGetLastError();
}

hipError_t launch_bwd_gather(const void* x, const void* dout, const int32_t* slot_token, float* slot_weight, const int32_t* expert_demand,
                             int H, int E, int C, int C_pad, int row_step, int dtype, void* xe, void* ge, const void* Wg, void* WgT, hipStream_t s) {
    const long long rows = (long long)E * C_pad, tiles = (long long)((H + 31) / 32) * ((E + 31) / 32);
    if (rows + tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 g((unsigned)(rows + tiles)), b(256);
    if (dtype == 0) hipLaunchKernelGGL(bwd_gather_kernel<F32>, g, b, 0, s, x, dout, slot_token, slot_weight, expert_demand, H, C, C_pad, row_step, xe, ge, (int)rows, Wg, WgT, E);
    else if (dtype == 1) hipLaunchKernelGGL(bwd_gather_kernel<BF16>, g, b, 0, s, x, dout, slot_token, slot_weight, expert_demand, H, C, C_pad, row_step, xe, ge, (int)rows, Wg, WgT, E);
    else hipLaunchKernelGGL(bwd_gather_kernel<F16>, g, b, 0, s, x, dout, slot_token, slot_weight, expert_demand, H, C, C_pad, row_step, xe, ge, (int)rows, Wg, WgT, E);
    return hipGetLastError();
}

hipError_t launch_bwd_act(const void* a, const float* dh, const void* ge, const void* b2, const int32_t* expert_demand,
                          const float* slot_weight, int E, int C, int C_pad, int row_step, int H, int I, int act, int dtype, void* h, void* da, float* p,
                          hipStream_t s) {
    const dim3 g((unsigned)((size_t)E * C_pad)), b(256);
#define MOE_BWD_ACT(S_) hipLaunchKernelGGL(bwd_act_kernel<S_>, g, b, 0, s, a, dh, ge, b2, expert_demand, slot_weight, C, C_pad, row_step, H, I, act, h, da, p)
    if (dtype == 0) MOE_BWD_ACT(F32);
    else if (dtype == 1) MOE_BWD_ACT(BF16);
    else MOE_BWD_ACT(F16);
#undef MOE_BWD_ACT
    return hipGetLastError();
}

hipError_t launch_bwd_gate(const float* p, const int32_t* topk_expert, const float* topk_weight, const int32_t* slot, int T, int T_pad,
                           int k, int E, int C, int C_pad, int ld, int dtype, float* dl, void* dL, hipStream_t s) {
    const dim3 g((unsigned)((T_pad + 3) / 4)), b(256);
    if (dtype == 0) hipLaunchKernelGGL(bwd_gate_kernel<F32>, g, b, 0, s, p, topk_expert, topk_weight, slot, T, T_pad, k, E, C, C_pad, ld, dl, dL);
    else if (dtype == 1) hipLaunchKernelGGL(bwd_gate_kernel<BF16>, g, b, 0, s, p, topk_expert, topk_weight, slot, T, T_pad, k, E, C, C_pad, ld, dl, dL);
    else hipLaunchKernelGGL(bwd_gate_kernel<F16>, g, b, 0, s, p, topk_expert, topk_weight, slot, T, T_pad, k, E, C, C_pad, ld, dl, dL);
    return hipGetLastError();
}

hipError_t launch_bwd_transpose(const float* in, float* out, int groups, int R, int Cc, int ld_out, const int32_t* expert_demand, int C,
                                hipStream_t s) {
    if (groups <= 0 || R <= 0 || Cc <= 0) return hipSuccess;
    if (groups > 65535 || (Cc + 63) / 64 > 65535 || (Cc & 3) || (ld_out & 3)) return hipErrorInvalidValue;
    const dim3 g((unsigned)((ld_out + 63) / 64), (unsigned)((Cc + 63) / 64), (unsigned)groups), b(256);
    hipLaunchKernelGGL(bwd_transpose_kernel, g, b, 0, s, in, out, R, Cc, ld_out, expert_demand, C);
    return hipGetLastError();
}

hipError_t launch_bwd_finish(BwdFinish a, int dtype, hipStream_t s) {
    const int vec = dtype == 0 ? 4 : 8;                  // elements of a 16-byte chunk; a workgroup of the column sums owns 64 chunks
    long long end = a.E;
    auto add = [&](long long n) {
        end += n;
        return end > 0x7fffffffLL ? 0x7fffffff : (int)end;
    };
    a.end_db2 = add((long long)a.E * ((a.H / vec + 63) / 64));
    a.end_db1 = add((long long)a.E * ((a.I / vec + 63) / 64));
    for (int q = 0; q < 3; ++q) a.end_sum[q] = add(a.sum[q].slices > 1 ? (a.sum[q].n / 4 + 255) / 256 : 0);
    add((a.T + 3ll) / 4);
    if (end > 0x7fffffffLL) return hipErrorInvalidValue;
    const dim3 g((unsigned)end), b(256);
    if (dtype == 0) hipLaunchKernelGGL(bwd_finish_kernel<F32>, g, b, 0, s, a);
    else if (dtype == 1) hipLaunchKernelGGL(bwd_finish_kernel<BF16>, g, b, 0, s, a);
    else hipLaunchKernelGGL(bwd_finish_kernel<F16>, g, b, 0, s, a);
    return hipGetLastError();
}

}  // namespace moe
