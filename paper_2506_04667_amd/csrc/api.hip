// C ABI of the MoE layer forward (see include/moe.h): argument validation,
// capacity arithmetic, workspace carving and the launch sequence
// gate -> dispatch -> expert FFN -> combine (Alg. 1 restricted to one GPU).
// Host code only; every step of the path runs in the kernels it launches.
#include "../../include/moe.h"

#include <algorithm>
#include <cmath>
#include <initializer_list>

#include "ffn_units.h"
#include "kernels.h"

// Scratch of moe_dispatch_noalloc, the entry point for callers that cannot allocate: a fixed array in device
// memory that every GPU the library runs on holds from the moment the code object is loaded there.  In host code
// this name is only a handle for hipGetSymbolAddress; the address it yields (one per device) is what kernels,
// fills and copies get.
constexpr size_t kStaticScratchBytes = 4u << 20;
static_assert(MOE_F32_BODY_64X256 == moe::kF32Body64x256 && MOE_F32_BODY_64 == moe::kF32Body64 && MOE_F32_BODY_128 == moe::kF32Body128 &&
                  MOE_F32_BODY_256 == moe::kF32Body256, "the header's numbers");
static_assert(MOE_KERNEL16_GENERIC == moe::kGemm16Generic && MOE_KERNEL16_128 == moe::kGemm16Narrow && MOE_KERNEL16_STREAM == moe::kGemm16Stream &&
                  MOE_KERNEL16_WGRAD == moe::kGemm16Wgrad, "the header's numbers");
static_assert(kStaticScratchBytes == MOE_STATIC_SCRATCH_BYTES, "the limit stated in the header");
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

// Device address of `scratch` on the current device, looked up once per device with that device current.
hipError_t static_scratch(void** out) {
    static std::atomic<void*> ptr[moe::kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= moe::kMaxDevices) return hipErrorInvalidDevice;
    void* p = ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        ptr[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return hipSuccess;
}

constexpr int kRowTile = 128;     // bM: per-expert buffers are aligned to this many rows
constexpr int kGatePad = 128;     // WgT rows are padded to a multiple of the gate GEMM's column tile
constexpr size_t kAlign = 256;

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

struct Plan {
    int C, C_pad, E_pad, elem;
    size_t off_wgt, off_logits, off_slot_token, off_slot_weight, off_counts, off_units, off_partials, off_h, off_y, total;
    int ldh;                                             // row pitch of h in elements
};

moe_status check_config(const moe_config* c) {
    if (!c) return MOE_ERR_INVALID_ARG;
    if (c->T <= 0 || c->H <= 0 || c->I <= 0 || c->E <= 0 || c->k <= 0 || c->k > c->E) return MOE_ERR_INVALID_ARG;
    if (c->capacity_override < 0) return MOE_ERR_INVALID_ARG;
    if (c->capacity_override == 0 && !(c->capacity_factor > 0.0f && std::isfinite(c->capacity_factor)))
        return MOE_ERR_INVALID_ARG;
    if (c->dtype < MOE_F32 || c->dtype > MOE_F16) return MOE_ERR_UNSUPPORTED;
    if (c->act < MOE_ACT_RELU || c->act > MOE_ACT_IDENTITY) return MOE_ERR_UNSUPPORTED;
    if (c->H % 8 != 0 || c->I % 8 != 0) return MOE_ERR_UNSUPPORTED;
    if (c->E > MOE_MAX_EXPERTS) return MOE_ERR_UNSUPPORTED;
    if (c->drop_policy < MOE_DROP_TOKEN_MAJOR || c->drop_policy > MOE_DROP_CHOICE_MAJOR) return MOE_ERR_UNSUPPORTED;
    if (c->capacity_mode < MOE_CAPACITY_PER_CHOICE || c->capacity_mode > MOE_CAPACITY_LAYOUT) return MOE_ERR_UNSUPPORTED;
    if (c->flags & ~(MOE_FLAG_FFN_SINGLE_LAUNCH | MOE_FLAG_DEBUG_DEPENDENCY_NEVER_MET | MOE_FLAG_LAYER_SINGLE_LAUNCH))
        return MOE_ERR_INVALID_ARG;
    if ((c->flags & MOE_FLAG_LAYER_SINGLE_LAUNCH) && (c->flags & ~MOE_FLAG_LAYER_SINGLE_LAUNCH)) return MOE_ERR_INVALID_ARG;
    if ((c->flags & MOE_FLAG_DEBUG_DEPENDENCY_NEVER_MET) && !(c->flags & MOE_FLAG_FFN_SINGLE_LAUNCH)) return MOE_ERR_INVALID_ARG;
    return MOE_OK;
}

moe_status capacity_of(const moe_config* c, int* C, int* C_pad) {
    long long cap;
    if (c->capacity_override > 0) {
        cap = c->capacity_override;
    } else {
        const double per_token = c->capacity_mode == MOE_CAPACITY_LAYOUT ? 1.0 : (double)c->k;
        const double v = std::ceil((double)c->capacity_factor * per_token * (double)c->T / (double)c->E);
        if (v > 2.0e9) return MOE_ERR_INVALID_ARG;
        cap = v < 1.0 ? 1 : (long long)v;
    }
    const long long pad = (cap + kRowTile - 1) / kRowTile * kRowTile;
    if (pad > 0x7fffffffLL) return MOE_ERR_INVALID_ARG;
    *C = (int)cap;
    *C_pad = (int)pad;
    return MOE_OK;
}

moe_status make_plan(const moe_config* c, Plan* p) {
    moe_status st = check_config(c);
    if (st != MOE_OK) return st;
    st = capacity_of(c, &p->C, &p->C_pad);
    if (st != MOE_OK) return st;
    p->elem = c->dtype == MOE_F32 ? 4 : 2;
    p->E_pad = (int)align_up((size_t)c->E, kGatePad);
    const size_t T = c->T, H = c->H, I = c->I, E = c->E, el = p->elem;
    const size_t rows = E * (size_t)p->C_pad;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, kAlign); return o; };
    p->off_wgt = take((size_t)p->E_pad * H * el);
    p->off_logits = take(T * E * 4);
    p->off_slot_token = take(E * (size_t)p->C * 4);
    p->off_slot_weight = take(E * (size_t)p->C * 4);
    p->off_counts = take((size_t)moe::route_chunks(c->T) * E * 4);
    // 16-bit storage: the two lists of live row tiles of the weight-streaming kernels; fp32: the list of live 256-row
    // tiles of the equal-span kernel and its partial tiles
    p->off_units = take((c->dtype == MOE_F32 ? moe::f32_units_ints(c->E, p->C) : moe::ffn_units_ints(c->E, p->C)) * 4);
    p->off_partials = take(c->dtype == MOE_F32 ? moe::f32_partials_bytes(c->E, p->C, c->H, c->I) : 0);
    p->ldh = c->I;                                       // (a pitch padded by one 128-byte line measured no different)
    p->off_h = take(rows * (size_t)p->ldh * el);
    p->off_y = take(rows * H * el);
    p->total = off;
    return MOE_OK;
}

bool misaligned(const void* p) { return ((uintptr_t)p & 15u) != 0; }

// MOE_FLAG_FFN_SINGLE_LAUNCH asks for both FFN tasks in one persistent launch; only shapes that the
// weight-streaming kernel takes for both tasks can run that way.  `gather`: the first task reads token rows
// through the routing table (moe_forward) instead of packed rows (moe_expert_ffn).
moe_status check_single_launch(const moe_config* c, const Plan& p, bool gather) {
    if (!(c->flags & MOE_FLAG_FFN_SINGLE_LAUNCH)) return MOE_OK;
    const bool ok = moe::stream_gemm_shape_ok(c->dtype, c->I, c->H, c->H, c->I, p.ldh, gather ? c->T : p.C_pad) &&
                    moe::stream_gemm_shape_ok(c->dtype, c->H, c->I, p.ldh, c->H, c->H, p.C_pad);
    return ok ? MOE_OK : MOE_ERR_UNSUPPORTED;
}

moe_status hip_status(hipError_t e) { return e == hipSuccess ? MOE_OK : MOE_ERR_HIP; }

char* ws_at(void* ws, size_t off) { return (char*)ws + off; }

// ---- stage launchers (arguments already validated) ---------------------------------

// the gate's slices; their sums lie where h and y go later
int gate_slices(const moe_config* c, const Plan& p) {
    return moe::gate_slices(c->T, c->H, c->dtype, moe::device_cu_count(), p.total - p.off_h, c->E);
}

moe_status run_gate(const moe_config* c, const Plan& p, void* ws, const void* x, const void* Wg,
                    const float* gate_bias, float* logits, int32_t* topk_expert, float* topk_weight,
                    bool* route_counts_written, hipStream_t s) {
    // route_counts_written != nullptr: the caller goes on to the slot assignment; the fused gate then writes
    // the per-chunk expert counts into the workspace and says so
    if (route_counts_written) *route_counts_written = false;
    if (moe::gate_fused_eligible(c->T, c->H, c->E, c->k, c->dtype)) {
        int32_t* counts = route_counts_written ? (int32_t*)ws_at(ws, p.off_counts) : nullptr;
        if (route_counts_written) *route_counts_written = true;
        return hip_status(moe::launch_gate_fused(x, Wg, gate_bias, c->T, c->H, c->E, c->k, c->dtype, logits, topk_expert, topk_weight,
                                                 counts, gate_slices(c, p), (float*)ws_at(ws, p.off_h), s));
    }
    void* wgt = ws_at(ws, p.off_wgt);
    hipError_t e = moe::launch_transpose_pad(Wg, wgt, c->H, c->E, p.E_pad, c->dtype, s);
    if (e != hipSuccess) return MOE_ERR_HIP;
    moe::GemmArgs g{};
    g.A = x; g.a_group_stride = 0; g.lda = c->H;
    g.a_row_index = nullptr; g.a_index_stride = 0; g.a_rows_total = c->T;
    g.B = wgt; g.b_group_stride = 0; g.ldb = c->H;
    g.C = logits; g.c_group_stride = 0; g.ldc = c->E;
    g.bias = gate_bias; g.bias_group_stride = 0;
    g.rows_dev = nullptr; g.rows_fixed = c->T; g.rows_cap = c->T;
    g.groups = 1; g.max_rows = c->T;
    g.N = c->E; g.K = c->H;
    g.act = MOE_ACT_IDENTITY; g.dtype = c->dtype; g.b_is_nk = true; g.c_f32 = true; g.fp32_mfma = true;
    e = moe::launch_grouped_gemm(g, s);
    if (e != hipSuccess) return MOE_ERR_HIP;
    return hip_status(moe::launch_topk(logits, c->T, c->E, c->k, topk_expert, topk_weight, s));
}

// counts: scratch of route_chunks(T) * E ints; units: the FFN kernels' scratch block to fill, or nullptr
moe_status run_dispatch(const moe_config* c, const Plan& p, int32_t* counts, int32_t* units, const void* x,
                        const int32_t* topk_expert, const float* topk_weight, int32_t* slot,
                        int32_t* expert_demand, int32_t* slot_token, float* slot_weight, void* xe,
                        bool counts_ready, hipStream_t s) {
    // the fused gate counts per chunk of 64 tokens, which is a chunk of the pair order only under token-major priority
    const bool choice_major = c->drop_policy == MOE_DROP_CHOICE_MAJOR;
    hipError_t e = moe::launch_route(topk_expert, topk_weight, c->T, c->E, c->k, p.C, choice_major,
                                     counts, counts_ready && !choice_major, slot, expert_demand,
                                     slot_token, slot_weight, units, c->dtype == MOE_F32, s);
    if (e != hipSuccess) return MOE_ERR_HIP;
    if (!xe) return MOE_OK;
    return hip_status(moe::launch_pack(x, topk_expert, slot, c->T, c->H, c->k, c->E, p.C, p.C_pad, c->dtype, xe, s));
}

// The two GEMMs of the expert FFN as grouped-GEMM arguments.
// xe: packed rows [E, C_pad, H]; or, with slot_token given, the token matrix x[T, H] whose rows the
// first GEMM gathers through slot_token[E, C] (no packed copy).
void ffn_gemms(const moe_config* c, const Plan& p, void* ws, const void* xe, const int32_t* slot_token,
               const int32_t* expert_demand, const void* W1, const void* b1, const void* W2, const void* b2, void* y,
               moe::GemmArgs* g1_out, moe::GemmArgs* g2_out) {
    void* h = ws_at(ws, p.off_h);
    const long long H = c->H, I = c->I;
    moe::GemmArgs g{};
    g.rows_dev = expert_demand; g.rows_fixed = 0; g.rows_cap = p.C;
    g.groups = c->E; g.max_rows = p.C; g.rows_likely = (long long)c->T * c->k;
    g.dtype = c->dtype; g.b_is_nk = false; g.c_f32 = false;
    // both tasks walk the same live (expert, row tile) units
    g.units = (int32_t*)ws_at(ws, p.off_units);
    if (c->dtype == MOE_F32) g.partials = (float*)ws_at(ws, p.off_partials);
    // task t1: h = phi1(xe W1 + b1)
    moe::GemmArgs g1 = g;
    g1.A = xe; g1.a_group_stride = (long long)p.C_pad * H; g1.lda = c->H;
    g1.a_row_index = slot_token; g1.a_index_stride = p.C;
    g1.a_rows_total = slot_token ? c->T : p.C_pad;
    g1.B = W1; g1.b_group_stride = H * I; g1.ldb = c->I;
    g1.C = h; g1.c_group_stride = (long long)p.C_pad * p.ldh; g1.ldc = p.ldh;
    g1.bias = b1; g1.bias_group_stride = I;
    g1.N = c->I; g1.K = c->H; g1.act = c->act;
    // task t2: y = h W2 + b2
    moe::GemmArgs g2 = g;
    g2.A = h; g2.a_group_stride = (long long)p.C_pad * p.ldh; g2.lda = p.ldh;
    g2.a_row_index = nullptr; g2.a_index_stride = 0;
    g2.a_rows_total = p.C_pad;
    g2.B = W2; g2.b_group_stride = I * H; g2.ldb = c->H;
    g2.C = y; g2.c_group_stride = (long long)p.C_pad * H; g2.ldc = c->H;
    g2.bias = b2; g2.bias_group_stride = H;
    g2.N = c->H; g2.K = c->I; g2.act = MOE_ACT_IDENTITY;
    *g1_out = g1;
    *g2_out = g2;
}

moe_status run_ffn(const moe_config* c, const Plan& p, void* ws, const void* xe, const int32_t* slot_token,
                   const int32_t* expert_demand, const void* W1, const void* b1, const void* W2,
                   const void* b2, void* y, bool units_ready, hipEvent_t between, hipStream_t s) {
    moe::GemmArgs g1, g2;
    ffn_gemms(c, p, ws, xe, slot_token, expert_demand, W1, b1, W2, b2, y, &g1, &g2);
    hipError_t e = hipSuccess;
    if (!units_ready) {
        e = c->dtype == MOE_F32 ? moe::launch_f32_units(expert_demand, p.C, c->E, p.C, g1.units, s)
                                : moe::launch_ffn_units(expert_demand, p.C, c->E, p.C, g1.units, s);
        if (e != hipSuccess) return MOE_ERR_HIP;
    }
    // Optional: one persistent launch for both tasks, a t2 tile starting when the t1 tiles it reads are stored
    // (the tile-level dependency of the paper's processors, Alg. 2).  No faster than two launches on one
    // MI355X at the paper's shapes, so it is opt-in (MOE_FLAG_FFN_SINGLE_LAUNCH; shapes checked by the caller).
    if (c->flags & MOE_FLAG_FFN_SINGLE_LAUNCH) {
        if (!moe::ffn_fused_eligible(g1, g2)) return MOE_ERR_UNSUPPORTED;
        e = moe::launch_ffn_stream_fused(g1, g2, (c->flags & MOE_FLAG_DEBUG_DEPENDENCY_NEVER_MET) != 0, s);
        if (e == hipSuccess && between) e = hipEventRecord(between, s);
        return hip_status(e);
    }
    e = moe::launch_grouped_gemm(g1, s);
    if (e != hipSuccess) return MOE_ERR_HIP;
    if (between && hipEventRecord(between, s) != hipSuccess) return MOE_ERR_HIP;
    return hip_status(moe::launch_grouped_gemm(g2, s));
}

moe_status run_combine(const moe_config* c, const Plan& p, const void* y, const int32_t* topk_expert,
                       const float* topk_weight, const int32_t* slot, void* out, hipStream_t s) {
    return hip_status(moe::launch_combine(y, topk_expert, topk_weight, slot, c->T, c->H, c->k, c->E, p.C,
                                          p.C_pad, c->dtype, out, s));
}

bool bad_required(std::initializer_list<const void*> ptrs) {
    for (const void* q : ptrs)
        if (!q || misaligned(q)) return true;
    return false;
}
bool bad_optional(std::initializer_list<const void*> ptrs) {
    for (const void* q : ptrs)
        if (q && misaligned(q)) return true;
    return false;
}

// The whole layer on one stream.  `ev` (optional, MOE_FORWARD_EVENTS events) are recorded on the stream at the
// stage boundaries: before the gate, after the gate, after the routing launches, after the first FFN launch,
// after the second (the same point as the first under the single-launch flag), after the combine.
moe_status forward_impl(const moe_config* cfg, void* workspace, size_t workspace_bytes, const void* x,
                        const void* Wg, const float* gate_bias, const void* W1, const void* b1,
                        const void* W2, const void* b2, void* out, float* gate_logits,
                        int32_t* topk_expert, float* topk_weight, int32_t* slot, int32_t* expert_demand,
                        const hipEvent_t* ev, hipStream_t s) {
    Plan p;
    moe_status st = make_plan(cfg, &p);
    if (st != MOE_OK) return st;
    if (bad_required({workspace, x, Wg, W1, W2, out, topk_expert, topk_weight, slot, expert_demand}) ||
        bad_optional({gate_bias, b1, b2, gate_logits}))
        return MOE_ERR_INVALID_ARG;
    if (workspace_bytes < p.total) return MOE_ERR_WORKSPACE_TOO_SMALL;
    st = check_single_launch(cfg, p, true);
    if (st != MOE_OK) return st;
    const bool one_launch = (cfg->flags & MOE_FLAG_LAYER_SINGLE_LAUNCH) != 0;
    if (one_launch && (cfg->drop_policy != MOE_DROP_TOKEN_MAJOR ||
                       !moe::layer_fused_eligible(cfg->T, cfg->H, cfg->I, p.ldh, cfg->E, cfg->k, p.C_pad, cfg->dtype)))
        return MOE_ERR_UNSUPPORTED;
    auto mark = [&](int i) { return !ev || hipEventRecord(ev[i], s) == hipSuccess; };
    float* logits = gate_logits ? gate_logits : (float*)ws_at(workspace, p.off_logits);
    int32_t* slot_token = (int32_t*)ws_at(workspace, p.off_slot_token);
    float* slot_weight = (float*)ws_at(workspace, p.off_slot_weight);
    void* y = ws_at(workspace, p.off_y);
    bool counts_ready = false;
    if (!mark(0)) return MOE_ERR_HIP;
    if (one_launch) {
        // Alg. 1 as one persistent kernel: the same stages from one launch, device-wide barriers in between
        moe::GemmArgs g1, g2;
        ffn_gemms(cfg, p, workspace, x, slot_token, expert_demand, W1, b1, W2, b2, y, &g1, &g2);
        if (moe::launch_layer_fused(x, Wg, gate_bias, cfg->T, cfg->H, cfg->E, cfg->k, p.C, p.C_pad, cfg->dtype, gate_slices(cfg, p), logits, topk_expert,
                                    topk_weight, (int32_t*)ws_at(workspace, p.off_counts), slot, expert_demand, slot_token,
                                    slot_weight, g1, g2, out, s) != hipSuccess)
            return MOE_ERR_HIP;
        for (int i = 1; i < MOE_FORWARD_EVENTS; ++i)
            if (!mark(i)) return MOE_ERR_HIP;
        return MOE_OK;
    }
    st = run_gate(cfg, p, workspace, x, Wg, gate_bias, logits, topk_expert, topk_weight, &counts_ready, s);
    if (st != MOE_OK) return st;
    if (!mark(1)) return MOE_ERR_HIP;
    // Dispatch builds the routing table only; the first FFN GEMM gathers its rows from x through
    // slot_token, so the packed copy xe is never materialised on this path.
    // the routing launch also lists the live FFN units
    st = run_dispatch(cfg, p, (int32_t*)ws_at(workspace, p.off_counts), (int32_t*)ws_at(workspace, p.off_units), x, topk_expert,
                      topk_weight, slot, expert_demand, slot_token, slot_weight, nullptr, counts_ready, s);
    if (st != MOE_OK) return st;
    if (!mark(2)) return MOE_ERR_HIP;
    st = run_ffn(cfg, p, workspace, x, slot_token, expert_demand, W1, b1, W2, b2, y, true, ev ? ev[3] : nullptr, s);
    if (st != MOE_OK) return st;
    if (!mark(4)) return MOE_ERR_HIP;
    st = run_combine(cfg, p, y, topk_expert, topk_weight, slot, out, s);
    if (st != MOE_OK) return st;
    return mark(5) ? MOE_OK : MOE_ERR_HIP;
}

// fp32 weight gradients after ReLU: sums over more slots than this are made in spans of it.  The split products round an
// accumulator 6 times per 32 slots whether or not half of the activations are zero, where fp32 products leave zeros out.
// Relative error of dW2 at 2048 / 4096 / 16384 slots (H = I = 512): 7.4e-7 / 9.9e-7 / 1.9e-6 in one sum, 5.8e-7 / 5.8e-7 /
// 6.0e-7 in spans, 7.0e-7 / 9.0e-7 / 1.7e-6 on the fp32 instruction (spans of 2048: 7.4e-7 from 2048 slots on).  The spans cost 3 to
// 11 % of the backward call (4.17 -> 4.65 ms at T = 8192, H = I = 2048, E = 4, top-2; fp32 instruction: 7.09), so the other
// activations, whose sums are as accurate as fp32 products' at every length (0.84 to 0.86 of their error), stay as they are.
constexpr int kReluGradSpan = 1024;

// ---- backward pass: workspace carving and launch order -------------------------------------------------------
struct BwdPlan {
    Plan p;
    int ldL, T_pad;
    int wg_slices, wg_slice_k;                           // dWg = x^T dL as wg_slices partial products over wg_slice_k tokens each
    size_t off_wg_part;
    size_t off_counts, off_units, off_slot_token, off_slot_weight, off_slot, off_demand, off_dl, off_dL, off_wgt, off_xe,
        off_ge, off_a, off_h, off_dh, off_da, off_dxe, off_row_p, off_sums, off_xT, off_wrows, off_wunits1, off_wunits2, total;
    bool w_stream;                                       // 16-bit storage: dW1 and dW2 on the weight-streaming kernel
    int row_step;                                        // the experts' rows are zero from the last live one to the next multiple of this
    int w_slices;                                        // 16-bit storage: slices of the weight gradients' sums over an expert's slots
};
constexpr long long kWgradWorkgroups = 512;              // two per CU

// The products over the experts' live rows
moe::GemmArgs bwd_gemm_args(const moe_config* c, const Plan& p, const int32_t* demand, int32_t* units) {
    moe::GemmArgs g{};
    g.rows_dev = demand; g.rows_fixed = 0; g.rows_cap = p.C; g.groups = c->E; g.max_rows = p.C; g.rows_likely = (long long)c->T * c->k;
    g.dtype = c->dtype; g.act = MOE_ACT_IDENTITY; g.a_rows_total = p.C_pad; g.units = units;
    return g;
}

// dh = ge W2^T in fp32 (of_h; W2[e] read as [N = I][K = H]) or dxe = da W1^T (W1[e] as [N = H][K = I])
moe::GemmArgs data_gradient_args(const moe_config* c, const Plan& p, const int32_t* demand, int32_t* units, const void* grad, const void* W,
                                 void* out, bool of_h) {
    const int K = of_h ? c->H : c->I, N = of_h ? c->I : c->H;
    moe::GemmArgs g = bwd_gemm_args(c, p, demand, units);
    g.A = grad; g.a_group_stride = (long long)p.C_pad * K; g.lda = K;
    g.B = W; g.b_group_stride = (long long)c->H * c->I; g.ldb = K; g.b_is_nk = true;
    g.C = out; g.c_group_stride = (long long)p.C_pad * N; g.ldc = N; g.N = N; g.K = K; g.c_f32 = of_h;
    return g;
}

// An expert's dW1 or dW2 as a GEMM of the weight-streaming kernel (its rows: `M` columns of h or xe, all C_pad slots as K)
moe::GemmArgs stream_wgrad_args(const moe_config* c, const Plan& p, const void* rows, int M, const void* grad, int N, float* out,
                                const int32_t* counts_dev, int32_t* units) {
    moe::GemmArgs w{};
    w.groups = c->E; w.dtype = c->dtype; w.act = MOE_ACT_IDENTITY; w.c_f32 = true; w.K = p.C_pad;
    w.A = rows; w.a_is_km = true; w.lda = M; w.a_group_stride = (long long)p.C_pad * M; w.a_rows_total = p.C_pad;
    w.rows_dev = counts_dev; w.units = units; w.rows_fixed = M; w.rows_cap = M; w.max_rows = M;
    w.B = grad; w.b_group_stride = (long long)p.C_pad * N; w.ldb = N;
    w.C = out; w.c_group_stride = (long long)c->H * c->I; w.ldc = N; w.N = N;
    return w;
}

// dW1 and dW2 in 16-bit storage on the weight-streaming kernel, or all weight gradients in one launch of wgrad.hip, whose sums stop
// at an expert's last live slot and which cuts tiles finer?  Both products, us, streaming / wgrad, H = I = 2048 (full slots): E = 128
// of 256 slots 1200 / 1351; E = 64 of 512 799 / 876; E = 16 of 2048 569 / 588; E = 8 of 4096 (two rounds of 256 x 256 tiles) 520 /
// 551.  E = 8 of 556, I = 768 (192 tiles): 69 / 49.  Slots a third empty, as at a capacity factor of 1.25: E = 128 of 384 1360 / 1290; E
// = 16, H = 1024, I = 4096 209 / 136.
bool wgrad_streams(const moe_config* c, const Plan& p) {
    if (c->dtype == MOE_F32) return false;
    int32_t some = 0;                                    // eligibility asks whether the lists are there, not what they hold
    if (!moe::stream_gemm_eligible(stream_wgrad_args(c, p, nullptr, c->I, nullptr, c->H, nullptr, &some, &some)) ||
        !moe::stream_gemm_eligible(stream_wgrad_args(c, p, nullptr, c->H, nullptr, c->I, nullptr, &some, &some)))
        return false;
    const long long tiles = (long long)c->E * ((c->H + 255) / 256) * ((c->I + 255) / 256);
    return tiles >= 512 && (long long)c->E * p.C_pad * 10 <= (long long)c->T * c->k * 12;
}

moe_status make_bwd_plan(const moe_config* c, BwdPlan* b) {
    moe_status st = make_plan(c, &b->p);
    if (st != MOE_OK) return st;
    if (c->k > 64) return MOE_ERR_UNSUPPORTED;          // the gate's Jacobian kernel keeps a token's choices in one wavefront
    if (c->flags != 0) return MOE_ERR_UNSUPPORTED;
    const Plan& p = b->p;
    const size_t T = c->T, H = c->H, I = c->I, E = c->E, k = c->k, el = p.elem;
    const size_t rows = E * (size_t)p.C_pad;
    b->ldL = (int)align_up(E, 8);
    // dWg has only (H / 128) x (E / 128) output tiles for a contraction over all T tokens: the tokens are cut into up to
    // 16 slices, each slice one "group" of the grouped GEMM, and the partial products added in slice order.  Slices of at least 1024 have
    // room of their own; those of fewer tokens see below
    b->wg_slices = (int)(T / 1024 < 1 ? 1 : (T / 1024 > 16 ? 16 : T / 1024));
    b->wg_slice_k = (int)align_up((T + b->wg_slices - 1) / b->wg_slices, 64);
    b->T_pad = b->wg_slices * b->wg_slice_k;             // >= T: x^T rows and dL are zero beyond T
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, kAlign); return o; };
    b->off_counts = take((size_t)moe::route_chunks(c->T) * E * 4);
    b->off_units = take(moe::ffn_units_ints(c->E, p.C) * 4);
    b->off_slot_token = take(E * (size_t)p.C * 4);
    b->off_slot_weight = take(E * (size_t)p.C * 4);
    b->off_slot = take(T * k * 4);
    b->off_demand = take(E * 4);
    b->off_dl = take(T * k * 4);
    b->off_dL = take((size_t)b->T_pad * b->ldL * el);
    b->off_wg_part = take(b->wg_slices > 1 ? (size_t)b->wg_slices * H * E * 4 : 0);
    b->off_wgt = take((size_t)p.E_pad * H * el);
    b->off_xe = take(rows * H * el);
    b->off_ge = take(rows * H * el);
    b->off_a = b->off_h = take(rows * I * el);           // the activation kernel writes h where it reads a
    b->off_row_p = take(rows * 4);
    const size_t h_bytes = align_up(rows * I * el, kAlign), x_bytes = align_up(rows * H * el, kAlign);
    // dxe, and behind it h^T and xe^T (fp32) or partial sums.  In 16-bit storage dh lies there before, which is read for the last time
    // when dxe begins, and the partial sums may take what makes this four buffers of H and four of I values per slot row with xe,
    // ge, h and da (more where dh needs more)
    const size_t most = c->dtype == MOE_F32 ? 2 * x_bytes + h_bytes : std::max(rows * I * 4, 2 * x_bytes + h_bytes);
    if (c->dtype == MOE_F32) {
        b->off_dh = b->off_da = take(rows * I * 4);      // and da in the place of dh, in fp32
        b->off_xT = take(H * (size_t)b->T_pad * el);
    } else {
        b->off_da = take(rows * I * el);
    }
    b->off_dxe = off;
    if (c->dtype != MOE_F32) b->off_dh = b->off_dxe;
    b->off_sums = b->off_dxe + x_bytes;
    b->w_slices = 1;
    b->w_stream = wgrad_streams(c, p);
    b->row_step = b->w_stream ? p.C_pad : 32;
    if (c->dtype != MOE_F32 && !b->w_stream) {
        // dW1 and dW2 have few output tiles where there are few experts or narrow layers: then an expert's slots are cut into
        // slices of at least 256, as many as give two workgroups per CU and as the partial sums have room for behind dxe
        const long long tiles = moe::wgrad_tiles(c->E, c->I, c->H) + moe::wgrad_tiles(c->E, c->H, c->I);
        const long long room = (long long)((align_up(most, kAlign) - x_bytes) / (2 * E * H * I * 4));
        b->w_slices = (int)std::max(1ll, std::min({kWgradWorkgroups / tiles, (long long)p.C_pad / 256, room}));
    }
    // Slices of at least 256 tokens, as many as make no more rows of x^T and dL and as the partial products have room for behind dxe
    // and the partial sums of dW1 and dW2 there: those of 1024 were 16 tiles each for 256 CUs in fp32 (T = 2048, H = 1024, E = 16:
    // 35.2 us, 13.8 in eight slices of 256), and in 16-bit storage the longest sums of the launch in small layers (whole call, T = 1024, H
    // = I = 256, E = 4 73.6 -> 60.9 us; T = 2048, H = 512, I = 1024, E = 8 126 -> 114; T = 8192, H = I = 2048, E = 32 1010 -> 1002).
    const size_t w_sums = b->w_slices > 1 ? 2 * (size_t)b->w_slices * E * H * I * 4 : 0;
    size_t live = c->dtype == MOE_F32 ? most : std::max(rows * I * 4, x_bytes + w_sums);      // bytes from dxe on
    for (int n = (int)std::min<size_t>(16, T / 256); n > b->wg_slices; --n) {
        const size_t slice = align_up((T + n - 1) / n, 64), end = x_bytes + w_sums + (size_t)n * H * E * 4;
        if (n * slice > (size_t)b->T_pad || (n - 1) * slice >= T || end > most) continue;
        b->wg_slices = n;
        b->wg_slice_k = (int)slice;
        b->T_pad = (int)(n * slice);
        b->off_wg_part = b->off_sums + w_sums;
        live = std::max(live, end);
        break;
    }
    take(live);
    if (b->w_stream) {
        b->off_wrows = take(2 * E * 4);
        b->off_wunits1 = take(moe::ffn_units_ints(c->E, c->H) * 4);
        b->off_wunits2 = take(moe::ffn_units_ints(c->E, c->I) * 4);
    }
    b->total = off;
    return MOE_OK;
}

moe_status run_backward(const moe_config* c, const BwdPlan& b, void* ws, const void* x, const void* Wg, const void* W1,
                        const void* b1, const void* W2, const void* b2, const int32_t* topk_expert, const float* topk_weight,
                        const void* dout, float* dx, float* dWg, float* dgate_bias, float* dW1, float* db1, float* dW2,
                        float* db2, hipStream_t s) {
    const Plan& p = b.p;
    const int T = c->T, H = c->H, I = c->I, E = c->E, k = c->k, C = p.C, C_pad = p.C_pad, dt = c->dtype;
    int32_t* counts = (int32_t*)ws_at(ws, b.off_counts);
    int32_t* units = dt != MOE_F32 ? (int32_t*)ws_at(ws, b.off_units) : nullptr;
    int32_t* slot_token = (int32_t*)ws_at(ws, b.off_slot_token);
    float* slot_weight = (float*)ws_at(ws, b.off_slot_weight);
    int32_t* slot = (int32_t*)ws_at(ws, b.off_slot);
    int32_t* demand = (int32_t*)ws_at(ws, b.off_demand);
    float* dl = (float*)ws_at(ws, b.off_dl);
    void *dL = ws_at(ws, b.off_dL), *wgt = ws_at(ws, b.off_wgt), *xe = ws_at(ws, b.off_xe), *ge = ws_at(ws, b.off_ge);
    void *a = ws_at(ws, b.off_a), *h = ws_at(ws, b.off_h), *da = ws_at(ws, b.off_da), *dxe = ws_at(ws, b.off_dxe);
    float *dh = (float*)ws_at(ws, b.off_dh), *row_p = (float*)ws_at(ws, b.off_row_p);
#define MOE_TRY(call) do { if ((call) != hipSuccess) return MOE_ERR_HIP; } while (0)
    // the routing tables again, from the selection the forward pass made (slots are a function of it)
    MOE_TRY(moe::launch_route(topk_expert, topk_weight, T, E, k, C, c->drop_policy == MOE_DROP_CHOICE_MAJOR, counts, false, slot,
                              demand, slot_token, slot_weight, units, false, s));
    MOE_TRY(moe::launch_bwd_gather(x, dout, slot_token, slot_weight, demand, H, E, C, C_pad, b.row_step, dt, xe, ge, Wg, wgt, s));
    // grouped GEMMs over the experts' live rows
    const long long rH = (long long)C_pad * H, rI = (long long)C_pad * I, HI = (long long)H * I;
    // the pre-activation again: a = xe W1 + b1
    moe::GemmArgs f1 = bwd_gemm_args(c, p, demand, units);
    f1.A = xe; f1.a_group_stride = rH; f1.lda = H; f1.B = W1; f1.b_group_stride = HI; f1.ldb = I;
    f1.C = a; f1.c_group_stride = rI; f1.ldc = I; f1.bias = b1; f1.bias_group_stride = I; f1.N = I; f1.K = H;
    MOE_TRY(moe::launch_grouped_gemm(f1, s));
    // dh = dout W2^T in fp32 (W2[e] read as [N = I][K = H]); h = w phi(a), da = w dh phi'(a); dxe = da W1^T (W1[e] as [N = H][K = I])
    MOE_TRY(moe::launch_grouped_gemm(data_gradient_args(c, p, demand, units, ge, W2, dh, true), s));
    MOE_TRY(moe::launch_bwd_act(a, dh, ge, b2, demand, slot_weight, E, C, C_pad, b.row_step, H, I, c->act, dt, h, da, row_p, s));
    // gate: w dL/dw of every kept pair is in row_p; the softmax Jacobian
    MOE_TRY(moe::launch_bwd_gate(row_p, topk_expert, topk_weight, slot, T, b.T_pad, k, E, C, C_pad, b.ldL, dt, dl, dL, s));
    MOE_TRY(moe::launch_grouped_gemm(data_gradient_args(c, p, demand, units, da, W1, dxe, false), s));
    // weight gradients: dW2[e] = h[e]^T ge[e], dW1[e] = xe[e]^T da[e] over the expert's slots, dWg = x^T dL over the tokens
    float* const wg_out = b.wg_slices > 1 ? (float*)ws_at(ws, b.off_wg_part) : dWg;
    moe::BwdFinish finish{};
    if (dt != MOE_F32) {
        float *dW1_out = dW1, *dW2_out = dW2;
        if (b.w_slices > 1) {
            dW1_out = (float*)ws_at(ws, b.off_sums);
            dW2_out = dW1_out + (size_t)b.w_slices * E * HI;
            finish.sum[0] = {dW1_out, b.w_slices, E * HI, dW1};
            finish.sum[1] = {dW2_out, b.w_slices, E * HI, dW2};
        }
        if (b.w_stream) {
            int32_t* wrows = (int32_t*)ws_at(ws, b.off_wrows);
            int32_t *wunits1 = (int32_t*)ws_at(ws, b.off_wunits1), *wunits2 = (int32_t*)ws_at(ws, b.off_wunits2);
            MOE_TRY(moe::launch_bwd_fill_rows(wrows, E, H, I, s));
            MOE_TRY(moe::launch_ffn_units(wrows, H, E, H, wunits1, s));
            MOE_TRY(moe::launch_ffn_units(wrows + E, I, E, I, wunits2, s));
            MOE_TRY(moe::launch_grouped_gemm(stream_wgrad_args(c, p, h, I, ge, H, dW2, wrows + E, wunits2), s));
            MOE_TRY(moe::launch_grouped_gemm(stream_wgrad_args(c, p, xe, H, da, I, dW1, wrows, wunits1), s));
        }
        const int experts = b.w_stream ? 0 : E;
        const moe::WgradProblem w[moe::kWgradProblems] = {
            {h, rI, I, C_pad, ge, rH, H, dW2_out, HI, H, demand, C, I, H, experts, b.w_slices},
            {xe, rH, H, C_pad, da, rI, I, dW1_out, HI, I, demand, C, H, I, experts, b.w_slices},
            {x, 0, H, T, dL, 0, b.ldL, wg_out, (long long)H * E, E, nullptr, T, H, E, 1, b.wg_slices}};
        MOE_TRY(moe::launch_wgrad(w, dt, s));
    } else {
        auto weight_grad = [&](const void* rows, int M, void* rowsT, const void* grad, int N, float* out) {
            if (hipError_t e = moe::launch_bwd_transpose((const float*)rows, (float*)rowsT, E, C_pad, M, C_pad, demand, C, s); e != hipSuccess) return e;
            moe::GemmArgs w{};
            w.groups = E; w.dtype = dt; w.act = MOE_ACT_IDENTITY; w.c_f32 = true; w.K = C_pad; w.k_dev = demand; w.k_cap = C;
            w.A = rowsT; w.lda = C_pad; w.a_group_stride = (long long)C_pad * M; w.a_rows_total = M;
            w.rows_fixed = M; w.rows_cap = M; w.max_rows = M;
            w.B = grad; w.b_group_stride = (long long)C_pad * N; w.ldb = N;
            w.C = out; w.c_group_stride = HI; w.ldc = N; w.N = N; w.k_span = c->act == MOE_ACT_RELU ? kReluGradSpan : 0;
            return moe::launch_grouped_gemm(w, s);
        };
        void *xeT = ws_at(ws, b.off_sums), *xT = ws_at(ws, b.off_xT);
        void* hT = (char*)xeT + align_up((size_t)E * rH * 4, kAlign);
        MOE_TRY(weight_grad(h, I, hT, ge, H, dW2));
        MOE_TRY(weight_grad(xe, H, xeT, da, I, dW1));
        MOE_TRY(moe::launch_bwd_transpose((const float*)x, (float*)xT, 1, T, H, b.T_pad, nullptr, 0, s));
        moe::GemmArgs wg{};
        wg.groups = b.wg_slices; wg.dtype = dt; wg.act = MOE_ACT_IDENTITY; wg.c_f32 = true;
        wg.A = xT; wg.lda = b.T_pad; wg.a_rows_total = H; wg.rows_fixed = H; wg.rows_cap = H; wg.max_rows = H;
        wg.a_group_stride = b.wg_slice_k;                // slice g of every row of x^T
        wg.B = dL; wg.ldb = b.ldL; wg.b_group_stride = (long long)b.wg_slice_k * b.ldL;
        wg.C = wg_out; wg.ldc = E; wg.c_group_stride = (long long)H * E; wg.N = E; wg.K = b.wg_slice_k;   // rows of both beyond T are zero
        MOE_TRY(moe::launch_grouped_gemm(wg, s));
    }
    // dWg from its slices, the bias gradients, and dx: the kept choices' rows of dxe plus the gate path
    finish.sum[2] = {wg_out, b.wg_slices, (long long)H * E, dWg};
    finish.topk_expert = topk_expert; finish.slot = slot; finish.expert_demand = demand; finish.dl = dl; finish.slot_weight = slot_weight;
    finish.dxe = dxe; finish.WgT = wgt; finish.ge = ge; finish.da = da;
    finish.dx = dx; finish.dgate_bias = dgate_bias; finish.db1 = db1; finish.db2 = db2;
    finish.T = T; finish.H = H; finish.I = I; finish.k = k; finish.E = E; finish.C = C; finish.C_pad = C_pad;
    MOE_TRY(moe::launch_bwd_finish(finish, dt, s));
#undef MOE_TRY
    return MOE_OK;
}

}  // namespace

extern "C" {

const char* moe_status_string(moe_status s) {
    switch (s) {
        case MOE_OK: return "ok";
        case MOE_ERR_INVALID_ARG: return "invalid argument";
        case MOE_ERR_UNSUPPORTED: return "unsupported configuration";
        case MOE_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
        case MOE_ERR_HIP: return "HIP launch error";
        case MOE_ERR_FFN_DEPENDENCY_TIMEOUT: return "single-launch FFN: a wait for first-task tiles gave up (results invalid)";
        case MOE_ERR_FFN_PLACEMENT: return "single-launch FFN: workgroups of one class ran on different XCDs (results may be stale)";
        case MOE_ERR_STATIC_SCRATCH_TOO_SMALL: return "configuration needs more than the fixed scratch of the no-allocation entry point";
    }
    return "unknown status";
}

int32_t moe_row_tile(void) { return kRowTile; }

moe_status moe_init(void) {
    hipError_t e = moe::prepare_gate_fused();
    if (e == hipSuccess) e = moe::prepare_grouped_gemm();
    if (e == hipSuccess) e = moe::prepare_grouped_gemm_stream();
    if (e == hipSuccess) e = moe::prepare_gemm_narrow();
    if (e == hipSuccess) e = moe::prepare_layer_fused();
    if (e == hipSuccess) e = moe::prepare_gemm_f32();
    if (e == hipSuccess) e = moe::prepare_wgrad();
    void* scratch_here = nullptr;
    if (e == hipSuccess) e = static_scratch(&scratch_here);
    if (e != hipSuccess) return MOE_ERR_HIP;
    (void)moe::device_cu_count();
    return MOE_OK;
}

int32_t moe_ffn_schedule(int32_t large_list, int32_t n_units_large, int32_t n_units_small, int32_t nrow_large,
                         int32_t ncol, int32_t xcd, int32_t wg, int32_t wgs, int32_t* list_index, int32_t* col_tile,
                         int32_t max_tasks) {
    if (n_units_large < 0 || n_units_small < 0 || nrow_large < 0 || ncol <= 0 || xcd < 0 || xcd >= moe::kXcds ||
        wgs <= 0 || wg < 0 || wg >= wgs || max_tasks < 0 || (max_tasks > 0 && (!list_index || !col_tile)))
        return -1;
    int unit0, unit_step, ux_l, ux;
    moe::ffn_xcd_share(true, n_units_large, nrow_large, xcd, unit0, unit_step, ux_l);
    int w = wg, handicap = 0;
    if (large_list) {
        ux = ux_l;
    } else {
        moe::ffn_xcd_share(false, n_units_small, 1, xcd, unit0, unit_step, ux);
        w = moe::ffn_small_list_rotation(wg, wgs, ux_l, ncol);
        handicap = moe::ffn_small_list_handicap(wgs, ux_l, ncol);
    }
    if ((long long)ux * ncol > 0x7fffffffLL - 2ll * wgs) return -1;
    const int n = moe::ffn_slot_count(w, wgs, handicap, ux * ncol);
    const int first = moe::ffn_first_slot(w, wgs, handicap);
    for (int j = 0; j < n && j < max_tasks; ++j)
        moe::ffn_task_at(moe::ffn_slot_position(first + j * wgs, wgs, handicap), ncol, unit0, unit_step, ux, large_list ? nrow_large : 1, list_index[j], col_tile[j]);
    return n;
}

int32_t moe_f32_ffn_schedule(const int32_t* rows, int32_t groups, int32_t capacity, int32_t N, int32_t K, int32_t workgroups,
                             int64_t* first_iteration, int64_t* fix_tile, int32_t* unit_id, int32_t* unit_cum, int32_t max_units) {
    if (!rows || groups <= 0 || capacity <= 0 || N <= 0 || K <= 0 || workgroups <= 0 || !first_iteration || !fix_tile || !unit_id ||
        !unit_cum || (long long)groups * moe::f32_units_nrow(capacity) > max_units)
        return -1;
    const int n = moe::f32_build_units_host(rows, capacity, groups, capacity, unit_id, unit_cum);
    const moe::F32Work k(unit_id, unit_cum, n, (N + moe::kF32TileCols - 1) / moe::kF32TileCols, (K + moe::kF32TileK - 1) / moe::kF32TileK);
    for (int w = 0; w <= workgroups; ++w) first_iteration[w] = k.boundary(w, workgroups);
    for (int w = 0; w < workgroups; ++w) fix_tile[w] = k.tile_to_fix(first_iteration[w], first_iteration[w + 1]);
    return n;
}

int32_t moe_f32_gemm_body(int32_t groups, int32_t max_rows, int32_t N, int32_t K, int32_t listed, int32_t cus) {
    if (groups <= 0 || max_rows <= 0 || N <= 0 || K <= 0 || cus <= 0) return -1;
    if (listed && moe::f32_spans_worth(groups, max_rows, N, K, cus)) return MOE_F32_BODY_SPANS;
    return moe::f32_tile_body(groups, max_rows, N, cus);
}

int32_t moe_gemm16_kernel(const moe_config* cfg, int32_t product, int32_t cus) {
    Plan p;
    if (make_plan(cfg, &p) != MOE_OK || cfg->dtype == MOE_F32 || cus <= 0) return -1;
    int32_t some = 0;                                    // the choice asks whether buffers are there, not what they hold
    switch (product) {
        case MOE_PRODUCT_FFN1:
        case MOE_PRODUCT_FFN2: {
            moe::GemmArgs g[2];
            ffn_gemms(cfg, p, &some, &some, nullptr, &some, &some, nullptr, &some, nullptr, &some, &g[0], &g[1]);
            return moe::gemm16_kernel(g[product], cus);
        }
        case MOE_PRODUCT_DH:
        case MOE_PRODUCT_DXE:
            return moe::gemm16_kernel(data_gradient_args(cfg, p, &some, &some, &some, &some, &some, product == MOE_PRODUCT_DH), cus);
        case MOE_PRODUCT_DW: return wgrad_streams(cfg, p) ? MOE_KERNEL16_STREAM : MOE_KERNEL16_WGRAD;
    }
    return -1;
}

moe_status moe_ffn_status(const moe_config* cfg, const void* workspace, size_t workspace_bytes, void* stream) {
    Plan p;
    moe_status st = make_plan(cfg, &p);
    if (st != MOE_OK) return st;
    if (!workspace || misaligned(workspace)) return MOE_ERR_INVALID_ARG;
    if (workspace_bytes < p.total) return MOE_ERR_WORKSPACE_TOO_SMALL;
    if (cfg->dtype == MOE_F32) return MOE_OK;            // the unit lists (and their fault words) belong to the 16-bit kernels
    long long w0 = 0, w1 = 0;
    moe::ffn_units_fault_words(cfg->E, p.C, &w0, &w1);
    const int32_t* units = (const int32_t*)((const char*)workspace + p.off_units);
    int32_t f0 = 0, f1 = 0;
    hipStream_t s = (hipStream_t)stream;
    if (hipMemcpyAsync(&f0, units + w0, sizeof(int32_t), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipMemcpyAsync(&f1, units + w1, sizeof(int32_t), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return MOE_ERR_HIP;
    const int32_t f = f0 | f1;
    if ((f & 1) && (cfg->flags & MOE_FLAG_LAYER_SINGLE_LAUNCH)) {
        // a device-wide barrier of the single-launch layer may have been left half-way: start the next launch clean
        if (moe::reset_layer_sync(s) != hipSuccess || hipStreamSynchronize(s) != hipSuccess) return MOE_ERR_HIP;
    }
    if (f & 1) return MOE_ERR_FFN_DEPENDENCY_TIMEOUT;
    if (f & 2) return MOE_ERR_FFN_PLACEMENT;
    return MOE_OK;
}

moe_status moe_layer_stage_ms(double* host_ms, int32_t n, void* stream) {
    if (!host_ms || n < 0 || n > MOE_LAYER_STAGES) return MOE_ERR_INVALID_ARG;
    return moe::layer_stage_ms(host_ms, n, (hipStream_t)stream) == hipSuccess ? MOE_OK : MOE_ERR_HIP;
}

moe_status moe_capacity(const moe_config* cfg, int32_t* C, int32_t* C_pad) {
    moe_status st = check_config(cfg);
    if (st != MOE_OK) return st;
    int c = 0, cp = 0;
    st = capacity_of(cfg, &c, &cp);
    if (st != MOE_OK) return st;
    if (C) *C = c;
    if (C_pad) *C_pad = cp;
    return MOE_OK;
}

moe_status moe_workspace_bytes(const moe_config* cfg, size_t* bytes) {
    if (!bytes) return MOE_ERR_INVALID_ARG;
    Plan p;
    moe_status st = make_plan(cfg, &p);
    if (st != MOE_OK) return st;
    *bytes = p.total;
    return MOE_OK;
}

moe_status moe_forward(const moe_config* cfg, void* workspace, size_t workspace_bytes, const void* x,
                       const void* Wg, const float* gate_bias, const void* W1, const void* b1,
                       const void* W2, const void* b2, void* out, float* gate_logits,
                       int32_t* topk_expert, float* topk_weight, int32_t* slot, int32_t* expert_demand,
                       void* stream) {
    return forward_impl(cfg, workspace, workspace_bytes, x, Wg, gate_bias, W1, b1, W2, b2, out, gate_logits, topk_expert,
                        topk_weight, slot, expert_demand, nullptr, (hipStream_t)stream);
}

moe_status moe_forward_timed(const moe_config* cfg, void* workspace, size_t workspace_bytes, const void* x,
                             const void* Wg, const float* gate_bias, const void* W1, const void* b1,
                             const void* W2, const void* b2, void* out, float* gate_logits,
                             int32_t* topk_expert, float* topk_weight, int32_t* slot, int32_t* expert_demand,
                             void* const* events, void* stream) {
    if (!events) return MOE_ERR_INVALID_ARG;
    for (int i = 0; i < MOE_FORWARD_EVENTS; ++i)
        if (!events[i]) return MOE_ERR_INVALID_ARG;
    return forward_impl(cfg, workspace, workspace_bytes, x, Wg, gate_bias, W1, b1, W2, b2, out, gate_logits, topk_expert,
                        topk_weight, slot, expert_demand, (const hipEvent_t*)events, (hipStream_t)stream);
}

moe_status moe_gate(const moe_config* cfg, void* workspace, size_t workspace_bytes, const void* x,
                    const void* Wg, const float* gate_bias, float* gate_logits, int32_t* topk_expert,
                    float* topk_weight, void* stream) {
    Plan p;
    moe_status st = make_plan(cfg, &p);
    if (st != MOE_OK) return st;
    if (bad_required({workspace, x, Wg, gate_logits, topk_expert, topk_weight}) || bad_optional({gate_bias}))
        return MOE_ERR_INVALID_ARG;
    if (workspace_bytes < p.total) return MOE_ERR_WORKSPACE_TOO_SMALL;
    return run_gate(cfg, p, workspace, x, Wg, gate_bias, gate_logits, topk_expert, topk_weight, nullptr, (hipStream_t)stream);
}

moe_status moe_route(const moe_config* cfg, const float* gate_logits, int32_t* topk_expert,
                     float* topk_weight, void* stream) {
    moe_status st = check_config(cfg);
    if (st != MOE_OK) return st;
    if (bad_required({gate_logits, topk_expert, topk_weight})) return MOE_ERR_INVALID_ARG;
    return hip_status(moe::launch_topk(gate_logits, cfg->T, cfg->E, cfg->k, topk_expert, topk_weight, (hipStream_t)stream));
}

moe_status moe_dispatch(const moe_config* cfg, void* workspace, size_t workspace_bytes, const void* x,
                        const int32_t* topk_expert, const float* topk_weight, int32_t* slot,
                        int32_t* expert_demand, int32_t* slot_token, float* slot_weight, void* xe,
                        void* stream) {
    Plan p;
    moe_status st = make_plan(cfg, &p);
    if (st != MOE_OK) return st;
    if (bad_required({workspace, topk_expert, topk_weight, slot, expert_demand, slot_token, slot_weight}) ||
        bad_optional({x, xe}) || (xe && !x))
        return MOE_ERR_INVALID_ARG;
    if (workspace_bytes < p.total) return MOE_ERR_WORKSPACE_TOO_SMALL;
    return run_dispatch(cfg, p, (int32_t*)ws_at(workspace, p.off_counts), nullptr, x, topk_expert, topk_weight, slot,
                        expert_demand, slot_token, slot_weight, xe, false, (hipStream_t)stream);
}

moe_status moe_dispatch_noalloc(const moe_config* cfg, const void* x, const int32_t* topk_expert,
                                const float* topk_weight, int32_t* slot, int32_t* expert_demand, int32_t* slot_token,
                                float* slot_weight, void* xe, void* stream) {
    Plan p;
    moe_status st = make_plan(cfg, &p);
    if (st != MOE_OK) return st;
    if (bad_required({topk_expert, topk_weight, slot, expert_demand, slot_token, slot_weight}) || bad_optional({x, xe}) ||
        (xe && !x))
        return MOE_ERR_INVALID_ARG;
    // the only scratch of the routing kernels: per-chunk expert counts (every entry is written before it is read,
    // so nothing of an earlier call has to be cleared)
    const size_t need = (size_t)moe::route_chunks(cfg->T) * (size_t)cfg->E * sizeof(int32_t);
    if (need > kStaticScratchBytes) return MOE_ERR_STATIC_SCRATCH_TOO_SMALL;
    void* counts = nullptr;
    if (static_scratch(&counts) != hipSuccess) return MOE_ERR_HIP;
    return run_dispatch(cfg, p, (int32_t*)counts, nullptr, x, topk_expert, topk_weight, slot, expert_demand, slot_token,
                        slot_weight, xe, false, (hipStream_t)stream);
}

moe_status moe_expert_ffn(const moe_config* cfg, void* workspace, size_t workspace_bytes, const void* xe,
                          const int32_t* expert_demand, const void* W1, const void* b1, const void* W2,
                          const void* b2, void* y, void* stream) {
    Plan p;
    moe_status st = make_plan(cfg, &p);
    if (st != MOE_OK) return st;
    if (bad_required({workspace, xe, expert_demand, W1, W2, y}) || bad_optional({b1, b2})) return MOE_ERR_INVALID_ARG;
    if (workspace_bytes < p.total) return MOE_ERR_WORKSPACE_TOO_SMALL;
    st = check_single_launch(cfg, p, false);
    if (st != MOE_OK) return st;
    return run_ffn(cfg, p, workspace, xe, nullptr, expert_demand, W1, b1, W2, b2, y, false, nullptr, (hipStream_t)stream);
}

moe_status moe_backward_workspace_bytes(const moe_config* cfg, size_t* bytes) {
    if (!bytes) return MOE_ERR_INVALID_ARG;
    BwdPlan b;
    moe_status st = make_bwd_plan(cfg, &b);
    if (st != MOE_OK) return st;
    *bytes = b.total;
    return MOE_OK;
}

moe_status moe_backward(const moe_config* cfg, void* workspace, size_t workspace_bytes, const void* x, const void* Wg,
                        const void* W1, const void* b1, const void* W2, const void* b2, const int32_t* topk_expert,
                        const float* topk_weight, const void* dout, float* dx, float* dWg, float* dgate_bias, float* dW1,
                        float* db1, float* dW2, float* db2, void* stream) {
    BwdPlan b;
    moe_status st = make_bwd_plan(cfg, &b);
    if (st != MOE_OK) return st;
    if (bad_required({workspace, x, Wg, W1, W2, topk_expert, topk_weight, dout, dx, dWg, dgate_bias, dW1, db1, dW2, db2}) ||
        bad_optional({b1, b2}))
        return MOE_ERR_INVALID_ARG;
    if (workspace_bytes < b.total) return MOE_ERR_WORKSPACE_TOO_SMALL;
    return run_backward(cfg, b, workspace, x, Wg, W1, b1, W2, b2, topk_expert, topk_weight, dout, dx, dWg, dgate_bias, dW1, db1,
                        dW2, db2, (hipStream_t)stream);
}

moe_status moe_combine(const moe_config* cfg, const void* y, const int32_t* topk_expert,
                       const float* topk_weight, const int32_t* slot, void* out, void* stream) {
    Plan p;
    moe_status st = make_plan(cfg, &p);
    if (st != MOE_OK) return st;
    if (bad_required({y, topk_expert, topk_weight, slot, out})) return MOE_ERR_INVALID_ARG;
    return run_combine(cfg, p, y, topk_expert, topk_weight, slot, out, (hipStream_t)stream);
}

}  // extern "C"
