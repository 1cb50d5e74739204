// Internal declarations shared by the translation units of libswapmoe.
// Nothing here is part of the C ABI (see include/swapmoe.h for that).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include <stddef.h>
#include <atomic>
#include <string>
#include <vector>

#include "swapmoe.h"

// Tokens handled by one workgroup of the sort kernels (histogram + ranking).
constexpr int SMOE_SORT_BLOCK = 1024;
// Upper bound on d_ff tiles / token tiles is derived from the config at bind time.

// What the second launch of a small batch finishes: ranking and importance sums.
struct smoe_step_tail {
    const float* expert_norm;
    const int32_t* orig_expert;
    const float* orig_gate;
    const float* xnorm;
    int32_t* count;
    float* gsum;
    float* score;
    int accumulate;
    int32_t* perm;
    int32_t* inv_perm;
    int32_t* offsets;
};

struct smoe_layer {
    smoe_config cfg;
    mutable smoe_step_tail tail{};           // left by a small batch's first launch for its second
    mutable bool hidden_by_token = false;    // ... with the layout in which it leaves the hidden activations
    bool bound = false;
    int slots_set = 0;                       // number of slots that hold an expert
    std::vector<int32_t> slot_to_expert;     // host copies of the maps
    std::vector<int32_t> expert_to_slot;
    std::vector<int32_t> phys;               // virtual slot -> physical weight slot (host copy)
    std::vector<int32_t> free_phys;          // physical slots no virtual slot maps to

    // asynchronous update: the plan, and one record per load in flight
    struct Staged {
        int slot = -1, expert = -1, phys = -1, stage = -1;
        hipEvent_t done = nullptr;           // recorded on the load stream after the pack
    };
    std::vector<std::pair<int, int>> plan;   // (slot, expert) changes not started yet, in order
    std::vector<Staged> staged;              // loads in flight
    std::vector<hipEvent_t> event_pool;      // spare events, owned by the handle
    std::vector<int> free_stage;             // staging areas (one per spare slot) not in use
    char* d_stage = nullptr;                 // [spare_slots][2 matrices], bank layout: landing area of host-bank copies
    std::vector<hipEvent_t> released;        // per physical slot: compute-stream event after which it may be overwritten
    const void* bank_seen[2] = {nullptr, nullptr};   // banks smoe_update_tick has validated
    bool bank_is_host = false;               // ... and whether they are pinned host memory
    int ffn_variant[2] = {-1, -1};           // SMOE_FFN_VARIANT read at smoe_create (tuning aid); -1: built-in choice

    // caller-owned device buffers
    const float* router_w = nullptr;
    void* slot_w1 = nullptr;
    void* slot_w2 = nullptr;
    const float* expert_norm = nullptr;
    char* workspace = nullptr;

    // carved out of the workspace (device)
    int32_t* d_expert_to_slot = nullptr;     // [E]
    int32_t* d_slot_to_expert = nullptr;     // [K]
    int32_t* d_phys = nullptr;               // [K] physical weight slot of each virtual slot
    int32_t* d_plan = nullptr;               // [1 + 2K] smoe_update_on_device: number of loads, their slots, their experts
    int32_t* d_sort_hist = nullptr;          // [sort blocks, K]
    int32_t* d_hist32 = nullptr;             // fused path: [ceil(max_tokens/32), K] from the router
    void* d_hidden = nullptr;                // activations of the FFN: [rows, d_ff], rows as in smoe_ws_plan
    float* d_norm_partial = nullptr;         // smoe_expert_norm: [E][64] partial sums of squares
    bool ws_ready = false;                   // device maps and counters initialised since the bind
    // smoe_update_on_device changes the device maps without the host: the host copies are then
    // stale until a call that needs them has fetched the device's (after waiting for that stream)
    bool maps_stale = false;
    hipStream_t maps_stream = nullptr;
    const void* dev_update_seen[3] = {nullptr, nullptr, nullptr};   // pointers smoe_update_on_device has checked
    bool dev_update_host = false;            // ... and whether a bank among them is pinned host memory
    bool load_from_host = false;             // set around a load's launch: its source is pinned host memory
    void* d_router_split = nullptr;          // bf16 path: router weights in matrix-operand order
    void* d_route_part = nullptr;            // small batches: partial logits and sums of squares of at most SMOE_FEW_T tokens
    bool router_split_done = false;          // made by the first smoe_route after a bind

    hipEvent_t prof_ev[4] = {nullptr, nullptr, nullptr, nullptr};   // one-shot FFN profiling events
    hipEvent_t bracket[2] = {nullptr, nullptr};                     // smoe_profile_begin / _end
    bool bracket_open = false;

    int slot_device = -1;                    // GPU of the layer's last load or pass, -1 before the first
    uint64_t slot_traffic_seen = 0;          // that GPU's slot traffic after the last pass, the layer's own loads since added

    // load-on-miss baseline: when each slot's expert was last some token's own choice
    std::vector<int64_t> last_use;
    int64_t use_clock = 0;
};

struct smoe_ws_layout {
    size_t e2s, s2e, phys, dplan, hist, hist32, hidden, rsplit, rpart, norm, stage, total;
};
smoe_ws_layout smoe_ws_plan(const smoe_config& c);

int smoe_fail(int code, const char* fmt, ...);
int smoe_check_hip(hipError_t e, const char* what);

inline size_t smoe_elem_size(int dtype) { return dtype == SMOE_BF16 ? 2 : 4; }
// smoe_forward takes at most this many tokens through its small-batch path (decode.hip), and at most those
// whose rows (8 elements of padding each) fit the dynamic LDS of a compute unit; the path keeps the hidden
// activations of every slot for every token of the batch, in blocks of 32 tokens.
constexpr int SMOE_SMALL_T = 128;
constexpr int SMOE_FEW_T = 16;                             // ... and at most this many take its launches for few tokens
constexpr int SMOE_SMALL_LDS = 160 * 1024 - 2048;          // the rest covers the static tables
inline size_t smoe_small_batch_rows(const smoe_config& c) {
    const int fit = SMOE_SMALL_LDS / (2 * (c.d_model + 8));
    const int t = c.max_tokens < SMOE_SMALL_T ? c.max_tokens : SMOE_SMALL_T;
    return c.dtype == SMOE_BF16 ? (size_t)c.K * (((t < fit ? t : fit) + 31) / 32 * 32) : 0;
}
inline int smoe_sort_blocks(int T) { return (T + SMOE_SORT_BLOCK - 1) / SMOE_SORT_BLOCK; }

// Kernel launchers, one per translation unit.  All validate nothing: the ABI
// layer has done that.  Each returns a smoe_status.
// hist32 (nullable): tokens per slot for every block of 32 tokens, [ceil(T/32)][K]
int smoe_launch_route(const smoe_layer* L, const void* x, int T, int32_t* orig_expert,
                      float* orig_gate, int32_t* slot, float* gate, float* xnorm, int32_t* hist32,
                      hipStream_t s);
// smoe_forward on a small batch, two or three launches (decode.hip): when it applies, the launches, and the names of its
// kernel instances
bool smoe_decode_first_applies(const smoe_layer* L, int T);
std::string smoe_describe_decode(const smoe_layer* L, int T, bool first);
int smoe_launch_decode_first(const smoe_layer* L, const void* x, int T, int32_t* orig_expert, float* orig_gate,
                             int32_t* slot, float* gate, float* xnorm, int32_t* count, float* gsum, float* score,
                             int accumulate, int32_t* perm, int32_t* inv_perm, int32_t* offsets, hipStream_t s,
                             hipEvent_t e0, hipEvent_t e1);
// Bytes of the layer's expert slots (both matrices, spare slots included) and of the slots of the other layers on its GPU
// that were loaded or passed over since its own last pass.
uint64_t smoe_slot_traffic(const smoe_layer* L);
// True when those are more than the 256 MB Infinity Cache can hold: its weights come from HBM then, and the small batch's kernels mark their loads
// non-temporal.  Measured with 16 slots of 768 x 3072: one layer stepped alone (151 MB, stays cached from
// step to step) is 15 % slower with such loads, six layers in turn (906 MB) are 7 % faster.  A captured
// graph keeps the choice of its capture; the results are the same bits either way.
bool smoe_weights_outgrow_cache(const smoe_layer* L);
// plain read of the first K slots of slot_w1 (which = 0) or slot_w2 (1): see smoe_profile_stream_read
int smoe_launch_stream_read(const smoe_layer* L, int which, hipStream_t s);
// true when the tile override, if any, leaves a T-token batch to the small-batch path
bool smoe_ffn_dense_path(const smoe_layer* L, int T);
int smoe_launch_ffn_bf16_dense_second(const smoe_layer* L, const int32_t* slot_of, const float* gate,
                                      const uint16_t* residual, int T, uint16_t* out, hipStream_t s);
int smoe_launch_rank_importance(const smoe_layer* L, const int32_t* orig_expert, const float* orig_gate,
                                const float* xnorm, const int32_t* slot, int T, int32_t* count, float* gsum,
                                float* score, int accumulate, int32_t* perm, int32_t* inv_perm,
                                int32_t* offsets, hipStream_t s);
int smoe_launch_ffn_bf16_fused(const smoe_layer* L, const uint16_t* x, const int32_t* perm, const int32_t* offsets,
                               const float* gate, const uint16_t* residual, int T, uint16_t* out, hipStream_t s);
int smoe_launch_importance(const smoe_layer* L, const int32_t* orig_expert, const float* orig_gate,
                           const float* xnorm, int T, int32_t* count, float* gsum, float* score,
                           int accumulate, hipStream_t s);
int smoe_launch_permute(const smoe_layer* L, const void* x, const int32_t* slot, int T, void* x_perm,
                        int32_t* perm, int32_t* inv_perm, int32_t* offsets, hipStream_t s);
// smoe_permute without a workspace: block histograms in the library's own fixed device array
int smoe_static_max_tokens();
int smoe_launch_permute_static(const smoe_config& c, const void* x, const int32_t* slot, int T, void* x_perm,
                               int32_t* perm, int32_t* inv_perm, int32_t* offsets, hipStream_t s);
int smoe_launch_ffn_f32(const smoe_layer* L, const float* x_perm, const int32_t* offsets, int T,
                        float* y_perm, hipStream_t s);
int smoe_launch_ffn_bf16(const smoe_layer* L, const uint16_t* x_perm, const int32_t* offsets, int T,
                         uint16_t* y_perm, hipStream_t s);
int smoe_describe_ffn_f32(const smoe_layer* L, int T, char* out, size_t n);
int smoe_describe_ffn_bf16(const smoe_layer* L, int T, int fused, char* out, size_t n);
int smoe_launch_combine(const smoe_layer* L, const void* y_perm, const int32_t* inv_perm,
                        const float* gate, const void* residual, int T, void* out, hipStream_t s);
// packs / copies one expert's two matrices into physical slot `phys`
int smoe_launch_pack_slot(const smoe_layer* L, int slot, const void* w1_src, const void* w2_src, hipStream_t s,
                          int map_slot = -1, int expert = -1, int old_expert = -1, int* map_done = nullptr);
// slot now serves `expert` from physical slot `phys` (old_expert, if any, leaves the maps)
int smoe_launch_set_map(const smoe_layer* L, int slot, int expert, int old_expert, int phys, hipStream_t s);
int smoe_launch_expert_norm(const smoe_layer* L, const void* w1, const void* w2, int n, float* out,
                            hipStream_t s);
int smoe_launch_clear_maps(const smoe_layer* L, hipStream_t s);
// update rule on the device from score [E] (device), then the planned loads from a device-readable bank
int smoe_launch_update_on_device(const smoe_layer* L, const float* score, const void* bank_w1, const void* bank_w2,
                                 hipStream_t s);
// brings the host copies of the maps up to date after smoe_update_on_device (waits for its stream)
int smoe_refresh_maps(smoe_layer* L);
int smoe_launch_split_router(const smoe_layer* L, hipStream_t s);

// Kernel launch that, when a pair of events is given, attaches them to the
// dispatch itself (start and end of the kernel's execution).
template <typename K, typename... Args>
inline void smoe_launch_timed_lds(K kernel, dim3 grid, dim3 block, size_t lds, hipStream_t s, hipEvent_t e0, hipEvent_t e1,
                                  Args... args) {
    if (e0 && e1) hipExtLaunchKernelGGL(kernel, grid, block, lds, s, e0, e1, 0, args...);
    else hipLaunchKernelGGL(kernel, grid, block, lds, s, args...);
}
template <typename K, typename... Args>
inline void smoe_launch_timed(K kernel, dim3 grid, dim3 block, hipStream_t s, hipEvent_t e0, hipEvent_t e1,
                              Args... args) {
    smoe_launch_timed_lds(kernel, grid, block, 0, s, e0, e1, args...);
}

// Raises a kernel's dynamic-LDS limit once per device, not on every launch (one object per kernel).
struct smoe_lds_raised {
    std::atomic<unsigned long long> mask{0};
    int ensure(const void* kern, size_t lds, int limit);
};

// 16-byte load of data that is read once per launch (the decode path's weight streams): marked
// non-temporal, so the caches do not keep it at the expense of data that is read again.
__device__ __forceinline__ uint4 smoe_load_stream(const uint4* p) {
    typedef unsigned int smoe_u32x4 __attribute__((ext_vector_type(4)));
    const smoe_u32x4 v = __builtin_nontemporal_load((const smoe_u32x4*)p);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Stores of data that this launch does not read, on their way past the caches likewise.
__device__ __forceinline__ void smoe_store_stream(uint2* p, uint2 v) {
    typedef unsigned int smoe_u32x2 __attribute__((ext_vector_type(2)));
    __builtin_nontemporal_store(smoe_u32x2{v.x, v.y}, (smoe_u32x2*)p);
}
__device__ __forceinline__ void smoe_store_stream(uint4* p, uint4 v) {
    typedef unsigned int smoe_u32x4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store(smoe_u32x4{v.x, v.y, v.z, v.w}, (smoe_u32x4*)p);
}

// Two values narrowed to bf16 by the conversion instruction (to nearest, ties to even) and packed, the first in the lower
// half: one instruction where shifts and additions took ten (4096 tokens of 4 slots of 768 x 3072, five calls: 80.5 -> 79.2 us).
__device__ __forceinline__ uint32_t smoe_pack_bf16(float a, float b) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {a, b};
    union { bf16x2 b; uint32_t u; } c;
    c.b = __builtin_convertvector(v, bf16x2);
    return c.u;
}

// Combine on 8 consecutive outputs of one token that are rounded to bf16 already: out = gate * y (+ residual) in fp32 with
// one final rounding, as smoe_apply_gate.
__device__ __forceinline__ uint4 smoe_gate_unit(uint4 y, float g, uint4 r, bool has_res) {
    uint32_t yw[4] = {y.x, y.y, y.z, y.w};
    const uint32_t rw[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float o0 = __uint_as_float(yw[q] << 16), o1 = __uint_as_float(yw[q] & 0xFFFF0000u);
        if (has_res) {
            o0 = fmaf(g, o0, __uint_as_float(rw[q] << 16));
            o1 = fmaf(g, o1, __uint_as_float(rw[q] & 0xFFFF0000u));
        } else {
            o0 *= g;
            o1 *= g;
        }
        yw[q] = smoe_pack_bf16(o0, o1);
    }
    return make_uint4(yw[0], yw[1], yw[2], yw[3]);
}

// Combine on 4 consecutive outputs of one token.  The product is first rounded to bf16 exactly as the
// separate calls store y_perm, so both give the same bits; then out = gate * y (+ residual) in fp32
// with one final rounding.
__device__ __forceinline__ void smoe_apply_gate(float& v0, float& v1, float& v2, float& v3, float g, uint2 r, bool has_res) {
    const uint32_t lo = smoe_pack_bf16(v0, v1), hi = smoe_pack_bf16(v2, v3);
    v0 = __uint_as_float(lo << 16); v1 = __uint_as_float(lo & 0xFFFF0000u);
    v2 = __uint_as_float(hi << 16); v3 = __uint_as_float(hi & 0xFFFF0000u);
    if (has_res) {
        v0 = fmaf(g, v0, __uint_as_float(r.x << 16)); v1 = fmaf(g, v1, __uint_as_float(r.x & 0xFFFF0000u));
        v2 = fmaf(g, v2, __uint_as_float(r.y << 16)); v3 = fmaf(g, v3, __uint_as_float(r.y & 0xFFFF0000u));
    } else {
        v0 *= g; v1 *= g; v2 *= g; v3 *= g;
    }
}
