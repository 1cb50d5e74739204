// smoe_forward on a small batch (bf16, at most SMALL_T tokens whose rows fit the LDS of a compute
// unit together): the whole layer in two launches, or three where most slots stay empty.
//
// With few tokens the layer is bound by reading the slots' weights once, so nothing that stands
// between the kernel's start and its weight stream is tolerated: no sort (every slot's workgroups
// multiply the batch in token order, an MFMA column depends on its own token only, so the bits are
// those of the sorted path), and no wait for the router.
//
//   first launch   one workgroup per 32 tokens is the router; all the others compute the first
//                  product of EVERY slot on EVERY token (hidden_layout).  The price is
//                  the first matrices of slots nobody was routed to, what it buys is the router's
//                  whole time.
//   second launch  one workgroup ranks the tokens and adds the importance sums (it needs only what
//                  the router left); the others compute the second product of the slots that got
//                  tokens, for those tokens, with the gate and the residual.
//
// Where the empty slots' first matrices cost more than the router (see sparse), the router is launched first
// and neither product reads a weight of a slot without a token; up to 16 tokens in a form of its own (see
// route_partial_kernel).

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "route_mfma.h"

namespace {

constexpr int SMALL_T = SMOE_SMALL_T;                      // the token lists below are two 64-lane ballots long
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int LDS_LIMIT = SMOE_SMALL_LDS;

// Where the hidden activations of a small batch are: unit u (8 features, 16 bytes) of token t of slot k is unit
// k * slot + t * token + u * unit.
struct hidden_strides {
    int slot, token, unit;
};

// ---------------------------------------------------------------------------
// First product for every slot and every token.  fbw waves of the workgroup own one 32-feature
// block each (all 8 waves stage the tokens); the token operands come from LDS (row pitch d_model + 8
// elements: conflict-free 16-byte reads), so the vector-memory pipe carries nothing but 1-KiB weight
// loads, 16 of them in flight per wave.  NBF: 32-token blocks the instance holds accumulators for.
// STREAM: the weight loads are marked non-temporal (see smoe_weights_outgrow_cache).
// served: the tokens' slots if the router has run already (then only slots with a token are computed), else NULL.
template <int NBF, bool STREAM>
__device__ __forceinline__ void dense_first_all(const uint16_t* __restrict__ x, const uint4* __restrict__ Wp, int T,
                                                uint16_t* __restrict__ h, const hidden_strides hs, int R, int N, const int32_t* __restrict__ phys,
                                                const int32_t* __restrict__ served, int block, int fbw, uint16_t* xs) {
    constexpr int G = 8;
    const int nfb = N >> 5, nrb = R >> 4, ldx = R + 8;
    const int ftiles = (nfb + fbw - 1) / fbw;
    const int slot = block / ftiles, ftile = block - slot * ftiles;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    if (served) {
        const bool own = served[min(lane, T - 1)] == slot || (NBF > 2 && served[min(lane + 64, T - 1)] == slot);
        if (!__ballot(own)) return;                        // uniform over the workgroup
    }
    const int fb = ftile * fbw + wave;
    const bool streams = wave < fbw && fb < nfb;           // the other waves help with the staging only
    const uint4* wp = Wp + ((size_t)(phys ? phys[slot] : slot) * nfb + min(fb, nfb - 1)) * nrb * 64 + lane;
    uint4 wA[G], wB[G];
    auto fetch_w = [&](uint4 (&w)[G], int g0) {
#pragma unroll
        for (int i = 0; i < G; ++i) {                      // past the end: reloaded, not used
            const uint4* src = wp + (size_t)min(g0 + i, nrb - 1) * 64;
            w[i] = STREAM ? smoe_load_stream(src) : *src;
        }
    };
    // The tokens are staged one chunk of 2 G reduction steps ahead of their use.  A wave's loads
    // complete in order, so each chunk of x is asked for before the weights that follow it: waiting
    // for the chunk then leaves two groups of weight loads in flight.
    constexpr int CC = 2 * G * 16, CPR = CC / 8;           // columns and 16-byte pieces per row of a chunk
    constexpr int XPT = NBF * 32 * CPR / 512;              // pieces per thread
    u32x4 xr[XPT];
    auto fetch_x = [&](u32x4 (&v)[XPT], int k0) {
#pragma unroll
        for (int q = 0; q < XPT; ++q) {
            const int idx = tid + q * 512, r = min(idx / CPR, T - 1), c = min(k0 + (idx % CPR) * 8, R - 8);
            v[q] = *(const u32x4*)(x + (size_t)r * R + c); // pieces outside the batch: read again, not stored
        }
    };
    auto stage_x = [&](u32x4 (&v)[XPT], int k0) {
#pragma unroll
        for (int q = 0; q < XPT; ++q) {
            const int idx = tid + q * 512, r = idx / CPR, c = k0 + (idx % CPR) * 8;
            if (r < T && c < R) *(u32x4*)&xs[r * ldx + c] = v[q];
        }
    };
    fetch_x(xr, 0);
    if (!streams) {                                        // a wave that only helps with the staging
        for (int g0 = 0; g0 < nrb; g0 += 2 * G) {
            stage_x(xr, g0 * 16);
            fetch_x(xr, g0 * 16 + CC);
            __syncthreads();
        }
        return;
    }
    __builtin_amdgcn_sched_barrier(0);
    fetch_w(wA, 0);
    const uint16_t* xrow[NBF];                             // columns past the batch repeat its last row, unstored
#pragma unroll
    for (int b = 0; b < NBF; ++b) xrow[b] = xs + min(b * 32 + (lane & 31), T - 1) * ldx + (lane >> 5) * 8;
    smoe_f32x16 acc[NBF];
#pragma unroll
    for (int b = 0; b < NBF; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[b][i] = 0.f;
    auto consume = [&](uint4 (&w)[G], int g0) {
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const bool in = g0 + i < nrb;                  // steps past the end multiply by a zero operand
#pragma unroll
            for (int b = 0; b < NBF; ++b) {
                uint4 xv = *(const uint4*)(xrow[b] + min(g0 + i, nrb - 1) * 16);
                if (!in) xv = make_uint4(0, 0, 0, 0);
                acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(smoe_frag(w[i]), smoe_frag(xv), acc[b], 0, 0, 0);
            }
        }
    };
    int g0 = 0;
    for (; nrb - g0 > 2 * G; g0 += 2 * G) {
        fetch_w(wB, g0 + G);
        stage_x(xr, g0 * 16);
        fetch_x(xr, g0 * 16 + CC);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        consume(wA, g0);
        __builtin_amdgcn_sched_barrier(0);
        fetch_w(wA, g0 + 2 * G);
        __builtin_amdgcn_sched_barrier(0);
        consume(wB, g0 + G);
        __builtin_amdgcn_sched_barrier(0);
    }
    fetch_w(wB, g0 + G);
    stage_x(xr, g0 * 16);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    consume(wA, g0);
    if (nrb - g0 > G) consume(wB, g0 + G);
    // accumulator register i of lane l: feature 8*(i/4) + 4*(l/32) + i%4, token l%32
#pragma unroll
    for (int b = 0; b < NBF; ++b) {
        const int tok = b * 32 + (lane & 31);
        if (tok >= T) continue;
        uint16_t* ydst = h + ((size_t)slot * hs.slot + (size_t)tok * hs.token + (size_t)fb * 4 * hs.unit) * 8 + (lane >> 5) * 4;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float v0 = fmaxf(acc[b][4 * g], 0.f), v1 = fmaxf(acc[b][4 * g + 1], 0.f), v2 = fmaxf(acc[b][4 * g + 2], 0.f),
                        v3 = fmaxf(acc[b][4 * g + 3], 0.f);
            uint2 o;
            o.x = smoe_pack_bf16(v0, v1);
            o.y = smoe_pack_bf16(v2, v3);
            *(uint2*)(ydst + (size_t)g * hs.unit * 8) = o;
        }
    }
}

// The router's workgroups come first: they are the launch's critical path.
template <int NEB, int NBF, bool STREAM>
__device__ __forceinline__ void decode_first_body(const smoe_route_args& ra, const uint4* W1, uint16_t* h, const hidden_strides hs, int d_ff,
                                                  const int32_t* phys, int fbw) {
    extern __shared__ __align__(16) float smem[];
    const int routers = (ra.T + SMOE_RT - 1) / SMOE_RT;
    if ((int)blockIdx.x < routers) smoe_route_mfma_body<NEB, 1, false>(blockIdx.x, ra, smem);
    else dense_first_all<NBF, STREAM>((const uint16_t*)ra.x, W1, ra.T, h, hs, ra.d, d_ff, phys, nullptr, blockIdx.x - routers, fbw, (uint16_t*)smem);
}

// Two kernels with one body: the second streams its weights past the caches.
template <int NEB, int NBF>
__global__ __launch_bounds__(512) void decode_first_kernel(const smoe_route_args ra, const uint4* __restrict__ W1, uint16_t* __restrict__ h,
                                                           const hidden_strides hs, int d_ff, const int32_t* __restrict__ phys, int fbw) {
    decode_first_body<NEB, NBF, false>(ra, W1, h, hs, d_ff, phys, fbw);
}

template <int NEB, int NBF>
__global__ __launch_bounds__(512) void decode_first_stream_kernel(const smoe_route_args ra, const uint4* __restrict__ W1,
                                                                  uint16_t* __restrict__ h, const hidden_strides hs, int d_ff,
                                                                  const int32_t* __restrict__ phys, int fbw) {
    decode_first_body<NEB, NBF, true>(ra, W1, h, hs, d_ff, phys, fbw);
}

// The same product behind a router launch of its own, for the slots that got tokens.
template <int NBF, bool STREAM>
__global__ __launch_bounds__(512) void dense_first_kernel(const uint16_t* __restrict__ x, const uint4* __restrict__ W1, int T,
                                                          uint16_t* __restrict__ h, const hidden_strides hs, int d, int d_ff,
                                                          const int32_t* __restrict__ phys, const int32_t* __restrict__ slot, int fbw) {
    extern __shared__ __align__(16) float smem[];
    dense_first_all<NBF, STREAM>(x, W1, T, h, hs, d, d_ff, phys, slot, blockIdx.x, fbw, (uint16_t*)smem);
}

// ---------------------------------------------------------------------------
// At most 16 tokens that reach few of the slots: three launches of short chains.  With one token a product is the
// 4.7 MB of one matrix, which the whole chip reads in a microsecond; what counts is how many compute units pull it and
// how many trips to memory follow one another.  So
//   route_partial_kernel       the partial logits of smoe_route_mfma_body, one wave on its own compute unit per (slice of
//                              the reduction, 32 experts) where that body's eight waves share one;
//   dense_first_kernel_served  every workgroup finishes the router for the whole batch by itself (the first one writes
//                              the results down), takes the served slots in order of their first token, and each wave
//                              streams 16 features of one with all its loads in flight;
//   dense_second_kernel_served the same for the second product, the reduction split four ways as in the other forms.
// Products of 16 x 16 x 32 halve the dependent chain of those of 32 x 32 x 16; the bits are the same.
// T = 1, 64 experts, 16 slots of 768 x 3072: 19.4 -> 14.5 us per layer (router, first and second launch took 5.8, 6.6
// and 7.6 us with one compute unit for the router, 96 and 24 with work for the products); 128 slots T = 5 36 -> 19 us.
constexpr int FEW_T = SMOE_FEW_T;

template <int NEB>
__global__ __launch_bounds__(64) void route_partial_kernel(const smoe_route_args a, float* __restrict__ part, float* __restrict__ sqp) {
    using S = smoe_route_shape<NEB, 1>;
    constexpr int NS = S::NS, EP = S::EP, G = 8;
    const int lane = threadIdx.x, slice = blockIdx.x % NS, eb = blockIdx.x / NS;
    const int nkb = a.d >> 4;
    const uint4* wp = a.wr + (size_t)eb * nkb * 2 * 64 + lane;
    const uint16_t* xp = (const uint16_t*)a.x + (size_t)min(lane & 31, a.T - 1) * a.d + (lane >> 5) * 8;
    smoe_f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    float sq = 0.f;
    for (int k0 = 0; k0 < a.d; k0 += SMOE_ROUTE_KC) {      // the same steps in the same order as smoe_route_mfma_body
        const int steps = min(SMOE_ROUTE_KC, a.d - k0) >> 4, per = (steps + NS - 1) / NS;
        const int lo = min(slice * per, steps), n = min(lo + per, steps) - lo, first = (k0 >> 4) + lo;
        if (n <= 0) continue;
        uint4 wA[G][2], wB[G][2], xA[G], xB[G];
        auto fetch = [&](uint4 (&w)[G][2], uint4 (&x)[G], int g0) {
#pragma unroll
            for (int i = 0; i < G; ++i) {                  // past the end: reloaded, not used
                const int k = first + min(g0 + i, n - 1);
                x[i] = *(const uint4*)(xp + k * 16);
#pragma unroll
                for (int hf = 0; hf < 2; ++hf) w[i][hf] = wp[(size_t)(k * 2 + hf) * 64];
            }
        };
        auto consume = [&](uint4 (&w)[G][2], uint4 (&x)[G], int g0) {
#pragma unroll
            for (int i = 0; i < G; ++i) {
                if (g0 + i >= n) break;                    // uniform
                smoe_add_squares(sq, x[i]);
                uint4 pc[3];
                smoe_cut_weights(w[i], pc);
#pragma unroll
                for (int s3 = 2; s3 >= 0; --s3)
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(smoe_frag(pc[s3]), smoe_frag(x[i]), acc, 0, 0, 0);
            }
        };
        fetch(wA, xA, 0);
        for (int g0 = 0; g0 < n; g0 += 2 * G) {
            fetch(wB, xB, g0 + G);
            __builtin_amdgcn_sched_barrier(0);
            consume(wA, xA, g0);
            if (g0 + 2 * G < n) fetch(wA, xA, g0 + 2 * G);
            consume(wB, xB, g0 + G);
        }
    }
    const int t = lane & 31;
    if (t >= a.T) return;
    float* row = part + ((size_t)slice * FEW_T + t) * EP + eb * 32 + 4 * (lane >> 5);
#pragma unroll
    for (int q = 0; q < 4; ++q) *(float4*)(row + 8 * q) = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
    if (eb == 0) sqp[(slice * 2 + (lane >> 5)) * FEW_T + t] = sq;
}

typedef float smoe_f32x4 __attribute__((ext_vector_type(4)));

// The rank-th distinct slot of the batch in order of its first token, -1 past the last; id = slot of token `lane` (T <= 64).
__device__ __forceinline__ int nth_served(int id, int T, int rank) {
    const int lane = threadIdx.x & 63;
    bool seen = lane >= T;
    for (int u = 0; u < T; ++u) seen |= u < lane && __builtin_amdgcn_readlane(id, u) == id;
    const unsigned long long firsts = __ballot(!seen);
    const unsigned long long at = __ballot(!seen && __popcll(firsts & ((1ull << lane) - 1ull)) == rank);
    return at ? __builtin_amdgcn_readlane(id, __ffsll(at) - 1) : -1;
}

// 16-byte units of a 16 x 32 operand out of fragment order (blocks of 16 reduction elements x 32 features):
// lane's feature n (of 32) and reduction units (lane / 16) of 8 elements each.
__device__ __forceinline__ int unit_of(int lane, int n) { return (lane >> 5) * 64 + ((lane >> 4) & 1) * 32 + n; }

template <int NEB, bool STREAM>
__global__ __launch_bounds__(256, 2) void dense_first_kernel_served(const smoe_route_args a, const float* __restrict__ part,
                                                                    const float* __restrict__ sqp, const uint4* __restrict__ W1,
                                                                    uint16_t* __restrict__ h, int d_ff, const int32_t* __restrict__ phys,
                                                                    int fbw) {
    using S = smoe_route_shape<NEB, 1>;
    constexpr int NS = S::NS, EP = S::EP, G = 16;
    extern __shared__ __align__(16) float smem[];
    __shared__ int32_t s_slot[FEW_T];
    uint16_t* xs = (uint16_t*)smem;                        // [T][ldx]
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int cpr = a.d >> 3, pieces = a.T * cpr, ldx = a.d + 8;
    for (int i0 = tid; i0 < pieces; i0 += 4 * 256) {
        u32x4 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = ((const u32x4*)a.x)[min(i0 + q * 256, pieces - 1)];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = min(i0 + q * 256, pieces - 1), r = i / cpr, c = i - r * cpr;
            *(u32x4*)&xs[r * ldx + c * 8] = v[q];
        }
    }
    const int sub = lane & 15;
    int sl[smoe_route_chunks(NEB)][4];
    smoe_route_slots<NEB>(sl, a, sub);
    for (int t0 = wave * 4; t0 < a.T; t0 += 16) {
        const int t = t0 + (lane >> 4), tc = min(t, a.T - 1);
        const smoe_choice c = smoe_route_token<NEB, NS>(part + tc * EP, FEW_T * EP, sl, a.E, a.gate_mode, sub);
        if (sub == 0 && t < a.T) {
            s_slot[t] = c.slot;
            if (blockIdx.x == 0) smoe_store_choice<NS>(a, t, c, sqp + t, FEW_T);
        }
    }
    __syncthreads();
    const int nhb = d_ff >> 4, nst = a.d >> 5, ftiles = (nhb + fbw - 1) / fbw;
    const int rank = blockIdx.x / ftiles, hb = (blockIdx.x - rank * ftiles) * fbw + wave;   // hb: 16 features
    const int slot = nth_served(s_slot[min(lane, a.T - 1)], a.T, rank);
    if (slot < 0 || wave >= fbw || hb >= nhb) return;      // (no barrier follows)
    const uint4* wp = W1 + ((size_t)(phys ? phys[slot] : slot) * (d_ff >> 5) + (hb >> 1)) * (a.d >> 4) * 64 +
                      unit_of(lane, (hb & 1) * 16 + (lane & 15));
    uint4 wA[G], wB[G];
    auto fetch = [&](uint4 (&w)[G], int g0) {
#pragma unroll
        for (int i = 0; i < G; ++i) {                      // past the end: reloaded, not used
            const uint4* src = wp + (size_t)min(g0 + i, nst - 1) * 128;
            w[i] = STREAM ? smoe_load_stream(src) : *src;
        }
    };
    smoe_f32x4 acc;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = 0.f;
    // columns past the batch repeat its last row, unstored
    const uint16_t* xrow = xs + min(lane & 15, a.T - 1) * ldx + (lane >> 4) * 8;
    auto consume = [&](uint4 (&w)[G], int g0) {
#pragma unroll
        for (int i = 0; i < G; ++i) {
            if (g0 + i >= nst) break;                      // uniform
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(smoe_frag(w[i]), smoe_frag(*(const uint4*)(xrow + (g0 + i) * 32)), acc, 0, 0, 0);
        }
    };
    fetch(wA, 0);
    for (int g0 = 0; g0 < nst; g0 += 2 * G) {
        fetch(wB, g0 + G);
        __builtin_amdgcn_sched_barrier(0);
        consume(wA, g0);
        if (g0 + 2 * G < nst) fetch(wA, g0 + 2 * G);
        consume(wB, g0 + G);
    }
    // accumulator register i of lane l: feature 4*(l/16) + i, token l%16
    const int tok = lane & 15;
    if (tok >= a.T) return;
    uint2 o;
    o.x = smoe_pack_bf16(fmaxf(acc[0], 0.f), fmaxf(acc[1], 0.f));
    o.y = smoe_pack_bf16(fmaxf(acc[2], 0.f), fmaxf(acc[3], 0.f));
    *(uint2*)(h + ((size_t)slot * a.T + tok) * d_ff + hb * 16 + 4 * (lane >> 4)) = o;
}

// ---------------------------------------------------------------------------
// Ranking (the index part of smoe_permute) and importance sums (Eq. 1) of at most SMALL_T tokens
// by one workgroup of 256 threads, from what the router left in memory.
__device__ __forceinline__ void finish_small(const smoe_step_tail& t, const int32_t* __restrict__ slot, int T, int E, int K) {
    __shared__ __align__(16) int32_t s_slot[SMALL_T];
    __shared__ int32_t s_oe[SMALL_T], s_cnt[256];
    __shared__ float s_og[SMALL_T], s_r[SMALL_T], s_gsum[256], s_rsum[256];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    int c0 = 0;
    float g0 = 0.f, r0 = 0.f, en = 0.f;
    if (tid < E) {                                         // asked for before anything else
        en = t.expert_norm[tid];
        if (t.accumulate) { c0 = t.count[tid]; g0 = t.gsum[tid]; r0 = t.score[tid]; }
    }
    if (tid < SMALL_T) {
        s_slot[tid] = tid < T ? slot[tid] : 0x7fffffff;    // past the batch: behind every slot, no expert's token
        s_oe[tid] = tid < T ? t.orig_expert[tid] : -1;
        const float og = tid < T ? t.orig_gate[tid] : 0.f;
        s_og[tid] = og;
        s_r[tid] = tid < T ? t.xnorm[tid] * og : 0.f;
    }
    __syncthreads();
    // stable position = tokens of lower slots + earlier tokens of the same slot
    const int nq = (T + 3) >> 2;
    if (tid < T) {
        const int my = s_slot[tid];
        int pos = 0;
        for (int q = 0; q < nq; ++q) {
            const int4 s = *(const int4*)&s_slot[4 * q];
            const int u = 4 * q;
            pos += (s.x < my) | ((s.x == my) & (u < tid));
            pos += (s.y < my) | ((s.y == my) & (u + 1 < tid));
            pos += (s.z < my) | ((s.z == my) & (u + 2 < tid));
            pos += (s.w < my) | ((s.w == my) & (u + 3 < tid));
        }
        t.perm[pos] = tid;
        t.inv_perm[tid] = pos;
    }
    for (int k = tid; k <= K; k += 256) {
        int before = 0;
        for (int q = 0; q < nq; ++q) {
            const int4 s = *(const int4*)&s_slot[4 * q];
            before += (s.x < k) + (s.y < k) + (s.z < k) + (s.w < k);
        }
        t.offsets[k] = before;
    }
    // importance: one wave per expert.  The tokens sit in leaves 0 .. 127 of the separate call's
    // 256-leaf summation tree and its other leaves are zero; token t + 64 first, then strides 32 .. 1,
    // are that tree's levels, so the sums have the same bits.
    const int oe0 = s_oe[lane], oe1 = s_oe[lane + 64];
    const float og0 = s_og[lane], og1 = s_og[lane + 64], rr0 = s_r[lane], rr1 = s_r[lane + 64];
    for (int e = wave; e < E; e += 4) {
        const bool h0 = oe0 == e, h1 = oe1 == e;
        const unsigned long long m0 = __ballot(h0), m1 = __ballot(h1);
        float g = 0.f, r = 0.f;
        if (m0 | m1) {
            g = (h0 ? og0 : 0.f) + (h1 ? og1 : 0.f);
            r = (h0 ? rr0 : 0.f) + (h1 ? rr1 : 0.f);
#pragma unroll
            for (int w = 32; w > 0; w >>= 1) { g += __shfl_xor(g, w); r += __shfl_xor(r, w); }
        }
        if (lane == 0) { s_cnt[e] = __popcll(m0) + __popcll(m1); s_gsum[e] = g; s_rsum[e] = r; }
    }
    __syncthreads();
    if (tid < E) {
        const float sc = en * s_rsum[tid];
        t.count[tid] = c0 + s_cnt[tid];
        t.gsum[tid] = t.accumulate ? g0 + s_gsum[tid] : s_gsum[tid];
        t.score[tid] = t.accumulate ? r0 + sc : sc;
    }
}

// ---------------------------------------------------------------------------
// Second product.  Workgroup (slot, feature block): 4 waves split the reduction four ways and meet
// in LDS (added in wave order: reproducible).  The first group of weight loads is issued before the
// slot ids have arrived, so the latency of the two overlaps; the workgroups of a slot nobody was
// routed to then simply leave.  The slot's own tokens are packed into columns; a batch of more than 32
// tokens (WIDE) has a workgroup for every 32 of them, the later ones at the end of the grid, where a slot
// with many tokens then keeps no workgroup longer than the others (one slot of 768 x 3072, T = 100 27.0 -> 18.3 us per
// layer with two blocks of columns at a time before).
struct second_args {
    const uint16_t* h;
    hidden_strides hs;
    const uint4* W2;
    const int32_t* slot;
    int T, E, K, R, N;
    const int32_t* phys;
    const float* gate;
    const uint16_t* residual;
    uint16_t* out;
    smoe_step_tail tail;
};

// EARLY: the first weights are asked for before the slot ids are there (an instance of its own: with a branch around
// the early loads the wait for the ids becomes a wait for everything, 0.8 us per layer).  Not behind a router launch of
// its own, where most slots are empty, and not with WIDE, where half of the workgroups and more have no token: early
// loads for the first 32 columns only gave nothing (1 to 20 slots, T = 33 .. 128: -0.3 .. 0.4 us).
template <bool WIDE, bool STREAM, bool EARLY>
__device__ __forceinline__ void decode_second_body(const second_args& a) {
    constexpr int KSPLIT = 4, G = 8;                       // G: reduction steps fetched together
    __shared__ __align__(16) float red[(KSPLIT - 1) * 16 * 64];
    __shared__ int32_t s_tok[KSPLIT][SMALL_T];
    if (blockIdx.x == 0) {
        finish_small(a.tail, a.slot, a.T, a.E, a.K);
        return;
    }
    const int nfb = a.N >> 5, nrb = a.R >> 4;
    const int pair = WIDE ? (blockIdx.x - 1) % (a.K * nfb) : blockIdx.x - 1;
    const int c0 = WIDE ? 32 * ((blockIdx.x - 1) / (a.K * nfb)) : 0;   // first of this workgroup's columns of the slot's token list
    const int slot = pair / nfb, fb = pair % nfb;
    // wave index as a scalar: MFMA loop bounds must be wave-uniform for the compiler too
    const int tid = threadIdx.x, part = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int per = (nrb + KSPLIT - 1) / KSPLIT;
    const int kb_lo = min(part * per, nrb), kb_hi = min(kb_lo + per, nrb);
    const uint4* wp = a.W2 + ((size_t)(a.phys ? a.phys[slot] : slot) * nfb + fb) * nrb * 64 + lane;
    auto fetch_w = [&](uint4 (&w)[G], int g0) {
#pragma unroll
        for (int i = 0; i < G; ++i) {                      // past the end: reloaded, not used
            const uint4* src = wp + (size_t)max(min(g0 + i, kb_hi - 1), 0) * 64;
            w[i] = STREAM ? smoe_load_stream(src) : *src;
        }
    };
    // A wave's loads complete in order: the slot ids are asked for first, so that waiting for them
    // does not wait for the weights, and the weights' first group right after, before anything is known.
    const int id0 = a.slot[min(lane, a.T - 1)], id1 = WIDE ? a.slot[min(lane + 64, a.T - 1)] : 0;
    __builtin_amdgcn_sched_barrier(0);
    uint4 wA[G], wB[G];
    if (EARLY) fetch_w(wA, kb_lo);
    __builtin_amdgcn_sched_barrier(0);
    const bool own0 = lane < a.T && id0 == slot, own1 = WIDE && lane + 64 < a.T && id1 == slot;
    const unsigned long long m0 = __ballot(own0), m1 = WIDE ? __ballot(own1) : 0ull;
    const int n0 = __popcll(m0), n = n0 + __popcll(m1);
    if (n <= c0) return;                                   // nothing routed to this slot, or no token left (uniform over the workgroup)
    if (!EARLY) fetch_w(wA, kb_lo);
    const unsigned long long below = (1ull << lane) - 1ull;
    if (own0) s_tok[part][__popcll(m0 & below)] = lane;
    if (own1) s_tok[part][n0 + __popcll(m1 & below)] = lane + 64;
    __syncthreads();                                       // the token lists are complete
    const int c = c0 + (lane & 31);
    const bool live = c < n;
    const int tok = s_tok[part][min(c, n - 1)];            // columns past the list repeat its last token
    const uint4* xp = (const uint4*)a.h + (size_t)slot * a.hs.slot + (size_t)tok * a.hs.token + (lane >> 5) * a.hs.unit;
    const int xstep = 2 * a.hs.unit;
    uint4 xA[G], xB[G];
    auto fetch_x = [&](uint4 (&xv)[G], int g0) {
#pragma unroll
        for (int i = 0; i < G; ++i) xv[i] = xp[(size_t)max(min(g0 + i, kb_hi - 1), 0) * xstep];
    };
    fetch_x(xA, kb_lo);
    float gmul = 1.f;
    uint2 rres[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) rres[g] = make_uint2(0, 0);
    if (live && part == 0) {                               // asked for now, used after the loop
        gmul = a.gate[tok];
        if (a.residual) {
            const uint16_t* rp = a.residual + (size_t)tok * a.N + fb * 32 + (lane >> 5) * 4;
#pragma unroll
            for (int g = 0; g < 4; ++g) rres[g] = *(const uint2*)(rp + g * 8);
        }
    }
    smoe_f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    auto consume = [&](uint4 (&w)[G], uint4 (&xv)[G], int g0) {
#pragma unroll
        for (int i = 0; i < G; ++i) {                      // steps past the end multiply by a zero operand
            const uint4 xz = g0 + i < kb_hi ? xv[i] : make_uint4(0, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(smoe_frag(w[i]), smoe_frag(xz), acc, 0, 0, 0);
        }
    };
    int g0 = kb_lo;
    for (; kb_hi - g0 > 2 * G; g0 += 2 * G) {
        fetch_w(wB, g0 + G);
        fetch_x(xB, g0 + G);
        __builtin_amdgcn_sched_barrier(0);
        consume(wA, xA, g0);
        __builtin_amdgcn_sched_barrier(0);
        fetch_w(wA, g0 + 2 * G);
        fetch_x(xA, g0 + 2 * G);
        __builtin_amdgcn_sched_barrier(0);
        consume(wB, xB, g0 + G);
        __builtin_amdgcn_sched_barrier(0);
    }
    fetch_w(wB, g0 + G);
    fetch_x(xB, g0 + G);
    __builtin_amdgcn_sched_barrier(0);
    consume(wA, xA, g0);
    __builtin_amdgcn_sched_barrier(0);
    consume(wB, xB, g0 + G);
    if (part > 0) {
#pragma unroll
        for (int i = 0; i < 16; ++i) red[((part - 1) * 16 + i) * 64 + lane] = acc[i];
    }
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int w2 = 0; w2 < KSPLIT - 1; ++w2)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] += red[(w2 * 16 + i) * 64 + lane];
    if (!live) return;
    // accumulator register i of lane l: feature 8*(i/4) + 4*(l/32) + i%4, column l%32
    uint16_t* ydst = a.out + (size_t)tok * a.N + fb * 32 + (lane >> 5) * 4;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        float v0 = acc[4 * g], v1 = acc[4 * g + 1], v2 = acc[4 * g + 2], v3 = acc[4 * g + 3];
        smoe_apply_gate(v0, v1, v2, v3, gmul, rres[g], a.residual != nullptr);
        uint2 o;
        o.x = smoe_pack_bf16(v0, v1);
        o.y = smoe_pack_bf16(v2, v3);
        *(uint2*)(ydst + g * 8) = o;
    }
}

// NB = 1: at most 32 tokens, 2: more.  Two workgroups to a compute unit and no third, for which there are registers:
// the units that get three are the last to finish (us per layer, three / two: 18 slots of 1024 x 4096, T = 33 64.4 / 60.2, T = 20
// 59.3 / 54.6; 16 of 512 x 3072, T = 128, four fifths of the tokens alike 44.7 / 40.9; 16 of 768 x 3072 alike; behind a router launch
// of its own 32 slots of 768 x 3072, T = 24 44.9 / 42.2, 64 of 512 x 2048, T = 32 34.7 / 32.5, 32 of 1024 x 4096, T = 20 63.2 / 58.4,
// but 64 of 768 x 3072, T = 32 56.3 / 58.2; 13 shapes, T = 17 .. 32: two 4 % ahead in the mean).
template <int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void decode_second_kernel(const second_args a) { decode_second_body<(NB > 1), false, NB == 1>(a); }

template <int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void decode_second_stream_kernel(const second_args a) { decode_second_body<(NB > 1), true, NB == 1>(a); }

// At most 32 tokens, few of the slots served.
template <bool STREAM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void dense_second_kernel(const second_args a) { decode_second_body<false, STREAM, false>(a); }

// Few tokens: workgroup (served slot, 16 features, or 8 of them while that leaves compute units idle: the lanes of
// the other 8 then read the same weights again).  4 waves split the reduction as above, each with 24 loads in flight.
template <bool STREAM>
__global__ __launch_bounds__(256, 2) void dense_second_kernel_served(const second_args a, int width) {
    constexpr int KSPLIT = 4, G = 12;
    __shared__ __align__(16) float red[(KSPLIT - 1) * 4 * 64];
    if (blockIdx.x == 0) {
        finish_small(a.tail, a.slot, a.T, a.E, a.K);
        return;
    }
    const int tid = threadIdx.x, part = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int cols = a.N / width, rank = (blockIdx.x - 1) / cols, f0 = ((blockIdx.x - 1) - rank * cols) * width;
    const int id = a.slot[min(lane, a.T - 1)];
    const int slot = nth_served(id, a.T, rank);
    if (slot < 0) return;                                  // uniform over the workgroup
    const int nrb = a.R >> 4, per = (nrb + KSPLIT - 1) / KSPLIT;
    const int kb_lo = min(part * per, nrb), nkb = min(kb_lo + per, nrb) - kb_lo, nst = (nkb + 1) >> 1;   // 16-deep blocks; steps of two
    const uint4* wp = a.W2 + (((size_t)(a.phys ? a.phys[slot] : slot) * (a.N >> 5) + (f0 >> 5)) * nrb + kb_lo) * 64 +
                      unit_of(lane, (f0 & 31) + (lane & (width - 1)));
    // the slot's tokens, packed into columns; columns past the list repeat its last token
    const unsigned long long mine = __ballot(lane < a.T && id == slot);
    const int n = __popcll(mine), col = lane & 15;
    int tok = 0;                                           // the col-th set bit
    for (int u = 0; u < a.T; ++u) tok = ((mine >> u) & 1) && __popcll(mine & ((1ull << u) - 1ull)) == min(col, n - 1) ? u : tok;
    const uint4* xp = (const uint4*)a.h + ((size_t)slot * a.T + tok) * (a.R >> 3) + 2 * kb_lo + (lane >> 4);
    uint4 wA[G], wB[G], xA[G], xB[G];
    // A range of an odd number of blocks ends in the middle of a step: the lanes of its upper half then read the lower
    // half again and multiply zeros.
    auto fetch = [&](uint4 (&w)[G], uint4 (&x)[G], int g0) {
#pragma unroll
        for (int i = 0; i < G; ++i) {                      // past the end: reloaded, not used
            const int st = min(g0 + i, nst - 1);
            const bool half = 2 * st + 1 >= nkb && lane >= 32;
            const uint4* src = wp + (size_t)st * 128 - (half ? 64 : 0);
            w[i] = STREAM ? smoe_load_stream(src) : *src;
            x[i] = xp[st * 4 - (half ? 2 : 0)];
        }
    };
    smoe_f32x4 acc;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] = 0.f;
    auto consume = [&](uint4 (&w)[G], uint4 (&x)[G], int g0) {
#pragma unroll
        for (int i = 0; i < G; ++i) {
            if (g0 + i >= nst) break;                      // uniform
            const bool half = 2 * (g0 + i) + 1 >= nkb && lane >= 32;
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(smoe_frag(w[i]), smoe_frag(half ? make_uint4(0, 0, 0, 0) : x[i]), acc, 0, 0, 0);
        }
    };
    const int f = f0 + 4 * (lane >> 4);                    // this lane's four features
    const bool store = part == 0 && 4 * (lane >> 4) < width && col < n;
    if (nst > 0) fetch(wA, xA, 0);
    float gmul = 1.f;
    uint2 rres = make_uint2(0, 0);
    if (store) {                                           // asked for now, used after the loop
        gmul = a.gate[tok];
        if (a.residual) rres = *(const uint2*)(a.residual + (size_t)tok * a.N + f);
    }
    for (int g0 = 0; g0 < nst; g0 += 2 * G) {
        fetch(wB, xB, g0 + G);
        __builtin_amdgcn_sched_barrier(0);
        consume(wA, xA, g0);
        if (g0 + 2 * G < nst) fetch(wA, xA, g0 + 2 * G);
        consume(wB, xB, g0 + G);
    }
    if (part > 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) red[((part - 1) * 4 + i) * 64 + lane] = acc[i];
    }
    __syncthreads();
    if (!store) return;
#pragma unroll
    for (int w2 = 0; w2 < KSPLIT - 1; ++w2)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] += red[(w2 * 4 + i) * 64 + lane];
    float v0 = acc[0], v1 = acc[1], v2 = acc[2], v3 = acc[3];
    smoe_apply_gate(v0, v1, v2, v3, gmul, rres, a.residual != nullptr);
    uint2 o;
    o.x = smoe_pack_bf16(v0, v1);
    o.y = smoe_pack_bf16(v2, v3);
    *(uint2*)(a.out + (size_t)tok * a.N + f) = o;
}

// 32-expert blocks rounded up to an instance of the router
int router_instance(int E) { return E <= 32 ? 1 : E <= 64 ? 2 : E <= 128 ? 4 : 8; }

size_t first_lds(const smoe_config& c, int T) {
    const int neb = router_instance(c.E), d = c.d_model;
    const size_t router = neb == 1   ? smoe_route_shape<1, 1>::lds_bytes(d)
                          : neb == 2 ? smoe_route_shape<2, 1>::lds_bytes(d)
                          : neb == 4 ? smoe_route_shape<4, 1>::lds_bytes(d)
                                     : smoe_route_shape<8, 1>::lds_bytes(d);
    return std::max(router, (size_t)T * (d + 8) * 2);
}

// Slots with a token, if T tokens are spread evenly.
double served_slots(const smoe_config& c, int T) { return c.K * (1.0 - std::pow(1.0 - 1.0 / c.K, T)); }

// Feature blocks per workgroup of the first product: as many of the 8 waves as leave at least
// three workgroups with work per four compute units.
int first_fbw(const smoe_config& c, double slots) {
    const int nfb = c.d_ff >> 5;
    int fbw = 8;
    while (fbw > 1 && slots * ((nfb + fbw - 1) / fbw) < 192) fbw >>= 1;
    return fbw;
}

// True when the router gets a launch (or two) in front of the first product, which then reads the weights
// of the slots with a token only.  Beside the router every slot's first matrix is read, so what that costs is
// the matrices of the slots that stay empty, at the 6 TB/s they stream with.
// More than 16 tokens: what it saves is the router's launch, 8 us up to 64 experts and 12 us above.  The line lies
// where the two meet, at 48 and 72 MB.  Measured per layer in stacks of 0.7 GB and more (beside the router / launch of
// its own, MB for nothing):
//   768 x 3072, E = 64    K = 64 T = 33 88 / 66 us (180 MB); K = 32 T = 32 48 / 48 us (55 MB)
//   768 x 3072, E = 128   K = 32 T = 32 51 / 55 us (55 MB); K = 128 T = 96 200 / 163 us (284 MB)
//   1024 x 4096, E = 128  K = 32 T = 64 108 / 108 us (35 MB)
//   512 x 2048, E = 200   K = 100 T = 64 74 / 64 us (110 MB)
// Up to 16 tokens the launches are those of route_partial_kernel, whose workgroups repeat the end of the router and
// the staging for every slot: the line rises with T, 16 MB + 2 MB a token (beside the router / launches of its own):
//   768 x 3072, E = 64    K = 16 T = 1 22.5 / 14.6 us (71 MB), T = 10 26.5 / 24.7 us (40 MB), T = 16 28.7 / 30.4 us (27 MB);
//                         K = 10 T = 4 17.8 / 17.2 us (31 MB), T = 6 18.1 / 20.1 us (25 MB)
//   768 x 3072, E = 32    K = 8 T = 1 16.3 / 14.1 us (33 MB), T = 6 16.7 / 17.7 us (17 MB); E = 8 K = 4 T = 1 13.7 / 14.0 us (14 MB)
//   1024 x 4096, E = 64   K = 16 T = 16 45.0 / 42.0 us (48 MB); E = 128 K = 16 T = 16 51.0 / 51.7 us (48 MB)
//   512 x 2048, E = 64    K = 20 T = 6 18.4 / 16.5 us (31 MB), T = 13 20.0 / 21.9 us (22 MB)
// These repeat their tokens.  With 64 batches in turn, whose experts do not stay in the cache, both columns hold: 768 x 3072,
// E = 64 K = 16 T = 1 22.2 / 14.7 us, T = 8 26.7 / 24.0, T = 16 28.6 / 32.1; E = 32 K = 8 T = 1 15.8 / 14.1, T = 4 16.4 / 17.0; 128
// slots T = 5 116 / 20; 1024 x 4096, E = 64 K = 16 T = 4 38.0 / 22.0; 512 x 2048, K = 20 T = 6 18.5 / 16.7.
bool sparse(const smoe_config& c, int T) {
    const double unused = (c.K - served_slots(c, T)) * 2.0 * c.d_model * c.d_ff;
    if (T <= FEW_T) return unused > 16e6 + 2e6 * T;
    return unused > (c.E <= 64 ? 48e6 : 72e6);
}

// Layout of the hidden activations between the two launches.  A wave of the second one reads 32 bytes of each of its
// tokens per step.  Token by token the steps of a token share lines, and only the slot's own tokens are touched: better
// where slots hold few of the batch's tokens.  Unit by unit neighbouring tokens share a line: better where slots hold most
// of them, and for rows of up to 4 KB.  What the extra requests of a slot with many tokens cost shows beside weights that
// come from the cache, and little beside weights from memory.  us per layer, [feature / 8][token] / [token][feature],
// clustered tokens:
//   from memory, d_ff > 2048   K = 4 768 x 3072 T = 32 17.0 / 16.1, T = 64 19.5 / 19.2; 6 T = 32 19.6 / 19.1; 16 T = 32 31.4 / 30.0,
//                              T = 64 37.1 / 34.6; 6 of 512 x 3072 T = 64 21.5 / 20.8; 5 of 1024 x 4096 T = 32 24.4 / 22.8
//   from the cache             K = 4 512 x 3072 T = 48 13.7 / 14.8, T = 64 14.6 / 15.7; 4 of 768 x 3072 T = 64 16.8 / 17.8; 5 of 640 x
//                              2560 T = 48 14.9 / 16.3; 6 of 256 x 3072 T = 48 14.0 / 15.0; but 8 of 768 x 3072 T = 32 17.6 / 17.0,
//                              10 T = 100 28.1 / 26.6; 8 of 512 x 2560 T = 64 18.1 / 17.1
//   fewer slots                two of 1024 x 4096 T = 32 16.4 / 18.3; three of 768 x 3072 T = 48 18.6 / 20.0
//   d_ff <= 2048               20 of 512 x 2048 T = 48 24.5 / 25.3; four of 768 x 2048 T = 48 17.0 / 18.0
// With four fifths of the tokens on one slot the second form is up to 10 % behind from 8 slots on as well.
bool hidden_by_token(const smoe_config& c, bool stream) { return c.d_ff > 2048 && c.K >= (stream ? 4 : 8); }

hidden_strides hidden_layout(const smoe_layer* L, int T) {
    const int units = L->cfg.d_ff >> 3, pitch = (T + 31) & ~31;
    return L->hidden_by_token ? hidden_strides{units * T, units, 1} : hidden_strides{units * pitch, 1, pitch};
}

template <int NEB, int NBF>
int launch_first(const smoe_layer* L, const smoe_route_args& ra, bool stream, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    const smoe_config& c = L->cfg;
    const size_t lds = first_lds(c, ra.T);
    const int fbw = first_fbw(c, c.K), ftiles = ((c.d_ff >> 5) + fbw - 1) / fbw;
    const dim3 grid(c.K * ftiles + (ra.T + SMOE_RT - 1) / SMOE_RT);
    const int32_t* phys = c.spare_slots > 0 ? L->d_phys : nullptr;
    auto kern = stream ? decode_first_stream_kernel<NEB, NBF> : decode_first_kernel<NEB, NBF>;
    static smoe_lds_raised raised[2];                      // per kernel: devices whose dynamic-LDS limit is up
    if (int rc = raised[stream].ensure((const void*)kern, lds, LDS_LIMIT)) return rc;
    if (e0 && e1)
        hipExtLaunchKernelGGL(kern, grid, dim3(512), lds, s, e0, e1, 0, ra, (const uint4*)L->slot_w1, (uint16_t*)L->d_hidden,
                              hidden_layout(L, ra.T), c.d_ff, phys, fbw);
    else
        hipLaunchKernelGGL(kern, grid, dim3(512), lds, s, ra, (const uint4*)L->slot_w1, (uint16_t*)L->d_hidden, hidden_layout(L, ra.T),
                           c.d_ff, phys, fbw);
    return smoe_check_hip(hipGetLastError(), "smoe_forward: decode launch");
}

template <int NEB>
int launch_first_nbf(const smoe_layer* L, const smoe_route_args& ra, bool stream, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    if (ra.T <= 32) return launch_first<NEB, 1>(L, ra, stream, s, e0, e1);
    if (ra.T <= 64) return launch_first<NEB, 2>(L, ra, stream, s, e0, e1);
    return launch_first<NEB, 4>(L, ra, stream, s, e0, e1);
}

// The first product by itself (see dense_first_kernel).
template <int NBF>
int launch_first_served(const smoe_layer* L, const smoe_route_args& ra, bool stream, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    const smoe_config& c = L->cfg;
    const size_t lds = (size_t)ra.T * (c.d_model + 8) * 2;
    const int fbw = first_fbw(c, served_slots(c, ra.T)), ftiles = ((c.d_ff >> 5) + fbw - 1) / fbw;
    const dim3 grid(c.K * ftiles);
    const int32_t* phys = c.spare_slots > 0 ? L->d_phys : nullptr;
    auto kern = stream ? dense_first_kernel<NBF, true> : dense_first_kernel<NBF, false>;
    static smoe_lds_raised raised[2];
    if (int rc = raised[stream].ensure((const void*)kern, lds, LDS_LIMIT)) return rc;
    if (e0 && e1)
        hipExtLaunchKernelGGL(kern, grid, dim3(512), lds, s, e0, e1, 0, (const uint16_t*)ra.x, (const uint4*)L->slot_w1, ra.T,
                              (uint16_t*)L->d_hidden, hidden_layout(L, ra.T), c.d_model, c.d_ff, phys, (const int32_t*)ra.slot, fbw);
    else
        hipLaunchKernelGGL(kern, grid, dim3(512), lds, s, (const uint16_t*)ra.x, (const uint4*)L->slot_w1, ra.T, (uint16_t*)L->d_hidden,
                           hidden_layout(L, ra.T), c.d_model, c.d_ff, phys, (const int32_t*)ra.slot, fbw);
    return smoe_check_hip(hipGetLastError(), "smoe_forward: first product launch");
}

// Few tokens on few slots: the three launches of route_partial_kernel's comment.
template <int NEB>
int launch_few(const smoe_layer* L, const smoe_route_args& ra, bool stream, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    using S = smoe_route_shape<NEB, 1>;
    const smoe_config& c = L->cfg;
    float* part = (float*)L->d_route_part;
    float* sqp = part + (size_t)S::NS * FEW_T * S::EP;
    hipLaunchKernelGGL(route_partial_kernel<NEB>, dim3(S::NS * ((c.E + 31) / 32)), dim3(64), 0, s, ra, part, sqp);
    if (int rc = smoe_check_hip(hipGetLastError(), "smoe_forward: router launch")) return rc;
    const size_t lds = (size_t)ra.T * (c.d_model + 8) * 2;
    const int nhb = c.d_ff >> 4, most = std::min(ra.T, c.K);
    const double slots = std::min<double>(served_slots(c, ra.T), most);
    int fbw = 4;                                           // waves of a workgroup that stream: fewer while compute units idle
    while (fbw > 1 && slots * ((nhb + fbw - 1) / fbw) < 192) fbw >>= 1;
    const dim3 grid(most * ((nhb + fbw - 1) / fbw));
    const int32_t* phys = c.spare_slots > 0 ? L->d_phys : nullptr;
    auto kern = stream ? dense_first_kernel_served<NEB, true> : dense_first_kernel_served<NEB, false>;
    static smoe_lds_raised raised[2];
    if (int rc = raised[stream].ensure((const void*)kern, lds, LDS_LIMIT)) return rc;
    smoe_launch_timed_lds(kern, grid, dim3(256), lds, s, e0, e1, ra, (const float*)part, (const float*)sqp, (const uint4*)L->slot_w1,
                          (uint16_t*)L->d_hidden, c.d_ff, phys, fbw);
    return smoe_check_hip(hipGetLastError(), "smoe_forward: first product launch");
}

}  // namespace

int smoe_lds_raised::ensure(const void* kern, size_t lds, int limit) {
    if (lds <= 48 * 1024) return SMOE_OK;
    int dev = 0;
    (void)hipGetDevice(&dev);
    if (dev < 0 || dev >= 64) return smoe_fail(SMOE_EINVAL, "device index %d outside [0,64)", dev);
    const unsigned long long bit = 1ull << dev;
    if (mask.load(std::memory_order_acquire) & bit) return SMOE_OK;
    int rc = smoe_check_hip(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, limit), "LDS size");
    if (!rc) mask.fetch_or(bit, std::memory_order_release);
    return rc;
}

bool smoe_decode_first_applies(const smoe_layer* L, int T) {
    return L->cfg.dtype == SMOE_BF16 && T >= 1 && T <= SMALL_T && first_lds(L->cfg, T) <= (size_t)LDS_LIMIT;
}

int smoe_launch_decode_first(const smoe_layer* L, const void* x, int T, int32_t* orig_expert, float* orig_gate,
                             int32_t* slot, float* gate, float* xnorm, int32_t* count, float* gsum, float* score,
                             int accumulate, int32_t* perm, int32_t* inv_perm, int32_t* offsets, hipStream_t s,
                             hipEvent_t e0, hipEvent_t e1) {
    if (!smoe_decode_first_applies(L, T)) return smoe_fail(SMOE_EINVAL, "smoe_forward: the fused decode launch does not apply");
    const smoe_config& c = L->cfg;
    L->tail = smoe_step_tail{L->expert_norm, orig_expert, orig_gate, xnorm, count, gsum, score, accumulate, perm, inv_perm, offsets};
    const smoe_route_args ra{x, (const uint4*)L->d_router_split, L->router_w, L->d_expert_to_slot, T, c.d_model, c.E, c.gate_mode,
                             orig_expert, orig_gate, slot, gate, xnorm, nullptr, c.K};
    const bool stream = smoe_weights_outgrow_cache(L);
    L->hidden_by_token = hidden_by_token(c, stream);
    if (sparse(c, T) && T <= FEW_T) {
        switch (router_instance(c.E)) {
            case 1: return launch_few<1>(L, ra, stream, s, e0, e1);
            case 2: return launch_few<2>(L, ra, stream, s, e0, e1);
            case 4: return launch_few<4>(L, ra, stream, s, e0, e1);
            default: return launch_few<8>(L, ra, stream, s, e0, e1);
        }
    }
    if (sparse(c, T)) {
        if (int rc = smoe_launch_route(L, x, T, orig_expert, orig_gate, slot, gate, xnorm, nullptr, s)) return rc;
        if (T <= 32) return launch_first_served<1>(L, ra, stream, s, e0, e1);
        if (T <= 64) return launch_first_served<2>(L, ra, stream, s, e0, e1);
        return launch_first_served<4>(L, ra, stream, s, e0, e1);
    }
    switch (router_instance(c.E)) {
        case 1: return launch_first_nbf<1>(L, ra, stream, s, e0, e1);
        case 2: return launch_first_nbf<2>(L, ra, stream, s, e0, e1);
        case 4: return launch_first_nbf<4>(L, ra, stream, s, e0, e1);
        default: return launch_first_nbf<8>(L, ra, stream, s, e0, e1);
    }
}

int smoe_launch_ffn_bf16_dense_second(const smoe_layer* L, const int32_t* slot_of, const float* gate,
                                      const uint16_t* residual, int T, uint16_t* out, hipStream_t s) {
    const smoe_config& c = L->cfg;
    const second_args a{(const uint16_t*)L->d_hidden, hidden_layout(L, T), (const uint4*)L->slot_w2, slot_of, T, c.E, c.K, c.d_ff, c.d_model,
                        c.spare_slots > 0 ? L->d_phys : nullptr, gate, residual, out, L->tail};
    const bool stream = smoe_weights_outgrow_cache(L);
    if (sparse(c, T) && T <= FEW_T) {
        const int most = std::min(T, c.K);
        const int width = most * (c.d_model >> 3) <= 256 ? 8 : 16;
        auto few = stream ? dense_second_kernel_served<true> : dense_second_kernel_served<false>;
        smoe_launch_timed(few, dim3(most * (c.d_model / width) + 1), dim3(256), s, L->prof_ev[2], L->prof_ev[3], a, width);
        L->tail = smoe_step_tail{};                        // the caller's pointers are not kept
        return smoe_check_hip(hipGetLastError(), "smoe_forward: FFN launch");
    }
    const dim3 grid((T + 31) / 32 * c.K * (c.d_model >> 5) + 1);
    auto kern = T <= 32 ? (stream ? decode_second_stream_kernel<1> : decode_second_kernel<1>)
                        : (stream ? decode_second_stream_kernel<2> : decode_second_kernel<2>);
    if (sparse(c, T) && T <= 32) kern = stream ? dense_second_kernel<true> : dense_second_kernel<false>;
    smoe_launch_timed(kern, grid, dim3(256), s, L->prof_ev[2], L->prof_ev[3], a);
    L->tail = smoe_step_tail{};                            // the caller's pointers are not kept
    return smoe_check_hip(hipGetLastError(), "smoe_forward: FFN launch");
}

std::string smoe_describe_decode(const smoe_layer* L, int T, bool first) {
    const std::string st = smoe_weights_outgrow_cache(L) ? "_stream" : "";
    const std::string tf = st.empty() ? "false>" : "true>";
    if (sparse(L->cfg, T) && T <= FEW_T) {
        return (first ? "dense_first_kernel_served<" + std::to_string(router_instance(L->cfg.E)) + ", " : std::string("dense_second_kernel_served<")) + tf;
    }
    if (sparse(L->cfg, T) && first) return std::string("dense_first_kernel<") + (T <= 32 ? "1, " : T <= 64 ? "2, " : "4, ") + tf;
    if (sparse(L->cfg, T) && T <= 32) return "dense_second_kernel<" + tf;
    if (!first) return "decode_second" + st + "_kernel<" + (T <= 32 ? "1>" : "2>");
    return "decode_first" + st + "_kernel<" + std::to_string(router_instance(L->cfg.E)) + ", " + (T <= 32 ? "1>" : T <= 64 ? "2>" : "4>");
}
