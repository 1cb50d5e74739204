// smoe_importance, smoe_permute and smoe_combine: the memory-bound steps
// around the expert FFN.
//
//  * importance (SwapMoE Eq. 1): one workgroup per expert walks all T tokens
//    and keeps those whose original choice is that expert; a fixed-shape LDS
//    tree gives the three sums, so the result is bit-reproducible (no atomics).
//  * permute: stable counting sort by slot -- per-block histograms, a ranking pass that
//    turns them into exact positions with wavefront ballots (no atomics on
//    positions, hence one unique, stable order), and the move of the rows; one to
//    three launches, by batch size.
//  * combine: out[t] = gate[t] * y_perm[inv_perm[t]] (+ residual); top-1 means
//    one source row per token, so this is a gather with 16-byte accesses.

#include <algorithm>
#include <mutex>

#include "smoe_internal.h"
#include "wave_ops.h"

namespace {

// ------------------------------------------------------------- importance
// One workgroup per expert walks all T tokens with coalesced, branch-free loads
// and keeps those whose original choice is that expert; per-thread sums in
// token order and a fixed-shape LDS tree give the three totals, so the result
// is bit-reproducible (no atomics, no dependence on scheduling).
constexpr int IMP_THREADS = 256;

// Thread tid's share of expert e's three sums: tokens tid, tid + 256, ... added
// in that order.  The loads of U tokens are issued together, the adds stay
// sequential, so the result does not depend on U.  What bounds it is the number
// of trips to the L2, one per group: 16 tokens a thread make one trip of a batch
// of 4096, 4 are enough up to 1024.  (rank_importance_kernel with this and the
// ranking's sums in registers: T = 16384, E = 128 11.7 -> 7.2 us.)
template <int U>
__device__ __forceinline__ void importance_groups(const int32_t* __restrict__ orig_expert,
                                                  const float* __restrict__ orig_gate,
                                                  const float* __restrict__ xnorm, int T, int e, int tid,
                                                  int& c, float& g, float& r) {
    for (int t = tid; t < T; t += U * IMP_THREADS) {
        int ev[U];
        float gv[U], xv[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {                      // past the batch: read again, not added
            const int u = min(t + i * IMP_THREADS, T - 1);
            ev[i] = orig_expert[u];
            gv[i] = orig_gate[u];
            xv[i] = xnorm[u];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const bool mine = ev[i] == e && t + i * IMP_THREADS < T;
            c += mine;
            g += mine ? gv[i] : 0.f;
            r += mine ? xv[i] * gv[i] : 0.f;
        }
    }
}

// The whole groups of 16 of a long batch without the checks against its end, which the adds would feel
// (smoe_importance, T = 65536: 16.0 us with them, 11.9 without); returns the tokens they cover.
__device__ __forceinline__ int importance_whole_groups(const int32_t* __restrict__ orig_expert,
                                                       const float* __restrict__ orig_gate,
                                                       const float* __restrict__ xnorm, int T, int e, int tid,
                                                       int& c, float& g, float& r) {
    constexpr int U = 16;
    int t0 = 0;
    for (; t0 + U * IMP_THREADS <= T; t0 += U * IMP_THREADS) {
        int ev[U];
        float gv[U], xv[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int u = t0 + tid + i * IMP_THREADS;
            ev[i] = orig_expert[u];
            gv[i] = orig_gate[u];
            xv[i] = xnorm[u];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const bool mine = ev[i] == e;
            c += mine;
            g += mine ? gv[i] : 0.f;
            r += mine ? xv[i] * gv[i] : 0.f;
        }
    }
    return t0;
}

// LONG: more than 4096 tokens.  An instance of its own: short batches (T = 4096) take 1 us more beside its
// code, and so does rank_importance_kernel.
template <bool LONG>
__device__ __forceinline__ void importance_share(const int32_t* __restrict__ orig_expert,
                                                 const float* __restrict__ orig_gate,
                                                 const float* __restrict__ xnorm, int T, int e, int tid,
                                                 int& c, float& g, float& r) {
    c = 0; g = 0.f; r = 0.f;
    if (LONG) {
        const int t0 = importance_whole_groups(orig_expert, orig_gate, xnorm, T, e, tid, c, g, r);
        importance_groups<16>(orig_expert + t0, orig_gate + t0, xnorm + t0, T - t0, e, tid, c, g, r);
    } else if (T <= 4 * IMP_THREADS) {
        importance_groups<4>(orig_expert, orig_gate, xnorm, T, e, tid, c, g, r);
    } else {
        importance_groups<16>(orig_expert, orig_gate, xnorm, T, e, tid, c, g, r);
    }
}

template <bool LONG>
__global__ __launch_bounds__(IMP_THREADS) void importance_kernel(
    const int32_t* __restrict__ orig_expert, const float* __restrict__ orig_gate,
    const float* __restrict__ xnorm, const float* __restrict__ expert_norm, int T,
    int32_t* __restrict__ count, float* __restrict__ gsum, float* __restrict__ score, int accumulate) {
    __shared__ int32_t s_c[IMP_THREADS];
    __shared__ float s_g[IMP_THREADS], s_r[IMP_THREADS];
    const int e = blockIdx.x, tid = threadIdx.x;
    int c;
    float g, r;
    importance_share<LONG>(orig_expert, orig_gate, xnorm, T, e, tid, c, g, r);
    s_c[tid] = c; s_g[tid] = g; s_r[tid] = r;
    __syncthreads();
    for (int w = IMP_THREADS / 2; w > 0; w >>= 1) {
        if (tid < w) { s_c[tid] += s_c[tid + w]; s_g[tid] += s_g[tid + w]; s_r[tid] += s_r[tid + w]; }
        __syncthreads();
    }
    if (tid == 0) {
        float sc = expert_norm[e] * s_r[0];
        if (accumulate) { count[e] += s_c[0]; gsum[e] += s_g[0]; score[e] += sc; }
        else { count[e] = s_c[0]; gsum[e] = s_g[0]; score[e] = sc; }
    }
}

// ------------------------------------------------------------- permute
constexpr int SB = SMOE_SORT_BLOCK;          // tokens (= threads) per sort block
constexpr int SB_WAVES = SB / 64;

__global__ __launch_bounds__(SB) void sort_hist_kernel(const int32_t* __restrict__ slot, int T, int K,
                                                       int32_t* __restrict__ hist) {
    extern __shared__ int32_t s_hist[];      // [K]
    for (int k = threadIdx.x; k < K; k += SB) s_hist[k] = 0;
    __syncthreads();
    int t = blockIdx.x * SB + threadIdx.x;
    if (t < T) {
        int k = slot[t];
        if ((unsigned)k < (unsigned)K) atomicAdd(&s_hist[k], 1);   // integer: order cannot matter
    }
    __syncthreads();
    for (int k = threadIdx.x; k < K; k += SB) hist[(size_t)blockIdx.x * K + k] = s_hist[k];
}

// Position of token t = offsets[slot] + (tokens of that slot in earlier blocks)
//                     + (in earlier waves of this block) + (in lower lanes of this wave).
__global__ __launch_bounds__(SB) void sort_rank_kernel(const int32_t* __restrict__ slot, int T, int K,
                                                       int nblk, const int32_t* __restrict__ hist,
                                                       int32_t* __restrict__ perm,
                                                       int32_t* __restrict__ inv_perm,
                                                       int32_t* __restrict__ offsets) {
    extern __shared__ int32_t sm[];
    int32_t* s_base = sm;                    // [K]  first position of this block's tokens per slot
    int32_t* s_total = sm + K;               // [K]  tokens per slot over all blocks
    int32_t* s_wave = sm + 2 * K;            // [SB_WAVES][K] per-wave counts -> exclusive prefix
    const int tid = threadIdx.x, blk = blockIdx.x;
    const int lane = tid & 63, wave = tid >> 6;

    for (int i = tid; i < SB_WAVES * K; i += SB) s_wave[i] = 0;
    __syncthreads();

    const int t = blk * SB + tid;
    int my = t < T ? slot[t] : -1;
    const bool live = (unsigned)my < (unsigned)K;   // out-of-contract slot values are skipped
    if (!live) my = 0;
    // lanes of this wave that hold the same slot: refine the live mask bit by bit
    unsigned long long peers = __ballot(live);
    for (int bit = 0; (1 << bit) < K; ++bit) {
        unsigned long long b = __ballot(live && ((my >> bit) & 1));
        peers &= ((my >> bit) & 1) ? b : ~b;
    }
    const unsigned long long below = (1ull << lane) - 1ull;
    const int rank_in_wave = __popcll(peers & below);
    if (live && rank_in_wave == 0) s_wave[wave * K + my] = __popcll(peers);
    __syncthreads();
    for (int k = tid; k < K; k += SB) {      // exclusive prefix over the waves, per slot
        int run = 0;
        for (int w = 0; w < SB_WAVES; ++w) {
            int c = s_wave[w * K + k];
            s_wave[w * K + k] = run;
            run += c;
        }
        int before = 0, total = 0;
        for (int b = 0; b < nblk; ++b) {
            int h = hist[(size_t)b * K + k];
            if (b < blk) before += h;
            total += h;
        }
        s_base[k] = before;
        s_total[k] = total;
    }
    __syncthreads();
    if (tid == 0) {                          // exclusive scan over slots (K <= 256)
        int run = 0;
        for (int k = 0; k < K; ++k) {
            int tot = s_total[k];
            if (blk == 0) offsets[k] = run;
            s_base[k] += run;
            run += tot;
        }
        if (blk == 0) offsets[K] = run;
    }
    __syncthreads();
    if (live) {
        int pos = s_base[my] + s_wave[wave * K + my] + rank_in_wave;
        perm[pos] = t;
        inv_perm[t] = pos;
    }
}

// Fused launch used by smoe_forward: blocks [0, nblk) rank the tokens exactly as
// sort_rank_kernel does, taking the per-32-token slot histograms the router
// wrote (so no histogram launch); blocks [nblk, nblk + E) are the importance
// reduction, one expert each.  The two halves are independent; sharing a launch
// only saves dispatch latency.
__global__ __launch_bounds__(SB) void rank_importance_kernel(
    const int32_t* __restrict__ slot, int T, int K, int nblk, const int32_t* __restrict__ hist32,
    int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm, int32_t* __restrict__ offsets,
    const int32_t* __restrict__ orig_expert, const float* __restrict__ orig_gate,
    const float* __restrict__ xnorm, const float* __restrict__ expert_norm,
    int32_t* __restrict__ count, float* __restrict__ gsum, float* __restrict__ score, int accumulate) {
    extern __shared__ int32_t sm[];
    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= nblk) {
        // ---- importance of expert e: the first IMP_THREADS threads repeat importance_kernel's
        // summation order exactly (thread j takes tokens j, j+256, ...; fixed LDS tree), so the
        // fused and the separate call give the same bits
        const int e = blockIdx.x - nblk;
        int32_t* s_c = sm;
        float* s_g = (float*)(sm + IMP_THREADS);
        float* s_r = (float*)(sm + 2 * IMP_THREADS);
        if (tid < IMP_THREADS) {
            int c;
            float g, r;
            importance_share<false>(orig_expert, orig_gate, xnorm, T, e, tid, c, g, r);
            s_c[tid] = c; s_g[tid] = g; s_r[tid] = r;
        }
        __syncthreads();
        for (int w = IMP_THREADS / 2; w > 0; w >>= 1) {
            if (tid < w) { s_c[tid] += s_c[tid + w]; s_g[tid] += s_g[tid + w]; s_r[tid] += s_r[tid + w]; }
            __syncthreads();
        }
        if (tid == 0) {
            const float sc = expert_norm[e] * s_r[0];
            if (accumulate) { count[e] += s_c[0]; gsum[e] += s_g[0]; score[e] += sc; }
            else { count[e] = s_c[0]; gsum[e] = s_g[0]; score[e] = sc; }
        }
        return;
    }
    // ---- stable rank of the tokens of sort block blk
    int32_t* s_base = sm;                    // [K]
    int32_t* s_total = sm + K;               // [K]
    int32_t* s_wave = sm + 2 * K;            // [SB_WAVES][K]
    const int blk = blockIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < (2 + SB_WAVES) * K; i += SB) sm[i] = 0;
    __syncthreads();
    // totals and "before this block" from the router's histograms (integer adds: order-free): SB / K rows
    // of K counts at a time, a thread stays with its slot and meets the others in LDS once
    const int rows = SB / K, k0 = tid % K, r0 = tid / K, nrb = (T + 31) / 32, first_rb = blk * (SB / 32);
    if (r0 < rows) {
        int total = 0, before = 0;
        constexpr int U = 8;                               // rows fetched together
        for (int rb = r0; rb < nrb; rb += U * rows) {
            int h[U];
#pragma unroll
            for (int i = 0; i < U; ++i) h[i] = hist32[(size_t)min(rb + i * rows, nrb - 1) * K + k0];
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int at = rb + i * rows;              // past the end: read again, not added
                total += at < nrb ? h[i] : 0;
                before += at < min(first_rb, nrb) ? h[i] : 0;
            }
        }
        if (total) atomicAdd(&s_total[k0], total);
        if (before) atomicAdd(&s_base[k0], before);
    }
    const int t = blk * SB + tid;
    int my = t < T ? slot[t] : -1;
    const bool live = (unsigned)my < (unsigned)K;
    if (!live) my = 0;
    unsigned long long peers = __ballot(live);
    for (int bit = 0; (1 << bit) < K; ++bit) {
        unsigned long long b = __ballot(live && ((my >> bit) & 1));
        peers &= ((my >> bit) & 1) ? b : ~b;
    }
    const unsigned long long below = (1ull << lane) - 1ull;
    const int rank_in_wave = __popcll(peers & below);
    if (live && rank_in_wave == 0) s_wave[wave * K + my] = __popcll(peers);
    __syncthreads();
    for (int k = tid; k < K; k += SB) {      // exclusive prefix over the waves, per slot
        int run = 0;
        for (int w = 0; w < SB_WAVES; ++w) {
            int c = s_wave[w * K + k];
            s_wave[w * K + k] = run;
            run += c;
        }
    }
    __syncthreads();
    if (wave == 0) {                         // exclusive scan over slots, 64 at a time
        int run = 0;
        for (int base = 0; base < K; base += 64) {
            const int k = base + lane, tot = k < K ? s_total[k] : 0;
            const int incl = run + smoe_wave_incl_scan(tot);
            if (k < K) {
                if (blk == 0) offsets[k] = incl - tot;
                s_base[k] += incl - tot;
            }
            run = __builtin_amdgcn_readlane(incl, 63);
        }
        if (blk == 0 && lane == 0) offsets[K] = run;
    }
    __syncthreads();
    if (live) {
        int pos = s_base[my] + s_wave[wave * K + my] + rank_in_wave;
        perm[pos] = t;
        inv_perm[t] = pos;
    }
}

// x_perm[pos, :] = x[perm[pos], :], 16 bytes per thread.
__global__ __launch_bounds__(256) void gather_rows_kernel(const uint4* __restrict__ x,
                                                          const int32_t* __restrict__ perm, int T,
                                                          int chunks_per_row, uint4* __restrict__ x_perm) {
    size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    size_t total = (size_t)T * chunks_per_row;
    if (idx >= total) return;
    int pos = (int)(idx / chunks_per_row), c = (int)(idx % chunks_per_row);
    int src = min(max(perm[pos], 0), T - 1);         // in range by construction; clamp guards misuse
    x_perm[idx] = x[(size_t)src * chunks_per_row + c];
}

// smoe_permute without a launch for the ranking and one for the rows: workgroup (b, part) ranks the 64
// tokens of block b and moves its share of them.  Counting is by ballots: the lanes of a wave that hold the
// same slot find each other, the lowest of them adds their number to the wave's own table, so nothing is
// contended, and the position of a token -- slot offset + tokens of its slot in front of it -- is that
// of the sorting kernels above.
//   T <= PERM_ONE_MAX    every workgroup looks at all the slot ids (hist == nullptr): one launch
//   beyond               at those of its 1024-token sort block, and takes the rest from the blocks'
//                        histograms: two launches
// Past PERM_TWO_MAX tokens or PERM_TWO_BYTES of rows, where adding up the histograms in every workgroup or
// moving rows with so few waves costs more than a launch, the three launches above.  Measured with K = 4, 128
// and 32 (fused / three launches, us): 65536 rows of 512 bytes 28, 45, 45 / 23, 39, 36; 32768 of 2 KB 29, 36,
// 34 / 29, 41, 37; 32768 of 4 KB 54, 61, 60 / 47, 60, 55; 16384 of 8 KB 51, 55, 54 / 46, 56, 52; 8192 of 8 KB
// 27, 30, 29 / 27, 36, 30.
// A block's rows are moved by four workgroups, rows of 4 KB and more by sixteen up to PERM_WIDE_MAX tokens,
// while that fills the chip (T = 2000 of 8 KB 19.0 -> 9.9 us, T = 8192 of 4 KB 17.8 -> 16.6, T = 16384 of 4 KB
// 27.7 -> 28.4).  K = 16, rows of 1.5 KB: T = 64 7.2 -> 4.4 us, T = 2048 10.1 -> 7.9 us against three launches.
constexpr int PERM_ONE_MAX = 2048, PERM_TWO_MAX = 32768, PERM_WIDE_MAX = 8192;
constexpr size_t PERM_TWO_BYTES = (size_t)64 << 20;

template <int PARTS>
__global__ __launch_bounds__(256) void permute_rows_kernel(const uint4* __restrict__ x, const int32_t* __restrict__ slot, int T, int K,
                                                          int chunks_per_row, uint4* __restrict__ x_perm, int32_t* __restrict__ perm,
                                                          int32_t* __restrict__ inv_perm, int32_t* __restrict__ offsets,
                                                          const int32_t* __restrict__ hist, int nblk) {
    __shared__ int32_t s_total[4][256], s_before[4][256];  // per wave: tokens of each slot, and those in front of the block
    __shared__ int32_t s_pos[64];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    constexpr int PER = 64 / PARTS;                        // rows to move
    const int blk = blockIdx.x / PARTS, part = blockIdx.x % PARTS, t0 = blk * 64;
    const int first = hist ? t0 / SB * SB : 0, end = hist ? t0 + 64 : T;   // the slot ids looked at
    {
        int total = 0, before = 0;                         // from the other sort blocks
        if (hist && tid < K)
            for (int b = 0; b < nblk; ++b) {
                const int h = hist[(size_t)b * K + tid];
                total += h;
                if (b < t0 / SB) before += h;
            }
#pragma unroll
        for (int w = 0; w < 4; ++w) { s_total[w][tid] = w ? 0 : total; s_before[w][tid] = w ? 0 : before; }
    }
    __syncthreads();
    const unsigned long long below = (1ull << lane) - 1ull;
    int my = -1, my_rank = 0;                              // of this block's token `lane`, in the wave that meets it
    constexpr int U = 4;                                   // ids fetched together
    for (int c0 = first + wave * 64; c0 < end; c0 += 256 * U) {
        int id[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = c0 + u * 256 + lane;
            id[u] = t < T ? slot[t] : -1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int base = c0 + u * 256;
            if (base >= end) break;                        // uniform
            const bool live = (unsigned)id[u] < (unsigned)K;   // out-of-contract slot values are skipped
            const int v = live ? id[u] : 0;
            unsigned long long peers = __ballot(live);
            for (int bit = 0; (1 << bit) < K; ++bit) {
                const unsigned long long b = __ballot(live && ((v >> bit) & 1));
                peers &= ((v >> bit) & 1) ? b : ~b;
            }
            const int rank = __popcll(peers & below);
            if (base == t0) { my = live ? v : -1; my_rank = rank; }
            if (live && rank == 0) {
                const int n = __popcll(peers);
                if (!hist) s_total[wave][v] += n;
                if (base < t0) s_before[wave][v] += n;
            }
        }
    }
    __syncthreads();
    if (wave == 0) {                                       // exclusive scan over the slots, 64 at a time
        int run = 0;
        for (int base = 0; base < K; base += 64) {
            const int k = base + lane;
            int n = 0, b = 0;
            if (k < K)
#pragma unroll
                for (int w = 0; w < 4; ++w) { n += s_total[w][k]; b += s_before[w][k]; }
            const int incl = run + smoe_wave_incl_scan(n);
            if (k < K) {
                s_before[0][k] = incl - n + b;             // first position of the block's tokens of slot k
                if (blockIdx.x == 0) offsets[k] = incl - n;
            }
            run = __builtin_amdgcn_readlane(incl, 63);
        }
        if (blockIdx.x == 0 && lane == 0) offsets[K] = run;
    }
    __syncthreads();
    if (wave == ((t0 >> 6) & 3)) {                         // the wave that met this block's tokens
        const int pos = my >= 0 ? s_before[0][my] + my_rank : -1;
        s_pos[lane] = pos;
        if (pos >= 0 && lane / PER == part) {
            perm[pos] = t0 + lane;
            inv_perm[t0 + lane] = pos;
        }
    }
    __syncthreads();
    const int r0 = part * PER, rows = min(PER, T - t0 - r0);
    for (int idx = tid; idx < rows * chunks_per_row; idx += 256) {
        const int r = idx / chunks_per_row, c = idx - r * chunks_per_row, pos = s_pos[r0 + r];
        if (pos >= 0) x_perm[(size_t)pos * chunks_per_row + c] = x[(size_t)(t0 + r0 + r) * chunks_per_row + c];
    }
}

bool permute_fused(const smoe_config& c, int T) {
    return T <= PERM_ONE_MAX || (T <= PERM_TWO_MAX && (size_t)T * c.d_model * smoe_elem_size(c.dtype) <= PERM_TWO_BYTES);
}

// hist: [blocks of SB tokens][K], needed above PERM_ONE_MAX tokens.
int launch_permute(const smoe_config& c, const void* x, const int32_t* slot, int T, void* x_perm, int32_t* perm, int32_t* inv_perm,
                   int32_t* offsets, int32_t* hist, hipStream_t s, const char* what) {
    const int K = c.K, cpr = (int)((size_t)c.d_model * smoe_elem_size(c.dtype) / 16), nblk = smoe_sort_blocks(T);
    if (T <= PERM_ONE_MAX) hist = nullptr;
    else hipLaunchKernelGGL(sort_hist_kernel, dim3(nblk), dim3(SB), K * sizeof(int32_t), s, slot, T, K, hist);
    if (permute_fused(c, T)) {
        const int parts = cpr >= 256 && T <= PERM_WIDE_MAX ? 16 : 4;
        const int blocks = std::max(1, (T + 63) / 64);     // T = 0 still writes offsets = 0
        hipLaunchKernelGGL(parts == 16 ? permute_rows_kernel<16> : permute_rows_kernel<4>, dim3(parts * blocks), dim3(256), 0, s,
                           (const uint4*)x, slot, T, K, cpr, (uint4*)x_perm, perm, inv_perm, offsets, hist, nblk);
    } else {
        hipLaunchKernelGGL(sort_rank_kernel, dim3(nblk), dim3(SB), (2 + SB_WAVES) * K * sizeof(int32_t), s, slot, T, K, nblk, hist, perm,
                           inv_perm, offsets);
        const size_t total = (size_t)T * cpr;
        hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, (const uint4*)x, perm, T, cpr,
                           (uint4*)x_perm);
    }
    return smoe_check_hip(hipGetLastError(), what);
}

// ------------------------------------------------------------- combine
template <bool BF16>
__global__ __launch_bounds__(256) void combine_kernel(const uint4* __restrict__ y_perm,
                                                      const int32_t* __restrict__ inv_perm,
                                                      const float* __restrict__ gate,
                                                      const uint4* __restrict__ residual, int T,
                                                      int chunks_per_row, uint4* __restrict__ out) {
    size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    size_t total = (size_t)T * chunks_per_row;
    if (idx >= total) return;
    int t = (int)(idx / chunks_per_row), c = (int)(idx % chunks_per_row);
    const float g = gate[t];
    int src = min(max(inv_perm[t], 0), T - 1);
    uint4 y = y_perm[(size_t)src * chunks_per_row + c];
    uint4 r = residual ? residual[idx] : make_uint4(0, 0, 0, 0);
    uint32_t yw[4] = {y.x, y.y, y.z, y.w}, rw[4] = {r.x, r.y, r.z, r.w}, ow[4];
    if (BF16) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float lo = __uint_as_float(yw[i] << 16), hi = __uint_as_float(yw[i] & 0xFFFF0000u);
            if (residual) {
                lo = fmaf(g, lo, __uint_as_float(rw[i] << 16));
                hi = fmaf(g, hi, __uint_as_float(rw[i] & 0xFFFF0000u));
            } else {
                lo *= g;
                hi *= g;
            }
            ow[i] = smoe_pack_bf16(lo, hi);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v = __uint_as_float(yw[i]);
            v = residual ? fmaf(g, v, __uint_as_float(rw[i])) : g * v;
            ow[i] = __float_as_uint(v);
        }
    }
    out[idx] = make_uint4(ow[0], ow[1], ow[2], ow[3]);
}

}  // namespace

int smoe_launch_importance(const smoe_layer* L, const int32_t* orig_expert, const float* orig_gate,
                           const float* xnorm, int T, int32_t* count, float* gsum, float* score,
                           int accumulate, hipStream_t s) {
    hipLaunchKernelGGL(T > 16 * IMP_THREADS ? importance_kernel<true> : importance_kernel<false>, dim3(L->cfg.E), dim3(IMP_THREADS), 0, s, orig_expert,
                       orig_gate, xnorm, L->expert_norm, T, count, gsum, score, accumulate);
    return smoe_check_hip(hipGetLastError(), "smoe_importance launch");
}

int smoe_launch_permute(const smoe_layer* L, const void* x, const int32_t* slot, int T, void* x_perm,
                        int32_t* perm, int32_t* inv_perm, int32_t* offsets, hipStream_t s) {
    return launch_permute(L->cfg, x, slot, T, x_perm, perm, inv_perm, offsets, L->d_sort_hist, s, "smoe_permute launch");
}

// ---------------------------------------------------------------------------
// smoe_permute for callers that may not allocate and have no workspace to bind:
// the per-block slot histograms, the one piece of device memory the sort needs
// beyond its inputs and outputs, live in a fixed array inside the library
// image instead of the bound workspace.  Every GPU the library runs on holds
// its own copy of the array (64 KiB) from the moment the code object is loaded
// until the process ends, at an address of its own, which is asked of the
// runtime once per device; host code never uses the array's name for anything
// else (the name is a host-side stand-in, not a device address).
constexpr int STATIC_MAX_TOKENS = 65536;                         // 64 sort blocks
constexpr int STATIC_MAX_SLOTS = 256;                            // K <= E <= 256 by the C ABI
constexpr int STATIC_HIST_INTS = (STATIC_MAX_TOKENS / SMOE_SORT_BLOCK) * STATIC_MAX_SLOTS;
static __device__ __align__(256) int32_t scratch[STATIC_HIST_INTS];

constexpr int MAX_DEVICES = 64;
static int32_t* g_scratch_ptr[MAX_DEVICES];                      // device address of `scratch`, per device
static std::mutex g_scratch_mu;

// Address of this device's copy of the array (the current device), or an error.
static int static_scratch(int32_t** out) {
    int dev = -1;
    int rc = smoe_check_hip(hipGetDevice(&dev), "smoe_permute_static: current device");
    if (rc) return rc;
    if (dev < 0 || dev >= MAX_DEVICES)
        return smoe_fail(SMOE_EINVAL, "smoe_permute_static: device index %d outside [0,%d)", dev, MAX_DEVICES);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        rc = smoe_check_hip(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "smoe_permute_static: scratch address");
        if (rc) return rc;
        if (!p) return smoe_fail(SMOE_EHIP, "smoe_permute_static: the runtime returned no address for the scratch array");
        g_scratch_ptr[dev] = (int32_t*)p;
    }
    *out = g_scratch_ptr[dev];
    return SMOE_OK;
}

int smoe_static_max_tokens() { return STATIC_MAX_TOKENS; }

// The launches of smoe_launch_permute; only the histogram buffer differs.  Nothing in the array has to
// start at zero: the histogram launch overwrites every entry the ranking reads ([blocks of this
// call][K]), so a smaller call after a larger one is safe.
int smoe_launch_permute_static(const smoe_config& c, const void* x, const int32_t* slot, int T, void* x_perm,
                               int32_t* perm, int32_t* inv_perm, int32_t* offsets, hipStream_t s) {
    int32_t* hist = nullptr;
    if (T > PERM_ONE_MAX)
        if (int rc = static_scratch(&hist)) return rc;
    return launch_permute(c, x, slot, T, x_perm, perm, inv_perm, offsets, hist, s, "smoe_permute_static launch");
}

int smoe_launch_rank_importance(const smoe_layer* L, const int32_t* orig_expert, const float* orig_gate,
                                const float* xnorm, const int32_t* slot, int T, int32_t* count, float* gsum,
                                float* score, int accumulate, int32_t* perm, int32_t* inv_perm,
                                int32_t* offsets, hipStream_t s) {
    const int K = L->cfg.K, E = L->cfg.E;
    const int nblk = smoe_sort_blocks(T);
    size_t lds = (size_t)(2 + SB_WAVES) * K * sizeof(int32_t);
    if (lds < 3 * IMP_THREADS * sizeof(int32_t)) lds = 3 * IMP_THREADS * sizeof(int32_t);
    hipLaunchKernelGGL(rank_importance_kernel, dim3(nblk + E), dim3(SB), lds, s, slot, T, K, nblk, L->d_hist32,
                       perm, inv_perm, offsets, orig_expert, orig_gate, xnorm, L->expert_norm, count, gsum,
                       score, accumulate);
    return smoe_check_hip(hipGetLastError(), "smoe_forward: sort/importance launch");
}

int smoe_launch_combine(const smoe_layer* L, const void* y_perm, const int32_t* inv_perm,
                        const float* gate, const void* residual, int T, void* out, hipStream_t s) {
    int cpr = (int)((size_t)L->cfg.d_model * smoe_elem_size(L->cfg.dtype) / 16);
    size_t total = (size_t)T * cpr;
    dim3 grid((unsigned)((total + 255) / 256));
    if (L->cfg.dtype == SMOE_BF16)
        hipLaunchKernelGGL(combine_kernel<true>, grid, dim3(256), 0, s, (const uint4*)y_perm, inv_perm,
                           gate, (const uint4*)residual, T, cpr, (uint4*)out);
    else
        hipLaunchKernelGGL(combine_kernel<false>, grid, dim3(256), 0, s, (const uint4*)y_perm, inv_perm,
                           gate, (const uint4*)residual, T, cpr, (uint4*)out);
    return smoe_check_hip(hipGetLastError(), "smoe_combine launch");
}
