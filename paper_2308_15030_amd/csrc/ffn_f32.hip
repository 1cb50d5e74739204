// smoe_expert_ffn, fp32 path: y = ReLU(x W1_k) W2_k per slot segment (the
// expert E_i(x) of SwapMoE's Background section, d_model -> d_ff -> ReLU ->
// d_model, no biases) as two grouped GEMMs with fp32 matrix products (fp32
// multiply and accumulate throughout).  Weights are the first operand, tokens
// the second, so an accumulator lane holds consecutive features of one token.
//
// Layouts.  Slots keep panels of 64 features (the last one narrower), each
// [R / 4][panel width][4]: four consecutive reduction elements of a feature are one 16-byte unit, a
// wave streams its panel contiguously.  The hidden activations are the same units,
// [row / 32][feature / 4][row % 32], with every segment re-based to a multiple of 32 rows: the first
// product's stores and the second's loads are runs of 512 bytes.
//
// One workgroup per (32-token row tile, range of 64, 32 or 16 features of a panel); its 8 waves split
// the reduction and meet in LDS (in wave order: reproducible).  v_mfma_f32_16x16x4 on one or two blocks
// of 16 tokens.  Operands come straight from memory, with no barrier in the loop: one 16-byte load per
// lane feeds four products, 24 bytes per cycle and compute unit at full rate.  (Tiles of 128 features x
// 64 tokens staged in LDS need half of that and were no faster up to T = 1024: 76 against 77 us at
// T = 512 on four slots of 768 x 3072.)  A lone product of 32 x 64 x 3072 keeps its workgroup busy for
// 21 us, so the feature range is narrowed until the items fill the chip.
//
// Both products, four slots of 768 x 3072 (LDS tiles of 32 x 64 with vector FMAs before): T = 512
// 280 -> 68 us (71 TFLOP/s; 40.0 + 34.4 in a kernel trace), T = 32 23 us, T = 4 16 us (75 MB of weights: 4.7 TB/s).  At
// T = 512 no unit is at its limit (trace and counters): the matrix cores are busy for 16.3 us of each launch, the L1 sees 0.30
// and 0.18 accesses per cycle (a token load of the first product is one per lane, 16 rows lying apart), 77 and 63 % of the L2
// requests hit, and a wave waits for its next instruction two thirds of the time, with two waves to a SIMD.  Items of
// 64 tokens halve the bytes per product and gave nothing (first product T = 512 35 us, both T = 1024 67 and 54 us).

#include <algorithm>
#include <cstdio>
#include <type_traits>

#include "smoe_internal.h"
#include "wave_ops.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int PW = 64;                                     // features of a full panel
constexpr int XCDS = 8;

// Slot and rows of row tile mt, counting ceil(len / bt) tiles per slot in slot order, and the tile's
// first row with every segment re-based to a multiple of 32; every wave works this out for itself.
// False when mt is past the last tile.
__device__ __forceinline__ bool find_tile(const int32_t* __restrict__ offsets, int nslots, int T, int mt, int bt, int& slot,
                                          int& m0, int& m_end, int& pm0) {
    const int lane = threadIdx.x & 63;
    int before = 0, pad_before = 0;
    for (int base = 0; base < nslots; base += 64) {
        const int k = base + lane;
        int a = 0, b = 0;
        if (k < nslots) {
            a = min(max(offsets[k], 0), T);                // clamps guard misuse
            b = max(min(max(offsets[k + 1], 0), T), a);
        }
        const int tiles = (b - a + bt - 1) / bt, pad = (b - a + 31) & ~31;
        const int incl = before + smoe_wave_incl_scan(tiles), pincl = pad_before + smoe_wave_incl_scan(pad);
        const unsigned long long past = __ballot(incl > mt);
        if (past) {
            const int who = __ffsll((long long)past) - 1;
            const int within = (mt - __builtin_amdgcn_readlane(incl - tiles, who)) * bt;
            slot = base + who;
            m0 = __builtin_amdgcn_readlane(a, who) + within;
            m_end = __builtin_amdgcn_readlane(b, who);
            pm0 = __builtin_amdgcn_readlane(pincl - pad, who) + within;
            return true;
        }
        before = __builtin_amdgcn_readlane(incl, 63);
        pad_before = __builtin_amdgcn_readlane(pincl, 63);
    }
    return false;
}

// Row tiles of all slots.
__device__ __forceinline__ int count_tiles(const int32_t* __restrict__ offsets, int nslots, int T, int bt) {
    const int lane = threadIdx.x & 63;
    int total = 0;
    for (int base = 0; base < nslots; base += 64) {
        const int k = base + lane;
        int a = 0, b = 0;
        if (k < nslots) {
            a = min(max(offsets[k], 0), T);
            b = max(min(max(offsets[k + 1], 0), T), a);
        }
        total += __builtin_amdgcn_readlane(smoe_wave_incl_scan((b - a + bt - 1) / bt), 63);
    }
    return total;
}

// The work items are (feature range, row tile) pairs, numbered with the row tile fastest.  Workgroups
// are dealt to the dies round-robin; die x owns the x-th eighth of the list, and the j-th of its n
// workgroups takes items j, j + n, ..: the row tiles of one feature range follow each other on one die,
// which then fetches the slot's weights once.  The grid holds what the chip keeps resident: a workgroup
// per item, most of them leaving at once, gets two workgroups with work onto one compute unit while
// others idle (measured on tiles of 128 x 64, T = 512: 119 us for both products against 76).
template <typename F>
__device__ __forceinline__ void for_items(const int32_t* __restrict__ offsets, int nslots, int T, int bt, int ranges, F&& body) {
    const int tiles = count_tiles(offsets, nslots, T, bt);
    const int G = tiles * ranges, die = blockIdx.x % XCDS, n = gridDim.x / XCDS;   // the grid is a multiple of 8
    const int lo = (int)((long long)G * die / XCDS), hi = (int)((long long)G * (die + 1) / XCDS);
    for (int g = lo + blockIdx.x / XCDS; g < hi; g += n) {
        const int range = g / tiles;
        int slot, m0, m_end, pm0;
        if (!find_tile(offsets, nslots, T, g - range * tiles, bt, slot, m0, m_end, pm0)) return;
        body(range, slot, m0, m_end, pm0);
    }
}

// ---------------------------------------------------------------------------
constexpr int PK_WAVES = 8;

// One wave's share of NC blocks of 16 features times NB blocks of 16 tokens: n steps of 16 reduction elements.  Lane l
// holds unit l / 16 of a step: of feature l % 16 of every 16-feature block, of token l % 16 of a block.
// CUT: two parts of the reduction in one stream of loads, the second part's operands on their way while the first is
// multiplied; cut(acc) takes the sums of the first part, cut_at steps (us, five calls: four slots of 768 x 3072, T = 512 89.7 ->
// 88.6, T = 1024 141.5 -> 139.2; two of 300 x 1200, T = 1024 53.3 -> 51.2).
template <int NB, int NC, bool CUT, typename F>
__device__ __forceinline__ void panel_tile(const float* const (&wp)[NC], const float* const (&xp)[NB], int wstep, int xstep, int u0,
                                           int n, int units, f32x4 (&acc)[NC][NB], int cut_at, F&& cut) {
    constexpr int G = NC == 4 ? (NB == 1 ? 3 : 2) : 4;     // steps fetched together; two such groups are in flight
    const int sub = (threadIdx.x & 63) >> 4;
    f32x4 wA[G][NC], wB[G][NC], xA[G][NB], xB[G][NB];
    auto fetch = [&](f32x4 (&w)[G][NC], f32x4 (&x)[G][NB], int g0) {
#pragma unroll
        for (int i = 0; i < G; ++i) {                      // past the end: read again, not used
            const int u = min(u0 + min(g0 + i, n - 1) * 4 + sub, units - 1);
#pragma unroll
            for (int b = 0; b < NB; ++b) x[i][b] = *(const f32x4*)(xp[b] + (size_t)u * xstep);
#pragma unroll
            for (int c = 0; c < NC; ++c) w[i][c] = *(const f32x4*)(wp[c] + (size_t)u * wstep);
        }
    };
    auto step = [&](f32x4 (&w)[NC], f32x4 (&x)[NB], int i) {
        if (CUT && i == cut_at) cut(acc);                  // uniform
        const bool in = u0 + i * 4 + sub < units;          // the reduction may end in the middle of a step
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const float xv = in ? x[b][q] : 0.f;
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[c][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[c][q], xv, acc[c][b], 0, 0, 0);
            }
    };
    fetch(wA, xA, 0);
    int g0 = 0;
    for (; n - g0 > 2 * G; g0 += 2 * G) {
        fetch(wB, xB, g0 + G);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < G; ++i) step(wA[i], xA[i], g0 + i);
        __builtin_amdgcn_sched_barrier(0);
        fetch(wA, xA, g0 + 2 * G);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < G; ++i) step(wB[i], xB[i], g0 + G + i);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (n - g0 > G) fetch(wB, xB, g0 + G);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < G; ++i)
        if (g0 + i < n) step(wA[i], xA[i], g0 + i);        // uniform; nothing is fetched after this
#pragma unroll
    for (int i = 0; i < G; ++i)
        if (g0 + G + i < n) step(wB[i], xB[i], g0 + G + i);
}

// FIRST: row-major x in, ReLU, hidden activations out; else hidden activations in, row-major y out.
// NC: 16-feature blocks of an item.  WAVES: 8, one part of the reduction each, or 4, which take two parts each.
// Either way the eight parts meet in LDS and are added in order: a row's bits do not depend on the batch around it.
template <bool FIRST, int NC, int WAVES>
__device__ __forceinline__ void panel_items(const float* __restrict__ X, const float* __restrict__ W, const int32_t* __restrict__ offsets,
                                            const int32_t* __restrict__ phys, int nslots, int T, float* __restrict__ Y, int R, int N,
                                            f32x4 (&red)[PK_WAVES][2 * NC][64]) {
    constexpr int PARTS = PK_WAVES / WAVES;
    for_items(offsets, nslots, T, 32, (N + 16 * NC - 1) / (16 * NC), [&](int range, int slot, int m0, int m_end, int pm0) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, col = lane & 15;
    const int n0 = range * 16 * NC, p0 = n0 & ~(PW - 1), nw = min(PW, N - p0), rows = min(32, m_end - m0);
    const int units = R >> 2, steps = (units + 3) >> 2, per = (steps + PK_WAVES - 1) / PK_WAVES;
    const float* wp[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) wp[c] = W + ((size_t)phys[slot] * N + p0) * R + min(n0 - p0 + c * 16 + col, nw - 1) * 4;
    const float* xp[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {                          // columns past the segment repeat its last row, unstored
        const int r = min(b * 16 + col, rows - 1);
        xp[b] = FIRST ? X + (size_t)(m0 + r) * R : X + ((size_t)(pm0 >> 5) * units * 32 + r) * 4;
    }
    const int xstep = FIRST ? 4 : 128;
    const bool two = rows > 16;                            // uniform
    auto run = [&](auto nbc) {
        constexpr int NB = decltype(nbc)::value;
        const float* xq[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) xq[b] = xp[b];
        const int lo = min(wave * PARTS * per, steps), n = min(lo + PARTS * per, steps) - lo;
        f32x4 acc[NC][NB];
        auto clear = [&](f32x4 (&acc)[NC][NB]) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int c = 0; c < NC; ++c) acc[c][b] = f32x4{0.f, 0.f, 0.f, 0.f};
        };
        auto put = [&](f32x4 (&acc)[NC][NB], int part) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int b = 0; b < NB; ++b) red[wave * PARTS + part][c * 2 + b][lane] = acc[c][b];
        };
        clear(acc);
        if (n > 0)
            panel_tile<NB, NC, (PARTS > 1)>(wp, xq, nw * 4, xstep, lo * 4, n, units, acc, per, [&](f32x4 (&acc)[NC][NB]) {
                put(acc, 0);
                clear(acc);
            });
        if (PARTS > 1 && n <= per) {                       // the second part is empty
            put(acc, 0);
            clear(acc);
        }
        put(acc, PARTS - 1);
    };
    if (two) run(std::integral_constant<int, 2>{});
    else run(std::integral_constant<int, 1>{});
    __syncthreads();
    // wave w finishes (feature block, token block) w, and w + 4 where there are 4 waves.  Accumulator register i of
    // lane l: feature 4*(l/16) + i of the block, token l%16
#pragma unroll
    for (int q = wave; q < 2 * NC; q += WAVES) {
        const int c = q >> 1, b = q & 1;
        const int r = b * 16 + col, f = n0 + c * 16 + (lane >> 4) * 4;
        if ((b == 0 || two) && r < rows && f < N) {
            f32x4 v = red[0][q][lane];
#pragma unroll
            for (int w = 1; w < PK_WAVES; ++w) v += red[w][q][lane];
            if (FIRST) {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = fmaxf(v[i], 0.f);
                *(f32x4*)&Y[((size_t)(pm0 >> 5) * (N >> 2) + (f >> 2)) * 128 + r * 4] = v;
            } else {
                *(f32x4*)&Y[(size_t)(m0 + r) * N + f] = v;
            }
        }
    }
    __syncthreads();                                       // the sums have been read
    });
}

template <bool FIRST, int NC>
__global__ __launch_bounds__(PK_WAVES * 64) void panel_gemm_f32(
    const float* __restrict__ X, const float* __restrict__ W, const int32_t* __restrict__ offsets,
    const int32_t* __restrict__ phys, int nslots, int T, float* __restrict__ Y, int R, int N) {
    __shared__ __align__(16) f32x4 red[PK_WAVES][2 * NC][64];
    if (blockDim.x == PK_WAVES * 64) panel_items<FIRST, NC, PK_WAVES>(X, W, offsets, phys, nslots, T, Y, R, N, red);
    else panel_items<FIRST, NC, PK_WAVES / 2>(X, W, offsets, phys, nslots, T, Y, R, N, red);
}

// 16-feature blocks of an item: the widest range that still gives three items per four compute units.
int feature_blocks(const smoe_config& c, int T, int N) {
    const int tiles = T / 32 + (std::min(c.K, T) + 1) / 2;                              // expected row tiles
    int nc = 4;
    while (nc > 1 && tiles * ((N + 16 * nc - 1) / (16 * nc)) < 192) nc >>= 1;
    return nc;
}

// As many workgroups as the chip keeps resident, fewer if the items run out: one of 8 waves on each of the 32 compute
// units of a die, or two of 4 waves where some compute units have two items and slots are filled.  Two that are at
// different places of their items hide the wait for an item's first operands and the meeting of its parts.  8 -> 4 waves:
// four slots of 768 x 3072, T = 1024 70 -> 60 and 59.5 -> 57 us, T = 512 first product 41 -> 36 us, T = 256 22.7 -> 21; two of
// 300 x 1200, T = 256 first product 10.9 -> 9.2 us.  But with 216 items (T = 512 second product) 31.4 -> 33.0, and with few
// tokens per slot, whose items are short, T = 128 13.4 -> 14.7 and eight slots of 512 x 2048, T = 64 11.4 -> 12.8.
template <bool FIRST>
void launch(const smoe_layer* L, const float* X, const void* W, const int32_t* offsets, int T, float* Y, int R, int N, hipStream_t s,
            hipEvent_t e0, hipEvent_t e1) {
    const int K = L->cfg.K, nc = feature_blocks(L->cfg, T, N), ranges = (N + 16 * nc - 1) / (16 * nc);
    const bool pairs = (long long)ranges * (T / 32 + (std::min(K, T) + 1) / 2) > 256 && T >= 48 * K;   // expected items
    const long long items = (long long)ranges * (T / 32 + std::min(K, T));              // upper bound
    const dim3 grid(XCDS * (unsigned)std::min<long long>((items + XCDS - 1) / XCDS, pairs ? 64 : 32));
    auto kern = nc == 4 ? panel_gemm_f32<FIRST, 4> : nc == 2 ? panel_gemm_f32<FIRST, 2> : panel_gemm_f32<FIRST, 1>;
    smoe_launch_timed(kern, grid, dim3(PK_WAVES * (pairs ? 32 : 64)), s, e0, e1, X, (const float*)W, offsets, (const int32_t*)L->d_phys, K, T, Y, R,
                      N);
}

}  // namespace

int smoe_launch_ffn_f32(const smoe_layer* L, const float* x_perm, const int32_t* offsets, int T,
                        float* y_perm, hipStream_t s) {
    const smoe_config& c = L->cfg;
    float* h = (float*)L->d_hidden;
    launch<true>(L, x_perm, L->slot_w1, offsets, T, h, c.d_model, c.d_ff, s, L->prof_ev[0], L->prof_ev[1]);
    launch<false>(L, h, L->slot_w2, offsets, T, y_perm, c.d_ff, c.d_model, s, L->prof_ev[2], L->prof_ev[3]);
    return smoe_check_hip(hipGetLastError(), "smoe_expert_ffn launch");
}

// Names of the two kernel instances of a T-token batch, as a profiler prints them.
int smoe_describe_ffn_f32(const smoe_layer* L, int T, char* out, size_t n) {
    const smoe_config& c = L->cfg;
    snprintf(out, n, "panel_gemm_f32<true, %d> | panel_gemm_f32<false, %d>", feature_blocks(c, T, c.d_ff), feature_blocks(c, T, c.d_model));
    return SMOE_OK;
}
