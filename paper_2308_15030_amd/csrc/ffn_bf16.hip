// smoe_expert_ffn, bf16 path: y = ReLU(x W1_k) W2_k per slot segment (the
// expert E_i(x) of SwapMoE's Background section; d_model -> d_ff -> ReLU ->
// d_model, no biases) as two grouped GEMMs on the matrix cores
// (v_mfma_f32_32x32x16_bf16, fp32 accumulation); the hidden activations are
// rounded to bf16 and kept in the workspace between the two.
//
// Shape of one GEMM:  Y[T, N] = act(X[T, R] . B_k[R, N])  for the rows of slot k.
//
// The weights are the MFMA's first operand and the tokens its second, so an
// accumulator lane ends up holding 4 consecutive output features of ONE token,
// and the token operand is 8 consecutive reduction elements of one row.
//
// Weights arrive in fragment order (see resident.hip): every wave streams its
// own feature blocks straight from HBM into registers with contiguous 1-KiB
// loads, prefetched PD reduction slices ahead in a register ring -- they never
// touch LDS, since no other wave of the workgroup needs them.  The token tile
// is what the waves share; it is staged through a three-stage LDS ring.
//
// The hidden activations h never leave the library, so they are kept in
// fragment order too: rows are re-based per segment to a multiple of 32
// ("padded rows"), and h is stored as 16-byte units [row/32][feature/8][row%32]
// of 8 features.  The first GEMM's accumulator layout then stores straight into
// 512-byte runs, and the second GEMM stages its token tile with a linear copy
// and reads operands from LDS without padding or bank conflicts.
//
// Workgroup = NW waves; tile = (32*MAXB tokens) x (NW*AF*32 features); wave w
// owns AF feature blocks and all token blocks: AF*NBF accumulators of 16 VGPRs.
// Token tiles are enumerated per slot from the device-side offsets; the tiled
// kernel runs as persistent workgroups that each walk a fixed share of the tiles.

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <string>
#include <type_traits>

#include "ffn_bf16.h"
#include "split_price.h"
#include "wave_ops.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int KPAD = 8;   // row-major token tile: LDS pitch (BKT+8)*2 B keeps b128 reads conflict-free

constexpr int XCDS = 8;   // MI355X: 8 accelerator dies, each with a private L2

// ---------------------------------------------------------------------------
// Work enumeration of the tiled kernel.  A work item is (row tile, feature
// tile); the row tiles of all slots form one list in slot order, ceil(len/bt)
// per slot.  Workgroups are dealt to the 8 XCDs round-robin by their linear id,
// so workgroup wg runs on XCD wg % 8.  The items are numbered slot by slot --
// inside a slot with the feature tile fastest (second product: g = mt * ftiles
// + ft) or with the row tile fastest (first product, see the kernel) -- and die
// x owns the x-th eighth of that list: the dies' shares differ by at most one
// item (a split by whole row tiles can leave one die with a fifth more work and
// a whole extra round of tiles) and a share still covers few slots, whose
// token or weight tiles the die's workgroups share through its L2.  The grid
// holds as many workgroups as the chip keeps resident; the j-th workgroup of a
// die takes the die's items j, j + n, j + 2n, ... (n workgroups per die).  Each
// workgroup builds the per-slot tables once, in LDS.
constexpr int MAX_SLOTS = 256;            // K <= E <= 256 by the C ABI

struct ItemMap {
    int first[MAX_SLOTS + 1];             // row tiles before slot k; [nslots] = all row tiles
    int pad[MAX_SLOTS];                   // padded rows (segments re-based to multiples of 32) before slot k
    int a[MAX_SLOTS], b[MAX_SLOTS];       // clamped segment bounds
};

// Called by every thread of the workgroup; ends with a barrier.
__device__ __forceinline__ void build_item_map(ItemMap& m, const int32_t* __restrict__ offsets, int nslots,
                                               int T, int bt) {
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        int tiles_before = 0, pad_before = 0;
        for (int base = 0; base < nslots; base += 64) {
            const int k = base + lane;
            int a = 0, b = 0, tiles = 0, pad = 0;
            if (k < nslots) {
                a = min(max(offsets[k], 0), T);                 // clamps guard misuse
                b = max(min(max(offsets[k + 1], 0), T), a);
                tiles = (b - a + bt - 1) / bt;
                pad = (b - a + 31) & ~31;
            }
            const int tin = smoe_wave_incl_scan(tiles), pin = smoe_wave_incl_scan(pad);
            if (k < nslots) {
                m.first[k] = tiles_before + tin - tiles;
                m.pad[k] = pad_before + pin - pad;
                m.a[k] = a;
                m.b[k] = b;
            }
            tiles_before += __shfl(tin, 63);
            pad_before += __shfl(pin, 63);
        }
        if (lane == 0) m.first[nslots] = tiles_before;
    }
    __syncthreads();
}

// Row tile mt of the global list: its slot, first row, segment end and padded
// first row.  Every wave works this out for itself; the results are scalars.
__device__ __forceinline__ void row_tile_at(const ItemMap& m, int nslots, int bt, int mt, int& slot, int& m0,
                                            int& m_end, int& pm0) {
    const int lane = threadIdx.x & 63;
    int nle = 0;                                               // slots whose first row tile is <= mt
    for (int base = 0; base < nslots; base += 64) {
        const int k = base + lane;
        nle += __popcll(__ballot(k < nslots && m.first[k] <= mt));
    }
    const int k = __builtin_amdgcn_readfirstlane(nle - 1);     // the last of them holds mt (empty slots repeat the next first)
    const int within = mt - __builtin_amdgcn_readfirstlane(m.first[k]);
    slot = k;
    m0 = __builtin_amdgcn_readfirstlane(m.a[k]) + within * bt;
    m_end = __builtin_amdgcn_readfirstlane(m.b[k]);
    pm0 = __builtin_amdgcn_readfirstlane(m.pad[k]) + within * bt;
}

__device__ __forceinline__ bf16x8 as_frag(uint4 v) {
    union { uint4 u; bf16x8 b; } c;
    c.u = v;
    return c.b;
}

__device__ __forceinline__ void apply_gate(float& v0, float& v1, float& v2, float& v3, float g,
                                           const uint16_t* res, bool fused) {
    if (fused) smoe_apply_gate(v0, v1, v2, v3, g, res ? *(const uint2*)res : make_uint2(0, 0), res != nullptr);
}

// One workgroup tile with NBF live token blocks.  Everything is compile-time
// shaped: no branch inside the reduction loop.
//   AF    feature blocks per wave          NW    waves per workgroup
//   BKT   reduction slice per LDS stage    PD    weight prefetch distance in slices
//   XFRAG token operand X is in fragment order (else row-major [T, R])
//   YFRAG output Y is written in fragment order (else row-major [T, N])
//   PAST  fragment-order output goes past the caches if fz.past
template <int AF, int NBF, int NW, int BKT, int PD, bool XFRAG, bool YFRAG, bool RELU, bool PAST>
__device__ __forceinline__ void run_tile(const uint16_t* __restrict__ X, const uint4* __restrict__ Wp,
                                         uint16_t* __restrict__ Y, int R, int N, int slot, int m0,
                                         int m_end, int pm0, int ftile, uint16_t* xs, int stage_elems,
                                         int* orow, float* ogate, const FuseArgs fz) {
    constexpr int THREADS = NW * 64;
    constexpr int KS = BKT / 16;
    constexpr int LDR = BKT + KPAD;
    constexpr int CPR = BKT / 8;                          // 16-byte pieces per token row and slice
    constexpr int PIECES = 32 * NBF * CPR;                // pieces of the token tile per slice
    constexpr int CPT = (PIECES + THREADS - 1) / THREADS;

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int nfb = N >> 5, nrb = R >> 4;
    const int fb0 = (ftile * NW + wave) * AF;
    const int nchunks = R / BKT;

    const uint4* wbase[AF];
#pragma unroll
    for (int a = 0; a < AF; ++a) {
        int fb = min(fb0 + a, nfb - 1);                   // surplus blocks recompute the last one, unstored
        wbase[a] = Wp + ((size_t)slot * nfb + fb) * nrb * 64 + lane;
    }
    // this thread's pieces of the token tile: global source, its stride per slice, LDS destination
    const uint16_t* tsrc[CPT];
    int tdst[CPT];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        int idx = min(tid + i * THREADS, PIECES - 1);     // surplus threads repeat the last piece
        if (XFRAG) {
            int b = idx / (CPR * 32), j = (idx / 32) % CPR, t = idx % 32;
            tsrc[i] = X + (((size_t)((pm0 >> 5) + b) * (R >> 3) + j) * 32 + t) * 8;
            tdst[i] = idx * 8;
        } else {
            int r = idx / CPR, c = idx % CPR;
            int row = min(m0 + r, m_end - 1);
            if (fz.perm) row = fz.perm[row];
            tsrc[i] = X + (size_t)row * R + c * 8;
            tdst[i] = r * LDR + c * 8;
        }
    }
    const size_t tstep = XFRAG ? (size_t)CPR * 32 * 8 : (size_t)BKT;     // elements per slice
    // this lane's operand inside token block 0, reduction step 0; per block / per step strides
    const int xoff = XFRAG ? ((lane >> 5) * 32 + (lane & 31)) * 8 : (lane & 31) * LDR + (lane >> 5) * 8;
    constexpr int XB = XFRAG ? CPR * 32 * 8 : 32 * LDR;   // token block stride in LDS
    constexpr int XK = XFRAG ? 2 * 32 * 8 : 16;           // reduction step stride in LDS

    // Row-major output: where each row of the tile goes (out[perm[row]] in the single-call
    // path, y_perm[row] otherwise; -1 past the segment's end) and its gate are fetched now,
    // a whole reduction before the epilogue needs them.
    if (!YFRAG) {
        for (int r = tid; r < 32 * NBF; r += THREADS) {
            int dst = -1;
            float g = 1.f;
            if (m0 + r < m_end) {
                dst = fz.perm ? fz.perm[m0 + r] : m0 + r;
                if (fz.perm) g = fz.gate[dst];
            }
            orow[r] = dst;
            ogate[r] = g;
        }
    }

    f32x16 acc[AF][NBF];
#pragma unroll
    for (int a = 0; a < AF; ++a)
#pragma unroll
        for (int b = 0; b < NBF; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

    // Software pipeline over the reduction slices c = 0 .. nchunks-1.
    //   weights: a ring of PD+1 slices in registers, loaded PD slices ahead;
    //   tokens:  TD register sets, loaded TD+1 slices ahead, written to LDS one
    //            slice ahead; LDS holds three stages (slice c in stage c % 3);
    //   operands: the next MFMA step's LDS reads are issued before the current
    //            step's MFMAs, across the slice boundary as well.
    // The one barrier per slice sits in the MIDDLE of the slice's MFMA steps: it
    // publishes stage (c+1)%3, written at the top of slice c, before the first
    // read of it at the bottom of slice c, and it orders the last reads of slice
    // c-1 (all issued before it) ahead of the writes that recycle that stage at
    // the top of slice c+1.  So no wave ever waits at a barrier with an empty
    // matrix pipe behind it.
    // Loads past the last slice are clamped to it (fetched again, never used),
    // so the loop body has no conditional loads.
    constexpr int TD = PD & 1 ? 2 : 1;
    static_assert(KS % 2 == 0, "the operand double buffer assumes an even number of steps per slice");
    uint4 tregA[CPT], tregB[CPT];                       // token register sets 0 and 1
    uint4 wbuf[PD + 1][KS][AF];
    bf16x8 xf[2][NBF];
#pragma unroll
    for (int i = 0; i < CPT; ++i) tregA[i] = *(const uint4*)tsrc[i];
#pragma unroll
    for (int p = 0; p < PD; ++p) {
        const int cp = min(p, nchunks - 1);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int a = 0; a < AF; ++a) wbuf[p][ks][a] = wbase[a][(size_t)(cp * KS + ks) * 64];
    }
    if (TD == 2) {
        const int c1 = min(1, nchunks - 1);
#pragma unroll
        for (int i = 0; i < CPT; ++i) tregB[i] = *(const uint4*)(tsrc[i] + (size_t)c1 * tstep);
    }
#pragma unroll
    for (int i = 0; i < CPT; ++i) *(uint4*)&xs[tdst[i]] = tregA[i];
    {   // set 0 is free again: it takes slice TD (the slice after the ones already loaded)
        const int c2 = min(TD, nchunks - 1);
#pragma unroll
        for (int i = 0; i < CPT; ++i) tregA[i] = *(const uint4*)(tsrc[i] + (size_t)c2 * tstep);
    }
    __syncthreads();
    // Row-major output, single-call path: the residual rows come from far away by now (two
    // weight streams have passed through the caches since x was read), so their pieces are asked for
    // here and carried through the reduction in registers.
    constexpr int OF = NW * AF * 32;                      // features of the workgroup tile
    constexpr int OCPR = OF / 8;                          // 16-byte pieces per output row
    constexpr int ONP = YFRAG ? 1 : 32 * NBF * OCPR / THREADS;   // pieces per thread (2 * NBF * AF)
    uint4 res[ONP];
    if (!YFRAG && fz.perm && fz.residual) {
#pragma unroll
        for (int i = 0; i < ONP; ++i) {
            const int idx = tid + i * THREADS, r = idx / OCPR, c = idx % OCPR;
            const int col = ftile * OF + c * 8, row = col < N ? orow[r] : -1;
            res[i] = make_uint4(0, 0, 0, 0);
            if (row >= 0) res[i] = *(const uint4*)(fz.residual + (size_t)row * N + col);
        }
    }
#pragma unroll
    for (int b = 0; b < NBF; ++b) xf[0][b] = as_frag(*(const uint4*)&xs[xoff + b * XB]);

    int st = 0;                                           // LDS stage of the current slice
    // nchunks is a multiple of PD+1 (the launcher picks PD so; PD is 0, 1 or 3),
    // and every ring index below is a compile-time constant.
    auto slice = [&](auto uc, int c0) {
        constexpr int u = decltype(uc)::value;            // position in the ring: compile-time
        const int c = c0 + u;
        const int cw = min(c + PD, nchunks - 1), ct = min(c + TD + 1, nchunks - 1);
        const int st1 = st == 2 ? 0 : st + 1;
        const uint16_t* tile = xs + st * stage_elems + xoff;
        const uint16_t* tile1 = xs + st1 * stage_elems + xoff;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int a = 0; a < AF; ++a)
                wbuf[(u + PD) % (PD + 1)][ks][a] = wbase[a][(size_t)(cw * KS + ks) * 64];
        // the set that holds slice c+1 goes to stage (c+1)%3 and is reloaded with slice c+TD+1
        uint16_t* dst = xs + st1 * stage_elems;
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            if constexpr ((u + 1) % TD == 0) *(uint4*)&dst[tdst[i]] = tregA[i];
            else *(uint4*)&dst[tdst[i]] = tregB[i];
        }
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            uint4 v = *(const uint4*)(tsrc[i] + (size_t)ct * tstep);
            if constexpr ((u + 1) % TD == 0) tregA[i] = v; else tregB[i] = v;
        }
        __builtin_amdgcn_sched_barrier(0);                // keep the prefetches ahead of the math
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks == KS / 2) __syncthreads();            // stage (c+1)%3 is complete from here on
            {   // operands of the next reduction step, or of the next slice's first
                const uint16_t* src = (ks + 1 == KS ? tile1 : tile) + (ks + 1) % KS * XK;
#pragma unroll
                for (int b = 0; b < NBF; ++b) xf[(ks + 1) & 1][b] = as_frag(*(const uint4*)&src[b * XB]);
            }
            __builtin_amdgcn_sched_barrier(0);            // next step's operands are on their way
#pragma unroll
            for (int b = 0; b < NBF; ++b)
#pragma unroll
                for (int a = 0; a < AF; ++a)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(wbuf[u][ks][a]), xf[ks & 1][b], acc[a][b], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        st = st1;
    };
    for (int c0 = 0; c0 < nchunks; c0 += PD + 1) {
        slice(std::integral_constant<int, 0>{}, c0);
        if constexpr (PD >= 1) slice(std::integral_constant<int, 1>{}, c0);
        if constexpr (PD >= 3) {
            slice(std::integral_constant<int, 2>{}, c0);
            slice(std::integral_constant<int, 3>{}, c0);
        }
    }
    __syncthreads();                                      // the next tile's first write may hit any stage

    // accumulator register i of lane l: feature 8*(i/4) + 4*(l/32) + i%4, token l%32
    if constexpr (YFRAG) {   // unit [(pm0/32 + b)][(fb0+a)*4 + g][lane%32], 8 bytes at half (lane/32)
#pragma unroll
        for (int a = 0; a < AF; ++a) {
            if (fb0 + a >= nfb) continue;
#pragma unroll
            for (int b = 0; b < NBF; ++b) {
                uint16_t* ydst = Y + (((size_t)((pm0 >> 5) + b) * (N >> 3) + (fb0 + a) * 4) * 32 + (lane & 31)) * 8 +
                                 (lane >> 5) * 4;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    float v0 = acc[a][b][4 * g], v1 = acc[a][b][4 * g + 1], v2 = acc[a][b][4 * g + 2],
                          v3 = acc[a][b][4 * g + 3];
                    if (RELU) { v0 = fmaxf(v0, 0.f); v1 = fmaxf(v1, 0.f); v2 = fmaxf(v2, 0.f); v3 = fmaxf(v3, 0.f); }
                    uint2 o;
                    o.x = smoe_pack_bf16(v0, v1);
                    o.y = smoe_pack_bf16(v2, v3);
                    if (PAST && fz.past) smoe_store_stream((uint2*)(ydst + g * 32 * 8), o);
                    else *(uint2*)(ydst + g * 32 * 8) = o;
                }
            }
        }
    } else {
        // Row-major output.  In the accumulator layout a store instruction would touch 32 rows
        // with 8 bytes each; the tile is turned through LDS instead (the ring is idle now), so
        // that 16 lanes write one row's 256 contiguous bytes.  The product is rounded to bf16
        // on the way in -- the value the plain path stores, and the one the fused path scales
        // by the gate (+ residual) in fp32 before its single final rounding.
        constexpr int F = OF, CPR8 = OCPR, NP = ONP;
        constexpr int LDO = F + 4;                        // LDS row pitch in elements (8-byte aligned rows)
        static_assert(32 * NBF * CPR8 % THREADS == 0, "pieces divide evenly");
#pragma unroll
        for (int a = 0; a < AF; ++a)
#pragma unroll
            for (int b = 0; b < NBF; ++b)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    float v0 = acc[a][b][4 * g], v1 = acc[a][b][4 * g + 1], v2 = acc[a][b][4 * g + 2],
                          v3 = acc[a][b][4 * g + 3];
                    if (RELU) { v0 = fmaxf(v0, 0.f); v1 = fmaxf(v1, 0.f); v2 = fmaxf(v2, 0.f); v3 = fmaxf(v3, 0.f); }
                    uint2 o;
                    o.x = smoe_pack_bf16(v0, v1);
                    o.y = smoe_pack_bf16(v2, v3);
                    *(uint2*)&xs[(b * 32 + (lane & 31)) * LDO + (wave * AF + a) * 32 + g * 8 + (lane >> 5) * 4] = o;
                }
        __syncthreads();
        const bool fused = fz.perm != nullptr, has_res = fused && fz.residual != nullptr;
        const int col0 = ftile * F;
        int prow[NP], pcol[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) {                    // every row first: one trip to LDS for all of them
            const int idx = tid + j * THREADS, r = idx / CPR8, c = idx % CPR8;
            pcol[j] = col0 + c * 8;
            prow[j] = pcol[j] < N ? orow[r] : -1;
        }
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            if (prow[j] < 0) continue;
            const int idx = tid + j * THREADS, r = idx / CPR8, c = idx % CPR8;
            const uint2 lo = *(const uint2*)&xs[r * LDO + c * 8], hi = *(const uint2*)&xs[r * LDO + c * 8 + 4];
            uint4 o = make_uint4(lo.x, lo.y, hi.x, hi.y);
            if (fused) o = smoe_gate_unit(o, ogate[r], res[j], has_res);
            *(uint4*)(Y + (size_t)prow[j] * N + pcol[j]) = o;
        }
        __syncthreads();                                  // the next tile's prologue reuses the ring
    }
}

template <int AF, int NBF, int MAXB, int NW, int BKT, int PD, bool XFRAG, bool YFRAG, bool RELU>
struct TileSwitch {
    static __device__ __forceinline__ void go(int nbf, const uint16_t* X, const uint4* Wp, uint16_t* Y, int R,
                                              int N, int slot, int m0, int m_end, int pm0, int ftile,
                                              uint16_t* xs, int* orow, float* ogate, const FuseArgs fz) {
        constexpr int stage = MAXB * 32 * (BKT + KPAD);
        if (nbf == NBF)
            run_tile<AF, NBF, NW, BKT, PD, XFRAG, YFRAG, RELU, (MAXB <= 2)>(X, Wp, Y, R, N, slot, m0, m_end, pm0, ftile, xs,
                                                               stage, orow, ogate, fz);
        else if constexpr (NBF > 1)
            TileSwitch<AF, NBF - 1, MAXB, NW, BKT, PD, XFRAG, YFRAG, RELU>::go(nbf, X, Wp, Y, R, N, slot, m0,
                                                                              m_end, pm0, ftile, xs, orow, ogate, fz);
    }
};

// FIRST = the d_model -> d_ff product: row-major x_perm in, ReLU, fragment-order h out.
// Otherwise the d_ff -> d_model product: fragment-order h in, row-major y_perm out.
// Persistent workgroups (see the enumeration above).
template <int AF, int MAXB, int NW, int BKT, int PD, int OCC, bool FIRST>
__global__ __launch_bounds__(NW * 64, OCC) void grouped_gemm_bf16(
    const uint16_t* __restrict__ X, const uint4* __restrict__ Wp, const int32_t* __restrict__ offsets,
    int nslots, int T, uint16_t* __restrict__ Y, int R, int N, const FuseArgs fz) {
    // the ring of token stages; the second product's epilogue turns its output tile through it
    constexpr int RING = 3 * MAXB * 32 * (BKT + KPAD), OUT_TILE = FIRST ? 0 : MAXB * 32 * (NW * AF * 32 + 4);
    __shared__ __align__(16) uint16_t xs[RING > OUT_TILE ? RING : OUT_TILE];
    __shared__ int s_orow[MAXB * 32];
    __shared__ float s_ogate[MAXB * 32];
    __shared__ ItemMap map;
    constexpr int BT = MAXB * 32;
    const int ftiles = ((N >> 5) + NW * AF - 1) / (NW * AF);
    build_item_map(map, offsets, nslots, T, BT);
    const long long G = (long long)__builtin_amdgcn_readfirstlane(map.first[nslots]) * ftiles;
    const int die = blockIdx.x % XCDS, nwg = gridDim.x / XCDS;   // the grid is a multiple of 8
    const long long lo = G * die / XCDS;
    const int cnt = (int)(G * (die + 1) / XCDS - lo);
    for (int j = blockIdx.x / XCDS; j < cnt; j += nwg) {
        const long long g = lo + j;
        int mt = (int)(g / ftiles), ftile = (int)(g % ftiles);
        int slot, m0, m_end, pm0;
        row_tile_at(map, nslots, BT, mt, slot, m0, m_end, pm0);
        if (FIRST) {
            // First product: inside a slot the items are numbered (feature tile, row tile) with the
            // row tile fastest.  A die's share of a large slot is then a range of feature tiles over
            // ALL the slot's rows, so no weight tile is fetched by two dies (the slot's token rows,
            // a quarter of the bytes, are what two dies may both read), and the workgroups that run
            // together read the same weight tile.  Measured on the Switch-base-64 shape: the L2s
            // request 93 MB per launch instead of 126 MB (the weights and tokens alone are 82 MB).
            // The second product keeps the row-tile-major numbering: its token tile (the hidden
            // activations of 128 rows) is as large as its weight tile, and the other order fetched
            // 15 % more at the Switch-large shape.
            const int first_k = __builtin_amdgcn_readfirstlane(map.first[slot]);
            const int tiles_k = __builtin_amdgcn_readfirstlane(map.first[slot + 1]) - first_k;
            const int local = (int)(g - (long long)first_k * ftiles);
            ftile = local / tiles_k;
            mt = first_k + (local - ftile * tiles_k);
            row_tile_at(map, nslots, BT, mt, slot, m0, m_end, pm0);
        }
        if (fz.phys) slot = __builtin_amdgcn_readfirstlane(fz.phys[slot]);   // from here on: where the weights live
        const int nbf = min(MAXB, (m_end - m0 + 31) >> 5);    // token blocks that hold real rows
        TileSwitch<AF, MAXB, MAXB, NW, BKT, PD, !FIRST, FIRST, FIRST>::go(nbf, X, Wp, Y, R, N, slot, m0, m_end,
                                                                         pm0, ftile, xs, s_orow, s_ogate, fz);
    }
}

// ---------------------------------------------------------------------------
// Small-batch (decode) variant: row tiles of 32 tokens, nothing but weight
// streaming.  With a handful of tokens per slot the FFN is bound by reading
// each active slot's weights once, so the kernel is built around keeping many
// 1-KiB weight loads in flight: no LDS staging and no barrier in the loop --
// the token operand (32 rows) is read straight from L2 -- and the operands of
// G reduction steps are fetched together, two groups in flight per wave.
// A workgroup of NWV waves covers NWV / KSPLIT neighbouring feature blocks;
// the KSPLIT waves that share a feature block split its reduction and meet in
// LDS at the end (added in wave order: reproducible).  Splitting shortens the
// stream each wave has to pull through its own queue of loads, which is what
// bounds a wave's share of the HBM bandwidth.
// Workgroup b serves (slot b / ftiles, feature tile b % ftiles): it knows its
// weights before it knows whether the slot has any tokens, so the first group
// of weight loads is issued ahead of the read of the offsets and the latency of
// the two overlaps; the workgroup of an empty slot then simply leaves.  That is
// a slot's first 32 rows.  The further row tiles of all slots are numbered
// through -- at most T / 32 of them -- and have workgroups behind those: one
// that worked off its slot 32 rows at a time streamed the same weights over and
// over while the others had left.  us per layer, before and after, with four
// fifths of the tokens alike: 4 slots of 768 x 3072, T = 170 42.5 / 27.8; 16
// slots, T = 200 64.3 / 50.9; 128 slots, T = 700 326 / 181; clustered tokens: 4
// slots, T = 200 38.9 / 28.0, of 1024 x 4096 51.9 / 40.1.  Two workgroups to a
// compute unit: a third, for which there are registers, gains 5 % on 32 slots
// (T = 180 73 / 69) and costs 4 % on 64 and 128 (T = 64 84.7 / 88.8) and 8 % on 4.
template <int NWV, int KSPLIT, bool FIRST>
__global__ __launch_bounds__(NWV * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void small_gemm_bf16(
    const uint16_t* __restrict__ X, const uint4* __restrict__ Wp, const int32_t* __restrict__ offsets,
    int nslots, int T, uint16_t* __restrict__ Y, int R, int N, const FuseArgs fz) {
    constexpr int G = 8;                                   // reduction steps fetched together
    constexpr int FBW = NWV / KSPLIT;                      // feature blocks per workgroup
    constexpr bool XFRAG = !FIRST, YFRAG = FIRST, RELU = FIRST;
    __shared__ __align__(16) float red[KSPLIT > 1 ? (KSPLIT - 1) * FBW * 16 * 64 : 1];
    const int nfb = N >> 5, nrb = R >> 4;
    const int ftiles = (nfb + FBW - 1) / FBW;
    const int item = blockIdx.x / ftiles, ftile = blockIdx.x % ftiles;
    const int extra = item - nslots;                       // >= 0: which of the further row tiles
    // the wave index as a scalar: the reduction range below must be wave-uniform in the
    // compiler's eyes too, because an MFMA under a lane mask still runs for every lane
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int fbi = wave / KSPLIT, part = wave % KSPLIT;   // feature block in the workgroup, share of the reduction
    const int fb = ftile * FBW + fbi;
    const bool fb_ok = fb < nfb;
    const int per = (nrb + KSPLIT - 1) / KSPLIT;
    const int kb_lo = min(part * per, nrb), kb_hi = min(kb_lo + per, nrb);
    auto weights_of = [&](int slot) {
        return Wp + ((size_t)(fz.phys ? fz.phys[slot] : slot) * nfb + min(fb, nfb - 1)) * nrb * 64 + lane;
    };
    int slot = min(item, nslots - 1);
    const uint4* wp = weights_of(slot);

    uint4 wA[G], xA[G], wB[G], xB[G];
    auto fetch_w = [&](uint4 (&w)[G], int g0) {
#pragma unroll
        for (int i = 0; i < G; ++i) w[i] = wp[(size_t)max(min(g0 + i, kb_hi - 1), 0) * 64];   // past the end: reloaded, not used
    };
    if (extra < 0) fetch_w(wA, kb_lo);                     // on its way before anything else is known

    // this slot's rows and the padded rows before it (segments re-based to multiples of 32)
    int seg_a = 0, seg_b = 0, pad_before = 0, more_before = 0, tile = 0;
    for (int base = 0; base < nslots; base += 64) {
        const int k = base + lane;
        int a = 0, b = 0;
        if (k < nslots) {
            a = min(max(offsets[k], 0), T);                 // clamps guard misuse
            b = max(min(max(offsets[k + 1], 0), T), a);
        }
        const int pad = (b - a + 31) & ~31;
        const int pin = smoe_wave_incl_scan(pad);
        int at = item - base;                              // this workgroup's lane of the chunk, if it is one of its lanes
        if (extra >= 0) {
            const int more = max((pad >> 5) - 1, 0), upto = smoe_wave_incl_scan(more);
            const unsigned long long past = __ballot(more_before + upto > extra);
            at = past ? __ffsll(past) - 1 : 64;
            tile = extra - more_before - __shfl(upto - more, at & 63) + 1;
            more_before += __shfl(upto, 63);
        }
        if (at < 64) {
            slot = base + at;
            seg_a = __shfl(a, at);
            seg_b = __shfl(b, at);
            pad_before += __shfl(pin - pad, at);
            break;
        }
        pad_before += __shfl(pin, 63);
    }
    seg_a = __builtin_amdgcn_readfirstlane(seg_a);
    seg_b = __builtin_amdgcn_readfirstlane(seg_b);
    pad_before = __builtin_amdgcn_readfirstlane(pad_before);
    if (seg_b <= seg_a) return;                            // nothing routed to this slot, or no further row tile
    if (extra >= 0) {
        slot = __builtin_amdgcn_readfirstlane(slot);
        tile = __builtin_amdgcn_readfirstlane(tile);
        wp = weights_of(slot);
        fetch_w(wA, kb_lo);
    }

    const int m0 = seg_a + 32 * tile, m_end = seg_b, pm0 = pad_before + 32 * tile;
    const uint4* xp;                                   // this lane's token operand at reduction step 0
    size_t xstep;                                      // in uint4 units per reduction step
    if (XFRAG) {
        xp = (const uint4*)X + ((size_t)(pm0 >> 5) * (R >> 3) + (lane >> 5)) * 32 + (lane & 31);
        xstep = 2 * 32;
    } else {
        int row = min(m0 + (lane & 31), m_end - 1);
        if (fz.perm) row = fz.perm[row];
        xp = (const uint4*)(X + (size_t)row * R + (lane >> 5) * 8);
        xstep = 2;
    }
    auto fetch_x = [&](uint4 (&xv)[G], int g0) {
#pragma unroll
        for (int i = 0; i < G; ++i) xv[i] = xp[(size_t)max(min(g0 + i, kb_hi - 1), 0) * xstep];
    };
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    auto consume = [&](uint4 (&w)[G], uint4 (&xv)[G], int g0) {
#pragma unroll
        for (int i = 0; i < G; ++i) {
            // steps past the end of the range multiply by a zero token operand
            const uint4 xz = g0 + i < kb_hi ? xv[i] : make_uint4(0, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(w[i]), as_frag(xz), acc, 0, 0, 0);
        }
    };
    // two groups of G reduction steps are always in flight: while one group's
    // MFMAs run, the next group's operands are already on their way
    fetch_x(xA, kb_lo);
    for (int g0 = kb_lo; g0 < kb_hi; g0 += 2 * G) {
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
    if (KSPLIT > 1) {
        if (part > 0) {
#pragma unroll
            for (int i = 0; i < 16; ++i) red[(((part - 1) * FBW + fbi) * 16 + i) * 64 + lane] = acc[i];
        }
        __syncthreads();
        if (part == 0) {
#pragma unroll
            for (int w2 = 0; w2 < KSPLIT - 1; ++w2)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[i] += red[((w2 * FBW + fbi) * 16 + i) * 64 + lane];
        }
    }
    if (part > 0 || !fb_ok) return;
    // accumulator register i of lane l: feature 8*(i/4) + 4*(l/32) + i%4, token l%32
    uint16_t* ydst;
    const uint16_t* rsrc = nullptr;
    float gmul = 1.f;
    if (YFRAG) {
        ydst = Y + (((size_t)(pm0 >> 5) * (N >> 3) + fb * 4) * 32 + (lane & 31)) * 8 + (lane >> 5) * 4;
    } else {
        int row = m0 + (lane & 31);
        if (row >= m_end) return;
        if (fz.perm) {
            row = fz.perm[row];
            gmul = fz.gate[row];
            if (fz.residual) rsrc = fz.residual + (size_t)row * N + fb * 32 + (lane >> 5) * 4;
        }
        ydst = Y + (size_t)row * N + fb * 32 + (lane >> 5) * 4;
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        float v0 = acc[4 * g], v1 = acc[4 * g + 1], v2 = acc[4 * g + 2], v3 = acc[4 * g + 3];
        if (!YFRAG) apply_gate(v0, v1, v2, v3, gmul, rsrc ? rsrc + g * 8 : nullptr, fz.perm != nullptr);
        if (RELU) { v0 = fmaxf(v0, 0.f); v1 = fmaxf(v1, 0.f); v2 = fmaxf(v2, 0.f); v3 = fmaxf(v3, 0.f); }
        uint2 o;
        o.x = smoe_pack_bf16(v0, v1);
        o.y = smoe_pack_bf16(v2, v3);
        *(uint2*)(ydst + (YFRAG ? g * 32 * 8 : g * 8)) = o;
    }
}

template <int NWV, int KSPLIT, bool FIRST>
void launch_small(const uint16_t* X, const void* Wp, const int32_t* offsets, int nslots, uint16_t* Y, int R,
                  int N, int T, const FuseArgs& fz, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    constexpr int FBW = NWV / KSPLIT;
    int nfb = N >> 5;
    int ftiles = (nfb + FBW - 1) / FBW;
    // one workgroup per (slot, feature tile), and as many further row tiles as T tokens can need
    dim3 grid((nslots + T / 32) * ftiles);
    smoe_launch_timed(small_gemm_bf16<NWV, KSPLIT, FIRST>, grid, dim3(NWV * 64), s, e0, e1, X, (const uint4*)Wp,
                      offsets, nslots, T, Y, R, N, fz);
}

// Compute units per die, asked of the runtime once.
int cus_per_die() {
    static int n = 0;
    if (n == 0) {
        int dev = 0, cus = 0;
        (void)hipGetDevice(&dev);
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < XCDS) {
            (void)hipGetLastError();
            cus = 256;
        }
        n = cus / XCDS;
    }
    return n;
}

template <int AF, int MAXB, int NW, int BKT, int PD, int OCC, bool FIRST>
void launch_gemm(const uint16_t* X, const void* Wp, const int32_t* offsets, int nslots, uint16_t* Y,
                 int R, int N, int T, const FuseArgs& fz, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    constexpr int BT = 32 * MAXB;
    const int mtiles = (T + BT - 1) / BT + nslots;         // upper bound on the row tiles of all slots
    const int ftiles = ((N >> 5) + NW * AF - 1) / (NW * AF);
    const long long items = (long long)mtiles * ftiles;
    // as many workgroups as the chip holds at once (OCC waves per SIMD), or fewer if the items run out
    const int resident = cus_per_die() * std::max(1, OCC * 4 / NW);
    const int per_die = (int)std::min<long long>((items + XCDS - 1) / XCDS, resident);
    dim3 grid(XCDS * std::max(per_die, 1));
    if ((R / BKT) % (PD + 1) == 0)
        smoe_launch_timed(grouped_gemm_bf16<AF, MAXB, NW, BKT, PD, OCC, FIRST>, grid, dim3(NW * 64), s, e0, e1, X,
                          (const uint4*)Wp, offsets, nslots, T, Y, R, N, fz);
    else   // slice count not a multiple of the ring length: same tile without weight prefetch
        smoe_launch_timed(grouped_gemm_bf16<AF, MAXB, NW, BKT, 0, OCC, FIRST>, grid, dim3(NW * 64), s, e0, e1, X,
                          (const uint4*)Wp, offsets, nslots, T, Y, R, N, fz);
}

// The kernels launch_variant knows; every one of them is chosen somewhere by pick_variants.
constexpr bool is_variant(int v) {
    return v == 1 || v == 3 || v == 4 || v == 5 || v == 6 || v == 8 || v == 9 || v == 10 || v == 11;
}

// What stands in where a kernel does not serve a product, as only a pair forced by hand can ask: the tiles of 64 and 32 rows (3, 4)
// are the first product's and the splitting kernel (11) the second's, which has it in their place; the ring kernel (9, 10) does not
// apply everywhere.
int standing_in(int v, bool first, int R, int T) {
    if (first && v == 11) return 1;
    if (!first && (v == 3 || v == 4)) return 11;
    if (v < 9 || v == 11 || smoe_ring_applies(first, R, T)) return v;
    return v == 9 ? 1 : 8;
}

template <bool FIRST>
int launch_variant(int v, const uint16_t* X, const void* Wp, const int32_t* offsets, int nslots,
                    uint16_t* Y, int R, int N, int T, const FuseArgs& fz, hipStream_t s, hipEvent_t e0,
                    hipEvent_t e1) {
    v = standing_in(v, FIRST, R, T);
    if (v == 11) return smoe_launch_split(X, Wp, offsets, nslots, Y, R, N, T, fz, cus_per_die(), s, e0, e1);
    if (v >= 9) return smoe_launch_ring(v == 9 ? 4 : 8, FIRST, X, Wp, offsets, nslots, Y, R, N, T, fz, cus_per_die(), s, e0, e1);
    if (R % 64 != 0 && v != 5 && v != 6) {   // d_model / d_ff are multiples of 32 by contract: 32-deep slices always fit
        launch_gemm<1, 4, 4, 32, 1, 2, FIRST>(X, Wp, offsets, nslots, Y, R, N, T, fz, s, e0, e1);
        return SMOE_OK;
    }
    // tokens x features of a workgroup  AF MAXB NW BKT PD OCC
    if (v == 1) launch_gemm<1, 4, 4, 64, 1, 2, FIRST>(X, Wp, offsets, nslots, Y, R, N, T, fz, s, e0, e1);        // 128 x 128
    else if (v == 8) launch_gemm<1, 4, 8, 64, 1, 2, FIRST>(X, Wp, offsets, nslots, Y, R, N, T, fz, s, e0, e1);   // 128 x 256, 8 waves
    else if (v == 5) launch_small<4, 1, FIRST>(X, Wp, offsets, nslots, Y, R, N, T, fz, s, e0, e1);               // 32 x 128, streaming
    else if (v == 6) launch_small<4, 4, FIRST>(X, Wp, offsets, nslots, Y, R, N, T, fz, s, e0, e1);               // 32 x 32, reduction split 4 ways
    else if constexpr (FIRST) {
        if (v == 3) launch_gemm<1, 2, 4, 64, 1, 4, FIRST>(X, Wp, offsets, nslots, Y, R, N, T, fz, s, e0, e1);    //  64 x 128
        else if (v == 4) launch_gemm<1, 1, 4, 64, 3, 4, FIRST>(X, Wp, offsets, nslots, Y, R, N, T, fz, s, e0, e1);   //  32 x 128
        else return smoe_fail(SMOE_EINVAL, "expert FFN: no first product %d", v);
    } else {
        return smoe_fail(SMOE_EINVAL, "expert FFN: no second product %d", v);
    }
    return SMOE_OK;
}

// Tile shape of the first product of a prefill batch, chosen by its predicted time: for every round of one item per compute
// unit the bytes of an item's weights and rows at the rate at which that tile takes them in.  A slot with x tiles' worth
// of tokens in the mean has about x + 1/2 tiles, and one where x is small.  The rates were fitted to 180 batches (13
// shapes from 4 slots of 256 x 768 to 32 of 1024 x 4096, T = 140 .. 6000, weights from HBM, every tile measured on each): the
// pick is 1.3 % slower than the best tile of each batch in the mean, where thresholds on the tokens per slot alone were 10 %
// slower.  us, those thresholds / this choice: 4 slots of 768 x 3072, T = 600 17.4 / 13.1; 16 of 768 x 2048, T = 4096 35.4 / 27.3.
int pick_first(int R, int N, int T, int K) {
    struct Rate { int v, rows, features; double gbs; };
    static constexpr Rate rates[] = {{4, 32, 128, 47.4}, {3, 64, 128, 56.7}, {1, 128, 128, 61.1}, {8, 128, 256, 48.4}};
    // slots of less than two blocks of rows: no wide tiles (each weight would pass through one compute
    // unit only, at the rate of cold lines: 16 slots of 1024 x 4096, T = 777 39.5, 31.0 with 128 features), and a count
    // that is nearer to the truth
    const bool thin = T / K < 60;
    const double cus = XCDS * cus_per_die();
    auto rounds = [&](int rows, int features) {
        const double x = (double)T / K / rows, tiles = K * (x + 0.5 + 0.5 * std::exp(-2 * x));
        return std::max(1.0, std::ceil(tiles * ((N + features - 1) / features) / cus - (thin ? 0.06 : 0.03)));
    };
    int best = 1;
    double least = 1e30;
    for (const Rate& r : rates) {
        if (thin && r.features > 128) continue;
        const double us = rounds(r.rows, r.features) * (r.rows + r.features) * 2e-3 * R / r.gbs;
        if (us < least) { least = us; best = r.v; }
    }
    if (!thin && smoe_ring_applies(true, R, T))
        for (int h = 1; h <= 8; ++h) {                     // the ring kernel chooses the height of its tiles
            const double us = -0.6 + rounds(32 * h, 256) * (256 + 32 * h) * 2e-3 * R / 38.4;
            if (us < least) { least = us; best = 10; }
        }
    return best;
}

// Kernel of the second product of a prefill batch, by predicted time likewise: tiled, ring, or splitting by the price that the kernel
// itself uses, with the expected number of tiles in the place of the counted.  Fitted to whole passes of 3720 batches, each of them with
// every kernel in turn (32 shapes from 2 slots of 768 x 3072 to 128 of 1024 x 4096, T = 130 .. 16384, clustered and even tokens,
// one layer alone and up to six): the pick takes 0.6 % more than the best of each batch in the mean, 3.8 % at the 95th percentile.
// us a layer with weights from memory, clustered tokens, splitting / 128 x 128 / 128 x 256 / large ring: 16 slots of 768 x 3072, T = 3000
// 78.0 / 80.1 / 92.1 / 93.6, T = 4000 86.5 / 84.9 / 97.6 / 97.8, T = 5500 105.4 / 105.3 / 103.5 / 108.4; 24 of 768 x 2048, T = 4500 87.3 / 90.5
// / 86.9 / 88.3; 128 of 1024 x 4096, T = 3000 411 / 402 / 398 / 398, T = 16384 615 / 596 / 584 / 560.
// Where the reduction is no multiple of 128 the tiled kernel has no weight prefetch, and the ring kernel stands for it (16 slots of 992
// x 3296, T = 800 77.0 and 42.6): its small tiles, two workgroups of them to a compute unit, while fewer than a hundred large ones
// exist (608 x 2912, T = 8000 44.5, 49.0 with large ones; 992 x 3296 70 with large ones, 96).
int pick_second(int R, int N, int T, int K) {
    struct Rate { int v, low, high, features, per_cu; double ends, slack, fixed, gbs; };   // heights in blocks of 32 rows
    static constexpr Rate rates[] = {{1, 4, 4, 128, 1, 0.48, 0, 2.3, 71.4}, {8, 4, 4, 256, 1, 0.48, 0, -1.0, 64.8},
                                     {9, 1, 4, 128, 2, 0.87, 0.19, 2.4, 39.7}, {10, 1, 8, 256, 1, 0.21, 0.23, 0.6, 55.6}};
    const double cus = XCDS * cus_per_die();
    auto rounds = [&](int h, int features, double n, double ends, double slack) {
        const double x = (double)T / K / (32 * h), tiles = K * (x + ends + (1 - ends) * std::exp(-2 * x));
        return std::max(1.0, std::ceil(tiles * ((N + features - 1) / features) / n - slack));
    };
    int best = 11;
    double least = 1e30;
    for (int w = 1; w <= 4; ++w)
        for (int h = 1; h <= 4; ++h)
            least = std::min(least, 2.2e-3 * smoe_split_price((float)rounds(h, 32 * w, cus, 0.57, 0.02), (float)((R + 63) / 64), w, h));
    const bool ring = smoe_ring_applies(false, R, T), whole = R % 128 == 0, many = (double)T * N / 65536 >= 100;
    for (const Rate& r : rates) {
        if (r.v == 1 || r.v == 8 ? ring && !whole : !ring || (r.v == 9 ? whole || many : !whole && !many)) continue;
        for (int h = r.low; h <= r.high; ++h) {
            const double us = r.fixed + rounds(h, r.features, cus * r.per_cu, r.ends, r.slack) * (r.features + 32 * h) * 2e-3 * R / r.gbs;
            if (us < least) { least = us; best = r.v; }
        }
    }
    return best;
}

// Where the ring kernel takes the first product in any case: 9 (at most 128 x 128) or 10 (at most 256 x 256), else 0.
//  * The reduction is no multiple of 128: the tiled kernel then has no weight prefetch.  us, tiled -> ring: 16 slots of
//    992 x 3296, T = 800 33.0 -> 29.8, T = 8000 107 -> 72; 11 of 416 x 1696, T = 800 12.5 -> 10.7.  With few tokens tiles of 64-deep
//    slices stay ahead (6 slots of 448 x 1280, T = 140 8.1, 9.2, T = 300 8.8, 9.4).  Under 6
//    tokens per slot the streaming kernel stays where rows are long and slots at most 64 (us per layer, streaming
//    / ring: 24 slots of 992 x 3296, T = 100 84 / 89, 48 T = 120 .. 264 2 .. 3 % ahead, 16 of 1184 x 4736 5 %; but 48 of 544 x
//    2176, T = 168 71 / 69, 128 of 928 x 3712, T = 192 1 .. 5 % behind).  The small tiles
//    serve where fewer than a hundred large ones exist.
//  * There are large tiles for the chip many times over, where the matrix products and the power they draw count
//    and not the bytes alone (128 x 128 tiles -> ring: 768 x 3072, T = 16384 108 -> 94; 32 slots of
//    1024 x 4096 190 -> 165; 16 of 768 x 2048 80 -> 68).
int ring_first(int R, int N, int T, int K, int tiled) {
    const double tiles = (double)T * N / 65536;            // full 256 x 256 tiles
    if (R % 128 != 0) {
        if ((tiled == 5 && R >= 900 && K <= 64) || (T / K < 60 && R % 64 == 0)) return 0;
        return tiles >= 100 ? 10 : 9;
    }
    return tiles >= 300 ? 10 : 0;
}

// Tile shapes for the two GEMMs.  A pair fixed at smoe_create (SMOE_FFN_VARIANT="v1,v2", a
// tuning aid; the indices are those of launch_variant) overrides the built-in choice.
void pick_variants(const smoe_layer* L, int T, int& v1, int& v2) {
    const int d = L->cfg.d_model, f = L->cfg.d_ff, K = L->cfg.K, per_slot = T / K;
    if (per_slot < 6) {                  // decode: a few tokens per slot, weight streaming
        v1 = 5;
        v2 = 6;
    } else {
        // The second product streams while its workgroups, one per 32 features and 32 rows of a slot, are little more than
        // the chip holds at once (two per compute unit): each then has a quarter of a reduction per wave in front of it,
        // where a tile has all of it.  Measured on 340 batches of 2 to 100 slots, T = 129 .. 2000, clustered and even tokens,
        // us per layer, streaming / best tile of the tiled kernel (the splitting kernel, which came later, is ahead of both on many of
        // them, 8 slots of 1024 x 4096, T = 400 55.5 / 47.9, and not yet part of this line).  700 workgroups: 25 .. 0 % ahead below (4
        // slots of 768 x 3072, T = 200 28 / 35; 6, T = 320 37 / 45; 4 of 2048 x 8192, T = 200 90 / 106), 3 % behind above (18 of 768 x 3072,
        // T = 668 69 / 67).  Under 28 tokens per slot, where most of a tile is empty, 780: 24 slots of 768 x 2048, T = 248 57.0 / 57.3, T = 400 54.9 / 53.4; 26 of 768 x
        // 3072, T = 263 71 / 69.  A long reduction makes the rounds of the tiles long, 850: 16 slots of 1024 x 4096, T = 300 73 / 76; 12
        // of 1280 x 5120, T = 300 88 / 93; 20 of 768 x 3072, T = 500 58.3 / 62.6 (even), 22 T = 480 66.7 / 66.1; but not with so few
        // tokens that the tiles are one round anyway (16 of 1280 x 5120, T = 160 104 / 101).
        // Not for short reductions, whose end the split lengthens (32 slots of 256 x 512, T = 260 23.5 / 22.4), and not for T = 640
        // and more, where the rows of the largest slots stream too often (one slot of 768 x 3072, T = 800 39.7 / 37.8).
        const int groups = (K + T / 32) * (d >> 5);
        const bool stream = T <= 512 && f >= 768 && groups <= (per_slot >= 28 ? 700 : per_slot >= 14 && f >= 3072 ? 850 : 780);
        v1 = d % 128 != 0 ? (per_slot < 28 ? 4 : 3) : pick_first(d, f, T, K);
        v2 = (f % 128 != 0 ? per_slot < 28 : stream) ? 6 : pick_second(f, d, T, K);
    }
    // the small-batch path of smoe_forward splits the second product's reduction four ways: the separate call does the
    // same, so that both give the same bits (the tiles of the first product all do)
    if (smoe_decode_first_applies(L, T)) {
        v2 = 6;
    } else {
        const int r1 = ring_first(d, f, T, K, v1);
        if (r1 && smoe_ring_applies(true, d, T)) v1 = r1;
        // The second product does not stream beside a hundred large tiles: rows of thousands of outputs, short reductions (128 slots of
        // 9216 x 256, T = 760 590 us a layer streaming, 345 through the ring)
        if (v2 == 6 && f % 128 == 0 && (double)T * d / 65536 >= 100 && smoe_ring_applies(false, f, T)) v2 = 10;
    }
    if (is_variant(L->ffn_variant[0]) && is_variant(L->ffn_variant[1])) {
        v1 = L->ffn_variant[0];
        v2 = L->ffn_variant[1];
    }
}

// Whether the first product (tile v1) stores the hidden activations past the caches.  Whole passes, past / plain in the mean, over 32
// shapes (4 MB to 2.1 GB of slots a layer), T = 130 .. 16384, one layer alone and up to six in turn; "all" are the slots that pass
// through memory from one pass of a layer to the next:
//  * Low tiles (3, 4): where weights come from memory, 100 MB or more of them a layer, whose stream h would displace: 0.965 .. 0.995 at
//    every such shape (16 slots of 768 x 3072, four layers, T = 777 56.4 -> 53.9 us a layer).  From the cache, one layer, 1.000 ..
//    1.02; six layers of 2 slots 1.05, of 8 of 768 x 2048 1.015.
//  * 256 x 256 tiles (10): 0.96 where a layer's slots are far more than the cache, which h would leave before it is read (0.94 at 64 slots
//    of 768 x 3072, 0.97 at 32 of 1024 x 4096; but 1.03 at 32 of 768 x 3072).  With less, large second products: 0.99 while all
//    slots stay in the cache; where they do not, 1.00 under 100 MB (in the separate calls 0.97: eight layers of 4 slots of 768 x 3072,
//    T = 4096 83.5 / 80.8) and 1.01 above.  Second products in smaller tiles read h more often: 1.02 .. 1.04, but
//    0.98 where all slots would stay in the cache beside each other and not beside h.
// Tiles of 128 rows store plainly.
bool h_past_caches(const smoe_layer* L, int v1, int v2) {
    const double own = 4.0 * L->cfg.K * L->cfg.d_model * L->cfg.d_ff * 1e-6, all = smoe_slot_traffic(L) * 1e-6;
    if (v1 == 3 || v1 == 4) return own >= 100 && smoe_weights_outgrow_cache(L);
    if (v1 != 10) return false;
    const bool large = v2 == 1 || v2 == 8 || v2 == 10;
    return own >= 400 || (large ? own < 100 || all <= 240 : own < 100 && all >= 100 && all <= 240);
}

}  // namespace

// Names of the two kernel instances the FFN of a T-token batch runs, as a profiler prints them
// (the benchmark uses this to check that a stored counter summary still describes the kernels
// it has just timed).
int smoe_describe_ffn_bf16(const smoe_layer* L, int T, int fused, char* out, size_t n) {
    int v[2];
    pick_variants(L, T, v[0], v[1]);
    std::string text;
    for (int i = 0; i < 2; ++i) {
        const bool first = i == 0;
        const int R = first ? L->cfg.d_model : L->cfg.d_ff;
        v[i] = standing_in(v[i], first, R, T);
        const char* shape = nullptr;                       // AF, MAXB, NW, BKT, PD, OCC of launch_variant
        std::string name;
        if (fused && smoe_decode_first_applies(L, T) && v[1] == 6) name = smoe_describe_decode(L, T, first);
        else if (v[i] == 5) name = std::string("small_gemm_bf16<4, 1, ") + (first ? "true>" : "false>");
        else if (v[i] == 6) name = std::string("small_gemm_bf16<4, 4, ") + (first ? "true>" : "false>");
        else if (v[i] == 11) name = "split_gemm_bf16";
        else if (v[i] == 10 && first && !h_past_caches(L, 10, v[1])) name = "ring_gemm_bf16_kept";
        else if (v[i] >= 9) name = std::string("ring_gemm_bf16<") + (v[i] == 9 ? "2, " : "4, ") + (first ? "true>" : "false>");
        else if (R % 64 != 0) shape = "1, 4, 4, 32, ";
        else if (v[i] == 1) shape = "1, 4, 4, 64, ";
        else if (v[i] == 3) shape = "1, 2, 4, 64, ";
        else if (v[i] == 4) shape = "1, 1, 4, 64, ";
        else if (v[i] == 8) shape = "1, 4, 8, 64, ";
        if (shape) {
            const int bkt = R % 64 != 0 ? 32 : 64, pd = (R % 64 == 0 && v[i] == 4) ? 3 : 1;
            const int occ = (R % 64 == 0 && (v[i] == 3 || v[i] == 4)) ? 4 : 2;
            const int pd_used = (R / bkt) % (pd + 1) == 0 ? pd : 0;
            name = std::string("grouped_gemm_bf16<") + shape + std::to_string(pd_used) + ", " + std::to_string(occ) + ", " +
                   (first ? "true>" : "false>");
        }
        text += (i ? " | " : "") + name;
    }
    if (!out || n == 0) return SMOE_EINVAL;
    snprintf(out, n, "%s", text.c_str());
    return SMOE_OK;
}

int smoe_launch_ffn_bf16(const smoe_layer* L, const uint16_t* x_perm, const int32_t* offsets, int T,
                         uint16_t* y_perm, hipStream_t s) {
    const smoe_config& c = L->cfg;
    int v1, v2;
    pick_variants(L, T, v1, v2);
    uint16_t* h = (uint16_t*)L->d_hidden;
    const int32_t* phys = L->cfg.spare_slots > 0 ? L->d_phys : nullptr;   // identity without spare slots
    const FuseArgs none{phys, nullptr, nullptr, nullptr, false}, first{phys, nullptr, nullptr, nullptr, h_past_caches(L, v1, v2)};
    if (int rc = launch_variant<true>(v1, x_perm, L->slot_w1, offsets, c.K, h, c.d_model, c.d_ff, T, first, s, L->prof_ev[0], L->prof_ev[1])) return rc;
    if (int rc = launch_variant<false>(v2, h, L->slot_w2, offsets, c.K, y_perm, c.d_ff, c.d_model, T, none, s, L->prof_ev[2], L->prof_ev[3])) return rc;
    return smoe_check_hip(hipGetLastError(), "smoe_expert_ffn launch");
}

bool smoe_ffn_dense_path(const smoe_layer* L, int T) {
    int v1, v2;
    pick_variants(L, T, v1, v2);
    return v2 == 6;
}

// Fused form used by smoe_forward: the first product gathers its rows from x
// through perm, the second scatters gate * y (+ residual) to out in token order.
int smoe_launch_ffn_bf16_fused(const smoe_layer* L, const uint16_t* x, const int32_t* perm, const int32_t* offsets,
                               const float* gate, const uint16_t* residual, int T, uint16_t* out, hipStream_t s) {
    const smoe_config& c = L->cfg;
    int v1, v2;
    pick_variants(L, T, v1, v2);
    uint16_t* h = (uint16_t*)L->d_hidden;
    const int32_t* phys = L->cfg.spare_slots > 0 ? L->d_phys : nullptr;   // identity without spare slots
    const FuseArgs gather{phys, perm, nullptr, nullptr, h_past_caches(L, v1, v2)}, scatter{phys, perm, gate, residual, false};
    if (int rc = launch_variant<true>(v1, x, L->slot_w1, offsets, c.K, h, c.d_model, c.d_ff, T, gather, s, L->prof_ev[0], L->prof_ev[1])) return rc;
    if (int rc = launch_variant<false>(v2, h, L->slot_w2, offsets, c.K, out, c.d_ff, c.d_model, T, scatter, s, L->prof_ev[2], L->prof_ev[3])) return rc;
    return smoe_check_hip(hipGetLastError(), "smoe_forward: FFN launch");
}
