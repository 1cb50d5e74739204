// Grouped bf16 products of prefill batches, both operands staged through a ring in LDS:
// Y[T, N] = act(X[T, R] . B_k[R, N]) for the rows of slot k, with the operand layouts, the rounding and the
// fusions of ffn_bf16.hip.  Used where there are large tiles for the chip many times over, and where the reduction is no
// multiple of 128: for every first product but with few tokens, for second products from where the splitting kernel no longer
// fills the chip better (ring_first and pick_second in ffn_bf16.hip have the rules and what they measured).
//
// What bounds these products on this chip, and what the kernel does about it:
//  * Power.  At the Switch-large prefill shape (16384 tokens, 32 slots of 1024 x 4096) random data pulls the clock
//    from 2.4 to 2.14 (first product) and 2.23 GHz.  v_mfma_f32_16x16x32 does the same work as
//    v_mfma_f32_32x32x16 at 12 % more (2008 against 1785 TFLOP/s from registers, 1707 against 1552 with the operand
//    reads), and a wave tile of 64 features x 128 tokens reads 0.75 KB of LDS per 32768 operations where one
//    feature block x 256 tokens reads 1.13.
//  * Latency.  Loads go from memory to LDS without passing through registers, three slices of 32 ahead, and the load
//    side runs on into the next tile while this one is multiplied and stored: a tile costs its reduction and the
//    issue of its stores, no prologue (256 x 256 tiles: 7 of 35 us before).  Any multiple of 32 is as good a
//    reduction length as another.
//  * Control.  The loop has no branch that is taken in ordinary steps: a wave without a block of its own loads one
//    lane's 16 bytes, so every slice has four loads to count.  With a branch for each of these the same loop without loads,
//    products and LDS reads took 40 and 55 us of launches of 168 and 177.
//  * Stores.  Without them the first product takes 134 of 156 us.  They stay on their way through the next tile's first
//    two steps, and the h of large tiles passes the caches by where that pays (h_past_caches in ffn_bf16.hip; here the second
//    product 169 -> 164 us).
//  * Balance.  Tile heights are chosen on the device from the segment lengths, and a slot's rows are cut evenly.
// Both products at that shape, from kernel traces: 168 + 188 -> 157 + 168 us; 8000 tokens, 16 slots of 992 x 3296: 241 ->
// 142 us.  What is left: launches of 156 and 164 us take 112 and 123 without their loads, 134 and 160 without the stores of h (traces of
// copies without the part): the loads bind.  The matrix cores are busy 0.47 and 0.46 of the time.
//
// Workgroup = 2 * NWF waves; tile = (64 * NWF features) x (at most 64 * NWF tokens), in blocks of 32.  Wave w loads
// feature block w and token block w of every slice; it multiplies the feature blocks 2 * (w % NWF) and the next with
// the token blocks of its parity w / NWF (waves w and w + NWF share a SIMD, so an odd block is no loss).
//
// A stage of the ring: feature blocks, then token blocks, 2 KB each.  Weights (fragment order) and hidden activations
// are linear copies, [8 reduction elements][32 rows] units of 16 bytes.  Row-major tokens land as rows of 64 bytes
// whose four units are permuted by (row / 2) % 4, which the lanes do by choosing what they load: operand reads
// of 8 neighbouring lanes then hit all banks.

#include <algorithm>
#include <type_traits>

#include "ffn_bf16.h"
#include "wave_ops.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int XCDS = 8;                   // accelerator dies, each with an L2 of its own
constexpr int MAX_SLOTS = 256;            // K <= E <= 256 by the C ABI
constexpr int ST = 4;                     // stages of the ring
constexpr int BLK = 2048;                 // bytes of 32 rows (or features) of one slice of 32 reduction elements
// A tile of h token blocks and 8 feature blocks takes 8 + h blocks through the compute unit per slice; 4 to 14 in the
// place of the 8 chose tiles of the same speed.
constexpr int TILE_COST0 = 8;

extern __shared__ __align__(16) char ring_lds[];

// Per-slot tables, in LDS behind the ring.
struct SlotMap {
    int first[MAX_SLOTS + 1];             // row tiles before slot k; [nslots] = all row tiles
    int pad[MAX_SLOTS];                   // 32-row blocks before slot k (segments are re-based to blocks)
    int a[MAX_SLOTS], b[MAX_SLOTS];       // clamped segment bounds
    int phys[MAX_SLOTS];                  // where the slot's weights are
};

struct Tile {
    int phys, nb, m0, m_end, pb0;         // slot's weights; token blocks (0: no tile); rows; first block in padded rows
    int fb0, width;                       // feature blocks
};

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ bf16x8 lds_frag(uint32_t off) { return *(const bf16x8*)(ring_lds + off); }

// Loads from memory to LDS: lane l's 16 (or 4) bytes land at off + 16 * l (4 * l).  Written out because the compiler,
// which cannot tell where the builtin's data lands, would wait for every LDS read in flight before each product.
// They have no result registers; whoever reads the data counts them (wait_vm) and then passes a barrier.
// Nothing else in the kernel uses m0.
__device__ __forceinline__ uint32_t lds_addr(uint32_t off) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)(ring_lds + off);
}
// A wave without a block of its own loads one lane's 16 bytes (of another wave's block, to a place that nobody reads): the loop
// then has no branch for it, and every slice the same number of loads to count.
__device__ __forceinline__ void load_1k(const char* base, uint32_t lo, uint32_t hi, uint32_t off, uint64_t lanes) {
    asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, %4\n\tglobal_load_lds_dwordx4 %1, %3\n\ts_add_u32 m0, %0, 0x400\n\t"
                 "s_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b64 exec, -1"
                 ::"s"(lds_addr(off)), "v"(lo), "v"(hi), "s"(base), "s"(lanes) : "memory", "scc");
}
__device__ __forceinline__ void load_2k(const char* base, uint32_t lane16, uint32_t off, uint64_t lanes) {   // the offset moves both sides
    asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, %3\n\tglobal_load_lds_dwordx4 %1, %2\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024\n\t"
                 "s_mov_b64 exec, -1"
                 ::"s"(lds_addr(off)), "v"(lane16), "s"(base), "s"(lanes) : "memory");
}
__device__ __forceinline__ void load_words(const void* src, uint32_t off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_addr(off)), "v"(src) : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vm() {   // at most the N youngest vector memory operations of this wave are outstanding
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <int NWF, bool FIRST>
struct RingShape {
    static constexpr int NB = 2 * NWF;                     // waves; feature blocks and most token blocks of a tile
    static constexpr int STAGE = 2 * NB * BLK;
    static constexpr uint32_t ROWS = ST * STAGE;           // row and gate tables of two tiles
    static constexpr uint32_t GATES = ROWS + 2 * NB * 32 * 4;
    static constexpr uint32_t MAP = GATES + (FIRST ? 0 : 2 * NB * 32 * 4);
    static constexpr size_t LDS = MAP + sizeof(SlotMap);
};

// FIRST = the d_model -> d_ff product: row-major tokens in (gathered through perm in the single-call path), ReLU,
// fragment-order h out.  Otherwise the d_ff -> d_model product: h in, row-major rows out (scattered through perm with
// gate and residual in the single-call path).  Items are numbered, dealt to the dies and walked as in
// grouped_gemm_bf16.
// PAST: hidden activations are stored past the caches.
template <int NWF, bool FIRST, bool PAST>
__device__ __forceinline__ void ring_body(
    const uint16_t* __restrict__ X, const uint4* __restrict__ Wp, const int32_t* __restrict__ offsets, int nslots,
    int T, uint16_t* __restrict__ Y, int R, int N, const FuseArgs fz) {
    using S = RingShape<NWF, FIRST>;
    constexpr int MAXB = S::NB, STAGE = S::STAGE;
    static_assert(ST == 4 && MAXB <= 8, "wait_slice counts two slices ahead");
    const int tid = threadIdx.x, wave = uni(tid >> 6), lane = tid & 63;
    const int wf = wave % NWF, wt = wave / NWF;
    const int nfb = N >> 5, ftiles = (nfb + MAXB - 1) / MAXB, nsub = R >> 5;
    SlotMap& map = *(SlotMap*)(ring_lds + S::MAP);
    const int* s_row = (const int*)(ring_lds + S::ROWS);
    const float* s_gate = (const float*)(ring_lds + S::GATES);

    struct Seg { int a, b; };
    auto segment = [&](int k) {
        Seg g{0, 0};
        if (k < nslots) {
            g.a = min(max(offsets[k], 0), T);              // clamps guard misuse
            g.b = max(min(max(offsets[k + 1], 0), T), g.a);
        }
        return g;
    };
    auto place = [&](int k) { return k < nslots && fz.phys ? fz.phys[k] : k; };
    const Seg seg0 = segment(lane);
    const int phys0 = place(lane);
    // tile height: the row tiles of at most 1, 2, .. blocks are counted, all take the best
    int tiles_of[MAXB] = {};
    for (int base = 0; base < nslots; base += 64) {
        const Seg g = base ? segment(base + lane) : seg0;
        const int nb = (g.b - g.a + 31) >> 5;
#pragma unroll
        for (int h = 1; h <= MAXB; ++h) tiles_of[h - 1] += __builtin_amdgcn_readlane(smoe_wave_incl_scan((nb + h - 1) / h), 63);
    }
    const int nwg = gridDim.x / XCDS;
    int H = MAXB, best = 0x7fffffff;
#pragma unroll
    for (int h = MAXB; h >= 1; --h) {
        const int per_die = (tiles_of[h - 1] * ftiles + XCDS - 1) / XCDS;
        const int cost = (per_die + nwg - 1) / nwg * (TILE_COST0 + h);
        if (cost < best) { best = cost; H = h; }
    }
    if (wave == 0) {
        int tiles_before = 0, pad_before = 0;
        for (int base = 0; base < nslots; base += 64) {
            const int k = base + lane;
            const Seg g = base ? segment(k) : seg0;
            const int pad = (g.b - g.a + 31) >> 5, tiles = (pad + H - 1) / H;
            const int tin = smoe_wave_incl_scan(tiles), pin = smoe_wave_incl_scan(pad);
            if (k < nslots) {
                map.first[k] = tiles_before + tin - tiles;
                map.pad[k] = pad_before + pin - pad;
                map.a[k] = g.a;
                map.b[k] = g.b;
                map.phys[k] = base ? place(k) : phys0;
            }
            tiles_before += __builtin_amdgcn_readlane(tin, 63);
            pad_before += __builtin_amdgcn_readlane(pin, 63);
        }
        if (lane == 0) map.first[nslots] = tiles_before;
    }
    __syncthreads();
    const int G = uni(map.first[nslots]) * ftiles;
    const int die = blockIdx.x % XCDS;
    const int lo = (int)((long long)G * die / XCDS), cnt = (int)((long long)G * (die + 1) / XCDS) - lo;

    auto tile_at = [&](int j) {
        Tile t;
        const int g = lo + j;
        int mt = g / ftiles, ft = g - mt * ftiles;
        int nle = 0;
        for (int base = 0; base < nslots; base += 64) {
            const int k = base + lane;
            nle += __popcll(__ballot(k < nslots && map.first[k] <= mt));
        }
        const int k = uni(nle - 1);
        const int fk = uni(map.first[k]), tiles = uni(map.first[k + 1]) - fk;
        if (FIRST) {                                       // row tile fastest inside a slot
            const int local = g - fk * ftiles;
            ft = local / tiles;
            mt = fk + local - ft * tiles;
        }
        const int a = uni(map.a[k]), b = uni(map.b[k]), nbk = (b - a + 31) >> 5, i = mt - fk;
        const int bq = nbk / tiles, br = nbk - bq * tiles, b0 = i * bq + min(i, br), b1 = b0 + bq + (i < br ? 1 : 0);
        t.phys = uni(map.phys[k]);
        t.nb = b1 - b0;
        t.m0 = a + 32 * b0;
        t.m_end = min(a + 32 * b1, b);
        t.pb0 = uni(map.pad[k]) + b0;
        const int fq = nfb / ftiles, fr = nfb - fq * ftiles;
        t.fb0 = ft * fq + min(ft, fr);
        t.width = fq + (ft < fr ? 1 : 0);
        return t;
    };

    int j = blockIdx.x / XCDS;
    if (j >= cnt) return;
    Tile cur = tile_at(j), nxt = cur;
    const bool gather = fz.perm != nullptr;
    int par = 0;                                           // which half of the tables the current tile has
    // load side: runs ST - 1 slices ahead of the products, across tiles
    int lc = 0, lpar = 0;                                  // slice of the tile; half of the tables
    uint32_t lst = 0;                                      // stage of the ring
    uint64_t lw = 1, lt = 1;                               // lanes that load weights and tokens
    const char *wsrc = nullptr, *tsrc = nullptr;           // scalar bases
    uint32_t to0 = 0, to1 = 0;                             // row-major tokens: this lane's two rows
    const uint32_t lane16 = lane * 16;
    auto weights_of = [&](const Tile& t) {
        lw = wave < t.width ? ~0ull : 1;
        wsrc = (const char*)Wp + ((size_t)t.phys * nfb + t.fb0 + min(wave, t.width - 1)) * (R >> 4) * 1024;
    };
    auto ask_rows = [&](const Tile& t, int p) {            // the rows of a tile's tokens, into half p of the table
        if (gather && wave * 64 < MAXB * 32)
            load_words(fz.perm + min(t.m0 + tid, t.m_end - 1), S::ROWS + (p * MAXB * 32 + wave * 64) * 4);
    };
    auto tokens_of = [&](const Tile& t, int p) {           // the rows are there
        lt = wave < t.nb ? ~0ull : 1;
        if (FIRST) {
            tsrc = (const char*)X;
            const int r0 = min(wave, t.nb - 1) * 32 + (lane >> 2);
            const uint32_t u = ((lane & 3) ^ ((lane >> 3) & 3)) * 16;
            const int g0 = gather ? s_row[p * MAXB * 32 + r0] : min(t.m0 + r0, t.m_end - 1);
            const int g1 = gather ? s_row[p * MAXB * 32 + r0 + 16] : min(t.m0 + r0 + 16, t.m_end - 1);
            to0 = (uint32_t)g0 * (uint32_t)(R * 2) + u;
            to1 = (uint32_t)g1 * (uint32_t)(R * 2) + u;
        } else {
            tsrc = (const char*)X + (size_t)(t.pb0 + min(wave, t.nb - 1)) * (R >> 3) * 512;
            if (gather && tid < MAXB * 32)                 // the rows' gates, for this tile's last step
                load_words(fz.gate + s_row[p * MAXB * 32 + tid], S::GATES + (p * MAXB * 32 + wave * 64) * 4);
        }
    };
    auto load_w = [&]() {
        load_2k(wsrc, lane16, lst + wave * BLK, lw);
        wsrc += 2048;
    };
    auto load_t = [&]() {
        const uint32_t st = lst + (wave + MAXB) * BLK;
        if (FIRST) load_1k(tsrc, to0, to1, st, lt);
        else load_2k(tsrc, lane16, st, lt);
        tsrc += FIRST ? 64 : 2048;
    };
    auto next_stage = [&]() { lst = (lst + STAGE) & (ST * STAGE - 1); };
    auto issue_t = [&]() {
        load_t();
        next_stage();
        if (__builtin_expect(++lc == nsub, 0)) {
            lc = 0;
            lpar ^= 1;
            if (nxt.nb > 0) {
                weights_of(nxt);
                tokens_of(nxt, lpar);
            } else {                                       // no tile left: the start of this one again, for one lane
                wsrc -= (size_t)nsub * 2048;
                tsrc -= (size_t)nsub * (FIRST ? 64 : 2048);
                lw = lt = 1;
            }
        }
    };

    // The first slices: weights on their way while the rows of the tokens are looked up.
    nxt.nb = 0;
    ask_rows(cur, 0);
    weights_of(cur);
#pragma unroll 1
    for (int i = 0; i < ST - 1; ++i) { load_w(); next_stage(); }
    wait_vm<2 * (ST - 1)>();                               // the rows
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    lst = 0;
    tokens_of(cur, 0);
#pragma unroll 1
    for (int i = 0; i < ST - 1; ++i) { load_t(); next_stage(); }
    lc = ST - 1;
    wait_vm<4>();                                          // the first slice
    __builtin_amdgcn_s_barrier();

    uint32_t cst = 0;                                      // stage that is multiplied
    int pend = -1;                                         // stores of this wave at the end of the tile before; -1: no such tile, the
                                                           // first slices' weights were asked for before their tokens
    // The next slice has landed: nothing but the four loads of the slice behind it is outstanding.  In a tile's first two
    // steps the last tile's stores, too, are younger than what is waited for, and stay on their way.
    auto wait_slice = [&](int c) {
        if (__builtin_expect(c < 2, 0)) {
            if (pend >= 16) wait_vm<20>();
            else if (pend >= 8) wait_vm<12>();
            else if (pend < 0 && c == 0) wait_vm<2>();
            else wait_vm<4>();
        } else {
            wait_vm<4>();
        }
    };
    auto run = [&](auto nbc) {
        constexpr int NB = decltype(nbc)::value;           // token blocks of this wave: wt, wt + 2, ...
        constexpr int NBA = NB ? NB : 1;
        f32x4 acc[4][2 * NBA];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 2 * NBA; ++b)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[a][b][i] = 0.f;
        const uint32_t frag = (lane >> 4) * 512 + (lane & 15) * 16;
        const uint32_t aoff = wf * 2 * BLK + frag;
        uint32_t boff = MAXB * BLK + wt * BLK;
        if (FIRST) boff += (lane & 15) * 64 + (((lane >> 4) ^ ((lane >> 1) & 3)) * 16);
        else boff += frag;
        constexpr uint32_t BH = FIRST ? 1024 : 256;        // the upper 16 tokens of a block
        bf16x8 fa[2][4], f0[NBA], f1[NBA];
        auto read_a = [&](bf16x8 (&f)[4], uint32_t st) {
#pragma unroll
            for (int a = 0; a < 4; ++a) f[a] = lds_frag(st + aoff + (a >> 1) * BLK + (a & 1) * 256);
        };
        auto read_b = [&](bf16x8 (&f)[NBA], uint32_t st, int half) {
#pragma unroll
            for (int i = 0; i < NB; ++i) f[i] = lds_frag(st + boff + ((half * NB + i) >> 1) * 2 * BLK + ((half * NB + i) & 1) * BH);
        };
        auto mul = [&](bf16x8 (&fa)[4], bf16x8 (&f)[NBA], int half, int lo, int hi) {   // products lo .. hi - 1 of a half step
#pragma unroll
            for (int i = lo; i < hi; ++i) {
                const int b = i >> 2, a = i & 3;
                acc[a][half * NB + b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[a], f[b], acc[a][half * NB + b], 0, 0, 0);
            }
        };
        constexpr int P = 4 * NB;
        if (NB) {
            read_a(fa[0], cst);
            read_b(f0, cst, 0);
        }
        auto step = [&](bf16x8 (&fa)[4], bf16x8 (&fn)[4], int c) {
            if (NB) {
                read_b(f1, cst, 1);
                __builtin_amdgcn_sched_barrier(0);
                mul(fa, f0, 0, 0, P);
                __builtin_amdgcn_sched_barrier(0);
            }
            wait_slice(c);
            __builtin_amdgcn_s_barrier();
            cst = (cst + STAGE) & (ST * STAGE - 1);
            if (NB) {
                read_a(fn, cst);
                read_b(f0, cst, 0);
                __builtin_amdgcn_sched_barrier(0);
                mul(fa, f1, 1, 0, P / 4);
                __builtin_amdgcn_sched_barrier(0);
            }
            // every wave is in this tile now, so nobody reads the rows of the one before any more
            if (__builtin_expect(c == 0, 0) && nxt.nb > 0) ask_rows(nxt, par ^ 1);
            load_w();
            if (NB) {
                __builtin_amdgcn_sched_barrier(0);
                mul(fa, f1, 1, P / 4, P / 2);
                __builtin_amdgcn_sched_barrier(0);
            }
            issue_t();
            if (NB) {
                __builtin_amdgcn_sched_barrier(0);
                mul(fa, f1, 1, P / 2, P);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        int c = 0;
#pragma unroll 1
        for (; c + 1 < nsub; c += 2) { step(fa[0], fa[1], c); step(fa[1], fa[0], c + 1); }
        if (c < nsub) step(fa[0], fa[1], c);
        if constexpr (NB > 0) {
            // accumulator register i of lane l: feature 4*(l/16) + i, token l%16.  Swapping rows of 16 lanes
            // between the two halves of a feature block gives every lane 8 consecutive features of its token.
            const int unit = ((lane >> 4) & 1) * 2 + (lane >> 5);
            uint4 rs[2][2 * NB];
            int row[2 * NB];
            float gate[2 * NB];
            pend = 0;
            if (!FIRST) {                                  // every piece of the residual is asked for before the first store
#pragma unroll
                for (int b = 0; b < 2 * NB; ++b) {
                    const int r = ((b >> 1) * 2 + wt) * 32 + (b & 1) * 16 + (lane & 15);
                    row[b] = cur.m0 + r;
                    gate[b] = 1.f;
                    if (gather) {                          // past the segment's end: its last row, not stored
                        row[b] = s_row[par * MAXB * 32 + r];
                        gate[b] = s_gate[par * MAXB * 32 + r];
                    }
                }
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2 * NB; ++b) {
                        rs[a][b] = make_uint4(0, 0, 0, 0);
                        if (gather && fz.residual)
                            rs[a][b] = *(const uint4*)(fz.residual + (size_t)row[b] * N + (cur.fb0 + min(wf * 2 + a, cur.width - 1)) * 32 + unit * 8);
                    }
            }
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                if (wf * 2 + a >= cur.width) continue;
                const int fbk = cur.fb0 + wf * 2 + a;
#pragma unroll
                for (int b = 0; b < 2 * NB; ++b) {
                    uint32_t w[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {          // w[0], w[1]: lower half of the block; w[2], w[3]: upper
                        float v0 = acc[2 * a + (q >> 1)][b][2 * (q & 1)], v1 = acc[2 * a + (q >> 1)][b][2 * (q & 1) + 1];
                        if (FIRST) { v0 = fmaxf(v0, 0.f); v1 = fmaxf(v1, 0.f); }
                        w[q] = smoe_pack_bf16(v0, v1);
                    }
                    const auto s0 = __builtin_amdgcn_permlane16_swap(w[0], w[2], false, false);
                    const auto s1 = __builtin_amdgcn_permlane16_swap(w[1], w[3], false, false);
                    uint4 o = make_uint4(s0[0], s1[0], s0[1], s1[1]);
                    if (FIRST) {
                        const size_t u = ((size_t)(cur.pb0 + (b >> 1) * 2 + wt) * (N >> 3) + fbk * 4 + unit) * 32 + (b & 1) * 16 + (lane & 15);
                        if (PAST) smoe_store_stream((uint4*)(Y + u * 8), o);
                        else *(uint4*)(Y + u * 8) = o;
                        ++pend;
                    } else {
                        const int r0 = cur.m0 + ((b >> 1) * 2 + wt) * 32 + (b & 1) * 16;
                        if (r0 >= cur.m_end) continue;     // uniform; else one store, of the lanes whose row is there
                        if (gather) o = smoe_gate_unit(o, gate[b], rs[a][b], fz.residual != nullptr);
                        if (r0 + (lane & 15) < cur.m_end) *(uint4*)(Y + (size_t)row[b] * N + fbk * 32 + unit * 8) = o;
                        ++pend;
                    }
                }
            }
        } else {
            pend = 0;
        }
    };
    while (true) {
        j += nwg;
        nxt.nb = 0;
        if (j < cnt) {
            nxt = tile_at(j);
        }
        const int mine = wf * 2 < cur.width ? (cur.nb + 1 - wt) >> 1 : 0;
        if (NWF == 4 && mine == 4) run(std::integral_constant<int, NWF>{});
        else if (NWF == 4 && mine == 3) run(std::integral_constant<int, NWF - 1>{});
        else if (mine == 2) run(std::integral_constant<int, 2>{});
        else if (mine == 1) run(std::integral_constant<int, 1>{});
        else run(std::integral_constant<int, 0>{});
        if (nxt.nb == 0) break;
        cur = nxt;
        par ^= 1;
    }
    wait_vm<0>();                                          // no load is on its way into LDS that is given back
}

// Large tiles store h past the caches; ring_gemm_bf16_kept is the instance for h that is better kept.  An instance of its own: one kernel
// with a branch at the end of a tile took 0.6 us more of 25 (4096 tokens, 4 slots of 768 x 3072), with one a store 1 to 3 %.
template <int NWF, bool FIRST>
__global__ __launch_bounds__(NWF * 128, 2) void ring_gemm_bf16(
    const uint16_t* __restrict__ X, const uint4* __restrict__ Wp, const int32_t* __restrict__ offsets, int nslots,
    int T, uint16_t* __restrict__ Y, int R, int N, const FuseArgs fz) {
    ring_body<NWF, FIRST, FIRST && NWF == 4>(X, Wp, offsets, nslots, T, Y, R, N, fz);
}
__global__ __launch_bounds__(4 * 128, 2) void ring_gemm_bf16_kept(
    const uint16_t* __restrict__ X, const uint4* __restrict__ Wp, const int32_t* __restrict__ offsets, int nslots,
    int T, uint16_t* __restrict__ Y, int R, int N, const FuseArgs fz) {
    ring_body<4, true, false>(X, Wp, offsets, nslots, T, Y, R, N, fz);
}

template <int NWF, bool FIRST, bool KEPT = false>
int launch(const uint16_t* X, const void* Wp, const int32_t* offsets, int nslots, uint16_t* Y, int R, int N, int T,
           const FuseArgs& fz, int cus_per_die, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    using S = RingShape<NWF, FIRST>;
    auto kern = ring_gemm_bf16<NWF, FIRST>;
    if constexpr (KEPT) kern = ring_gemm_bf16_kept;
    static smoe_lds_raised raised;
    if (int rc = raised.ensure((const void*)kern, S::LDS, (int)S::LDS)) return rc;
    const int ftiles = ((N >> 5) + S::NB - 1) / S::NB;
    const long long items = ((long long)(T + 31) / 32 + nslots) * ftiles;   // if every tile were one block high
    const int resident = cus_per_die * (8 / S::NB);        // two waves per SIMD
    const int per_die = (int)std::min<long long>((items + XCDS - 1) / XCDS, resident);
    smoe_launch_timed_lds(kern, dim3(XCDS * std::max(per_die, 1)), dim3(NWF * 128), S::LDS, s, e0, e1, X, (const uint4*)Wp,
                          offsets, nslots, T, Y, R, N, fz);
    return SMOE_OK;
}

}  // namespace

// The load side looks up the next tile's rows three slices before this tile ends, from a table that is asked for in
// the tile's first slice and complete two slices later; row-major tokens are addressed by 32-bit offsets.
bool smoe_ring_applies(bool first, int R, int T) {
    return R >= 256 && (!first || (unsigned long long)T * R * 2 < (1ull << 32));
}

int smoe_launch_ring(int blocks, bool first, const uint16_t* X, const void* Wp, const int32_t* offsets, int nslots,
                     uint16_t* Y, int R, int N, int T, const FuseArgs& fz, int cus_per_die, hipStream_t s, hipEvent_t e0,
                     hipEvent_t e1) {
    if (blocks == 8)
        return !first    ? launch<4, false>(X, Wp, offsets, nslots, Y, R, N, T, fz, cus_per_die, s, e0, e1)
               : fz.past ? launch<4, true>(X, Wp, offsets, nslots, Y, R, N, T, fz, cus_per_die, s, e0, e1)
                         : launch<4, true, true>(X, Wp, offsets, nslots, Y, R, N, T, fz, cus_per_die, s, e0, e1);
    return first ? launch<2, true>(X, Wp, offsets, nslots, Y, R, N, T, fz, cus_per_die, s, e0, e1)
                 : launch<2, false>(X, Wp, offsets, nslots, Y, R, N, T, fz, cus_per_die, s, e0, e1);
}
