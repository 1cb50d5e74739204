// Second products of middle-sized batches, reduction split over the four waves of a workgroup:
// Y[T, N] = X[T, R] . B_k[R, N] for the rows of slot k, X the hidden activations, both operands in fragment order, with
// the rounding and the fusions of ffn_bf16.hip.
//
// A second product has few outputs and a long reduction (4096 x 768 outputs of 3072 terms): tiles that fill the chip are
// small, and what bounds them is bytes, a tile of w feature and h token blocks takes (w + h) KB per 16 terms through its
// compute unit, and the time until they arrive.  So every wave holds the whole tile, a quarter of the reduction each: each
// byte passes through the compute unit once, straight into registers, with no LDS traffic and no barrier in the loop, and
// one wave per SIMD has 512 registers, 256 of accumulators and room for 32 KB of operands in flight (128 KB per compute
// unit, where a tile of the tiled kernel has 48).  The parts meet in LDS at the end and are added in order.
// The tile shape, up to 4 x 4 blocks, is chosen on the device from the segment lengths: every lane prices one shape.
//
// us a layer, whole passes, weights from memory, clustered tokens, with tiled or ring kernel / with this one: 16 slots of 768 x 3072 (first
// d_model, then d_ff), T = 777 61.0 / 55.2, T = 3000 81.1 / 77.3; 4 slots, T = 600 39.3 / 32.7, T = 3000 70.8 / 63.0; 11 of
// 416 x 1696, T = 1213 40.3 / 31.2; 10 of 992 x 3296, T = 777 79.0 / 63.7; 32 of 1024 x 4096, T = 600 144 / 129; 64 of 768 x
// 3072, T = 2000 154 / 150.  The launch of 16 slots, T = 777, takes 23.1 us, without its products 22.9, without its loads 10.5,
// without either 7.3 (until the shape is chosen and the operands have come, the meeting and the stores): the loads bind it, 90 MB
// at 3.7 TB/s.  With 4 x 4 tiles (4 slots, T = 4096) 33.4, 29.7, 25.4 and 14.1: one wave per SIMD does not overlap products
// and loads wholly.

#include <algorithm>
#include <type_traits>

#include "ffn_bf16.h"
#include "split_price.h"
#include "wave_ops.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int XCDS = 8;                   // accelerator dies, each with an L2 of its own
constexpr int MAXW = 4, MAXH = 4;         // 32-feature and 32-token blocks of the largest tile
constexpr int PARTS = 4;                  // waves of a workgroup: each has a quarter of the reduction
constexpr int PHASE = 8;                  // 32 x 32 blocks that meet in LDS together

extern __shared__ __align__(16) char split_lds[];
constexpr int MEET_BYTES = PHASE * PARTS * 4096;
constexpr int LDS_BYTES = MEET_BYTES + MAXH * 32 * 4;

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

struct TileArgs {
    const char *w, *x;                    // first feature block, first token block
    size_t wstride;                       // bytes from one block to the next, both operands
    int lo, n;                            // this wave's steps of 16
    int m0, rows, col0, N;                // first row and live rows; first column
    uint16_t* Y;
    const int32_t* perm;
    const float* gate;
    const uint16_t* residual;
};

template <int W, int H>
__device__ __forceinline__ void run_tile(const TileArgs& t) {
    constexpr int NL = W + H;
    const int tid = threadIdx.x, part = uni(tid >> 6), lane = tid & 63;
    const uint32_t lane16 = lane * 16;
    int* s_row = (int*)(split_lds + MEET_BYTES);
    const int mine = t.m0 + min(tid, t.rows - 1);
    const int dst = t.perm ? t.perm[mine] : mine;          // asked for before the operands, needed behind them
    const char* src[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) src[i] = (i < W ? t.w + i * t.wstride : t.x + (i - W) * t.wstride) + (size_t)t.lo * 1024;
    f32x16 acc[W][H];
#pragma unroll
    for (int a = 0; a < W; ++a)
#pragma unroll
        for (int b = 0; b < H; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
    auto frag = [&](const u32x4& v) {
        union { u32x4 u; bf16x8 b; } c;
        c.u = v;
        return c.b;
    };
    auto load = [&](u32x4 (&v)[NL], int s) {               // past the end: read again, not used
        const size_t at = (size_t)max(min(s, t.n - 1), 0) * 1024;
#pragma unroll
        for (int q = 0; q < NL; ++q) v[q] = *(const u32x4*)(src[q] + at + lane16);
    };
    auto mul = [&](const u32x4 (&v)[NL]) {
#pragma unroll
        for (int p = 0; p < W * H; ++p)
            acc[p / H][p % H] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(v[p / H]), frag(v[W + p % H]), acc[p / H][p % H], 0, 0, 0);
    };
    if constexpr (NL >= 7 || NL == 2) {                    // one set of steps, each refilled behind its products
        // One block either way needs many steps in flight, and two sets of twelve did not fit the half of the register file that
        // products read from: 96 copies, three operands of every round through scratch, all loads waited for.
        constexpr int D = NL == 2 ? 12 : 4;
        u32x4 buf[D][NL];
#pragma unroll
        for (int i = 0; i < D; ++i) load(buf[i], i);
        int s0 = 0;
#pragma unroll 1
        for (; t.n - s0 > D; s0 += D) {
#pragma unroll
            for (int i = 0; i < D; ++i) {
                mul(buf[i]);
                __builtin_amdgcn_sched_barrier(0);
                load(buf[i], s0 + D + i);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int i = 0; i < D; ++i)
            if (s0 + i < t.n) mul(buf[i]);                 // uniform
    } else {                                               // two sets in turn: with few products the compiler moves the loads in
        // front of them and copies the registers
        constexpr int D = NL >= 5 ? 4 : NL == 4 ? 6 : 8;
        u32x4 A[D][NL], B[D][NL];
#pragma unroll
        for (int i = 0; i < D; ++i) load(A[i], i);
        int s0 = 0;
#pragma unroll 1
        for (; t.n - s0 > 2 * D; s0 += 2 * D) {
#pragma unroll
            for (int i = 0; i < D; ++i) load(B[i], s0 + D + i);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < D; ++i) mul(A[i]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < D; ++i) load(A[i], s0 + 2 * D + i);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < D; ++i) mul(B[i]);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (t.n - s0 > D)                                  // uniform
#pragma unroll
            for (int i = 0; i < D; ++i) load(B[i], s0 + D + i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < D; ++i)
            if (s0 + i < t.n) mul(A[i]);                   // uniform
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < D; ++i)
            if (s0 + D + i < t.n) mul(B[i]);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (tid < MAXH * 32) s_row[tid] = tid < t.rows ? dst : -1;
    __syncthreads();
    // The four parts meet in LDS, PHASE blocks at a time, and are added in order.  Accumulator register i of lane l:
    // feature 8*(i/4) + 4*(l/32) + i%4, token l%32.  A thread finishes 8 features of a token at a time.
    constexpr int NP = W * H, UNITS = (NP * 128 + 255) / 256, PU = PHASE * 128 / 256;
    u32x4 rs[UNITS];
    int row[UNITS];
    float gate[UNITS];
#pragma unroll
    for (int j = 0; j < UNITS; ++j) {
        const int u = tid + j * 256, p = u >> 7, g = (u >> 5) & 3;
        row[j] = p < NP ? s_row[(p % H) * 32 + (u & 31)] : -1;
        rs[j] = u32x4{0, 0, 0, 0};
        gate[j] = 1.f;
        if (t.perm && row[j] >= 0) {
            gate[j] = t.gate[row[j]];
            if (t.residual) rs[j] = *(const u32x4*)(t.residual + (size_t)row[j] * t.N + t.col0 + (p / H) * 32 + g * 8);
        }
    }
#pragma unroll
    for (int ph = 0; ph < NP; ph += PHASE) {
        if (ph) __syncthreads();
#pragma unroll
        for (int p = ph; p < NP && p < ph + PHASE; ++p)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *(float4*)(split_lds + (((p - ph) * PARTS + part) * 4 + g) * 1024 + lane16) =
                    make_float4(acc[p / H][p % H][4 * g], acc[p / H][p % H][4 * g + 1], acc[p / H][p % H][4 * g + 2], acc[p / H][p % H][4 * g + 3]);
        __syncthreads();
#pragma unroll
        for (int j = ph * 128 / 256; j < UNITS && j < ph * 128 / 256 + PU; ++j) {
            if (row[j] < 0) continue;
            const int u = tid + j * 256, p = u >> 7, g = (u >> 5) & 3;
            const char* m = split_lds + ((p - ph) * PARTS * 4 + g) * 1024 + (u & 31) * 16;
            float4 lo = *(const float4*)m, hi = *(const float4*)(m + 512);
#pragma unroll
            for (int q = 1; q < PARTS; ++q) {
                const float4 l = *(const float4*)(m + q * 4096), h = *(const float4*)(m + q * 4096 + 512);
                lo.x += l.x; lo.y += l.y; lo.z += l.z; lo.w += l.w;
                hi.x += h.x; hi.y += h.y; hi.z += h.z; hi.w += h.w;
            }
            uint4 o = make_uint4(smoe_pack_bf16(lo.x, lo.y), smoe_pack_bf16(lo.z, lo.w), smoe_pack_bf16(hi.x, hi.y), smoe_pack_bf16(hi.z, hi.w));
            if (t.perm) o = smoe_gate_unit(o, gate[j], make_uint4(rs[j][0], rs[j][1], rs[j][2], rs[j][3]), t.residual != nullptr);
            *(uint4*)(t.Y + (size_t)row[j] * t.N + t.col0 + (p / H) * 32 + g * 8) = o;
        }
    }
    __syncthreads();                                       // the next tile writes the tables
}

template <int W, int H>
__device__ __forceinline__ void pick_w(int w, int h, const TileArgs& t) {
    if (w == W && h == H) run_tile<W, H>(t);
    else if constexpr (H > 1) pick_w<W, H - 1>(w, h, t);
    else if constexpr (W > 1) pick_w<W - 1, MAXH>(w, h, t);
}

// Lane k of a chunk of 64 slots: the slot's rows, and the 32-row blocks in front of it (segments are re-based to blocks).
struct Lane { int a, b, pad; };

// Items (row tile, feature tile) are numbered slot by slot; die x owns the x-th eighth of the list, the j-th of its n workgroups
// takes items j, j + n, ...  Inside a slot the row tile is fastest, so that the slot's weights are fetched by one die, while its
// rows are fewer bytes than they; else the feature tile.

__global__ __launch_bounds__(256, 1) void split_gemm_bf16(const uint16_t* __restrict__ X, const uint4* __restrict__ Wp,
                                                          const int32_t* __restrict__ offsets, int nslots, int T, uint16_t* __restrict__ Y,
                                                          int R, int N, const FuseArgs fz) {
    const int tid = threadIdx.x, part = uni(tid >> 6), lane = tid & 63;
    const int nfb = N >> 5, nrb = R >> 4, per = (nrb + PARTS - 1) / PARTS;
    const int nwg = gridDim.x / XCDS;
    auto slots = [&](int base, int before) {               // slots base .. base + 63
        Lane s{0, 0, 0};
        if (base + lane < nslots) {
            s.a = min(max(offsets[base + lane], 0), T);    // clamps guard misuse
            s.b = max(min(max(offsets[base + lane + 1], 0), T), s.a);
        }
        const int nb = (s.b - s.a + 31) >> 5;
        s.pad = before + smoe_wave_incl_scan(nb) - nb;
        return s;
    };
    const Lane first = slots(0, 0);
    // tile shape: lane (W - 1) * 4 + H - 1 prices its shape, the cheapest wins
    int tl[MAXH] = {0, 0, 0, 0};
    for (int base = 0; base < nslots; base += 64) {
        const Lane s = base ? slots(base, 0) : first;
        const int nb = (s.b - s.a + 31) >> 5;
#pragma unroll
        for (int h = 1; h <= MAXH; ++h) tl[h - 1] += __builtin_amdgcn_readlane(smoe_wave_incl_scan((nb + h - 1) / h), 63);
    }
    const int cw = ((lane >> 2) & 3) + 1, ch = (lane & 3) + 1;
    const int mine = (lane & 3) == 0 ? tl[0] : (lane & 3) == 1 ? tl[1] : (lane & 3) == 2 ? tl[2] : tl[3];
    const int cft = (nfb + cw - 1) / cw;
    const int rounds = ((mine * cft + XCDS - 1) / XCDS + nwg - 1) / nwg;
    const float price = smoe_split_price((float)rounds, (float)per, cw, ch);
    float best = price;
#pragma unroll
    for (int d = 8; d; d >>= 1) best = fminf(best, __shfl_xor(best, d));
    const int id = __ffsll((long long)__ballot(price == best)) - 1, W = (id >> 2) + 1, H = (id & 3) + 1;
    const int ftiles = (nfb + W - 1) / W;
    const int G = (H == 1 ? tl[0] : H == 2 ? tl[1] : H == 3 ? tl[2] : tl[3]) * ftiles;
    const int die = blockIdx.x % XCDS;
    const int lo = (int)((long long)G * die / XCDS), cnt = (int)((long long)G * (die + 1) / XCDS) - lo;
    for (int j = blockIdx.x / XCDS; j < cnt; j += nwg) {
        const int g = lo + j;
        int before = 0, pad_before = 0, slot = 0, a = 0, b = 0, tiles = 1, fk = 0, pad = 0;
        for (int base = 0; base < nslots; base += 64) {
            const Lane s = base ? slots(base, pad_before) : first;
            const int nb = (s.b - s.a + 31) >> 5, mt = (nb + H - 1) / H;
            const int tin = before + smoe_wave_incl_scan(mt);
            const unsigned long long past = __ballot(tin * ftiles > g);
            if (past) {
                const int who = __ffsll((long long)past) - 1;
                slot = base + who;
                a = __builtin_amdgcn_readlane(s.a, who);
                b = __builtin_amdgcn_readlane(s.b, who);
                tiles = __builtin_amdgcn_readlane(mt, who);
                fk = __builtin_amdgcn_readlane(tin - mt, who);
                pad = __builtin_amdgcn_readlane(s.pad, who);
                break;
            }
            before = __builtin_amdgcn_readlane(tin, 63);
            pad_before = __builtin_amdgcn_readlane(s.pad + nb, 63);
        }
        const int local = g - fk * ftiles;
        int i, ft;
        if (b - a < N) { ft = local / tiles; i = local - ft * tiles; }
        else { i = local / ftiles; ft = local - i * ftiles; }
        const int nb = (b - a + 31) >> 5, bq = nb / tiles, br = nb - bq * tiles, b0 = i * bq + min(i, br), h = bq + (i < br ? 1 : 0);
        const int fq = nfb / ftiles, fr = nfb - fq * ftiles, f0 = ft * fq + min(ft, fr), w = fq + (ft < fr ? 1 : 0);
        const int phys = fz.phys ? uni(fz.phys[slot]) : slot;
        TileArgs t;
        t.wstride = (size_t)nrb * 1024;
        t.w = (const char*)Wp + ((size_t)phys * nfb + f0) * t.wstride;
        t.x = (const char*)X + (size_t)(pad + b0) * t.wstride;
        t.lo = min(part * per, nrb);
        t.n = min(t.lo + per, nrb) - t.lo;
        t.lo = t.n > 0 ? t.lo : 0;
        asm volatile("" : "+s"(t.n), "+s"(t.lo));          // known per item only: else every shape's first addresses are computed in
        // front of the items' loop, and 43 scalars kept in vector registers (2 now)
        t.m0 = a + 32 * b0;
        t.rows = min(32 * h, b - t.m0);
        t.col0 = f0 * 32;
        t.N = N;
        t.Y = Y;
        t.perm = fz.perm;
        t.gate = fz.gate;
        t.residual = fz.perm ? fz.residual : nullptr;
        pick_w<MAXW, MAXH>(w, h, t);
    }
}

}  // namespace

// Any reduction of a multiple of 16; parts past its end stay empty.
int smoe_launch_split(const uint16_t* X, const void* Wp, const int32_t* offsets, int nslots, uint16_t* Y, int R, int N, int T,
                      const FuseArgs& fz, int cus_per_die, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    static smoe_lds_raised raised;
    if (int rc = raised.ensure((const void*)split_gemm_bf16, LDS_BYTES, LDS_BYTES)) return rc;
    const long long items = ((long long)T / 32 + nslots) * (N >> 5);
    const int per_die = (int)std::min<long long>((items + XCDS - 1) / XCDS, cus_per_die);
    smoe_launch_timed_lds(split_gemm_bf16, dim3(XCDS * std::max(per_die, 1)), dim3(256), LDS_BYTES, s, e0, e1, X, (const uint4*)Wp, offsets,
                          nslots, T, Y, R, N, fz);
    return SMOE_OK;
}
