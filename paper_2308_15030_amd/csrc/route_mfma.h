// The router for bf16 activations: product, softmax, original top-1, masked top-1 and |x|,
// as a device function shared by smoe_route's kernel and the small batch's first launch.
//
// x is exactly bf16, and an fp32 router weight is exactly the sum of three bf16 numbers
// (8 + 8 + 8 significand bits): w = hi + mid + lo, each the upper half of what the one before left.
// Every product x * {hi, mid, lo} is exact in fp32, so three bf16 MFMA passes with fp32 accumulation
// give the fp32-weight logits up to accumulation rounding -- the same error class as an fp32 FMA
// chain, at matrix-core speed.  The workspace holds the fp32 weights in MFMA operand order (made on
// the first smoe_route after smoe_bind); they are cut in registers, eleven vector instructions a
// pair, because what bounds the kernel is the bytes a compute unit can take in (one workgroup needs
// the whole router): four per weight instead of the six of three stored pieces.
//
// One workgroup = 8 waves = TB blocks of 32 tokens x all experts.  The tokens are staged in LDS
// (read straight into operand order, an instruction would touch 32 rows with 32 bytes each: twice
// the cache accesses of the weights per byte).  The reduction (d_model) is cut into NS slices (8 up
// to 32 experts, 4 above) and, above 32 experts, the expert blocks into two groups: wave = (slice,
// group).  The partial logits meet in LDS, token by token with the experts side by side, and are
// added in slice order (fixed, so results are reproducible).
//
// Epilogue: 16 lanes per token, so a wave finishes four tokens at once; the maximum, the masked
// maximum, their lowest indexes and the softmax sums are rotations within the 16 lanes, without a
// barrier.
#pragma once

#include "smoe_internal.h"
#include "wave_ops.h"

typedef __bf16 smoe_bf16x8 __attribute__((ext_vector_type(8)));
typedef float smoe_f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ smoe_bf16x8 smoe_frag(uint4 v) {
    union { uint4 u; smoe_bf16x8 b; } c;
    c.u = v;
    return c.b;
}

constexpr int SMOE_RT = 32;       // tokens per token block (one MFMA operand)

struct smoe_route_args {
    const void* x;                // bf16 or fp32 [T, d]
    const uint4* wr;              // bf16 layers: fp32 [expert block][reduction step][2 halves][lane][4]
    const float* wrow;            // fp32 layers: the caller's [E, d]
    const int32_t* e2s;
    int T, d, E, gate_mode;
    int32_t* orig_expert;
    float* orig_gate;
    int32_t* slot;
    float* gate;
    float* xnorm;
    int32_t* hist32;              // tokens per slot of every 32-token block, or NULL
    int K;
};

constexpr int SMOE_ROUTE_KC = 1024;   // columns of x staged together

// NEB: 32-expert blocks the instance is compiled for (1, 2, 4 or 8; surplus blocks are skipped).
template <int NEB, int TB>
struct smoe_route_shape {
    static constexpr int NS = NEB == 1 ? 8 : 4;            // slices of the reduction
    static constexpr int NEBH = NEB * NS / 8;              // expert blocks per group
    static constexpr int EP = NEB * 32;
    static constexpr int LDP = EP + 4;                     // padded token row of partial logits: 16-byte stores hit all banks
    static constexpr int NTOK = TB * SMOE_RT;
    // the staged tokens, and after them the partial logits and sums of squares, in the same place
    static size_t lds_bytes(int d) {
        const size_t part = (size_t)(NS * NTOK * LDP + NS * 2 * NTOK) * 4;
        const size_t xs = (size_t)NTOK * ((d < SMOE_ROUTE_KC ? d : SMOE_ROUTE_KC) + 8) * 2;
        return part > xs ? part : xs;
    }
};

// What the router finds for one token.
struct smoe_choice {
    int expert, slot;
    float orig_gate, gate;
};

constexpr int smoe_route_chunks(int NEB) { return (NEB * 32 + 63) / 64; }   // chunks of 64 experts; a lane of the epilogue has 4 of each

// Slots of this lane's experts, -1 if not resident; sub = the lane's place among the 16 of its token.
template <int NEB>
__device__ __forceinline__ void smoe_route_slots(int (&sl)[smoe_route_chunks(NEB)][4], const smoe_route_args& a, int sub) {
#pragma unroll
    for (int c = 0; c < smoe_route_chunks(NEB); ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int e = 64 * c + 4 * sub + j;
            sl[c][j] = e < a.E ? a.e2s[e] : -1;
        }
}

// Choice of one token by its 16 lanes: row = its partial logits of slice 0, those of the next slice slice_stride further.
template <int NEB, int NS>
__device__ __forceinline__ smoe_choice smoe_route_token(const float* row, int slice_stride, const int (&sl)[smoe_route_chunks(NEB)][4],
                                                        int E, int gate_mode, int sub) {
    constexpr int EC = smoe_route_chunks(NEB), EP = NEB * 32;
    float v[EC][4];
#pragma unroll
    for (int c = 0; c < EC; ++c) {
        const int e = 64 * c + 4 * sub;
        const float* col = row + min(e, EP - 4);
        float4 s = *(const float4*)col;
#pragma unroll
        for (int q = 1; q < NS; ++q) {                     // fixed order
            const float4 o = *(const float4*)(col + q * slice_stride);
            s.x += o.x; s.y += o.y; s.z += o.z; s.w += o.w;
        }
        v[c][0] = s.x; v[c][1] = s.y; v[c][2] = s.z; v[c][3] = s.w;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[c][j] = e + j < E ? v[c][j] : -INFINITY;   // past E: never wins, adds exp(-inf) = 0
    }
    float best = -INFINITY, rbest = -INFINITY;
#pragma unroll
    for (int c = 0; c < EC; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            best = fmaxf(best, v[c][j]);
            rbest = fmaxf(rbest, sl[c][j] >= 0 ? v[c][j] : -INFINITY);
        }
    best = smoe_row_max(best);
    rbest = smoe_row_max(rbest);
    int bi = 0x7fffffff, rb = 0x7fffffff;                  // lowest expert id that holds the maximum; (id, slot) of the masked one
    float z = 0.f, zr = 0.f;
#pragma unroll
    for (int c = EC - 1; c >= 0; --c)
#pragma unroll
        for (int j = 3; j >= 0; --j) {
            const int e = 64 * c + 4 * sub + j;
            bi = v[c][j] == best ? e : bi;
            rb = sl[c][j] >= 0 && v[c][j] == rbest ? (e << 8 | sl[c][j]) : rb;
            const float p = expf(v[c][j] - best);
            z += p;
            zr += sl[c][j] >= 0 ? p : 0.f;
        }
    bi = smoe_row_min(bi);
    rb = smoe_row_min(rb);
    z = smoe_row_sum(z);
    if (gate_mode == SMOE_GATE_RENORM) zr = smoe_row_sum(zr);
    smoe_choice r;
    r.expert = bi;
    r.slot = rb == 0x7fffffff ? 0 : rb & 255;              // a token whose logits are all NaN: slot 0, a NaN gate
    r.orig_gate = 1.0f / z;
    r.gate = expf(rbest - best) / (gate_mode == SMOE_GATE_RENORM ? zr : z);
    return r;
}

// Writes a token's results; sq = its partial sums of squares, stride apart, two halves of every slice.
template <int NS>
__device__ __forceinline__ void smoe_store_choice(const smoe_route_args& a, int tok, const smoe_choice& c, const float* sq, int stride) {
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < 2 * NS; ++q) ss += sq[q * stride];
    a.orig_expert[tok] = c.expert;
    a.orig_gate[tok] = c.orig_gate;
    a.slot[tok] = c.slot;
    a.gate[tok] = c.gate;
    a.xnorm[tok] = sqrtf(ss);
}

// The partial logits of the 8 waves meet in LDS and every token's results are written.
template <int NEB, int TB>
__device__ __forceinline__ void smoe_route_finish(const int block, const smoe_route_args& a,
                                                  smoe_f32x16 (&acc)[smoe_route_shape<NEB, TB>::NEBH][TB], float (&sq)[TB],
                                                  float* smem) {
    using S = smoe_route_shape<NEB, TB>;
    constexpr int NS = S::NS, NEBH = S::NEBH, LDP = S::LDP, RT = SMOE_RT, NTOK = S::NTOK;
    float* part = smem;                                    // [NS][NTOK][LDP] partial logits
    float* sqp = smem + NS * NTOK * LDP;                   // [NS][2 halves][NTOK] partial sums of squares
    __shared__ int32_t s_hist[TB * 256];                   // tokens per block and slot
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int slice = wave % NS, group = wave / NS;
    const int tw0 = block * NTOK, neb = (a.E + 31) >> 5;
    if (a.hist32)
        for (int i = tid; i < TB * 256; i += 512) s_hist[i] = 0;
    const int sub = lane & 15;                             // the 16 lanes of a token
    int sl[smoe_route_chunks(NEB)][4];
    smoe_route_slots<NEB>(sl, a, sub);

    __syncthreads();                                       // the partial logits take the staged tokens' place
    // accumulator register i of lane l: expert 8*(i/4) + 4*(l/32) + i%4 (+32 per block), token l%32
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
        float* row = part + (slice * NTOK + tb * RT + (lane & 31)) * LDP + 4 * (lane >> 5);
#pragma unroll
        for (int b = 0; b < NEBH; ++b) {
            if (group * NEBH + b >= neb) continue;         // a surplus block
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(float4*)(row + (group * NEBH + b) * 32 + 8 * q) =
                    make_float4(acc[b][tb][4 * q], acc[b][tb][4 * q + 1], acc[b][tb][4 * q + 2], acc[b][tb][4 * q + 3]);
        }
        if (group == 0) sqp[(slice * 2 + (lane >> 5)) * NTOK + tb * RT + (lane & 31)] = sq[tb];
    }
    __syncthreads();

    // epilogue: lanes 16q .. 16q + 15 of wave w own token 4w + q of every 32-token block
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
        const int t = tb * RT + wave * 4 + (lane >> 4), tok = tw0 + t;
        const smoe_choice c = smoe_route_token<NEB, NS>(part + t * LDP, NTOK * LDP, sl, a.E, a.gate_mode, sub);
        if (sub == 0 && tok < a.T) {
            smoe_store_choice<NS>(a, tok, c, sqp + t, NTOK);
            if (a.hist32) atomicAdd(&s_hist[tb * 256 + c.slot], 1);   // integer: order cannot matter
        }
    }
    if (a.hist32) {                                        // tokens per slot in each block, for the ranking that follows
        __syncthreads();
        for (int i = tid; i < TB * a.K; i += 512) {
            const int tb = i / a.K, k = i - tb * a.K;
            if (tw0 + tb * RT < a.T) a.hist32[((size_t)block * TB + tb) * a.K + k] = s_hist[tb * 256 + k];
        }
    }
}

// Eight fp32 weights -> their hi, mid and lo pieces as three operands of a bf16 product.
__device__ __forceinline__ void smoe_cut_weights(const uint4 (&w)[2], uint4 (&pc)[3]) {
    const uint32_t f[8] = {w[0].x, w[0].y, w[0].z, w[0].w, w[1].x, w[1].y, w[1].z, w[1].w};
    uint32_t p[3][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float u = __uint_as_float(f[2 * q]), v = __uint_as_float(f[2 * q + 1]);
#pragma unroll
        for (int s3 = 0; s3 < 3; ++s3) {                   // upper halves packed; the remainders are exact
            p[s3][q] = __builtin_amdgcn_perm(__float_as_uint(v), __float_as_uint(u), 0x07060302u);
            u -= __uint_as_float(__float_as_uint(u) & 0xFFFF0000u);
            v -= __uint_as_float(__float_as_uint(v) & 0xFFFF0000u);
        }
    }
#pragma unroll
    for (int s3 = 0; s3 < 3; ++s3) pc[s3] = make_uint4(p[s3][0], p[s3][1], p[s3][2], p[s3][3]);
}

// Adds the squares of eight bf16 values to sq, in order.
__device__ __forceinline__ void smoe_add_squares(float& sq, const uint4& xv) {
    const uint32_t xw[4] = {xv.x, xv.y, xv.z, xv.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float l = __uint_as_float(xw[q] << 16), h = __uint_as_float(xw[q] & 0xFFFF0000u);
        sq = fmaf(l, l, sq);
        sq = fmaf(h, h, sq);
    }
}

// MULTI: d_model takes more than one chunk; the first round of the next chunk's loads is then in flight
// while this one is multiplied.
template <int NEB, int TB, bool MULTI>
__device__ __forceinline__ void smoe_route_mfma_body(const int block, const smoe_route_args& a, float* smem) {
    using S = smoe_route_shape<NEB, TB>;
    constexpr int NS = S::NS, NEBH = S::NEBH, RT = SMOE_RT, NTOK = S::NTOK;
    constexpr int KC = SMOE_ROUTE_KC;
    // Reduction steps whose weights are fetched together; two such groups are in flight.  More of them only queue at the
    // compute unit's memory path: groups of 4 and 3 took 0.3 .. 1.2 us more a layer (16384 tokens, 128 experts, four layers 1384
    // and 1376 us), two groups of 6 asked for before the tokens are staged 1.4 us more (T = 777, 64 experts).
    constexpr int G = NEBH == 1 ? 3 : 2;
    uint16_t* xs = (uint16_t*)smem;                        // [NTOK][ldx] columns of x

    // wave index as a scalar: loop bounds that guard MFMAs must be wave-uniform for the
    // compiler as well (an MFMA under a lane mask still runs for every lane)
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int slice = wave % NS, group = wave / NS;
    const int tw0 = block * NTOK;                          // first token of the workgroup
    const int neb = (a.E + 31) >> 5, nkb = a.d >> 4;
    const uint4* wp[NEBH];
#pragma unroll
    for (int b = 0; b < NEBH; ++b) wp[b] = a.wr + (size_t)min(group * NEBH + b, neb - 1) * nkb * 2 * 64 + lane;

    smoe_f32x16 acc[NEBH][TB];
    float sq[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
        sq[tb] = 0.f;
#pragma unroll
        for (int b = 0; b < NEBH; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[b][tb][i] = 0.f;
    }
    const int ldx = min(a.d, KC) + 8;                      // conflict-free 16-byte operand reads
    constexpr int PPT = 8;                                 // 16-byte pieces of x a thread fetches together
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // (an array of uint4 would live in scratch memory across chunks)
    u32x4 v[PPT];
    const int rows = min(NTOK, a.T - tw0);                 // rows past the batch stay as they are: their logits are not used
    auto fetch_x = [&](int k0, int i0) {                   // pieces past the end repeat the last one
        const int cpr = min(KC, a.d - k0) >> 3;            // pieces per row
#pragma unroll
        for (int q = 0; q < PPT; ++q) {
            const int idx = min(i0 + q * 512, rows * cpr - 1), r = idx / cpr, c = idx - r * cpr;
            v[q] = *(const u32x4*)((const uint16_t*)a.x + (size_t)(tw0 + r) * a.d + k0 + c * 8);
        }
    };
    for (int k0 = 0; k0 < a.d; k0 += KC) {                 // (one pass up to d_model = 1024)
        const int kc = min(KC, a.d - k0), steps = kc >> 4;
        const int per = (steps + NS - 1) / NS;
        const int lo = min(slice * per, steps), hi = min(lo + per, steps);   // this wave's steps of the chunk
        const int n = hi - lo;
        const uint4* w0[NEBH];
#pragma unroll
        for (int b = 0; b < NEBH; ++b) w0[b] = wp[b] + (size_t)((k0 >> 4) + lo) * 2 * 64;
        uint4 wA[G][NEBH][2], wB[G][NEBH][2];
        auto fetch = [&](uint4 (&w)[G][NEBH][2], int g0) {
#pragma unroll
            for (int i = 0; i < G; ++i)                    // past the end: reloaded, not used
#pragma unroll
                for (int b = 0; b < NEBH; ++b)
#pragma unroll
                    for (int h = 0; h < 2; ++h) w[i][b][h] = w0[b][(size_t)(max(min(g0 + i, n - 1), 0) * 2 + h) * 64];
        };
        // A slice may have no step of this chunk (n = 0): its w0 is then one step past the expert block, so
        // nothing is fetched and nothing multiplied (whatever lies there times a zero operand need not be zero).
        if (n > 0) fetch(wA, 0);                           // on their way while the tokens are staged
        if (k0) __syncthreads();                           // the previous chunk has been used up
        const int cpr = kc >> 3;                           // 16-byte pieces per row
        for (int i0 = tid; i0 < rows * cpr; i0 += 512 * PPT) {
            if (!MULTI || !k0 || i0 != tid) fetch_x(k0, i0);
#pragma unroll
            for (int q = 0; q < PPT; ++q) {
                const int idx = min(i0 + q * 512, rows * cpr - 1), r = idx / cpr, c = idx - r * cpr;
                *(u32x4*)&xs[r * ldx + c * 8] = v[q];
            }
        }
        __syncthreads();
        if (MULTI && k0 + KC < a.d) fetch_x(k0 + KC, tid);
        const uint16_t* xrow = xs + (lane & 31) * ldx + (lane >> 5) * 8 + lo * 16;
        auto consume = [&](uint4 (&w)[G][NEBH][2], int g0) {
#pragma unroll
            for (int i = 0; i < G; ++i) {
                smoe_bf16x8 xf[TB];
#pragma unroll
                for (int tb = 0; tb < TB; ++tb) {
                    uint4 xv = *(const uint4*)(xrow + tb * RT * ldx + max(min(g0 + i, n - 1), 0) * 16);
                    if (g0 + i >= n) xv = make_uint4(0, 0, 0, 0);   // steps past the end multiply by a zero operand
                    xf[tb] = smoe_frag(xv);
                    if (group == 0) smoe_add_squares(sq[tb], xv);   // the groups read the same tokens: one of them adds the squares
                }
#pragma unroll
                for (int b = 0; b < NEBH; ++b) {
                    uint4 pc[3];
                    smoe_cut_weights(w[i][b], pc);
                    // smallest terms first, so they are not absorbed by the large partial sums
#pragma unroll
                    for (int s3 = 2; s3 >= 0; --s3)
#pragma unroll
                        for (int tb = 0; tb < TB; ++tb)
                            acc[b][tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                smoe_frag(pc[s3]), xf[tb], acc[b][tb], 0, 0, 0);
                }
            }
        };
        int g0 = 0;
        for (; n - g0 > 2 * G; g0 += 2 * G) {
            fetch(wB, g0 + G);
            __builtin_amdgcn_sched_barrier(0);             // the next group's loads are issued first
            consume(wA, g0);
            __builtin_amdgcn_sched_barrier(0);
            fetch(wA, g0 + 2 * G);
            __builtin_amdgcn_sched_barrier(0);
            consume(wB, g0 + G);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (n - g0 > G) {
            fetch(wB, g0 + G);
            __builtin_amdgcn_sched_barrier(0);
            consume(wA, g0);
            __builtin_amdgcn_sched_barrier(0);
            consume(wB, g0 + G);
        } else if (n > 0) {
            consume(wA, g0);
        }
    }
    smoe_route_finish<NEB, TB>(block, a, acc, sq, smem);
}

// fp32 activations: the same split of the work with fp32 matrix products (v_mfma_f32_32x32x2_f32).
// A lane holds four consecutive reduction elements of its row, the two halves of the wave eight: one
// 16-byte load per operand feeds four MFMAs.  A product of 32 x 32 x 2 takes 64 cycles, so the operands
// come straight from memory.
template <int NEB>
__device__ __forceinline__ void smoe_route_f32_body(const int block, const smoe_route_args& a, float* smem) {
    using S = smoe_route_shape<NEB, 1>;
    constexpr int NS = S::NS, NEBH = S::NEBH;
    constexpr int G = NEBH == 1 ? 6 : NEBH == 2 ? 4 : 2;   // steps of 8 reduction elements fetched together
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int slice = wave % NS, group = wave / NS, half4 = (lane >> 5) * 4;
    const int steps = (a.d + 7) >> 3, per = (steps + NS - 1) / NS;
    const int lo = min(slice * per, steps), n = min(lo + per, steps) - lo;
    const float* xp = (const float*)a.x + (size_t)min(block * SMOE_RT + (lane & 31), a.T - 1) * a.d;
    const float* wp[NEBH];
    smoe_f32x16 acc[NEBH][1];
#pragma unroll
    for (int b = 0; b < NEBH; ++b) {
        wp[b] = a.wrow + (size_t)min((group * NEBH + b) * 32 + (lane & 31), a.E - 1) * a.d;   // experts past E: computed, not used
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[b][0][i] = 0.f;
    }
    float sq[1] = {0.f};
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    f32x4 xA[G], wA[G][NEBH], xB[G], wB[G][NEBH];
    auto fetch = [&](f32x4 (&xv)[G], f32x4 (&w)[G][NEBH], int g0) {
#pragma unroll
        for (int i = 0; i < G; ++i) {                      // past the end: read again, not used
            const int k = min((lo + max(min(g0 + i, n - 1), 0)) * 8 + half4, a.d - 4);
            xv[i] = *(const f32x4*)(xp + k);
#pragma unroll
            for (int b = 0; b < NEBH; ++b) w[i][b] = *(const f32x4*)(wp[b] + k);
        }
    };
    auto step = [&](f32x4& xv, f32x4 (&w)[NEBH], int k) {
        const bool in = k + half4 < a.d;                   // d_model may end in the middle of a step
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float xj = in ? xv[j] : 0.f;
            sq[0] = fmaf(xj, xj, sq[0]);
#pragma unroll
            for (int b = 0; b < NEBH; ++b) acc[b][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[b][j], xj, acc[b][0], 0, 0, 0);
        }
    };
    auto consume = [&](f32x4 (&xv)[G], f32x4 (&w)[G][NEBH], int g0) {
#pragma unroll
        for (int i = 0; i < G; ++i) step(xv[i], w[i], (lo + g0 + i) * 8);
    };
    auto consume_tail = [&](f32x4 (&xv)[G], f32x4 (&w)[G][NEBH], int g0) {   // nothing is fetched after this
#pragma unroll
        for (int i = 0; i < G; ++i) {
            if (g0 + i >= n) break;                        // uniform
            step(xv[i], w[i], (lo + g0 + i) * 8);
        }
    };
    fetch(xA, wA, 0);
    int g0 = 0;
    for (; n - g0 > 2 * G; g0 += 2 * G) {
        fetch(xB, wB, g0 + G);
        __builtin_amdgcn_sched_barrier(0);
        consume(xA, wA, g0);
        __builtin_amdgcn_sched_barrier(0);
        fetch(xA, wA, g0 + 2 * G);
        __builtin_amdgcn_sched_barrier(0);
        consume(xB, wB, g0 + G);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (n - g0 > G) {
        fetch(xB, wB, g0 + G);
        __builtin_amdgcn_sched_barrier(0);
        consume(xA, wA, g0);
        __builtin_amdgcn_sched_barrier(0);
        consume_tail(xB, wB, g0 + G);
    } else {
        consume_tail(xA, wA, g0);
    }
    smoe_route_finish<NEB, 1>(block, a, acc, sq, smem);
}
