// smoe_route: router product, softmax, original top-1, masked top-1 and |x|.
//
// For every token:  logit = x . Wr^T,  p = softmax(logit) over all E experts,
// e* = argmax logit (SwapMoE, Background: the expert with max G(x)_i), and the
// Masked-Gating choice s = argmax over resident experts only (Section 3.1,
// Figure 4(b)).  |x|_2 is produced on the way because x is already in flight
// (it is the first factor of the importance score, Eq. 1).
//
// The kernels' bodies are in route_mfma.h: one workgroup owns 32 tokens (64 in large bf16 batches)
// and all E experts.

#include "route_mfma.h"

namespace {

// Wr [E, d] fp32 -> units [eb][kb][half][lane] of 4 fp32: expert eb*32 + lane%32, reduction index
// kb*16 + (lane/32)*8 + half*4 + i.  Experts past E are zero.
__global__ __launch_bounds__(256) void pack_router_kernel(const float* __restrict__ Wr, int E, int d,
                                                          float4* __restrict__ out, int neb) {
    const int unit = blockIdx.x * 256 + threadIdx.x;       // ((eb * nkb + kb) * 2 + half) * 64 + lane
    const int nkb = d >> 4;
    if (unit >= neb * nkb * 128) return;
    const int lane = unit & 63, half = (unit >> 6) & 1, kb = (unit >> 7) % nkb, eb = (unit >> 7) / nkb;
    const int e = eb * 32 + (lane & 31), k0 = kb * 16 + (lane >> 5) * 8 + half * 4;
    out[unit] = e < E ? *(const float4*)&Wr[(size_t)e * d + k0] : make_float4(0, 0, 0, 0);
}

template <int NEB, int TB, bool MULTI>
__global__ __launch_bounds__(512) void route_mfma_kernel(const smoe_route_args a) {
    extern __shared__ __align__(16) float smem[];
    smoe_route_mfma_body<NEB, TB, MULTI>(blockIdx.x, a, smem);
}

template <int NEB, int TB, bool MULTI>
int launch_mfma_multi(const smoe_route_args& a, hipStream_t s) {
    using S = smoe_route_shape<NEB, TB>;
    const size_t lds = S::lds_bytes(a.d);
    static smoe_lds_raised raised;
    if (int rc = raised.ensure((const void*)route_mfma_kernel<NEB, TB, MULTI>, lds, (int)S::lds_bytes(SMOE_ROUTE_KC))) return rc;
    constexpr int NTOK = SMOE_RT * TB;
    hipLaunchKernelGGL((route_mfma_kernel<NEB, TB, MULTI>), dim3((a.T + NTOK - 1) / NTOK), dim3(512), lds, s, a);
    return smoe_check_hip(hipGetLastError(), "smoe_route launch");
}

template <int NEB, int TB>
int launch_mfma_tb(const smoe_route_args& a, hipStream_t s) {
    // The prefetch across chunks pays for two token blocks, whose staging takes two rounds (E = 8, T = 16384: d_model =
    // 2048 26.1 -> 22.7 us, 4096 46.6 -> 38.1), not for one (d_model = 2048, T = 32 10.0 -> 10.5), and takes registers that
    // more than 64 experts do not leave (E = 128, d_model = 1056, T = 16384 27.8 us without, 33.1 with)
    if constexpr (TB == 2 && NEB <= 2) {
        if (a.d > SMOE_ROUTE_KC) return launch_mfma_multi<NEB, TB, true>(a, s);
    }
    return launch_mfma_multi<NEB, TB, false>(a, s);
}

template <int NEB>
int launch_mfma(const smoe_route_args& a, hipStream_t s) {
    // more 32-token blocks than compute units (256): two blocks per workgroup, so that the router's
    // weights are fetched half as often, while the partial-logit tile of 64 tokens still fits the
    // LDS (up to 128 experts)
    if constexpr (NEB <= 4) {
        if ((a.T + SMOE_RT - 1) / SMOE_RT > 256) return launch_mfma_tb<NEB, 2>(a, s);
    }
    return launch_mfma_tb<NEB, 1>(a, s);
}

template <int NEB>
__global__ __launch_bounds__(512) void route_f32_kernel(const smoe_route_args a) {
    extern __shared__ __align__(16) float smem[];
    smoe_route_f32_body<NEB>(blockIdx.x, a, smem);
}

template <int NEB>
int launch_f32(const smoe_route_args& a, hipStream_t s) {
    const size_t lds = smoe_route_shape<NEB, 1>::lds_bytes(0);
    static smoe_lds_raised raised;
    if (int rc = raised.ensure((const void*)route_f32_kernel<NEB>, lds, (int)lds)) return rc;
    hipLaunchKernelGGL(route_f32_kernel<NEB>, dim3((a.T + SMOE_RT - 1) / SMOE_RT), dim3(512), lds, s, a);
    return smoe_check_hip(hipGetLastError(), "smoe_route launch");
}

}  // namespace

int smoe_launch_split_router(const smoe_layer* L, hipStream_t s) {
    const int neb = (L->cfg.E + 31) / 32;
    const int units = neb * (L->cfg.d_model >> 4) * 128;
    hipLaunchKernelGGL(pack_router_kernel, dim3((units + 255) / 256), dim3(256), 0, s, L->router_w, L->cfg.E,
                       L->cfg.d_model, (float4*)L->d_router_split, neb);
    return smoe_check_hip(hipGetLastError(), "smoe_route: router re-layout launch");
}

int smoe_launch_route(const smoe_layer* L, const void* x, int T, int32_t* orig_expert,
                      float* orig_gate, int32_t* slot, float* gate, float* xnorm, int32_t* hist32,
                      hipStream_t s) {
    const smoe_config& c = L->cfg;
    const smoe_route_args a{x, (const uint4*)L->d_router_split, L->router_w, L->d_expert_to_slot, T, c.d_model, c.E, c.gate_mode,
                            orig_expert, orig_gate, slot, gate, xnorm, hist32, c.K};
    const bool f32 = c.dtype == SMOE_F32;
    if (c.E <= 32) return f32 ? launch_f32<1>(a, s) : launch_mfma<1>(a, s);
    if (c.E <= 64) return f32 ? launch_f32<2>(a, s) : launch_mfma<2>(a, s);
    if (c.E <= 128) return f32 ? launch_f32<4>(a, s) : launch_mfma<4>(a, s);
    return f32 ? launch_f32<8>(a, s) : launch_mfma<8>(a, s);
}
