// Declarations shared by the grouped bf16 products (ffn_bf16.hip, ffn_ring.hip, ffn_split.hip).
#pragma once

#include "smoe_internal.h"

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Optional fusion of the permute and combine steps into the two products
// (perm == nullptr: plain products on x_perm / y_perm).
//   first product:  row r of the sorted order is read from x[perm[r]] (no x_perm);
//   second product: row r is written to out[perm[r]] = gate[perm[r]] * y (+ residual[perm[r]]),
//                   i.e. y = G(x)_i E_i(x) lands in token order (no y_perm).
struct FuseArgs {
    const int32_t* phys;      // virtual slot -> physical weight slot, [nslots]; NULL = identity (no spare slots)
    const int32_t* perm;
    const float* gate;
    const uint16_t* residual;
    bool past;                // first product: hidden activations are stored past the caches (kernels that know how to)
};

// ffn_ring.hip: tiles of at most `blocks` x 32 tokens and `blocks` x 32 features, blocks = 4 or 8
bool smoe_ring_applies(bool first, int R, int T);
int smoe_launch_ring(int blocks, bool first, const uint16_t* X, const void* Wp, const int32_t* offsets, int nslots,
                     uint16_t* Y, int R, int N, int T, const FuseArgs& fz, int cus_per_die, hipStream_t s, hipEvent_t e0,
                     hipEvent_t e1);

// ffn_split.hip: second product, reduction split over the waves, tiles of up to 128 x 128
int smoe_launch_split(const uint16_t* X, const void* Wp, const int32_t* offsets, int nslots, uint16_t* Y, int R, int N, int T,
                      const FuseArgs& fz, int cus_per_die, hipStream_t s, hipEvent_t e0, hipEvent_t e1);
