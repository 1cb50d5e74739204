// Price of a tile shape of the splitting kernel (ffn_split.hip).  The kernel picks its shape by it; plain C++, for the host as well.
#pragma once

// `rounds` of items per workgroup, tiles of w feature and h token blocks of 32, `per` steps of 16 in a wave's part of the reduction:
// a step's blocks and products, and the meeting of the parts, in 2.2 ns.  Fitted to 150 batches (13 shapes from 5 slots of 256 x 768
// to 64 of 768 x 3072, T = 132 .. 8192; 4 % off at the median).  Not an integer: 2^24 tokens of 2^16 x 2^18 are 2^40.
constexpr float smoe_split_price(float rounds, float per, int w, int h) {
    return rounds * (per * (float)(15 * (w + h) + 4 * w * h) + (float)(157 * w * h));
}
