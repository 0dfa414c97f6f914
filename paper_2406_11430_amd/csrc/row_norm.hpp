// Squared norm of one cached row in the library's fixed summation order (16 chunks of consecutive elements,
// each left to right, then a balanced tree over neighbouring chunks), for the lane layouts in
// which the kernels hold rows.  All lanes of a row group must be active.
#pragma once
#include "l2kv_device.hpp"

namespace l2kv {

// Rows of 256 and 512 bytes, one per 16 lanes in 16-byte pieces (Pieces): the same sum in all 16 lanes.
template <typename E, int D>
__device__ __forceinline__ float chunked_sum_of_squares(const float (&x)[Slice<E, D>::kElems]) {
#pragma clang fp contract(off)
    using S = Slice<E, D>;
    using P = Pieces<S::kWords>;
    static_assert(P::kCount <= 2, "rows of at most 512 bytes");
    if constexpr (P::kCount == 1) {
        float acc = x[0] * x[0];
#pragma unroll
        for (int e = 1; e < S::kElems; ++e) {
            float sq = x[e] * x[e];
            acc = acc + sq;
        }
        return row16_tree_sum(acc);
    } else {
        constexpr int n = S::kElems / 2;              // elements per piece; x[s * n ..] = piece slot s
        float t[2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            // first half of a chunk (valid in even lanes): 0 + x0^2 is x0^2 exactly
            float acc = 0.f;
#pragma unroll
            for (int e = 0; e < n; ++e) {
                float sq = x[s * n + e] * x[s * n + e];
                acc = acc + sq;
            }
            // second half (valid in odd lanes): continue from the even neighbour's sum.  Even
            // lanes continue from their own sum; their result is overwritten below.  (No
            // select on the lane parity here: the cross-lane read must run with all lanes
            // active.)
            float full = dpp_read<kDppQuadEven>(acc);
#pragma unroll
            for (int e = 0; e < n; ++e) {
                float sq = x[s * n + e] * x[s * n + e];
                full = full + sq;
            }
            // chunk sums sit in the odd lanes: copy to the even neighbour, then the tree
            // over the 8 chunks of this slot
            float v = dpp_read<kDppQuadOdd>(full);
            v = v + dpp_read<kDppXor2>(v);
            v = v + dpp_read<kDppHalfMirror>(v);
            v = v + dpp_read<kDppMirror>(v);
            t[s] = v;
        }
        return t[0] + t[1];
    }
}

// Rows of 128 bytes (bf16, 64 elements), two per 16 lanes: the sum of a row in all of its 8 lanes.  A lane holds
// two of the 16 chunks (4 elements each).
__device__ __forceinline__ float row_pair_sum_of_squares(const Words<4>& raw) {
#pragma clang fp contract(off)
    float x[8];
    widen<BF16, 128>(raw, x);             // 4 words -> 8 values in element order
    float a = x[0] * x[0];
    float b = x[4] * x[4];
#pragma unroll
    for (int e = 1; e < 4; ++e) {
        float sa = x[e] * x[e];
        float sb = x[4 + e] * x[4 + e];
        a = a + sa;
        b = b + sb;
    }
    float v = a + b;                      // chunks 2j and 2j+1
    v = v + dpp_read<kDppXor1>(v);
    v = v + dpp_read<kDppXor2>(v);
    v = v + dpp_read<kDppHalfMirror>(v);  // the 8 lanes of this row
    return v;
}

}  // namespace l2kv
