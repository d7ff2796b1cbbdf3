// Exchanges between the lanes of a wave without LDS (device code, gfx950).
#pragma once
#include <hip/hip_runtime.h>

namespace hdg {
namespace {

// Lane pairs (l, l ^ 16) or (l, l ^ 32) by the gfx950 row swaps: with both
// operands the same register, the two results hold, lane by lane, the lane's own
// value and its partner's (in some order), which is all a symmetric combine needs.
template <int W> __device__ inline void swap_pair(unsigned x, unsigned &a, unsigned &b) {
    const auto p = (W == 16) ? __builtin_amdgcn_permlane16_swap(x, x, false, false)
                             : __builtin_amdgcn_permlane32_swap(x, x, false, false);
    a = p[0];
    b = p[1];
}

// Maximum over groups of N lanes (a power of two): quad permutations and rotations inside
// each 16-lane row, then the row swaps.  No step goes through LDS.
template <int CTRL> __device__ inline unsigned max_dpp(unsigned v) {
    return max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, true));
}
template <int W> __device__ inline unsigned max_swap(unsigned v) {
    unsigned a, b;
    swap_pair<W>(v, a, b);
    return max(a, b);
}
template <int N> __device__ inline unsigned lanes_max(unsigned v) {
    if (N > 1) v = max_dpp<0xB1>(v);
    if (N > 2) v = max_dpp<0x4E>(v);
    if (N > 4) v = max_dpp<0x124>(v);
    if (N > 8) v = max_dpp<0x128>(v);
    if (N > 16) v = max_swap<16>(v);
    if (N > 32) v = max_swap<32>(v);
    return v;
}
// The upper word of a value >= 0: a larger one is a larger value.
__device__ inline unsigned upper_word(double x) { return (unsigned)((unsigned long long)__double_as_longlong(x) >> 32); }
__device__ inline unsigned upper_word(float x) { return __float_as_uint(x); }

}  // namespace
}  // namespace hdg
