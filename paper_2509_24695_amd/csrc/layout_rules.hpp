// What a token tensor's strides mean for the kernels: whether 32-bit offsets reach its heads, and in which order workgroups
// are dealt to it.  Plain C++ (no device code), shared by the launcher and a host-side test.
#pragma once

#include <stdint.h>

namespace sv {

// The matrix-core kernels address a head's tokens with 32-bit byte offsets below 2^31: what a head spans, and what one tile of 64 rows
// spans (rows past the end are reached by address before they are dropped).
inline bool head_offsets_fit(int64_t N, int64_t stride_n, int elem_bytes)
{
    constexpr int64_t kLimit = int64_t(1) << 31;
    const int64_t rows = N > 64 ? N : 64;
    return stride_n <= (kLimit - 1) / (rows * elem_bytes);   // rows * stride_n * elem_bytes < kLimit, without overflow
}

}  // namespace sv
