// Shared device-side helpers for the gfx950 linear-attention kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "layout_rules.hpp"
#include "tile_walk.hpp"

namespace sv {

constexpr int kWave = 64;            // CDNA wavefront width
constexpr int kThreads = 256;        // four waves, the workgroup of the kernels that name no other

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Element strides of a [B][H][N][d] token tensor (d contiguous).
struct TokStrides {
    int64_t b, h, n;
};

// ---- bf16 <-> fp32 on raw bit patterns -------------------------------------------------

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float bf16_bits_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Round to nearest even (hardware conversion on gfx950).
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float x) {
    return __builtin_bit_cast(uint16_t, (__bf16)x);
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    f32x2 f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}

// ReLU feature map on two packed bf16 values: a negative bf16 is a negative
// int16, so a signed 16-bit max with zero clears it (and turns -0 into +0).
__device__ __forceinline__ uint32_t relu_bf16x2(uint32_t w) {
    const s16x2 zero = {0, 0};
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, w), zero));
}
__device__ __forceinline__ u32x4 relu_bf16x8(u32x4 v) {
    v.x = relu_bf16x2(v.x); v.y = relu_bf16x2(v.y); v.z = relu_bf16x2(v.z); v.w = relu_bf16x2(v.w);
    return v;
}

// ---- RoPE after ReLU (numerator of the Sec. 3.2 equation) ----------------------------------------
// A rotation table row holds d/2 (cos, sin) fp32 pairs of one token; feature pair
// (2p, 2p+1) is turned by angle p:  y[2p] = x[2p] cos - x[2p+1] sin,  y[2p+1] = x[2p] sin + x[2p+1] cos.
// A 32-bit word of a bf16 token row is exactly one such pair.
__device__ __forceinline__ uint32_t rope_rotate_pair(uint32_t w, float c, float s) {
    const float a = bf16_lo(w), b = bf16_hi(w);
    return pack_bf16x2(a * c - b * s, a * s + b * c);
}
// ---- range-checked streaming access ------------------------------------------------------------
//
// Token tiles are addressed through buffer resources: the hardware compares each
// lane's byte offset with the resource's size, returns zeros for loads at or past
// it and drops such stores.  Ragged tails and tiles past the end of a wave's share
// therefore need no branch, every stage of a software pipeline issues the same
// number of memory instructions, and the compiler can wait for exactly the
// loads it needs (s_waitcnt vmcnt(n)) while later ones stay in flight.  Offsets are
// 32-bit: the host routes tensors whose heads span 2 GiB or more to other kernels.
using rsrc_t = __amdgpu_buffer_rsrc_t;

// `p` must be wave-uniform.  Bytes [0, bytes) are addressable.
__device__ __forceinline__ rsrc_t make_rsrc(const void *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000);
}

// Tokens are read once and outputs written once, so both are marked non-temporal (NT) - except where the cache
// lines of a row are shared with the neighbouring heads of a [B][N][H][d] tensor (see TokenLayout in
// layout_rules.hpp): there the neighbours' accesses have to meet in the L2.
template <bool NT = true> __device__ __forceinline__ u32x4 load_stream16(rsrc_t r, uint32_t off) {
    return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, NT ? 2 : 0);
}
template <bool NT = true> __device__ __forceinline__ void store_stream16(rsrc_t r, uint32_t off, u32x4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, NT ? 2 : 0);
}
// Cached 16-byte load (rotation table: shared by all heads, worth keeping in L2).
__device__ __forceinline__ f32x4 load_cached16(rsrc_t r, uint32_t off) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

// x + the sums of the other lanes of a row of 16: every lane ends with the row's total.  Quad, half-row and row permutations of the vector
// ALU in place of four trips through the LDS crossbar; the same pairs are added.
template <int CTRL> __device__ __forceinline__ float dpp_add(float x)
{
    return x + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float row16_sum(float x)
{
    x = dpp_add<0xb1>(x);      // quad_perm 1,0,3,2
    x = dpp_add<0x4e>(x);      // quad_perm 2,3,0,1
    x = dpp_add<0x141>(x);     // row_half_mirror: the other quad of eight lanes
    return dpp_add<0x140>(x);  // row_mirror: the other eight lanes
}

// ---- typed scalar access used by the generic (any dtype) kernels --------------------------

template <typename T> struct Elem;
template <> struct Elem<float> {
    static __device__ __forceinline__ float load(const float *p) { return *p; }
    static __device__ __forceinline__ void store(float *p, float x) { *p = x; }
};
template <> struct Elem<uint16_t> {   // bf16 bit patterns
    static __device__ __forceinline__ float load(const uint16_t *p) { return bf16_bits_to_f32(*p); }
    static __device__ __forceinline__ void store(uint16_t *p, float x) { *p = f32_to_bf16_bits(x); }
};

// How a grid's workgroups are dealt to (chunk, head) and the heads' walks staggered (kernel argument `order`, see layout_rules.hpp):
constexpr int kDies = 8;              // MI355X: accelerator dies (XCDs), one L2 each; workgroup ids go round them
struct WgRole {
    int c, bh;
    __device__ __forceinline__ WgRole(int C, int order) : c(blockIdx.x), bh(blockIdx.y) {
        if (order & kOrderChunkMajor) chunk_major_role((int)(blockIdx.y * gridDim.x + blockIdx.x), C, (int)gridDim.y, kDies, c, bh);
    }
    // phase key of the walk (see TileWalk)
    __device__ __forceinline__ int phase(int b, int order) const { return order & kOrderLockstep ? 5 * b : bh; }
};

// Tiles of a token range are dealt to chunks as evenly as integers allow:
// chunk c of C owns tiles [c*T/C, (c+1)*T/C).
__host__ __device__ __forceinline__ int chunk_tile_begin(int c, int C, int T) {
    return (int)(((int64_t)c * T) / C);
}

// Orders this wave's LDS traffic for the compiler; the hardware already executes
// one wave's LDS instructions in issue order, so no s_barrier is involved.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Workgroup barrier for handing LDS over between waves.  __syncthreads() alone does not do: the compiler
// has been seen to move LDS reads that stand before it to behind it (two barriers in a row, the reads
// after both), where another wave, already past the barrier, may have overwritten the memory.  The
// assembly statement is opaque to the compiler (no memory operation crosses it in either direction) and
// waits for this wave's LDS traffic, reads included, before the waves meet; the fences keep the meaning
// that __syncthreads() has for global memory.
__device__ __forceinline__ void wg_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// All LDS traffic of this wave is done, then all waves of the workgroup meet.
// Global memory traffic is not waited for.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

}  // namespace sv
