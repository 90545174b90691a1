// State reduction for d = 112 and 128: eight waves on shared tiles, a block of the state each.
//
//   S[k][v] (+)= sum_j phi(K[j][k]) V[j][v],   z[k] (+)= sum_j phi(K[j][k])
//
// (brackets of the linear-attention equation of Sec. 3.2; with ROPE the keys that meet V are
// rotated after the ReLU, the key sum is not).
//
// With the whole state in every wave (wide_state.hpp) the waves' states have to be added up at the end: 192 KB through LDS, 2.3 of the
// 19 to 22 us that 20 heads, 4 680 tokens take.  Here a tile of 64 tokens is loaded once per workgroup, whole rows, eight per wave,
// handed over in LDS, and wave w sums key features 32 (w / 2) .. +32 by value features 64 (w % 2) .. +64 of all its tokens: two 32 x 32
// accumulators per running sum, nothing to add up between waves, two waves to a SIMD.  One barrier per tile: the tiles
// alternate between two buffers.  Two tiles in flight per wave: a third gained 0.3 us with factored tables and lost as much without.
//
// 20 heads of 112, 4 680 tokens 18.6 -> 16.6 us (42 MB, 2.5 TB/s), token-major 22.7 -> 21.3, factored tables 21.0 -> 19.4; 256 heads, 1 560 tokens
// 41.0 -> 35.6 (179 MB, 5.0 TB/s); 20 heads of 128, 14 040 tokens, factored tables 37.4 -> 35.6.  Short ranges are bound by the launch, the first
// loads' latency and the exchange among a head's workgroups.  Longer shares (coop_state_pays) are left to wide_state.hpp, whose waves wait
// for each other once, not at every tile.
#pragma once

#include "wide_state.hpp"

namespace sv {

constexpr int kCoopWaves = 8, kCoopThreads = 64 * kCoopWaves, kCoopTokens = 64;
// Running sums of a wave, taken in turn by the tile's four groups of 16 tokens: none is longer than where four waves shared the tokens.
constexpr int kCoopSets = 4;
// LDS (bytes): two buffers of a K and a V tile, the waves' key sums, the epoch word, the rotation tables
constexpr int kCoopTileBytes = kCoopTokens * kWideRow, kCoopZOffset = 4 * kCoopTileBytes;
constexpr int kCoopEpochOffset = kCoopZOffset + kCoopWaves * 128 * 4, kCoopTabOffset = kCoopEpochOffset + kEpochLdsBytes;
template <int ROPE> constexpr int coop_state_lds() { return kCoopTabOffset + (ROPE == kRope3D ? kRope3dLdsBytes : 0); }

// A wave's rows of the workgroup's tiles: rows 8 wave + lane / 16 + 4 j, DEPTH tiles in flight.
template <int DEPTH, int ROPE, bool NT>
struct CoopStateStream {
    static constexpr int NLD = kCoopTokens / kCoopWaves / 4;
    rsrc_t rK, rV;
    uint32_t row_bytes, lane_off;
    bool valid;
    TileWalk walk;
    u32x4 k[DEPTH][NLD], v[DEPTH][NLD];
    Rotator<ROPE, NLD, DEPTH> rot;

    __device__ __forceinline__ CoopStateStream(const uint16_t *Kh, const uint16_t *Vh, const RopeArg &rope, const unsigned char *lds_tab,
                                               int64_t stride_n, int t1, int d, int wave, int lane, const TileWalk &w)
        : rK(make_rsrc(Kh, (uint32_t)t1 * (uint32_t)stride_n * 2u)), rV(make_rsrc(Vh, (uint32_t)t1 * (uint32_t)stride_n * 2u)),
          row_bytes((uint32_t)stride_n * 2u),
          lane_off((uint32_t)(8 * wave + (lane >> 4)) * (uint32_t)stride_n * 2u + (uint32_t)(lane & 15) * 16u),
          valid((lane & 15) * 8 < d), walk(w), rot(rope, t1, d, 8 * wave + (lane >> 4), 4, 4 * (lane & 15), 1, lds_tab) {}

    __device__ __forceinline__ void request(int s, int i)
    {
        const uint32_t base = valid ? walk.offset<kCoopTokens>(i, row_bytes) : kOutOfRange;
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            k[s][j] = load_stream16<NT>(rK, base + lane_off + (uint32_t)j * 4u * row_bytes);
            v[s][j] = load_stream16<NT>(rV, base + lane_off + (uint32_t)j * 4u * row_bytes);
        }
        rot.request(s, i < walk.count, walk.token<kCoopTokens>(i));
    }
};

// Sums the workgroup's share, whose first DEPTH tiles are requested and whose rotation is at the first one (begin_tile): wave w ends with S of key features 32 (w / 2) .. +32 by value features
// 64 (w % 2) .. +64 in `fin`, and with its rows' key sums in zw[w][128] (LDS).  The tiles pass through `lds`.  Called by all waves; a
// barrier has to follow before the key sums are read or the tiles' memory is used again.
template <int DEPTH, int ROPE, bool NT>
__device__ __forceinline__ void coop_state_sum(CoopStateStream<DEPTH, ROPE, NT> &stream, unsigned char *lds, float *zw, int wave, int lane,
                                               f32x16 (&fin)[2])
{
    const int kb = wave >> 1, vb = wave & 1;
    f32x16 acc[kCoopSets][2] = {};
    float zs[8] = {};
    const int wr_off = (8 * wave + (lane >> 4)) * kWideRow + (lane & 15) * 16;
    // tile i0 + s, staged in registers s, through buffer (i0 + s) % 2
    auto tile = [&](int i, int s) __attribute__((always_inline)) {
        constexpr int NLD = CoopStateStream<DEPTH, ROPE, NT>::NLD;
        __builtin_amdgcn_sched_barrier(0);       // stages stay in program order
        unsigned char *bufK = lds + (i & 1) * 2 * kCoopTileBytes, *bufV = bufK + kCoopTileBytes;
        f32x2 cs[NLD][4];
#pragma unroll
        for (int j = 0; j < NLD; ++j) stream.rot.fetch(s, j, cs[j]);
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            const u32x4 kk = relu_bf16x8(stream.k[s][j]);
            zs[0] += bf16_lo(kk.x);  zs[1] += bf16_hi(kk.x);
            zs[2] += bf16_lo(kk.y);  zs[3] += bf16_hi(kk.y);
            zs[4] += bf16_lo(kk.z);  zs[5] += bf16_hi(kk.z);
            zs[6] += bf16_lo(kk.w);  zs[7] += bf16_hi(kk.w);
            *reinterpret_cast<u32x4 *>(bufK + wr_off + 4 * j * kWideRow) = stream.rot.rotate_with(kk, cs[j]);
            *reinterpret_cast<u32x4 *>(bufV + wr_off + 4 * j * kWideRow) = stream.v[s][j];
        }
        stream.request(s, i + DEPTH);            // refill this stage
        // The tile is complete.  It is overwritten two tiles on, by waves that have passed the next tile's barrier, which every wave
        // reaches after its reads of this one.
        lds_barrier();
        stream.rot.template begin_tile<kCoopTokens>(stream.walk, i + 1);
#pragma unroll
        for (int ks = 0; ks < kCoopTokens / 16; ++ks) {
            const bf16x8 a = lds_tr_operand<kWideRow>(bufK, 16 * ks, 32 * kb, lane);
            const bf16x8 b0 = lds_tr_operand<kWideRow>(bufV, 16 * ks, 64 * vb, lane), b1 = lds_tr_operand<kWideRow>(bufV, 16 * ks, 64 * vb + 32, lane);
            f32x16(&x)[2] = acc[ks % kCoopSets];
            x[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b0, x[0], 0, 0, 0);
            x[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b1, x[1], 0, 0, 0);
        }
    };
    // Tiles past the share hold zeros and add nothing; all waves take the same number.
    for (int i0 = 0; i0 < stream.walk.count; i0 += DEPTH) {
#pragma unroll
        for (int s = 0; s < DEPTH; ++s)
            if (i0 + s < stream.walk.count) tile(i0 + s, s);
    }

#pragma unroll
    for (int cb = 0; cb < 2; ++cb) fin[cb] = (acc[0][cb] + acc[1][cb]) + (acc[2][cb] + acc[3][cb]);
#pragma unroll
    for (int e = 0; e < 8; ++e) {                               // lanes with equal lane % 16 hold the same eight features
        float x = zs[e];
        x += __shfl_xor(x, 16);
        x += __shfl_xor(x, 32);
        if (lane < 16) zw[wave * 128 + lane * 8 + e] = x;
    }
}

// The workgroup's sum of key k, from the waves' rows in zw.
__device__ __forceinline__ float coop_key_sum(const float *zw, int k)
{
    float x[kCoopWaves];
#pragma unroll
    for (int w = 0; w < kCoopWaves; ++w) x[w] = zw[w * 128 + k];
#pragma unroll
    for (int s = kCoopWaves / 2; s >= 1; s /= 2)
#pragma unroll
        for (int w = 0; w < s; ++w) x[w] += x[w + s];
    return x[0];
}

// grid = (C, B*H), block = kCoopThreads; chunk c owns tiles c + C i of the ceil((t1 - t0) / 64) tiles.  FINALIZE as in state_mfma_d64.
// Partials are laid out by wide_word.
template <int DEPTH, bool FINALIZE, int ROPE, bool NT>
__global__ __launch_bounds__(kCoopThreads, 2) void state_mfma_coop(
    const uint16_t *__restrict__ K, const uint16_t *__restrict__ V, RopeArg rope, TokStrides st,
    int H, int d, int t0, int t1, int C, const float *S_in, const float *z_in, float *S_out, float *z_out,
    void *__restrict__ ws, unsigned long long epoch, uint32_t spin_limit, int order)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const WgRole role(C, order);
    const int c = role.c, bh = role.bh, BH = gridDim.y;
    const int b = bh / H, h = bh % H;
    const int elems = d * d + d;
    const int n_tiles = (t1 - t0 + kCoopTokens - 1) / kCoopTokens;
    EpochSource es;
    if (FINALIZE) es.begin(ws, BH, elems, epoch, bh, c, C);

    CoopStateStream<DEPTH, ROPE, NT> stream(K + b * st.b + h * st.h, V + b * st.b + h * st.h, rope, lds + kCoopTabOffset, st.n, t1, d,
                                            wave, lane, TileWalk(t0, c, C, n_tiles, role.phase(b, order)));
    Rope3dFill tabs;
    if (ROPE == kRope3D) rope3d_lds_fill_begin(rope.r3, tabs);   // the first loads of the kernel
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) {
        stream.request(s, s);
        __builtin_amdgcn_sched_barrier(0);
    }
    stream.rot.template begin_tile<kCoopTokens>(stream.walk, 0);   // while the tables and the first tiles are on their way
    if (ROPE == kRope3D) {
        rope3d_lds_fill_end(lds + kCoopTabOffset, rope.r3, tabs);
        wg_barrier();
    }
    f32x16 fin[2];
    float *zw = reinterpret_cast<float *>(lds + kCoopZOffset);  // [wave][128]
    coop_state_sum(stream, lds, zw, wave, lane, fin);
    lds_barrier();
    const WideTarget target{S_in ? S_in + (size_t)bh * d * d : nullptr, z_in + (size_t)bh * d, S_out + (size_t)bh * d * d,
                            z_out + (size_t)bh * d, static_cast<float *>(ws) + (size_t)bh * kMaxChunks * elems, d, c, C};
    wide_store_block<2>(fin, wave >> 1, 2 * (wave & 1), FINALIZE && C == 1, target, lane);
    if (FINALIZE && C == 1) {
        if (tid < d) target.z_out[tid] = (target.S_in ? target.z_in[tid] : 0.f) + coop_key_sum(zw, tid);
        return;
    }
    if (tid < d / 2) store_coherent(target.partials + (size_t)c * elems + (size_t)d * d + 2 * tid, f32x2{coop_key_sum(zw, 2 * tid), coop_key_sum(zw, 2 * tid + 1)});
    if (FINALIZE) {
        epoch = es.resolve(reinterpret_cast<unsigned long long *>(lds + kCoopEpochOffset));
        auto wait = [&]() __attribute__((always_inline)) {
            return state_publish_and_wait(ws, BH, elems, bh, c, C, 0, epoch, spin_limit, lane);
        };
        if (C <= 2) wide_fold<kCoopThreads, 4, 2>(target, wait);
        else if (C <= 4) wide_fold<kCoopThreads, 3, 4>(target, wait);
        else if (C <= 8) wide_fold<kCoopThreads, 2, 8>(target, wait);
        else wide_fold<kCoopThreads, 1, 16>(target, wait);
    }
}

}  // namespace sv
