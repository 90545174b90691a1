// State reduction for d = 112 and 128 by quadrants of the state.
//
//   S[k][v] (+)= sum_j phi(K[j][k]) V[j][v],   z[k] (+)= sum_j phi(K[j][k])
//
// (brackets of the linear-attention equation of Sec. 3.2; with ROPE the keys that meet V are
// rotated after the ReLU, the key sum is not).
//
// A workgroup sums one 64 x 64 quadrant of a head's state over its chunk of the tokens, so it reads half of each K row
// and half of each V row.  The four workgroups of a chunk run on one die and read the same rows at about the same time: memory sees
// every row once, the L2 twice.  What that buys is everything behind the token loop: a wave holds 64 registers of state
// instead of 256, so two of them share a SIMD, the waves' sums are a quarter as much to add up, and a workgroup's
// partial is 16 KB instead of 50 or 65.
#pragma once

#include "state_mfma.hpp"

namespace sv {

constexpr int kQuadWaves = 8;                        // per workgroup, two to a SIMD
constexpr int kQuadWords = 64 * 64 / 4;              // 16-byte words of a quadrant: four rows of one column
constexpr int kQuadZWords = 64 / 4;                  // ... and of its key sums
constexpr int kQuadElems = 4 * (kQuadWords + kQuadZWords);   // floats of a partial in the workspace
static_assert(4 * kQuadMaxChunks <= 2 * kMaxChunks, "a flag per quadrant and chunk");
static_assert(4 * kQuadMaxChunks * kQuadElems <= kMaxChunks * (112 * 112 + 112), "the partials fit where whole states do");

template <int TILE_, int ROPE> struct QuadShape {
    static constexpr int WAVES = kQuadWaves, TILE = TILE_, THREADS = 64 * WAVES, kTileBytes = TILE * kRowBytes;
    // LDS map (bytes): the waves' K/V tiles, then the rotation tables; once the token loop is over, the waves'
    // accumulators as words and their key sums; the epoch word
    static constexpr int kTabOffset = WAVES * 2 * kTileBytes, kLoop = kTabOffset + (ROPE == kRope3D ? kRope3dLdsBytes : 0);
    static constexpr int kZOffset = WAVES * kQuadWords * 16, kSums = kZOffset + WAVES * 64 * 4;
    static constexpr int kEpochOffset = kLoop > kSums ? kLoop : kSums, kLdsBytes = kEpochOffset + kEpochLdsBytes;
};

// Where word v of a quadrant's sums belongs: in the order in which the accumulators hold them, element i of block (rb, cb) of lane l
// being row 32 rb + 8 (i / 4) + 4 (l / 32) + i % 4, column 32 cb + l % 32: v = (2 rb + cb) * 256 + (i / 4) * 64 + l.  The 16 words
// of the key sums follow.
struct QuadWordAt {
    int row, col;
    __device__ __forceinline__ QuadWordAt(int v, int kb, int vb)
        : row(64 * kb + 32 * (v >> 9) + 8 * ((v >> 6) & 3) + 4 * ((v >> 5) & 1)), col(64 * vb + 32 * ((v >> 8) & 1) + (v & 31)) {}
};

// One head's carried state (null: none) and new state, and a quadrant of it.
struct QuadTarget {
    const float *S_in, *z_in;
    float *S_out, *z_out;
    int d, kb, vb;
    // rows come in fours and 112 is a multiple of four: a word exists as a whole or not at all
    __device__ __forceinline__ bool exists(int v) const
    {
        if (v >= kQuadWords) return vb == 0 && v < kQuadWords + kQuadZWords && 64 * kb + 4 * (v - kQuadWords) < d;
        const QuadWordAt w(v, kb, vb);
        return w.row < d && w.col < d;
    }
    __device__ __forceinline__ f32x4 carried(int v) const       // of a word that exists
    {
        if (!S_in) return f32x4{0.f, 0.f, 0.f, 0.f};
        if (v >= kQuadWords) return *reinterpret_cast<const f32x4 *>(z_in + 64 * kb + 4 * (v - kQuadWords));
        const QuadWordAt w(v, kb, vb);
        const float *p = S_in + w.row * d + w.col;
        return f32x4{p[0], p[d], p[2 * d], p[3 * d]};
    }
    __device__ __forceinline__ void store(int v, f32x4 x) const
    {
        if (v >= kQuadWords) {
            *reinterpret_cast<f32x4 *>(z_out + 64 * kb + 4 * (v - kQuadWords)) = x;
            return;
        }
        const QuadWordAt w(v, kb, vb);
        float *p = S_out + w.row * d + w.col;
        p[0] = x.x;  p[d] = x.y;  p[2 * d] = x.z;  p[3 * d] = x.w;
    }
};

// One wave's input stream: rows lane/8 + 8 j of every tile of its walk, the 64 key features of half kb and the 64 value
// features of half vb, DEPTH tiles in flight.  Lanes whose features lie past d (d = 112) address out of range: zeros.
template <int TILE, int DEPTH, int ROPE>
struct QuadStream {
    static constexpr int NLD = TILE / 8;
    rsrc_t rK, rV;
    uint32_t row_bytes, offK, offV;
    bool okK, okV;
    TileWalk walk;
    u32x4 k[DEPTH][NLD], v[DEPTH][NLD];
    Rotator<ROPE, NLD, DEPTH> rot;

    __device__ __forceinline__ QuadStream(const uint16_t *Kh, const uint16_t *Vh, const RopeArg &rope, const unsigned char *lds_tab,
                                          int64_t stride_n, int t1, int d, int kb, int vb, int lane, const TileWalk &w)
        : rK(make_rsrc(Kh, (uint32_t)t1 * (uint32_t)stride_n * 2u)), rV(make_rsrc(Vh, (uint32_t)t1 * (uint32_t)stride_n * 2u)),
          row_bytes((uint32_t)stride_n * 2u), offK((uint32_t)(lane >> 3) * row_bytes + (uint32_t)(64 * kb + 8 * (lane & 7)) * 2u),
          offV((uint32_t)(lane >> 3) * row_bytes + (uint32_t)(64 * vb + 8 * (lane & 7)) * 2u), okK(64 * kb + 8 * (lane & 7) < d),
          okV(64 * vb + 8 * (lane & 7) < d), walk(w), rot(rope, t1, d, lane >> 3, 8, 32 * kb + 4 * (lane & 7), 1, lds_tab) {}

    __device__ __forceinline__ void request(int s, int i)
    {
        const uint32_t base = walk.offset<TILE>(i, row_bytes), bk = okK ? base : kOutOfRange, bv = okV ? base : kOutOfRange;
#pragma unroll
        for (int j = 0; j < NLD; ++j) {
            k[s][j] = load_stream16<false>(rK, bk + offK + (uint32_t)j * 8u * row_bytes);
            v[s][j] = load_stream16<false>(rV, bv + offV + (uint32_t)j * 8u * row_bytes);
        }
        rot.request(s, i < walk.count, walk.token<TILE>(i));
    }
};

struct QuadAcc {
    // Two running sums, so that none is longer than in the kernel of whole rows (a workgroup has a quarter of the chunks and twice
    // the waves): the error of S against 64 bits stays where it was (1.1e-7 of 20 heads, 4 680 tokens with either).
    static constexpr int SETS = 2;
    f32x16 s[SETS][2][2];   // [running sum][key feature block][value feature block]
    float z[8];             // features 8 (lane % 8) + e of the tokens this lane loaded
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int t = 0; t < SETS; ++t)
#pragma unroll
            for (int rb = 0; rb < 2; ++rb)
#pragma unroll
                for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) s[t][rb][cb][i] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) z[e] = 0.f;
    }
};

// Accumulates the wave's share (its first DEPTH tiles are requested); stage s adds to running sum s % 2.
template <int TILE, int DEPTH, int ROPE>
__device__ __forceinline__ void quad_accumulate(QuadStream<TILE, DEPTH, ROPE> &st, unsigned char *tileK, unsigned char *tileV,
                                                int lane, QuadAcc &acc)
{
    constexpr int NLD = TILE / 8;
    const int wr_off = (lane >> 3) * kRowBytes + (lane & 7) * 16;
    for (int i0 = 0; i0 < st.walk.count; i0 += DEPTH) {
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) {
            __builtin_amdgcn_sched_barrier(0);   // stages stay in program order
            st.rot.template begin_tile<TILE>(st.walk, i0 + s);
            f32x2 cs[NLD][4];
#pragma unroll
            for (int j = 0; j < NLD; ++j) st.rot.fetch(s, j, cs[j]);
#pragma unroll
            for (int j = 0; j < NLD; ++j) {
                const u32x4 kk = relu_bf16x8(st.k[s][j]);
                acc.z[0] += bf16_lo(kk.x);  acc.z[1] += bf16_hi(kk.x);
                acc.z[2] += bf16_lo(kk.y);  acc.z[3] += bf16_hi(kk.y);
                acc.z[4] += bf16_lo(kk.z);  acc.z[5] += bf16_hi(kk.z);
                acc.z[6] += bf16_lo(kk.w);  acc.z[7] += bf16_hi(kk.w);
                st.k[s][j] = kk;
            }
#pragma unroll
            for (int j = 0; j < NLD; ++j) st.k[s][j] = st.rot.rotate_with(st.k[s][j], cs[j]);
            wave_lds_fence();
#pragma unroll
            for (int j = 0; j < NLD; ++j) {
                *reinterpret_cast<u32x4 *>(tileK + wr_off + 8 * j * kRowBytes) = st.k[s][j];
                *reinterpret_cast<u32x4 *>(tileV + wr_off + 8 * j * kRowBytes) = st.v[s][j];
            }
            st.request(s, i0 + s + DEPTH);       // refill this stage: DEPTH tiles ahead
            __builtin_amdgcn_sched_barrier(0);
            wave_lds_fence();
#pragma unroll
            for (int ks = 0; ks < TILE / 16; ++ks) {
                const bf16x8 a0 = lds_tr_operand(tileK, 16 * ks, 0, lane), a1 = lds_tr_operand(tileK, 16 * ks, 32, lane);
                const bf16x8 b0 = lds_tr_operand(tileV, 16 * ks, 0, lane), b1 = lds_tr_operand(tileV, 16 * ks, 32, lane);
                f32x16(&a)[2][2] = acc.s[s % QuadAcc::SETS];
                a[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b0, a[0][0], 0, 0, 0);
                a[0][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b1, a[0][1], 0, 0, 0);
                a[1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b0, a[1][0], 0, 0, 0);
                a[1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b1, a[1][1], 0, 0, 0);
            }
        }
    }
}

// All threads: the waves' sums as words in LDS, wave w's at [w][v]; the key sums at zs[w][64].  The tiles and tables are dead.
template <class P>
__device__ __forceinline__ void quad_words_to_lds(QuadAcc &acc, unsigned char *lds, int wave, int lane)
{
    float *zs = reinterpret_cast<float *>(lds + P::kZOffset) + wave * 64;
#pragma unroll
    for (int e = 0; e < 8; ++e) {                       // lanes with equal lane % 8 hold the same eight features
        float x = acc.z[e];
        x += __shfl_xor(x, 8);
        x += __shfl_xor(x, 16);
        x += __shfl_xor(x, 32);
        acc.z[e] = x;
    }
    wg_barrier();                                       // all waves are done with their tiles
    f32x4 *mine = reinterpret_cast<f32x4 *>(lds) + wave * kQuadWords + lane;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            f32x4 x;
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = acc.s[0][b >> 1][b & 1][4 * q + i] + acc.s[1][b >> 1][b & 1][4 * q + i];
            mine[b * 256 + q * 64] = x;
        }
    if (lane < 8) {
#pragma unroll
        for (int e = 0; e < 8; ++e) zs[lane * 8 + e] = acc.z[e];
    }
    wg_barrier();
}
// Word v of the workgroup's sums: a fixed tree over the waves.
template <class P> __device__ __forceinline__ f32x4 quad_sum(const unsigned char *lds, int v)
{
    const f32x4 *src = v < kQuadWords ? reinterpret_cast<const f32x4 *>(lds) + v
                                      : reinterpret_cast<const f32x4 *>(lds + P::kZOffset) + (v - kQuadWords);
    const int step = v < kQuadWords ? kQuadWords : kQuadZWords;
    f32x4 x[P::WAVES];
#pragma unroll
    for (int w = 0; w < P::WAVES; ++w) x[w] = src[w * step];
#pragma unroll
    for (int h = P::WAVES / 2; h >= 1; h /= 2)
#pragma unroll
        for (int w = 0; w < h; ++w) x[w] += x[w + h];
    return x[0];
}

// Chunk c's slice of the quadrant, once all C partials are there (`wait`): the carried values plus the partials in chunk
// order.  UNITS words per thread and round, GROUP partials in flight per word.
template <int THREADS, int UNITS, int GROUP, class WaitFn>
__device__ __forceinline__ void quad_fold(const QuadTarget &t, const float *partials, int c, int C, int words, WaitFn wait)
{
    const int per = (words + C - 1) / C, lo = c * per, hi = lo + per < words ? lo + per : words, tid = (int)threadIdx.x;
    constexpr uint32_t kStride = 4u * kQuadElems * 4u;                          // bytes from chunk to chunk
    const rsrc_t rP = make_rsrc(partials, (uint32_t)(C - 1) * kStride + kQuadElems * 4u);
    f32x4 x[UNITS];
    bool there[UNITS];
    auto carried = [&](int v0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            const int v = v0 + u * THREADS;
            there[u] = v < hi && t.exists(v);
            x[u] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (there[u]) x[u] = t.carried(v);
        }
    };
    carried(lo + tid);
    if (!wait()) return;                                                        // timed out: this wave's part of S, z stays as it was
    for (int v0 = lo + tid; v0 < hi; v0 += THREADS * UNITS) {
        if (v0 != lo + tid) carried(v0);
        for (int c0 = 0; c0 < C; c0 += GROUP) {
            f32x4 p[UNITS][GROUP];
#pragma unroll
            for (int cc = 0; cc < GROUP; ++cc)
#pragma unroll
                for (int u = 0; u < UNITS; ++u)                                // past the last partial and the slice: nothing is read
                    p[u][cc] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                   rP, there[u] && c0 + cc < C ? 16u * (uint32_t)(v0 + u * THREADS) + (uint32_t)(c0 + cc) * kStride : kOutOfRange, 0,
                                   16 /* sc1 */));
#pragma unroll
            for (int u = 0; u < UNITS; ++u)
#pragma unroll
                for (int cc = 0; cc < GROUP; ++cc)
                    if (c0 + cc < C) x[u] += p[u][cc];
        }
#pragma unroll
        for (int u = 0; u < UNITS; ++u)
            if (there[u]) t.store(v0 + u * THREADS, x[u]);
    }
}

// grid = quad_grid(C, BH, kDies), block = 64 * kQuadWaves.  Wave w of chunk c owns tiles WAVES c + w + WAVES C i of the ceil((t1 - t0) / TILE)
// tiles.  With C > 1 the workgroups of a head's quadrant wait for each other: all must be resident.
template <int TILE, int DEPTH, int ROPE>
__global__ __launch_bounds__(64 * kQuadWaves, 2) void state_mfma_quad(
    const uint16_t *__restrict__ K, const uint16_t *__restrict__ V, RopeArg rope, TokStrides st, int H, int BH, int d, int t0, int t1,
    int C, const float *S_in, const float *z_in, float *S_out, float *z_out, void *__restrict__ ws, unsigned long long epoch,
    uint32_t spin_limit, int order)
{
    using P = QuadShape<TILE, ROPE>;
    constexpr int WAVES = P::WAVES;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int c, bh, q;
    if (!quad_role((int)blockIdx.x, C, BH, kDies, (order & kOrderChunkMajor) != 0, c, bh, q)) return;
    const int kb = q & 1, vb = q >> 1;
    const int b = bh / H, h = bh % H, elems = d * d + d;
    const uint16_t *Kh = K + b * st.b + h * st.h, *Vh = V + b * st.b + h * st.h;
    const int n_tiles = (t1 - t0 + TILE - 1) / TILE;
    EpochSource es;
    if (C > 1) es.begin(ws, BH, elems, epoch, bh, 4 * c + q, 4 * C);

    QuadAcc acc;
    acc.clear();
    const int phase = order & kOrderLockstep ? 5 * b : bh;
    QuadStream<TILE, DEPTH, ROPE> stream(Kh, Vh, rope, lds + P::kTabOffset, st.n, t1, d, kb, vb, lane,
                                             TileWalk(t0, WAVES * c + wave, WAVES * C, n_tiles, phase));
    Rope3dFill tabs;
    if (ROPE == kRope3D) rope3d_lds_fill_begin(rope.r3, tabs);   // the first loads of the kernel
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) {
        stream.request(s, s);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (ROPE == kRope3D) {
        rope3d_lds_fill_end(lds + P::kTabOffset, rope.r3, tabs);
        wg_barrier();
    }
    unsigned char *tileK = lds + wave * 2 * P::kTileBytes;
    quad_accumulate(stream, tileK, tileK + P::kTileBytes, lane, acc);
    quad_words_to_lds<P>(acc, lds, wave, lane);

    const QuadTarget target{S_in ? S_in + (size_t)bh * d * d : nullptr, z_in + (size_t)bh * d, S_out + (size_t)bh * d * d,
                            z_out + (size_t)bh * d, d, kb, vb};
    const int words = kQuadWords + (vb == 0 ? kQuadZWords : 0);
    if (C == 1) {
        for (int v = tid; v < words; v += P::THREADS)
            if (target.exists(v)) target.store(v, target.carried(v) + quad_sum<P>(lds, v));
        return;
    }
    float *partials = static_cast<float *>(ws) + (size_t)bh * kMaxChunks * elems + (size_t)q * kQuadElems;
    const rsrc_t rOut = make_rsrc(partials + (size_t)c * 4 * kQuadElems, kQuadElems * 4u);
    constexpr int kRounds = (kQuadWords + kQuadZWords + P::THREADS - 1) / P::THREADS;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int v = tid + r * P::THREADS;
        const bool there = v < words && target.exists(v);
        const f32x4 x = quad_sum<P>(lds, v < words ? v : 0);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), rOut, there ? 16u * (uint32_t)v : kOutOfRange, 0, 16 /* sc1 */);
    }
    epoch = es.resolve(reinterpret_cast<unsigned long long *>(lds + P::kEpochOffset));
    auto wait = [&]() __attribute__((always_inline)) {
        unsigned long long *flags = ws_flags(ws, BH, elems, bh, 0) + q * kQuadMaxChunks;
        coherent_stores_done();
        wg_barrier();
        if (tid == 0) flag_publish(flags + c, epoch);
        const bool ok = flags_wait_all(flags, C, epoch, spin_limit, lane);
        if (!ok && lane == 0) __hip_atomic_store(ws_error(ws, BH, elems), kWsTimeoutMark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return ok;
    };
    if (C <= 2) quad_fold<P::THREADS, 2, 2>(target, partials, c, C, words, wait);
    else if (C <= 4) quad_fold<P::THREADS, 1, 4>(target, partials, c, C, words, wait);
    else quad_fold<P::THREADS, 1, 16>(target, partials, c, C, words, wait);
}

}  // namespace sv
