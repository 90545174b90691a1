// State reduction and apply in fp32 arithmetic on the matrix cores (v_mfma_f32_16x16x4_f32): the fp32 mode at every head
// dimension, and bf16 at d = 32.
//
//   S[k][v] (+)= sum_j phi(K[j][k]) V[j][v],  z[k] (+)= sum_j phi(K[j][k])          (Sec. 3.2, brackets)
//   O[i][v] = (sum_k phi(Q[i][k]) S[k][v]) / (sum_k phi(Q[i][k]) z[k] + eps)        (Sec. 3.2, right-hand form)
//
// Bound by HBM: 4 d flops per byte of fp32 tokens, the fp32 matrix rate allows about 20 times what the streams
// need at d = 32 and 5 times at d = 128.  One MFMA takes a 16 x 4 and a 4 x 16 operand, one element per lane (row or
// column lane % 16, contraction index lane / 16), which is what lets both kernels go without LDS:
//
//   state   the contraction runs over tokens: lane (m, g) loads VEC consecutive features VEC*m .. of token g of
//           a group of four with one 4- to 16-byte load (16 lanes make a row), and element e of that vector IS
//           the operand of feature block e, whose 16 features are e, VEC + e, 2 VEC + e, ...
//   apply   the contraction runs over features: lane (n, g) holds chunks of 4 consecutive features of a token, chunk j
//           from feature(j, g) on, and element q is the operand of the step that contracts the features
//           feature(j, 0) + q .. feature(j, 3) + q; the state is kept in registers in the matching order.  Output block b holds features NB*n + b, so that a
//           lane ends up with NB consecutive features of a token and stores them as they are.
//
// Measured (a layer, in turn: plain FMAs out of LDS; this with four waves in the state kernel; with eight, and the state in pieces and the last workgroup's fold
// for bf16): fp32, 32 heads of 64, 4 680 tokens 120 -> 45.6 -> 43.4 us (3.5 TB/s); bf16, 128 heads of 32, 4 096 tokens 130 -> 40.4 -> 33.0 us (4.1 TB/s).
// What is left above the streams' time is the start of the kernels and adding the partial states up.
//
// d <= 64: a wave holds the whole state and works alone on its tiles.  d = 112, 128: the waves of a workgroup
// share the tiles, in the state kernel as 64 x 64 quadrants (each half row is loaded by two waves, the second out
// of the caches), in the apply kernel as 32 output features each.
#pragma once

#include "rope.hpp"
#include "state_mfma.hpp"

namespace sv {

// W 32-bit words from / to a buffer resource, non-temporal.
template <int W> struct Words { uint32_t w[W]; };
template <int W> __device__ __forceinline__ Words<W> load_words(rsrc_t r, uint32_t off)
{
    Words<W> x;
    if constexpr (W == 4) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 2);
        x.w[0] = v.x; x.w[1] = v.y; x.w[2] = v.z; x.w[3] = v.w;
    } else if constexpr (W == 2) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 2);
        x.w[0] = v[0]; x.w[1] = v[1];
    } else {
        x.w[0] = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 2);
    }
    return x;
}
template <int W> __device__ __forceinline__ void store_words(rsrc_t r, uint32_t off, const Words<W> &x)
{
    if constexpr (W == 4) {
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{x.w[0], x.w[1], x.w[2], x.w[3]}, r, off, 0, 2);
    } else if constexpr (W == 2) {
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{x.w[0], x.w[1]}, r, off, 0, 2);
    } else {
        __builtin_amdgcn_raw_buffer_store_b32(x.w[0], r, off, 0, 2);
    }
}
// N values of type T as fp32, from and to the words that hold them.
template <typename T, int N> constexpr int kWords = N * (int)sizeof(T) / 4;
template <typename T, int N> __device__ __forceinline__ void widen(const Words<kWords<T, N>> &x, float (&f)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if constexpr (sizeof(T) == 4) f[i] = __uint_as_float(x.w[i]);
        else f[i] = i & 1 ? bf16_hi(x.w[i / 2]) : bf16_lo(x.w[i / 2]);
    }
}
template <typename T, int N> __device__ __forceinline__ Words<kWords<T, N>> narrow(const float (&f)[N])
{
    Words<kWords<T, N>> x;
#pragma unroll
    for (int i = 0; i < kWords<T, N>; ++i) {
        if constexpr (sizeof(T) == 4) x.w[i] = __float_as_uint(f[i]);
        else x.w[i] = pack_bf16x2(f[2 * i], f[2 * i + 1]);
    }
    return x;
}

// Position of token `tok` in the factored tables' grid.  Quotients by a product with the rounded reciprocal: exact
// for fewer than 2^20 tokens, which the host checks ((x + 0.5) / n is 0.5 / n away from an integer).
struct GridPos {
    int f, r, c;
    __device__ __forceinline__ GridPos(const Rope3D &R, int tok, float inv_rc, float inv_cols)
    {
        const int rc = R.rows * R.cols;
        f = (int)(((float)tok + 0.5f) * inv_rc);
        const int rem = tok - f * rc;
        r = (int)(((float)rem + 0.5f) * inv_cols);
        c = rem - r * R.cols;
        f = f < R.frames ? f : R.frames - 1;      // tokens past the last: any valid entry, their features are zero
    }
};
// (cos, sin) of feature pair p at that position, from the tables in LDS.
__device__ __forceinline__ f32x2 rope3d_entry_lds(const unsigned char *tab, const Rope3D &R, const GridPos &g, int p)
{
    const int nt = R.frames * R.n_t, nh = R.rows * R.n_h;
    int e = g.f * R.n_t + p;
    if (p >= R.n_t) e = nt + g.r * R.n_h + (p - R.n_t);
    if (p >= R.n_t + R.n_h) e = nt + nh + g.c * R.n_w + (p - R.n_t - R.n_h);
    return reinterpret_cast<const f32x2 *>(tab)[e];
}
// Turns the N / 2 feature pairs in f by the entries in cs.
template <int N> __device__ __forceinline__ void rotate_pairs(float (&f)[N], const f32x2 (&cs)[N / 2])
{
#pragma unroll
    for (int p = 0; p < N / 2; ++p) {
        const float a = f[2 * p], b = f[2 * p + 1];
        f[2 * p] = a * cs[p].x - b * cs[p].y;
        f[2 * p + 1] = a * cs[p].y + b * cs[p].x;
    }
}

// ---- state ----------------------------------------------------------------------------------------------------

// How a head's tokens and its state are shared out (HOW):
//   kF32Shared    C workgroups, a share of the tokens each; the last of them or state_reduce adds their partial states up.
//   kF32Sole      one workgroup, which stores the new state.
//   kF32Quarters  four workgroups, all tokens and a quarter of the state each (d = 32 and 64): half of the 16 x 16 blocks in either direction.  They load
//                 what one would, the second to fourth time out of their die's L2, but the matrix products, of which one compute unit needs
//                 3.5 us for 1 024 tokens of 32 features or 256 of 64, are shared out and nothing has to be added up: the same bits as one workgroup's.  (Layers: 2 heads of 32,
//                 1 024 tokens 13.7 -> 12.4 us, 64 heads of 64, 192 tokens 15.4 -> 12.1; with the quarters on four dies 8 heads, 640
//                 tokens had taken 13.3 us instead of 11.8, on one 11.0.)
// Eight waves, two to a SIMD, so that one multiplies while the other converts and requests (four waves with three tiles in flight each,
// before: 32 heads of 64, 4 680 tokens, layer 45.6 -> 43.5 us; 20 heads of 112 88.6 -> 83.1; 128 heads of 32, bf16, 4 096 tokens, rotated 48.5 -> 45.0).  At d = 32
// a head that is not shared by its tokens gets sixteen waves in the 128 registers that leaves each (2 heads, 1 024 tokens, one workgroup: 11.6 -> 10.0 us).
constexpr int kF32Shared = 0, kF32Sole = 1, kF32Quarters = 2;
template <typename T, int D, int HOW, int ROPE> struct StateF32 {
    static constexpr bool kSplit = D > 64;                 // quadrants instead of whole states
    static constexpr bool kAlone = HOW != kF32Shared, kQuarter = HOW == kF32Quarters;
    static_assert(!kQuarter || !kSplit, "wide heads are dealt to the waves as quadrants already");
    static constexpr bool kMany = kAlone && D == 32;
    static constexpr int kWaves = kMany ? 16 : 8;
    static constexpr int F = kSplit ? 64 : D;              // features of a wave's part, on both axes
    static constexpr int VEC = F / 16, W = kWords<T, VEC>;
    static constexpr int NB = kQuarter ? VEC / 2 : VEC;    // blocks of 16 features that a wave multiplies, on both axes
    // Groups of four tokens per tile: what the registers hold (three or four at d = 64 and more: level to 5 % slower, and rotated they spill).
    // The two forms of the rotation keep the same tiles and give the same bits.
    static constexpr int U = D > 32 ? 2 : kMany && ROPE == kRopeNone ? 8 : 4;
    static constexpr int TILE = 4 * U;
    static constexpr int DEPTH = kMany ? 1 : D == 32 ? 3 : 2;    // tiles in flight per wave
    // Running sums: a set per stage, and at d = 32 (few registers) one for each parity of the token group.  An fp32 sum's error grows
    // with the root of its length; one set for the whole share had S up to 1.8 times as far from 64-bit sums as the scalar kernel, whose
    // chunks are shorter (2 heads of 32, 1 024 tokens: 2.1e-7 against 1.3e-7; 160 heads of 112, 4 680 tokens: 8.7e-7 against
    // 5.0e-7).  With these it is no further off at any size measured (1.0e-7, 4.9e-7), for less than 0.5 us per launch.  Adding
    // every tile's products to the share's sum instead was as exact and up to 20 % slower.
    static constexpr int kChains = VEC == 2 ? 2 : 1;
    static constexpr int FQ = kQuarter ? F / 2 : F;        // features of the part that is summed, on both axes
    static constexpr int kSlot = FQ * FQ + F;              // a wave's part in LDS: state, then key sums
    static constexpr int kParts = kSplit ? kWaves / 4 : kWaves;   // waves that hold the same part of the state
    static constexpr int kWgTokens = kParts * TILE;
    // tokens that a running sum takes of the longest head that one workgroup sums at d = 112 and 128 (see f32_sole_tokens)
    static constexpr int kSoleTiles = (kF32WideSoleTokens + kWgTokens - 1) / kWgTokens;      // of a wave
    static_assert(!kSplit || (kSoleTiles + DEPTH * kChains - 1) / (DEPTH * kChains) * TILE == kF32WideSumTokens, "f32_sole_tokens counts on it");
    static constexpr int lds_bytes() {
        constexpr int slots = kWaves * kSlot * 4, tab = ROPE == kRope3D ? kRope3dLdsBytes : 0;   // tables, then slots
        return slots > tab ? slots : tab;
    }
};

// A head's C workgroups count themselves in a word of the workspace, whose contents are undefined before the call: the one that finds all others
// counted is the last and adds the partials up.  Nobody waits.  The word holds tag + workgroups that have stored their partial; `tag` is the
// call's own, its low six bits zero.  Every workgroup sees to the word early on, while its first tiles are on their way: if it holds no count of this call,
// it is replaced, provided that it is still what was seen (otherwise another workgroup of the call has been there, and nobody else writes it).  The last one
// leaves zero, so that a replayed launch, whose tag is the same, starts anew.
struct LastFold {
    unsigned long long seen = 0;                   // thread 0's only, like all that follows but arrive()'s result
    __device__ __forceinline__ void look(unsigned long long *word)
    {
        if (threadIdx.x == 0) seen = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ void open(unsigned long long *word, unsigned long long tag)
    {
        if (threadIdx.x != 0) return;
        unsigned long long was = seen;
        asm volatile("" : "+v"(was));              // looked at here, behind the requests of the first tiles, and not before
        if ((was & ~63ull) != tag)
            (void)__hip_atomic_compare_exchange_strong(word, &was, tag, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // Called by all threads when the workgroup's partial is stored (coherently): is this the head's last workgroup?  `lds_word` may be in use until then.
    __device__ __forceinline__ bool arrive(unsigned long long *word, int C, int *lds_word) const
    {
        coherent_stores_done();
        wg_barrier();
        if (threadIdx.x == 0) {
            const unsigned long long n = __hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 63ull;
            *lds_word = (int)n == C - 1;
            if ((int)n == C - 1) __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        wg_barrier();
        return *lds_word != 0;
    }
};
// What state_reduce does with TREE, in the same order: the carried state, then sixteen partials at a time.
template <int THREADS, int D> __device__ __forceinline__ void fold_partials(const HeadState &hs, const float *partials, int C, int tid)
{
    constexpr int elems = D * D + D, kWords = elems / 4, kS = D * D / 4, UNITS = (kWords + THREADS - 1) / THREADS;
    const rsrc_t rP = make_rsrc(partials, (uint32_t)C * (uint32_t)(elems * 4));
    f32x4 x[UNITS];
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
        const int v = tid + u * THREADS;
        x[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (hs.S_in && v < kWords) x[u] = *reinterpret_cast<const f32x4 *>(v < kS ? hs.S_in + 4 * v : hs.z_in + 4 * (v - kS));
    }
    for (int c0 = 0; c0 < C; c0 += 16) {
        f32x4 p[UNITS][8];
        auto load = [&](int u, int c) __attribute__((always_inline)) {        // past the last partial and past the state: zeros, nothing is read
            const int v = tid + u * THREADS;
            return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                rP, v < kWords && c < C ? 16u * (uint32_t)v + (uint32_t)c * (uint32_t)(elems * 4) : kOutOfRange, 0, 16 /* sc1 */));
        };
#pragma unroll
        for (int u = 0; u < UNITS; ++u)
#pragma unroll
            for (int j = 0; j < 8; ++j) p[u][j] = load(u, c0 + j);
        if (c0 + 8 < C)
#pragma unroll
            for (int u = 0; u < UNITS; ++u) {
                f32x4 q[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) q[j] = load(u, c0 + 8 + j);
#pragma unroll
                for (int j = 0; j < 8; ++j) p[u][j] += q[j];
            }
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
#pragma unroll
            for (int h = 4; h >= 1; h /= 2)
#pragma unroll
                for (int j = 0; j < h; ++j) p[u][j] += p[u][j + h];
            x[u] += p[u][0];
        }
    }
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
        const int v = tid + u * THREADS;
        if (v < kWords) *reinterpret_cast<f32x4 *>(v < kS ? hs.S_out + 4 * v : hs.z_out + 4 * (v - kS)) = x[u];
    }
}

// grid = (C, B*H), block = 64 * kWaves; arguments and the partials in the workspace as in state_mfma_d64.  No workgroup waits for another:
// with kF32Sole (C = 1) and kF32Quarters (grid = quad_grid(1, B*H, kDies), C = 1) the new state is stored; otherwise the head's last workgroup adds the
// partials up (LastFold; tag != 0, see f32_last_folds) or state_reduce does.  These calls stay
// free of waits because they always were: they may run beside anything on other streams, and be replayed without preparation.
template <typename T, int D, int HOW, int ROPE>
__global__ __launch_bounds__((64 * StateF32<T, D, HOW, ROPE>::kWaves), (StateF32<T, D, HOW, ROPE>::kWaves / 4)) void state_f32(
    const T *__restrict__ K, const T *__restrict__ V, RopeArg rope, TokStrides st, int H, int BH, int t0, int t1, int C,
    const float *S_in, const float *z_in, float *S_out, float *z_out, void *__restrict__ ws, unsigned long long tag, int order)
{
    using P = StateF32<T, D, HOW, ROPE>;
    constexpr int kThreads = 64 * P::kWaves, kParts = P::kParts, VEC = P::VEC, NB = P::NB, W = P::W, U = P::U, TILE = P::TILE, DEPTH = P::DEPTH, F = P::F, E = (int)sizeof(T);
    constexpr int elems = D * D + D;
    constexpr bool kCanFold = HOW == kF32Shared && D <= 64;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, g = lane >> 4;
    const WgRole role(C, order);
    int c = role.c, bh = role.bh, quarter = 0;
    if (P::kQuarter && !quad_role((int)blockIdx.x, 1, BH, kDies, (order & kOrderChunkMajor) != 0, c, bh, quarter)) return;
    const int b = bh / H, h = bh % H;
    const bool hi_k = quarter & 1, hi_v = quarter & 2;      // the upper half of the blocks

    const int kb = P::kSplit ? wave & 1 : 0, vb = P::kSplit ? (wave >> 1) & 1 : 0;
    const int n_tiles = (t1 - t0 + TILE - 1) / TILE;
    const int phase = order & kOrderLockstep ? 5 * b : bh;       // of the head worked on: a quarter's is not the grid's
    const TileWalk walk(t0, kParts * c + (P::kSplit ? wave >> 2 : wave), kParts * C, n_tiles, phase);
    const uint32_t row_bytes = (uint32_t)st.n * E;
    const rsrc_t rK = make_rsrc(K + b * st.b + h * st.h, (uint32_t)t1 * row_bytes);
    const rsrc_t rV = make_rsrc(V + b * st.b + h * st.h, (uint32_t)t1 * row_bytes);
    const int fk = F * kb + VEC * m, fv = F * vb + VEC * m;         // the lane's first features
    const uint32_t offK = fk < D ? (uint32_t)g * row_bytes + (uint32_t)fk * E : kOutOfRange;
    const uint32_t offV = fv < D ? (uint32_t)g * row_bytes + (uint32_t)fv * E : kOutOfRange;
    const rsrc_t rT = make_rsrc(rope.table, ROPE == kRopeTable ? (uint32_t)t1 * (uint32_t)(D * 4) : 0u);
    const uint32_t offT = fk < D ? (uint32_t)g * (uint32_t)(D * 4) + (uint32_t)fk * 4u : kOutOfRange;

    Words<W> kw[DEPTH][U], vw[DEPTH][U];
    Words<ROPE == kRopeTable ? VEC : 1> tw[DEPTH][U];
    // Requests the wave's i-th tile into stage s; past the share every address is out of range and reads zeros.
    auto request = [&](int s, int i) __attribute__((always_inline)) {
        const uint32_t base = walk.offset<TILE>(i, row_bytes);
        const uint32_t bk = fk < D ? base : 0u, bv = fv < D ? base : 0u;      // kOutOfRange once, not twice
#pragma unroll
        for (int u = 0; u < U; ++u) {
            kw[s][u] = load_words<W>(rK, offK + bk + (uint32_t)(4 * u) * row_bytes);
            vw[s][u] = load_words<W>(rV, offV + bv + (uint32_t)(4 * u) * row_bytes);
        }
        if constexpr (ROPE == kRopeTable) {
            const uint32_t bt = fk < D ? walk.offset<TILE>(i, (uint32_t)(D * 4)) : 0u;
#pragma unroll
            for (int u = 0; u < U; ++u) tw[s][u] = load_words<VEC>(rT, offT + bt + (uint32_t)(4 * u) * (uint32_t)(D * 4));
        }
    };

    LastFold fold;
    if (kCanFold && tag) fold.look(ws_flags(ws, BH, elems, bh, 0));
    Rope3dFill tabs;
    if (ROPE == kRope3D) rope3d_lds_fill_begin(rope.r3, tabs);
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) request(s, s);
    if (kCanFold && tag) fold.open(ws_flags(ws, BH, elems, bh, 0), tag);
    if (ROPE == kRope3D) {
        rope3d_lds_fill_end(lds, rope.r3, tabs);
        wg_barrier();
    }
    const float inv_rc = ROPE == kRope3D ? 1.0f / (float)(rope.r3.rows * rope.r3.cols) : 0.f;
    const float inv_cols = ROPE == kRope3D ? 1.0f / (float)rope.r3.cols : 0.f;

    f32x4 acc[DEPTH][P::kChains][NB][NB] = {};
    float zs[VEC] = {};
    for (int i0 = 0; i0 < walk.count; i0 += DEPTH) {
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) {
            // short shares: the rest of the round would be code and no work (the wide ones skip only the products: leaving the loop costs registers there)
            if (D == 32 && i0 + s >= walk.count) break;
            __builtin_amdgcn_sched_barrier(0);   // stages stay in program order
            float kf[U][VEC], vf[U][VEC], zt[VEC];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                widen<T, VEC>(kw[s][u], kf[u]);
                widen<T, VEC>(vw[s][u], vf[u]);
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    kf[u][e] = fmaxf(kf[u][e], 0.f);
                    zt[e] = u == 0 ? kf[u][e] : zt[e] + kf[u][e];          // the key sum is never rotated
                }
                if constexpr (ROPE != kRopeNone) {
                    f32x2 cs[VEC / 2];
                    if constexpr (ROPE == kRopeTable) {
#pragma unroll
                        for (int p = 0; p < VEC / 2; ++p)
                            cs[p] = f32x2{__uint_as_float(tw[s][u].w[2 * p]), __uint_as_float(tw[s][u].w[2 * p + 1])};
                    } else {
                        const GridPos pos(rope.r3, walk.token<TILE>(i0 + s) + 4 * u + g, inv_rc, inv_cols);
#pragma unroll
                        for (int p = 0; p < VEC / 2; ++p) {
                            const int pair = fk / 2 + p;
                            cs[p] = rope3d_entry_lds(lds, rope.r3, pos, pair < D / 2 ? pair : D / 2 - 1);
                        }
                    }
                    rotate_pairs<VEC>(kf[u], cs);
                }
            }
#pragma unroll
            for (int e = 0; e < VEC; ++e) zs[e] += zt[e];
            request(s, i0 + s + DEPTH);
            __builtin_amdgcn_sched_barrier(0);
            if (D == 32 || i0 + s < walk.count)
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int i = 0; i < NB; ++i)
#pragma unroll
                        for (int j = 0; j < NB; ++j) {
                            f32x4 &a = acc[s][u % P::kChains][i][j];
                            const float k0 = kf[u][i], k1 = kf[u][VEC - NB + i], v0 = vf[u][j], v1 = vf[u][VEC - NB + j];
                            a = __builtin_amdgcn_mfma_f32_16x16x4f32(hi_k ? k1 : k0, hi_v ? v1 : v0, a, 0, 0, 0);
                        }
        }
    }
    f32x4 sum[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            f32x4 x[DEPTH];
#pragma unroll
            for (int s = 0; s < DEPTH; ++s) {
                x[s] = acc[s][0][i][j];
                if (P::kChains == 2) x[s] += acc[s][P::kChains - 1][i][j];
            }
            sum[i][j] = x[0];
#pragma unroll
            for (int s = 1; s < DEPTH; ++s) sum[i][j] += x[s];
        }

    // The wave's part in [k][v] order in its LDS slot: element r of block (i, j) is key feature VEC (4 g + r) + i, value
    // feature VEC m + j, so a lane's blocks j make VEC consecutive floats.  (A quarter's: NB in the place of VEC.)
    float *slots = reinterpret_cast<float *>(lds), *mine = slots + wave * P::kSlot;
    wg_barrier();                                   // everybody is done with the tables
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float *row = mine + (NB * (4 * g + r) + i) * P::FQ + NB * m;
#pragma unroll
            for (int j = 0; j < NB; ++j) row[j] = sum[i][j][r];
        }
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        float x = zs[e];
        x += __shfl_xor(x, 16);
        x += __shfl_xor(x, 32);
        if (lane < 16) mine[P::FQ * P::FQ + VEC * m + e] = x;
    }
    wg_barrier();
    float *partials = static_cast<float *>(ws) + (size_t)bh * kMaxChunks * elems, *out = partials + (size_t)c * elems;
    const HeadState hs{S_in ? S_in + (size_t)bh * D * D : nullptr, z_in + (size_t)bh * D, S_out + (size_t)bh * D * D,
                       z_out + (size_t)bh * D};
    if constexpr (P::kQuarter) {
        auto total = [&](const float *src) __attribute__((always_inline)) {
            float x[kParts];
#pragma unroll
            for (int p = 0; p < kParts; ++p) x[p] = src[p * P::kSlot];
#pragma unroll
            for (int h = kParts / 2; h >= 1; h /= 2)
#pragma unroll
                for (int p = 0; p < h; ++p) x[p] += x[p + h];
            return x[0];
        };
        for (int e = tid; e < P::FQ * P::FQ; e += kThreads) {
            const int kk = e / P::FQ, vv = e % P::FQ;
            const int at = (VEC * (kk / NB) + (hi_k ? VEC - NB : 0) + kk % NB) * D + VEC * (vv / NB) + (hi_v ? VEC - NB : 0) + vv % NB;
            hs.S_out[at] = (hs.S_in ? hs.S_in[at] : 0.f) + total(slots + e);
        }
        if (quarter == 0 && tid < D) hs.z_out[tid] = (hs.S_in ? hs.z_in[tid] : 0.f) + total(slots + P::FQ * P::FQ + tid);
        return;
    }
    auto unit = [&](int u) __attribute__((always_inline)) {
        const float *src = slots + 2 * u;
        if constexpr (P::kSplit) {
            const int k = (2 * u) / D, v = 2 * u - k * D, kz = 2 * u - D * D;
            src = u < D * D / 2 ? slots + ((k >> 6) + 2 * (v >> 6)) * P::kSlot + (k & 63) * 64 + (v & 63)
                                : slots + (kz >> 6) * P::kSlot + F * F + (kz & 63);
        }
        f32x2 x[kParts];
#pragma unroll
        for (int p = 0; p < kParts; ++p) x[p] = *reinterpret_cast<const f32x2 *>(src + p * (P::kSplit ? 4 : 1) * P::kSlot);
#pragma unroll
        for (int h = kParts / 2; h >= 1; h /= 2)
#pragma unroll
            for (int p = 0; p < h; ++p) x[p] += x[p + h];
        return x[0];
    };
    if (P::kAlone) {
        state_store_sole<kThreads, D>(hs, tid, unit);
        return;
    }
    if constexpr (kCanFold)
        if (tag) {
            for (int u = tid; u < elems / 2; u += kThreads) store_coherent(out + 2 * u, unit(u));
            if (fold.arrive(ws_flags(ws, BH, elems, bh, 0), C, reinterpret_cast<int *>(lds))) fold_partials<kThreads, D>(hs, partials, C, tid);
            return;
        }
    for (int u = tid; u < elems / 2; u += kThreads) *reinterpret_cast<f32x2 *>(out + 2 * u) = unit(u);
}

// ---- apply ----------------------------------------------------------------------------------------------------

template <int D> struct ApplyF32 {
    static constexpr bool kSplit = D > 64;                  // 32 output features per wave, the waves share the tiles
    static constexpr int NB = D == 64 ? 4 : 2;              // blocks of 16 output features per wave
    static constexpr int NJ = D / 16;
    static constexpr int TILE = 16;
    // first of the four features that lane (n, g) holds in chunk j: whole 64-byte runs of a row per load
    template <typename T> static __device__ __forceinline__ int feature(int j, int g) {
        return sizeof(T) == 2 ? 8 * g + 4 * j : 16 * j + 4 * g;
    }
    // tiles in flight per wave; the rotation of wide heads leaves registers for one
    template <int ROPE> static constexpr int kDepth = ROPE != kRopeNone && D > 64 ? 1 : 2;
    static constexpr int kWgTokens = kSplit ? TILE : 4 * TILE;
};

// What apply_f32 does.  bf16 tokens: false where denominators or a state were met that want the loop with checks, CHECKED, which does all of the wave's share again.
// (Checks in every tile cost the kernel 1 to 3 %, a look at state and key sums before the loop 0.2 to 0.3 us.)
template <typename T, int D, int ROPE, bool CHECKED>
__device__ __forceinline__ bool apply_f32_tiles(
    unsigned char *lds, const T *__restrict__ Q, T *__restrict__ O, const RopeArg &rope, const TokStrides &st, int H, int t0, int t1, int C,
    const float *__restrict__ S, const float *__restrict__ z, float eps, int order)
{
    using P = ApplyF32<D>;
    constexpr int NB = P::NB, NJ = P::NJ, TILE = P::TILE, DEPTH = P::template kDepth<ROPE>, E = (int)sizeof(T);
    // a lane's features of a token come in NL loads of LC chunks (16 bytes)
    constexpr int LC = E == 2 ? 2 : 1, NL = NJ / LC;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, g = lane >> 4;
    const WgRole role(C, order);
    const int c = role.c, bh = role.bh;
    const int b = bh / H, h = bh % H;
    const int n_tiles = (t1 - t0 + TILE - 1) / TILE;
    const TileWalk walk(t0, P::kSplit ? c : 4 * c + wave, P::kSplit ? C : 4 * C, n_tiles, role.phase(b, order));
    const uint32_t row_bytes = (uint32_t)st.n * E;
    const rsrc_t rQ = make_rsrc(Q + b * st.b + h * st.h, (uint32_t)t1 * row_bytes);
    const rsrc_t rO = make_rsrc(O + b * st.b + h * st.h, (uint32_t)t1 * row_bytes);
    const rsrc_t rT = make_rsrc(rope.table, ROPE == kRopeTable ? (uint32_t)t1 * (uint32_t)(D * 4) : 0u);
    // MFMA row i is token 4 (i % 4) + i / 4 of the tile: element r of an accumulator in lane group g is then token 4 r + g,
    // and a store instruction writes four consecutive rows
    const int tok = 4 * (n & 3) + (n >> 2);
    const uint32_t offQ = (uint32_t)tok * row_bytes + (uint32_t)(P::template feature<T>(0, g) * E);
    const uint32_t offT = (uint32_t)tok * (uint32_t)(D * 4) + (uint32_t)(P::template feature<T>(0, g) * 4);
    const int f_out = (P::kSplit ? 32 * wave : 0) + NB * n;               // the lane's first output feature
    const uint32_t offO = (uint32_t)g * row_bytes + (uint32_t)(f_out * E);

    Words<4> qw[DEPTH][NL];
    Words<ROPE == kRopeTable ? 4 : 1> tw[DEPTH][NJ];
    auto request = [&](int s, int i) __attribute__((always_inline)) {
        const uint32_t base = walk.offset<TILE>(i, row_bytes) + offQ;
#pragma unroll
        for (int l = 0; l < NL; ++l) qw[s][l] = load_words<4>(rQ, base + (uint32_t)(64 * l));
        if constexpr (ROPE == kRopeTable) {
            const uint32_t bt = walk.offset<TILE>(i, (uint32_t)(D * 4)) + offT;
#pragma unroll
            for (int j = 0; j < NJ; ++j) tw[s][j] = load_words<4>(rT, bt + (uint32_t)((E == 2 ? 16 : 64) * j));
        }
    };
    Rope3dFill tabs;
    if (ROPE == kRope3D && !CHECKED) rope3d_lds_fill_begin(rope.r3, tabs);
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) request(s, s);
    if (ROPE == kRope3D && !CHECKED) {                                   // they are there the second time
        rope3d_lds_fill_end(lds, rope.r3, tabs);
        wg_barrier();
    }
    const float inv_rc = ROPE == kRope3D ? 1.0f / (float)(rope.r3.rows * rope.r3.cols) : 0.f;
    const float inv_cols = ROPE == kRope3D ? 1.0f / (float)rope.r3.cols : 0.f;

    // the state and the key sums, in the order in which the contraction meets the features
    float sr[NJ][4][NB], zr[NJ][4];
    const float *Sh = S + (size_t)bh * D * D, *zh = z + (size_t)bh * D;
    const bool exists = f_out < D;                                      // NB divides D: all of a lane's features or none
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = P::template feature<T>(j, g) + q;
            zr[j][q] = zh[k];
            typedef float vec __attribute__((ext_vector_type(NB)));
            const vec x = *reinterpret_cast<const vec *>(Sh + k * D + (exists ? f_out : 0));
#pragma unroll
            for (int e = 0; e < NB; ++e) sr[j][q][e] = x[e];            // columns that do not exist are never stored
        }

    // bf16 tokens without a rotation (d = 32): the state in three bf16 pieces, which hold all of its 24 bits, so the products stay those of
    // fp32, at a fifth of the matrix core's time.  Lane (n, g)'s eight features of a token are the operand of one 16 x 16 x 32 product.
    // (Layer of 128 heads, 4 096 tokens 36.2 -> 34.4 us; rotated features are fp32 values and stay with fp32 products.)
    // An entry below 2^-110 has bits below 2^-133, the last of bf16's denormal numbers (which the products take as they are): a wave that meets one
    // takes fp32 products.
    constexpr bool kPieces = E == 2 && ROPE == kRopeNone;
    bf16x8 piece[kPieces ? 3 : 1][NB];
    bool whole = false;                                         // wave-uniform: the pieces hold the state
    if constexpr (kPieces) {
        uint32_t least = ~0u;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < NB; ++e) {
                    const uint32_t twice = 2u * __float_as_uint(sr[j][q][e]) - 1u;     // magnitudes in order, zero behind all others
                    least = twice < least ? twice : least;
                }
        whole = __all(least >= 2u * __float_as_uint(0x1p-110f) - 1u);
#pragma unroll
        for (int e = 0; e < NB; ++e) {
            uint32_t w[3][4];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const int j = p >> 1, q = 2 * (p & 1);
                uint32_t half[2][3];
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    float x = sr[j][q + a][e];
#pragma unroll
                    for (int l = 0; l < 3; ++l) {
                        half[a][l] = __float_as_uint(x) >> 16;          // the leading eight bits
                        const float y = __uint_as_float(half[a][l] << 16);
                        x = x == y ? 0.f : x - y;                       // (an infinity is its first piece)
                    }
                }
#pragma unroll
                for (int l = 0; l < 3; ++l) w[l][p] = half[0][l] | half[1][l] << 16;
            }
#pragma unroll
            for (int l = 0; l < 3; ++l) piece[l][e] = __builtin_bit_cast(bf16x8, u32x4{w[l][0], w[l][1], w[l][2], w[l][3]});
        }
    }

    // bf16 results take a row's reciprocal, once per token, in place of quotients (a layer of 128 heads of 32, 4 096 tokens 39.4 -> 36.2 us): the
    // product's error is far below the result's rounding.  Not where it may be infinite: the quotients themselves.
    float low = 1.f;                                                    // smallest denominator met
    for (int i0 = 0; i0 < walk.count; i0 += DEPTH) {
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) {
            const int i = i0 + s;
            if (i >= walk.count) break;
            __builtin_amdgcn_sched_barrier(0);
            float qf[NJ][4], den = 0.f;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if constexpr (E == 2) {
                    const Words<2> half = {{qw[s][0].w[2 * j], qw[s][0].w[2 * j + 1]}};
                    widen<T, 4>(half, qf[j]);
                } else {
                    widen<T, 4>(qw[s][j], qf[j]);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    qf[j][q] = fmaxf(qf[j][q], 0.f);
                    den = fmaf(qf[j][q], zr[j][q], den);                // the denominator takes the plain features
                }
            }
            if constexpr (ROPE == kRopeTable) {
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const f32x2 cs[2] = {{__uint_as_float(tw[s][j].w[0]), __uint_as_float(tw[s][j].w[1])},
                                         {__uint_as_float(tw[s][j].w[2]), __uint_as_float(tw[s][j].w[3])}};
                    rotate_pairs<4>(qf[j], cs);
                }
            } else if constexpr (ROPE == kRope3D) {
                const GridPos pos(rope.r3, walk.token<TILE>(i) + tok, inv_rc, inv_cols);
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    const f32x2 cs[2] = {rope3d_entry_lds(lds, rope.r3, pos, P::template feature<T>(j, g) / 2),
                                         rope3d_entry_lds(lds, rope.r3, pos, P::template feature<T>(j, g) / 2 + 1)};
                    rotate_pairs<4>(qf[j], cs);
                }
            }
            request(s, i + DEPTH);
            __builtin_amdgcn_sched_barrier(0);
            den += __shfl_xor(den, 16);
            den += __shfl_xor(den, 32);                                 // that of MFMA row n, in all its lanes
            const float dn = den + eps;
            const bool reciprocal = E == 2 && (!CHECKED || __all(fabsf(dn) >= 0x1p-126f));
            const float scale = reciprocal ? 1.0f / dn : dn;
            if (E == 2 && !CHECKED) low = fminf(low, fabsf(dn));
            f32x4 acc[NB] = {};
            if (kPieces && (!CHECKED || whole)) {
                const u32x4 w = {pack_bf16x2(qf[0][0], qf[0][1]), pack_bf16x2(qf[0][2], qf[0][3]), pack_bf16x2(qf[1][0], qf[1][1]), pack_bf16x2(qf[1][2], qf[1][3])};
#pragma unroll
                for (int l = 2; l >= 0; --l)                            // small terms first
#pragma unroll
                    for (int e = 0; e < NB; ++e)
                        acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), piece[l][e], acc[e], 0, 0, 0);
            } else
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int e = 0; e < NB; ++e)
                        acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(qf[j][q], sr[j][q][e], acc[e], 0, 0, 0);
            // element r of block e: MFMA row 4 g + r, token 4 r + g, feature f_out + e
            const uint32_t out = exists ? walk.offset<TILE>(i, row_bytes) + offO : kOutOfRange;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float dd = __shfl(scale, 4 * g + r);
                float o[NB];
#pragma unroll
                for (int e = 0; e < NB; ++e) o[e] = reciprocal ? acc[e][r] * dd : acc[e][r] / dd;
                store_words(rO, out + (uint32_t)(4 * r) * row_bytes, narrow<T, NB>(o));
            }
        }
    }
    return E != 2 || CHECKED || (__all(low >= 0x1p-126f) && (whole || !kPieces));
}

// grid = (C, B*H), block = 256; dynamic LDS: kRope3dLdsBytes with kRope3D.
template <typename T, int D, int ROPE>
__global__ __launch_bounds__(kThreads, 2) void apply_f32(
    const T *__restrict__ Q, T *__restrict__ O, RopeArg rope, TokStrides st, int H, int t0, int t1, int C,
    const float *__restrict__ S, const float *__restrict__ z, float eps, int order)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const bool done = apply_f32_tiles<T, D, ROPE, false>(lds, Q, O, rope, st, H, t0, t1, C, S, z, eps, order);
    if constexpr (sizeof(T) == 2)
        if (__builtin_expect(!done, 0)) apply_f32_tiles<T, D, ROPE, true>(lds, Q, O, rope, st, H, t0, t1, C, S, z, eps, order);
}

}  // namespace sv
