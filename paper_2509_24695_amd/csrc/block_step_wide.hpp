// One-launch block step for d = 112 and 128 (Sec. 3.3.1; cache update and use of Alg. 1):
//
//   S += phi(K_b)^T V_b,  z += sum phi(K_b),  O_b = phi(Q_b) S / (phi(Q_b) z + eps)
//
// with O_b computed from the UPDATED state.  The state phase is that of coop_state.hpp, the apply phase that of coop128.hpp for eight waves, so
// one workgroup shape serves both: eight waves that share tiles of 64 tokens, one workgroup per compute unit, all of them resident.
//
// What two launches lose at block size is the gap between them, the second one's start (its tables, its first tiles, 50 KB of state for each of
// three workgroups per compute unit) and, above all, the exchange of 50 KB of sums per workgroup through the memory that all dies share: at
// 20 heads of 112 and 4 680 tokens the first of the following took 4.3 us of a 32 us step, at the 2.8 TB/s at which all stores together go out.
//   - A head whose workgroups are on one die (wide_roles) exchanges its sums through that die's L2: plain stores, coherent loads, as in
//     block_step_mfma.  Step 32.0 -> 27.8 us, with factored tables 38.0 -> 33.0.
//   - The new state travels in the order in which the operands of the apply phase need it (wide_word): workgroup c puts its slice in place of
//     slice c of partial 0, which nobody else reads, and an operand is two 16-byte loads per lane.
//   - A workgroup that has a head to itself (SOLE) keeps the new state in LDS: no partial, no flag, no wait.
//   - The first two tiles of Q are requested with the first tiles of K and V.  Four and six, or the later ones during the exchange: level to 1 us slower.
// Timeline (medians over workgroups, us after the first workgroup's entry, plain / factored tables): state summed 9.6 / 11.8, partial stored 11.4 /
// 13.6, all partials of the head in 12.5 / 15.0, slice folded 13.8 / 16.3, all slices in 14.9 / 17.7, operands in registers 15.8 / 18.7, O stored
// 24.5 / 29.6 (the last workgroup 27.2 / 32.5).  The token phases run at 5 to 6.7 TB/s between their ends; with factored tables vector
// instructions bound them.
// Stream of four such blocks 133 -> 120 us, factored tables 154 -> 137 (2.5 TB/s over all); 160 heads of 128, 1 560 tokens, a workgroup each: 62 -> 57 us a step
// (4.5 TB/s); 400 heads of 112, 240 tokens 159 -> 53.  wide_step_serves says where two launches stay ahead.
#pragma once

#include "coop128.hpp"
#include "coop_state.hpp"

namespace sv {

// The 128 x 32 panel of S of value block vb as MFMA operands, from words in the order of wide_word: word(v) fetches word v.  (Row F of the
// panel and its place in the accumulators: ApplyOperands.)
template <class WordFn>
__device__ __forceinline__ void wide_operands(ApplyOperands<128, true, 1, false> &A, int d, int vb, int lane, WordFn word)
{
    const int m = lane & 31, g = lane >> 5;
    const int F = 32 * vb + 16 * ((m >> 2) & 1) + 4 * (m >> 3) + (m & 3);
    f32x4 x[8][2];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int R = 2 * ks + g;
            x[ks][q] = word(8 * R < d && F < d ? wide_word(d, R, q, F) : -1);
        }
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
        uint32_t hi[4], lo[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const float a = x[ks][p >> 1][2 * (p & 1)], b = x[ks][p >> 1][2 * (p & 1) + 1];
            hi[p] = pack_bf16x2(a, b);
            lo[p] = pack_bf16x2(a - bf16_lo(hi[p]), b - bf16_hi(hi[p]));
        }
        const u32x4 h4 = {hi[0], hi[1], hi[2], hi[3]}, l4 = {lo[0], lo[1], lo[2], lo[3]};
        A.s[0][0][ks] = __builtin_bit_cast(bf16x8, h4);
        A.s[1][0][ks] = __builtin_bit_cast(bf16x8, l4);
    }
}

template <int ROPE> constexpr int block_step_wide_lds()
{
    static_assert(step_apply_lds_bytes() <= kCoopZOffset, "the apply's tiles fit where the state's were");
    static_assert(128 * 128 * 4 <= kCoopZOffset, "so does the state of a head");
    return coop_state_lds<ROPE>();
}

// grid: see WideRoles, or (C, B*H) with C chunks per head; block = kCoopThreads.  With several workgroups per head all have to be resident: they wait for each
// other, a bounded number of polls (a wait that runs out is recorded in the workspace and its wave stores nothing more).
// ROPE: keys and queries are rotated after the ReLU in the numerator path.  NT: see load_stream16.
template <int ROPE, bool NT, bool SOLE>
__global__ __launch_bounds__(kCoopThreads, 2) void block_step_mfma_wide(
    const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K, const uint16_t *__restrict__ V, uint16_t *__restrict__ O, RopeArg rope,
    TokStrides st, int H, int d, int N, int C, const float *S_in, const float *z_in, float *S_out, float *z_out, float eps,
    void *__restrict__ ws, unsigned long long epoch, uint32_t spin_limit, int order, WideRoles roles)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int DEPTH_S = 2, DEPTH_A = 2;      // tiles of K and V, and of Q, in flight
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const WgRole role(C, order);
    int c = role.c, bh = role.bh, BH = gridDim.y;
    bool local = false;
    if (!SOLE && roles.dies) {
        BH = roles.BH;
        if (!wide_role((int)blockIdx.x, roles, c, C, bh, local)) return;
    }
    const int b = bh / H, h = bh % H;
    // The state kernels' phase keys, wherever the head lives.  With keys dealt die by die (die_local_phase_key) the eight neighbouring heads of the dies walked
    // in phase; where as many head strides come near a power of two (4 680, 9 360, 18 720 tokens) their streams met on the same DRAM
    // resources (128 heads of 128, 9 360 tokens 261 -> 225 us a block, 80 heads 162 -> 140, 128 heads of 112, 18 720 tokens 426 -> 356; nothing slower).
    const int phase = order & kOrderLockstep ? 5 * b : bh;
    const int64_t head_off = b * st.b + h * st.h;
    const int elems = d * d + d;
    const int n_tiles = (N + kCoopTokens - 1) / kCoopTokens;
    const WideTarget target{S_in + (size_t)bh * d * d, z_in + (size_t)bh * d, S_out + (size_t)bh * d * d, z_out + (size_t)bh * d,
                            static_cast<float *>(ws) + (size_t)bh * kMaxChunks * elems, d, c, C};
    EpochSource es;
    if (!SOLE) es.begin(ws, BH, elems, epoch, bh, c, C);

    // The first tiles of Q arrive during the state phase; with a full table their rows would take registers that phase needs.
    constexpr bool kEarlyQ = ROPE != kRopeTable;
    // Both phases walk the same tiles of 64 tokens.
    const TileWalk walk(0, c, C, n_tiles, phase);
    static_assert(CoopApplyStream<DEPTH_A, ROPE, kCoopWaves, 1, NT>::STEP == kCoopTokens, "both phases walk tiles of the same size");
    CoopApplyStream<DEPTH_A, ROPE, kCoopWaves, 1, NT> qstream(Q + head_off, O + head_off, rope, lds + kCoopTabOffset, st.n, N, d, wave, lane, walk);
    CoopStateStream<DEPTH_S, ROPE, NT> kvstream(K + head_off, V + head_off, rope, lds + kCoopTabOffset, st.n, N, d, wave, lane, walk);
    Rope3dFill tabs;
    if (ROPE == kRope3D) rope3d_lds_fill_begin(rope.r3, tabs);   // the first loads of the kernel
#pragma unroll
    for (int s = 0; s < DEPTH_S; ++s) {
        kvstream.request(s, s);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (kEarlyQ) coop_apply_prefetch<0, DEPTH_A>(qstream);
    kvstream.rot.template begin_tile<kCoopTokens>(walk, 0);        // while the tables and the first tiles are on their way
    if (ROPE == kRope3D) {
        rope3d_lds_fill_end(lds + kCoopTabOffset, rope.r3, tabs);
        wg_barrier();
    }
    // The queries' positions are worked out when the state phase is over: the compiler would keep them in registers all along.  Factored tables
    // only: with a full table the rotator holds the rows requested with the first tiles of Q.
    auto q_positions = [&]() __attribute__((always_inline)) {
        if constexpr (ROPE == kRope3D) {
            int l = lane;
            asm volatile("" : "+v"(l));
            qstream.rot = decltype(qstream.rot)(rope, N, d, 8 * wave + (l >> 4), 4, 4 * (l & 15), 1, lds + kCoopTabOffset);
            qstream.rot.template begin_tile<kCoopTokens>(walk, 0);
        }
    };
    float *zw = reinterpret_cast<float *>(lds + kCoopZOffset);  // [wave][128]
    ApplyOperands<128, true, 1, false> A;
    float zr[8];
    if constexpr (SOLE) {
        f32x16 fin[2];
        const int kb = wave >> 1, vb = wave & 1;
        coop_state_sum(kvstream, lds, zw, wave, lane, fin);
        lds_barrier();
        if (!kEarlyQ) coop_apply_prefetch<0, DEPTH_A>(qstream);
        wide_store_sole<2>(fin, kb, 2 * vb, target, lane);
        // the new state stays in LDS, in the order of wide_word, the key sums behind it
        f32x4 *words = reinterpret_cast<f32x4 *>(lds);
        float *z_lds = reinterpret_cast<float *>(lds + 128 * 128 * 4);
        const int n = lane & 31, g = lane >> 5;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (32 * kb + 8 * q < d && 64 * vb + 32 * cb + n < d)
                    words[wide_word(d, 4 * kb + q, g, 64 * vb + 32 * cb + n)] = f32x4{fin[cb][4 * q], fin[cb][4 * q + 1], fin[cb][4 * q + 2], fin[cb][4 * q + 3]};
        if (tid < 128) {
            const float x = tid < d ? target.z_in[tid] + coop_key_sum(zw, tid) : 0.f;
            z_lds[tid] = x;
            if (tid < d) target.z_out[tid] = x;
        }
        lds_barrier();
        wide_operands(A, d, wave & 3, lane, [&](int v) __attribute__((always_inline)) {
            const f32x4 x = words[v >= 0 ? v : 0];
            return v >= 0 ? x : f32x4{0.f, 0.f, 0.f, 0.f};
        });
#pragma unroll
        for (int e = 0; e < 8; ++e) zr[e] = z_lds[8 * (lane & 15) + e];
        q_positions();
        lds_barrier();                           // the tiles of the apply phase go where the state was
    } else {
        {
            f32x16 fin[2];
            coop_state_sum(kvstream, lds, zw, wave, lane, fin);
            lds_barrier();
            float *zp = target.partials + (size_t)c * elems + (size_t)d * d + 2 * tid;
            const f32x2 zs = tid < d / 2 ? f32x2{coop_key_sum(zw, 2 * tid), coop_key_sum(zw, 2 * tid + 1)} : f32x2{0.f, 0.f};
            if (local) {
                wide_store_block<2, true>(fin, wave >> 1, 2 * (wave & 1), false, target, lane);
                if (tid < d / 2) store_coherent<true>(zp, zs);
            } else {
                wide_store_block<2>(fin, wave >> 1, 2 * (wave & 1), false, target, lane);
                if (tid < d / 2) store_coherent(zp, zs);
            }
        }
        // ---- the head agrees on its new state ------------------------------------------------------
        int *failed = reinterpret_cast<int *>(lds + kCoopEpochOffset + 8);
        if (tid == 0) failed[0] = failed[1] = 0;
        epoch = es.resolve(reinterpret_cast<unsigned long long *>(lds + kCoopEpochOffset));
        const uint32_t my_die = local ? die_id() : 0u;
        // tells the head's other workgroups that this one's stores are done; waits for theirs
        auto publish = [&](int phase) __attribute__((always_inline)) {
            unsigned long long *flag = ws_flags(ws, BH, elems, bh, 0) + wide_flag_word(local, phase, c, C, kMaxChunks);
            if (tid != 0) return;
            if (local) flag_publish<true>(flag, flag_with_die(epoch, my_die));
            else flag_publish(flag, epoch);
        };
        auto wait = [&](int phase) __attribute__((always_inline)) {
            if (!local) return state_wait(ws, BH, elems, bh, C, phase, epoch, spin_limit, lane);
            bool same_die;
            const bool ok = flags_wait_all_local(ws_flags(ws, BH, elems, bh, 0) + wide_flag_word(local, phase, 0, C, kMaxChunks), C, epoch, spin_limit, lane, my_die, &same_die) && same_die;
            if (!ok && lane == 0) __hip_atomic_store(ws_error(ws, BH, elems), kWsTimeoutMark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return ok;
        };
        const WideSlice sl(c, C, d);
        const rsrc_t rP = make_rsrc(target.partials, (uint32_t)C * (uint32_t)elems * 4u);
        const bool folds = sl.lo + 64 * wave < sl.hi;               // waves past the slice have nothing to fold
        auto fold = [&](auto units, auto group) __attribute__((always_inline)) {
            f32x4 x[units()];
            wide_carried<kCoopThreads>(target, sl, sl.lo + tid, x);
            coherent_stores_done();
            wg_barrier();
            publish(0);
            if (!folds) return;
            if (!wait(0)) {
                failed[0] = 1;
                return;
            }
            // Slice c of partial 0 is read by this workgroup alone: its words of the new state take their place there, for the others.
            wide_fold_slice<kCoopThreads, units(), group()>(target, sl, x, [&](int v, f32x4 y) __attribute__((always_inline)) {
                if (local) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, y), rP, 16u * (uint32_t)v, 0, 0);
                else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, y), rP, 16u * (uint32_t)v, 0, 16 /* sc1 */);
                wide_store_word(target, sl, v, y);
            });
        };
        using std::integral_constant;
        if (C <= 2) fold(integral_constant<int, 4>{}, integral_constant<int, 2>{});
        else if (C <= 4) fold(integral_constant<int, 3>{}, integral_constant<int, 4>{});
        else if (C <= 8) fold(integral_constant<int, 2>{}, integral_constant<int, 8>{});
        else fold(integral_constant<int, 1>{}, integral_constant<int, 16>{});
        if (folds) coherent_stores_done();
        wg_barrier();
        if (failed[0]) return;
        publish(1);
        if (!kEarlyQ) coop_apply_prefetch<0, DEPTH_A>(qstream);
        q_positions();
        if (!wait(1)) failed[1] = 1;
        wg_barrier();
        if (failed[1]) return;

        // ---- its operands ----
        {
            f32x4 z4[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int k = 8 * (lane & 15) + 4 * q;
                z4[q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rP, k < d ? 4u * (uint32_t)(d * d + k) : kOutOfRange, 0, 16));
            }
            wide_operands(A, d, wave & 3, lane, [&](int v) __attribute__((always_inline)) {
                return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rP, v >= 0 ? 16u * (uint32_t)v : kOutOfRange, 0, 16));
            });
#pragma unroll
            for (int e = 0; e < 8; ++e) zr[e] = z4[e >> 2][e & 3];
        }
    }
    // ---- apply the updated state to this workgroup's share of Q_b --------------------------------
    apply_tiles_steps(qstream, lds, wave, lane, A, zr, eps);
}

}  // namespace sv
