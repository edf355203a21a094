// The K-step kernel for batches of at most one 64-environment tile per SIMD: two waves per
// tile, one forming the thrust of the steps ahead, the other advancing pose and velocity.
//
// What bounds the one-wave form there: a wave issues at most one vector instruction per four
// cycles, while a SIMD with two waves issues one in little more than two, so a lone wave per
// SIMD leaves issue slots empty whatever its instructions are (1,049 cycles for the step's
// 203; 616 per tile once the SIMD holds several waves). Rotor lag, thrust and layout (54 of
// the 203 for six thrusters) need nothing of the pose or velocity, so a second wave runs them
// ahead of the first, without any exchange back, and hands each step's wrench over in LDS.
// The arithmetic is the one-wave form's, value for value. 1000 steps in one launch: 437 -> 387
// us for 65,536 environments (both waves on each SIMD), 407 -> 335 for 8,192; in double 567
// -> 428 for 1,024 (builds with other register allocations of the same source 379 to 429). (The layout on the matrix cores, v_mfma_f32_4x4x1 with the layout's
// columns broadcast, gives the same bits but holds the SIMD's other wave up: 466 us.)
#pragma once
#include <hip/hip_runtime.h>

#include "env_loop.hpp"
#include "kernels.hpp"

namespace mgx {

constexpr int kAheadTiles = 4;  // tiles per block at most

// Steps are handed over in groups, one block barrier each: of four in a long float launch
// (1000 steps of 8,192 environments: 346 us in groups of two, 335 us), of two in a short one,
// where the rigid-body wave waits for the first group (16-step launches of 65,536: 10.3 us,
// 10.7 in groups of four, 10.75 in the one-wave form), and of two in double (no difference).
// A step's hand-over is the propellers' wrench and, with fins, the sines and cosines of the M
// deflections. The ring holds two groups per tile: 12 KB, or up to 22 KB with fins in groups
// of two (four tiles in groups of four would not fit a compute unit's LDS).
template <typename T, int M, bool kFins>
struct AheadRing {
    static constexpr int kGroup = sizeof(T) == 4 && !kFins ? 4 : 2;
    static constexpr int kRows = 6 + (kFins ? 2 * M : 0);
    T x[2][kGroup][kRows][kWave];
    static __device__ __forceinline__ int group(int K) { return K > 32 ? kGroup : 2; }
};

// End of the hand-over group that starts at step k0: `group` steps on, or the end of the
// stretch of `seg` steps (which both waves keep in `end`) or of the launch.
__device__ __forceinline__ int ahead_group_end(int k0, int group, int seg, int K, int& end) {
    if (k0 == end) end += seg;
    if (end > K) end = K;
    return k0 + group < end ? k0 + group : end;
}

// The thrust wave: rotor states, command rows and their bookkeeping as in env_steps.
template <typename T, int M, bool kOut, bool kShaped, bool kFins, bool kSeg>
__device__ __forceinline__ void ahead_thrust(const StepArgs& A, const ClassT<T>& Cs, int64_t env, int lane, bool live,
                                             int64_t t0, int seg, AheadRing<T, M, kFins>& ring) {
    const int group = ring.group(A.K);
    const int64_t np = A.npad;
    T* S = (T*)A.state + kStateFixed * np + env;
    T n[M], cur[M], nxt[M];
#pragma unroll
    for (int i = 0; i < M; ++i) n[i] = S[i * np];
    const ClassT<T> C = class_in_vgpr<T, M, false, kFins>(Cs);
    const int K = A.K;
    const int64_t hold = A.hold, nrows = A.n_rows, rstride = A.row_stride;
    const T* abase = (const T*)A.actions + env;
    auto clamp_row = [nrows](int64_t x) { return x < 0 ? (int64_t)0 : (x >= nrows ? nrows - 1 : x); };
    const int64_t rowa = floor_div(t0, hold);
    int phase = (int)(t0 - rowa * hold);
    int64_t r = rowa - A.row0;
    bool bad = (r < 0 || r >= nrows);
    const T* p0 = abase + clamp_row(r) * rstride;
#pragma unroll
    for (int i = 0; i < M; ++i) cur[i] = p0[i * np];
    const T* p1 = abase + clamp_row(r + 1) * rstride;
#pragma unroll
    for (int i = 0; i < M; ++i) nxt[i] = p1[i * np];
    if (hold - phase < K && r + 1 >= nrows) bad = true;
    __builtin_amdgcn_s_waitcnt(0);
#pragma unroll
    for (int i = 0; i < M; ++i) cur[i] = clip1(cur[i]);
    [[clang::code_align(64)]] for (int k0 = 0, buf = 0, end = seg; k0 < K; buf ^= 1) {
        const int k1 = kSeg ? ahead_group_end(k0, group, seg, K, end) : k0 + group < K ? k0 + group : K;
        [[clang::code_align(64)]] for (int k = k0; k < k1; ++k) {
            constexpr int kRows = AheadRing<T, M, kFins>::kRows;
            T nl[M], x[kRows];
            thrust_part<T, M, kShaped, kFins>(C, n, cur, nl, x);
            if constexpr (kFins) fin_angles<T, M>(C, nl, x + 6);
#pragma unroll
            for (int j = 0; j < kRows; ++j) ring.x[buf][k - k0][j][lane] = x[j];
#pragma unroll
            for (int i = 0; i < M; ++i) n[i] = nl[i];
            if constexpr (kOut) {
                if (A.traj && live) {
                    T* to = (T*)A.traj + k * A.traj_stride + kStateFixed * np + env;
#pragma unroll
                    for (int i = 0; i < M; ++i) to[i * np] = n[i];
                }
            }
            if (++phase == hold) {
                phase = 0;
                ++r;
#pragma unroll
                for (int i = 0; i < M; ++i) cur[i] = clip1(nxt[i]);
                const T* pn = abase + clamp_row(r + 1) * rstride;
#pragma unroll
                for (int i = 0; i < M; ++i) nxt[i] = pn[i * np];
                if (k + 1 + hold < K && r + 1 >= nrows) bad = true;
            }
        }
        k0 = kSeg ? k1 : k0 + group;
        __syncthreads();
    }
    if (bad && lane == 0) atomicOr(&A.misc->err, kErrActionRow);
    if (live) {
#pragma unroll
        for (int i = 0; i < M; ++i) S[i * np] = n[i];
    }
}

// The rigid-body wave.
template <typename T, int M, bool kOut, bool kFins, bool kPayload, bool kSeg>
__device__ __forceinline__ void ahead_rigid(const StepArgs& A, const ClassT<T>& Cs, int64_t env, int lane, bool live,
                                            int seg, const AheadRing<T, M, kFins>& ring) {
    const int group = ring.group(A.K);
    const int64_t np = A.npad;
    MGX_WAVE_TS(ts_entry);
    RigidT<T> s;
    EnvT<T> E;
    T IA2[3], Brb[3];
    float st[kStats];  // launches with statistics run the one-wave form
    load_rigid<T>((const T*)A.state, np, env, s);
    load_record<T, kPayload>((const T*)A.rec, np, env, Cs.flags, E);
    const ClassT<T> C = fins_in_vgpr<T, M, kFins>(Cs);
    // classes with fins carry the attitude's low-order words through a stretch (float)
    constexpr bool kComp = kFins && std::is_same<T, float>::value;
    StateLo<T> lo;
#pragma unroll
    for (int j = 0; j < 4; ++j) lo.q[j] = T(0);
    env_prologue<T, kPayload>(C, E, IA2, Brb);
    __builtin_amdgcn_s_waitcnt(0);
    MGX_WAVE_TS(ts_loaded);
    const int K = A.K;
    [[clang::code_align(64)]] for (int k0 = 0, buf = 0, end = seg; k0 < K; buf ^= 1) {
        const int k1 = kSeg ? ahead_group_end(k0, group, seg, K, end) : k0 + group < K ? k0 + group : K;
        __syncthreads();
        [[clang::code_align(64)]] for (int k = k0; k < k1; ++k) {
            constexpr int kRows = AheadRing<T, M, kFins>::kRows;
            T x[kRows];
#pragma unroll
            for (int j = 0; j < kRows; ++j) x[j] = ring.x[buf][k - k0][j][lane];
            if constexpr (kOut) {
                T f[kForceLen];
                rigid_part<T, M, true, kFins, kPayload, kComp, false, true>(C, E, IA2, Brb, s, x + 6, x, f, &lo);
                if (live) {
                    if (A.forces) {
                        T* fo = (T*)A.forces + k * A.force_stride + env;
#pragma unroll
                        for (int c = 0; c < kForceLen; ++c) fo[c * np] = f[c];
                    }
                    if (A.traj) store_rigid<T>((T*)A.traj + k * A.traj_stride, np, env, s);
                }
            } else {
                rigid_part<T, M, false, kFins, kPayload, kComp, false, true>(C, E, IA2, Brb, s, x + 6, x, nullptr, &lo);
            }
        }
        k0 = kSeg ? k1 : k0 + group;
        if constexpr (kSeg) {
            if (k1 == end && k1 < K) {
                renorm_attitude<T>(s, st);
#pragma unroll
                for (int j = 0; j < 4; ++j) lo.q[j] = T(0);
            }
        }
    }
    MGX_WAVE_TS(ts_stepped);
    renorm_attitude<T>(s, st);
    if (live) store_rigid<T>((T*)A.state, np, env, s);
#ifdef MGX_WAVE_TIMESTAMPS
    __builtin_amdgcn_s_waitcnt(0);
    MGX_WAVE_TS(ts_stored);
    if (lane == 0 && live && env / kWave < kWaveTsMax) {
        g_wave_ts[env / kWave][0] = ts_entry;
        g_wave_ts[env / kWave][1] = ts_loaded;
        g_wave_ts[env / kWave][2] = ts_stepped;
        g_wave_ts[env / kWave][3] = ts_stored;
    }
#endif
}

// Blocks of up to kAheadTiles tiles: the first half of a block's waves are the rigid-body
// waves, so that with four tiles each SIMD of the compute unit holds one wave of either
// kind. Waves past the segment run its last tile and store nothing.
// kSeg: the launch holds several stretches of L.seg steps (a kernel of its own: the cut of
// the hand-over groups at the stretches' ends costs a double launch of one stretch 10%).
template <typename T, int M, bool kOut, bool kShaped, bool kFins, bool kPayload, bool kSeg>
__global__ void __launch_bounds__(2 * kAheadTiles * kWave) k_step_ahead(StepLaunch<T> L) {
    __shared__ AheadRing<T, M, kFins> rings[kAheadTiles];
    const StepArgs& A = L.a;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int tiles = blockDim.x / (2 * kWave), wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int slot = wv < tiles ? wv : wv - tiles;
    const int64_t tile = (int64_t)blockIdx.x * tiles + slot, last = A.npad / kWave - 1;
    const bool live = tile <= last;
    const int64_t env = (live ? tile : last) * kWave + lane;
    const int64_t t0 = A.misc->t[A.rd];
    if (blockIdx.x == 0 && tid == 0) {
        if (A.advance) A.misc->t[A.wr] = t0 + A.advance;
        prepare_next_slot(A.misc, A.wr);
    }
    if (wv >= tiles)
        ahead_thrust<T, M, kOut, kShaped, kFins, kSeg>(A, L.cls, env, lane, live, t0, L.seg, rings[slot]);
    else
        ahead_rigid<T, M, kOut, kFins, kPayload, kSeg>(A, L.cls, env, lane, live, L.seg, rings[slot]);
}

}  // namespace mgx
