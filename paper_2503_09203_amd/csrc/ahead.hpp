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
// -> 379 for 1,024. (The layout on the matrix cores, v_mfma_f32_4x4x1 with the layout's
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
// The ring holds two groups per tile, 12 KB.
template <typename T>
struct AheadRing {
    static constexpr int kGroup = sizeof(T) == 4 ? 4 : 2;
    T tau[2][kGroup][6][kWave];
    static __device__ __forceinline__ int group(int K) { return K > 32 ? kGroup : 2; }
};

// The thrust wave: rotor states, command rows and their bookkeeping as in env_steps.
template <typename T, int M, bool kOut, bool kShaped>
__device__ __forceinline__ void ahead_thrust(const StepArgs& A, const ClassT<T>& Cs, int64_t env, int lane, bool live,
                                             int64_t t0, AheadRing<T>& ring, bool* fin_out) {
    const int group = AheadRing<T>::group(A.K);
    const int64_t np = A.npad;
    T* S = (T*)A.state + kStateFixed * np + env;
    T n[M], cur[M], nxt[M];
#pragma unroll
    for (int i = 0; i < M; ++i) n[i] = S[i * np];
    const ClassT<T> C = class_in_vgpr<T, M>(Cs);
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
    for (int k0 = 0, buf = 0; k0 < K; k0 += group, buf ^= 1) {
        const int k1 = k0 + group < K ? k0 + group : K;
        [[clang::code_align(64)]] for (int k = k0; k < k1; ++k) {
            T nl[M], tau[6];
            thrust_part<T, M, kShaped>(C, n, cur, nl, tau);
#pragma unroll
            for (int j = 0; j < 6; ++j) ring.tau[buf][k - k0][j][lane] = tau[j];
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
        __syncthreads();
    }
    if (bad && lane == 0) atomicOr(&A.misc->err, kErrActionRow);
    bool fin = true;
#pragma unroll
    for (int i = 0; i < M; ++i) fin &= finite_(n[i]);
    *fin_out = fin;
    if (live) {
#pragma unroll
        for (int i = 0; i < M; ++i) S[i * np] = n[i];
    }
}

// The rigid-body wave.
template <typename T, int M, bool kOut, bool kPayload>
__device__ __forceinline__ void ahead_rigid(const StepArgs& A, const ClassT<T>& C, int64_t env, int lane, bool live,
                                            const AheadRing<T>& ring, EnvT<T>& E, T IA2[3], RigidT<T>& s,
                                            float st[kStats]) {
    const int group = AheadRing<T>::group(A.K);
    const int64_t np = A.npad;
    MGX_WAVE_TS(ts_entry);
    load_rigid<T>((const T*)A.state, np, env, s);
    load_record<T, kPayload>((const T*)A.rec, np, env, C.flags, E);
    T Brb[3];
    env_prologue<T, kPayload>(C, E, IA2, Brb);
    __builtin_amdgcn_s_waitcnt(0);
    MGX_WAVE_TS(ts_loaded);
    const int K = A.K;
    for (int k0 = 0, buf = 0; k0 < K; k0 += group, buf ^= 1) {
        const int k1 = k0 + group < K ? k0 + group : K;
        __syncthreads();
        [[clang::code_align(64)]] for (int k = k0; k < k1; ++k) {
            T tau[6];
#pragma unroll
            for (int j = 0; j < 6; ++j) tau[j] = ring.tau[buf][k - k0][j][lane];
            if constexpr (kOut) {
                T f[kForceLen];
                rigid_part<T, M, true, false, kPayload>(C, E, IA2, Brb, s, nullptr, tau, f);
                if (live) {
                    if (A.forces) {
                        T* fo = (T*)A.forces + k * A.force_stride + env;
#pragma unroll
                        for (int c = 0; c < kForceLen; ++c) fo[c * np] = f[c];
                    }
                    if (A.traj) store_rigid<T>((T*)A.traj + k * A.traj_stride, np, env, s);
                }
            } else {
                rigid_part<T, M, false, false, kPayload>(C, E, IA2, Brb, s, nullptr, tau);
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
template <typename T, int M, bool kOut, bool kShaped, bool kPayload>
__global__ void __launch_bounds__(2 * kAheadTiles * kWave) k_step_ahead(StepLaunch<T> L) {
    __shared__ AheadRing<T> rings[kAheadTiles];
    __shared__ float red[2 * kAheadTiles][kStats];
    __shared__ uint8_t rotors_finite[kAheadTiles][kWave];
    __shared__ int is_last;
    const StepArgs& A = L.a;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int tiles = blockDim.x / (2 * kWave), wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int slot = wv < tiles ? wv : wv - tiles;
    const int64_t tile = (int64_t)blockIdx.x * tiles + slot, last = A.npad / kWave - 1;
    const bool live = tile <= last;
    const int64_t env = (live ? tile : last) * kWave + lane;
    float st[kStats];
#pragma unroll
    for (int j = 0; j < kStats; ++j) st[j] = 0.0f;
    const int64_t t0 = A.misc->t[A.rd];
    if (blockIdx.x == 0 && tid == 0) {
        if (A.advance) A.misc->t[A.wr] = t0 + A.advance;
        prepare_next_slot(A.misc, A.wr);
    }
    if (wv >= tiles) {
        bool fin;
        ahead_thrust<T, M, kOut, kShaped>(A, L.cls, env, lane, live, t0, rings[slot], &fin);
        if (!A.partials) return;
        rotors_finite[slot][lane] = fin ? 1 : 0;
        __syncthreads();
    } else {
        EnvT<T> E;
        RigidT<T> s;
        T IA2[3];
        ahead_rigid<T, M, kOut, kPayload>(A, L.cls, env, lane, live, rings[slot], E, IA2, s, st);
        if (!A.partials) return;
        __syncthreads();
        T m = T(0);
#pragma unroll
        for (int j = 0; j < 3; ++j) m = __builtin_elementwise_maximum(m, abs_(s.p[j]));
#pragma unroll
        for (int j = 0; j < 4; ++j) m = __builtin_elementwise_maximum(m, abs_(s.q[j]));
#pragma unroll
        for (int j = 0; j < 6; ++j) m = __builtin_elementwise_maximum(m, abs_(s.nu[j]));
        env_stats<T, kPayload>(E, IA2, s, m <= (T)3.0e38 && rotors_finite[slot][lane], live && env < A.nvalid, st);
        if (!live) {
#pragma unroll
            for (int j = 0; j < kStats; ++j) st[j] = 0.0f;
        }
    }
    finish_stats(A, st, red, &is_last);
}

}  // namespace mgx
