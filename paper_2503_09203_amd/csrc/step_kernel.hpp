// The step kernel and its launchers, shared by the translation units that instantiate it
// per element type (the step kernels are most of the build's compile time).
#pragma once
#include <hip/hip_runtime.h>

#include "ahead.hpp"
#include "env_loop.hpp"
#include "kernels.hpp"

namespace mgx {

// ----------------------------------------------------------------------------- step

// K steps of every environment of one class segment; state in registers throughout.
// kShaped: the class has dead zones or direction-dependent gains; kFins: it has fins;
// kPayload: its centre of gravity is off the body origin (fin and payload classes take the
// shaped propeller body too). Each is a separate instantiation (chosen
// on the host from the class) rather than a branch in one kernel, so that the plain
// body's register allocation does not pay for the others.
template <typename T, int M, bool kOut, bool kSingle, bool kShaped, bool kFins, bool kPayload>
__global__ void __launch_bounds__(256) k_step(StepLaunch<T> L) {
    const StepArgs& A = L.a;
    const int tid = threadIdx.x;
    const int64_t env = (int64_t)blockIdx.x * blockDim.x + tid;
    float st[kStats];
#pragma unroll
    for (int j = 0; j < kStats; ++j) st[j] = 0.0f;
    if constexpr (kSingle) {
        // Every lane runs (lanes past the segment on its last slot, without storing), so the
        // loads sit outside any branch; the step reads the counter itself, and the counter
        // update of slot wr comes after the environment work, so that no store precedes
        // (and may alias) the state and record loads. (Done that way in the K-step form, the
        // 16-step launch measured slower: 12.05 against 11.55 us.)
        int64_t t0 = 0;
        env_steps<T, M, kOut, kShaped, kSingle, kFins, kPayload>(A, L.cls, env, 0, A.K, st, &t0);
        if (blockIdx.x == 0 && tid == 0) {
            if (A.advance) A.misc->t[A.wr] = t0 + A.advance;
            prepare_next_slot(A.misc, A.wr);
        }
    } else {
        const int64_t t0 = A.misc->t[A.rd];
        if (blockIdx.x == 0 && tid == 0) {
            if (A.advance) A.misc->t[A.wr] = t0 + A.advance;
            prepare_next_slot(A.misc, A.wr);  // the next launch may be a persistent one
        }
        if (env < A.npad) env_steps<T, M, kOut, kShaped, kSingle, kFins, kPayload>(A, L.cls, env, t0, A.K, st);
    }
    if (!A.partials) return;
    // Statistics: block partials, then the last block to finish reduces them in order.
    __shared__ float red[256 / kWave][kStats];
    __shared__ int is_last;
    block_reduce_stats(st, red, A.partials + (int64_t)blockIdx.x * kStats);
    __threadfence();
    __syncthreads();
    if (tid == 0) {
        const unsigned prev = atomicAdd(&A.misc->done[A.class_index], 1u);
        is_last = (prev == gridDim.x - 1);
    }
    __syncthreads();
    if (is_last) {
        __threadfence();
        if (tid < kStats) final_reduce_stats(A.partials, gridDim.x, tid, A.stats);
        if (tid == 0) atomicExch(&A.misc->done[A.class_index], 0u);
    }
}

template <typename T, int M, bool kShaped, bool kFins, bool kPayload = false>
static void launch_step_body(const StepLaunch<T>& L, unsigned grid, int block, bool out, bool single,
                             int n_cu, hipStream_t s) {
    constexpr bool kDoubleFins = kFins && std::is_same<T, double>::value;
    if constexpr (!kDoubleFins) {
        // Launches with outputs: both waves store, and those of the short hand-over groups only
        // wait for each other (4,571 environments with the trajectory: 8 steps 8.4 -> 9.3 us,
        // 64 steps 42.6 -> 45.1), so they take two waves only for longer launches of the float
        // bodies with more to do per step, up to two tiles per compute unit. The thrust of seven
        // or eight actuators pays for the hand-over by itself (64 steps of 1,024 to 32,768, eight
        // shaped: 6 to 8% less). With fewer, what pays is the command rows, which wait for
        // another wave's stores no more: 64 steps of six, a row every step 20 to 30% less, every
        // 4 steps 4 to 9%, every 10 with a payload 3% less and without 2% less to 1% more, held
        // throughout up to 5% more; of four, a row every step 10% less, every 4 steps 2 to 7%
        // more.
        constexpr bool kAheadOut = kShaped && !kFins && sizeof(T) == 4;
        constexpr int64_t kOutHold = M >= 7 ? INT64_MAX : M == 6 ? (kPayload ? 16 : 8) : 1;
        if (!L.a.partials && two_waves(L.a.npad, L.a.K, kDoubleFins, n_cu) &&
            (!out || (kAheadOut && L.a.K > 32 && L.a.hold <= kOutHold && L.a.npad / kWave <= 2 * (int64_t)n_cu))) {
            // One block per compute unit, the tiles spread over all units: a block's waves go
            // round its unit's SIMDs, so no SIMD holds two rigid-body waves. (In blocks of four,
            // 33,000 environments left half the units idle: 8-step launches 7.06 us, 6.49 so,
            // 6.77 with one wave per tile.) Up to two tiles per unit, float bodies without outputs
            // stay at one per block where the LDS of two blocks fits a unit (16-step launches of
            // 20,000 8.61 us, 8.91 in blocks of two; with a trajectory, 64 steps 54.3, 49.1 in
            // blocks of two). Where it does not (eight actuators with fins), half the
            // blocks would wait for the others to end: 100 steps of 20,000 187 us, 96 so, 129
            // with one wave per tile. In double, two blocks' waves share SIMDs: 56.5 us, 48.2 so.
            constexpr size_t kUnitLds = 160 * 1024;
            constexpr bool kTwoBlocks =
                sizeof(T) == 4 && 2 * kAheadTiles * sizeof(AheadRing<T, M, kFins>) < kUnitLds;
            const int64_t tiles = L.a.npad / kWave;
            const int per = kTwoBlocks && !out && tiles <= 2 * (int64_t)n_cu ? 1 : (int)((tiles + n_cu - 1) / n_cu);
            const dim3 g((unsigned)((tiles + per - 1) / per)), b(2 * per * kWave);
            if (out) {
                if constexpr (kAheadOut)
                    hipLaunchKernelGGL((k_step_ahead<T, M, true, kShaped, kFins, kPayload, false>), g, b, 0, s, L);
            } else if (L.seg < L.a.K)
                hipLaunchKernelGGL((k_step_ahead<T, M, false, kShaped, kFins, kPayload, true>), g, b, 0, s, L);
            else
                hipLaunchKernelGGL((k_step_ahead<T, M, false, kShaped, kFins, kPayload, false>), g, b, 0, s, L);
            return;
        }
    }
    if (out)
        hipLaunchKernelGGL((k_step<T, M, true, false, kShaped, kFins, kPayload>), dim3(grid), dim3(block), 0, s, L);
    else if (single)
        hipLaunchKernelGGL((k_step<T, M, false, true, kShaped, kFins, kPayload>), dim3(grid), dim3(block), 0, s, L);
    else
        hipLaunchKernelGGL((k_step<T, M, false, false, kShaped, kFins, kPayload>), dim3(grid), dim3(block), 0, s, L);
}

// Five bodies: plain; shaped propellers; fins (with shaped propellers); payload (with
// shaped propellers); payload with fins and shaped propellers, the most general one. The
// payload body without fins keeps the fin geometry out of its registers.
template <typename T, int M>
static void launch_step_m(const StepLaunch<T>& L, unsigned grid, int block, bool out, bool single, bool shaped,
                          bool fins, bool payload, int n_cu, hipStream_t s) {
    if (payload && fins)
        launch_step_body<T, M, true, true, true>(L, grid, block, out, single, n_cu, s);
    else if (payload)
        launch_step_body<T, M, true, false, true>(L, grid, block, out, single, n_cu, s);
    else if (fins)
        launch_step_body<T, M, true, true>(L, grid, block, out, single, n_cu, s);
    else if (shaped)
        launch_step_body<T, M, true, false>(L, grid, block, out, single, n_cu, s);
    else
        launch_step_body<T, M, false, false>(L, grid, block, out, single, n_cu, s);
}

#define MGX_STEP_CASE(MM)                                                     \
    case MM:                                                                  \
        launch_step_m<T, MM>(L, grid, block, out, single, shaped, fins, payload, n_cu, s);   \
        break;

template <typename T>
hipError_t launch_step(const StepLaunch<T>& L, int m, int block, int n_cu, hipStream_t s) {
    const unsigned grid = (unsigned)((L.a.npad + block - 1) / block);
    const bool out = L.a.traj != nullptr || L.a.forces != nullptr;
    // The single-step instantiation fetches the action row the host expects beside the
    // state; a one-step launch without that expectation (in a graph replayed from another
    // step than it was captured at) runs the K-step one, which reads the counter first.
    const bool single = L.a.K == 1 && L.a.t_hint >= 0;
    const bool shaped = L.cls.shaped != 0;
    const bool fins = L.cls.fin_mask != 0;
    const bool payload = L.cls.payload != 0;
    switch (m) {
        MGX_STEP_CASE(1)
        MGX_STEP_CASE(2)
        MGX_STEP_CASE(3)
        MGX_STEP_CASE(4)
        MGX_STEP_CASE(5)
        MGX_STEP_CASE(6)
        MGX_STEP_CASE(7)
        MGX_STEP_CASE(8)
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace mgx
