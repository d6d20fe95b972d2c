// Held-command step kernels: K steps per launch with each drone's state in
// registers (K = 1 is the plain single-step kernel), in three lane mappings
// (per-lane world, one world per tile, persistent work queue over tiles).
#include "cf_device.hpp"
#include "cf_dispatch.hpp"
#include "cf_internal.hpp"

namespace cfk {

constexpr int STEP_PARTS = 3;

// One drone, K steps with a held command; state rows st[i*D + d].
// MR: variant for an onboard controller slower than the physics; ONE: for a single step
template <int MODEL, int CTRL, int INTEG, bool AERO, bool MR, bool ONE, class R>
__device__ __forceinline__ void run_held(const R& rec, const StepArgs& a, size_t d, int w) {
    const size_t D = (size_t)a.D;
    const int K = ONE ? 1 : a.K;
    bool bad = false;
    if constexpr (MODEL == MODEL_FP) {
        constexpr int S = (CTRL == CTRL_PID) ? S_PID : S_FP;
        const FpParams P = load_fp<AERO>(rec);
        float x[S], u[4], comp[S_FP];
#pragma unroll
        for (int i = 0; i < S; ++i) x[i] = a.st[i * D + d];
        rotors_to_dev(x, P);
#pragma unroll
        for (int i = 0; i < S_FP; ++i) comp[i] = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = a.cmd[i * D + d];
        float rc[4] = {0.f, 0.f, 0.f, 0.f};   // held rotor commands
        int phase = 0;                        // launches start on a controller step
        // the controller's gains are read where it runs (scalar loads of the world's
        // record) rather than held in registers through the integration; with a world
        // per lane they would be 33 vector loads a step, so there they stay in
        // registers (131 072 position-controlled worlds, 100 steps: 200 -> 173 us)
        constexpr bool HOLD_GAINS = ONE || std::is_same<R, SoaRec>::value;
        PidParams C;
        if constexpr (CTRL != CTRL_ROTOR && HOLD_GAINS) C = load_pid(rec, CTRL == CTRL_POSITION);
        for (int k = 0; k < K; ++k) {
            const bool ctrl_now = MR ? phase == 0 : true;
            if constexpr (CTRL != CTRL_ROTOR && !HOLD_GAINS) {
                if (ctrl_now) C = load_pid(laundered(rec), CTRL == CTRL_POSITION);
            }
            fp_step<CTRL, INTEG>(x, comp, u, P, C, a.dt, a.dtc, a.inv_dtc, a.renorm, rc, ctrl_now);
            if constexpr (MR) {
                if (++phase == a.ctrl_every) phase = 0;
            }
        }
        rotors_from_dev(x, P);
        // the row addresses are formed again here rather than kept from the loads
        // through the step loop (where they would take registers or scratch)
        size_t ds = d;
        asm volatile("" : "+v"(ds));
#pragma unroll
        for (int i = 0; i < S; ++i) {
            a.st[i * D + ds] = x[i];
            bad |= !isfinite(x[i]);
        }
    } else {
        const IdParams P = load_id<AERO>(rec);
        float x[S_ID], u[4], comp[S_ID];
#pragma unroll
        for (int i = 0; i < S_ID; ++i) { x[i] = a.st[i * D + d]; comp[i] = 0.f; }
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = a.cmd[i * D + d];
        EulerBase B;
        for (int k = 0; k < K; ++k) {
            id_begin_step(x, B, k);
            id_step_base<INTEG>(x, comp, u, P, a.dt, B);
        }
        size_t ds = d;
        asm volatile("" : "+v"(ds));
#pragma unroll
        for (int i = 0; i < S_ID; ++i) {
            a.st[i * D + ds] = x[i];
            bad |= !isfinite(x[i]);
        }
    }
    if (a.nonfinite && bad) atomicOr(a.nonfinite + w, 1u);
}

template <int MODELS, int CTRL, int INTEG, bool AERO, bool MR, bool ONE, class R>
__device__ __forceinline__ void run_model(int model, const R& rec, const StepArgs& a, size_t d, int w) {
    if constexpr (MODELS == MS_FP) {
        run_held<MODEL_FP, CTRL, INTEG, AERO, MR, ONE>(rec, a, d, w);
    } else if constexpr (MODELS == MS_ID) {
        run_held<MODEL_ID, CTRL, INTEG, AERO, MR, ONE>(rec, a, d, w);
    } else {
        if (model == MODEL_FP) run_held<MODEL_FP, CTRL, INTEG, AERO, MR, ONE>(rec, a, d, w);
        else run_held<MODEL_ID, CTRL, INTEG, AERO, MR, ONE>(rec, a, d, w);
    }
}

// A packed tile: `count` consecutive entries of the drone list from `first`, all
// of one model, possibly of several worlds (every tile but each model's last is
// full, so no lanes idle at world ends). A wave whose lanes share one world
// reads that world's parameters with scalar loads into scalar registers; a wave
// across a world boundary reads each lane's own with vector loads.
template <int MODELS, int CTRL, int INTEG, bool AERO, bool MR, bool ONE>
__device__ __forceinline__ void run_tile(const StepArgs& a, int4 td) {
    // td = {first list entry, drone count, model, 0}, uniform over the workgroup
    const int first = __builtin_amdgcn_readfirstlane(td.x);
    const int cnt = __builtin_amdgcn_readfirstlane(td.y);
    const int model = __builtin_amdgcn_readfirstlane(td.z);
    const int lane = threadIdx.x;
    if (lane >= cnt) return;
    const size_t d = (size_t)a.plist[first + lane];
    const int w = a.drone_world[d];
    const int w0 = __builtin_amdgcn_readfirstlane(w);
    if (__builtin_amdgcn_ballot_w64(w != w0) == 0) {
        run_model<MODELS, CTRL, INTEG, AERO, MR, ONE>(model, AosRec{a.par_aos + (size_t)w0 * NREC}, a, d, w0);
    } else {
        run_model<MODELS, CTRL, INTEG, AERO, MR, ONE>(model, LaneRec{a.par_aos + (size_t)w * NREC}, a, d, w);
    }
}

template <int MODELS, int CTRL, int INTEG, bool AERO, bool MR, bool ONE>
__global__ __launch_bounds__(256) void k_step_lane(StepArgs a) {
    const size_t d = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= (size_t)a.D) return;
    const int w = a.drone_world[d];
    constexpr int MODEL = MODELS == MS_FP ? MODEL_FP : MODEL_ID;
    if constexpr (ONE) {
        if (soa_quads(a.D, a.M)) {
            run_held<MODEL, CTRL, INTEG, AERO, MR, ONE>(QuadRec{a.par_soa, a.M, w}, a, d, w);
            return;
        }
    }
    run_held<MODEL, CTRL, INTEG, AERO, MR, ONE>(SoaRec(a.par_soa, a.D, a.M, w), a, d, w);
}

template <int MODELS, int CTRL, int INTEG, bool AERO, bool MR, bool ONE>
__global__ __launch_bounds__(256) void k_step_tile(StepArgs a, const int4* __restrict__ tiles) {
    run_tile<MODELS, CTRL, INTEG, AERO, MR, ONE>(a, tiles[blockIdx.x]);
}

// Persistent work queue: each workgroup pops the next tile index from *counter
// until the tiles run out; every workgroup exits after one failed pop.
template <int MODELS, int CTRL, int INTEG, bool AERO, bool MR>
__device__ __forceinline__ void run_queue(const StepArgs& a, const int4* __restrict__ tiles, int n_tiles,
                                          unsigned* counter) {
    __shared__ int s_next;
    for (;;) {
        if (threadIdx.x == 0) s_next = (int)atomicAdd(counter, 1u);
        __syncthreads();
        const int t = __builtin_amdgcn_readfirstlane(s_next);
        __syncthreads();
        if (t >= n_tiles) break;
        run_tile<MODELS, CTRL, INTEG, AERO, MR, false>(a, tiles[t]);
    }
}

template <int MODELS, int CTRL, int INTEG, bool AERO, bool MR>
__global__ __launch_bounds__(256) void k_step_wq(StepArgs a, const int4* __restrict__ tiles, int n_tiles,
                                                 unsigned* counter) {
    run_queue<MODELS, CTRL, INTEG, AERO, MR>(a, tiles, n_tiles, counter);
}



template <int MODELS, int CTRL, int INTEG, bool AERO, bool MR, bool ONE>
static hipError_t launch_step_k(const KernelSel& ks, const StepArgs& a, const int4* tiles, int n_tiles,
                                unsigned* counter, int wq_blocks, hipStream_t s) {
    if (ks.mode == LM_LANE) {
        if constexpr (MODELS == MS_BOTH) return hipErrorInvalidValue;
        const int bs = ks.tile;
        const unsigned grid = (unsigned)((a.D + bs - 1) / bs);
        hipLaunchKernelGGL((k_step_lane<MODELS, CTRL, INTEG, AERO, MR, ONE>), dim3(grid), dim3(bs), 0, s, a);
    } else if (ks.mode == LM_TILE) {
        hipLaunchKernelGGL((k_step_tile<MODELS, CTRL, INTEG, AERO, MR, ONE>), dim3(n_tiles), dim3(ks.tile), 0, s, a, tiles);
    } else if constexpr (!ONE) {
        // work-queue workgroups that do not fit at once start later, find the
        // queue empty and exit
        hipLaunchKernelGGL((k_step_wq<MODELS, CTRL, INTEG, AERO, MR>), dim3(wq_blocks), dim3(ks.tile), 0, s, a, tiles,
                           n_tiles, counter);
    }
    return hipGetLastError();
}

// the slow-controller variant exists only where there is an onboard controller
template <int MODELS, int CTRL, int INTEG, bool AERO>
static hipError_t launch_step_t(const KernelSel& ks, const StepArgs& a, const int4* tiles, int n_tiles,
                                unsigned* counter, int wq_blocks, hipStream_t s) {
    if constexpr (MODELS != MS_ID && CTRL != CTRL_ROTOR) {
        if (a.ctrl_every > 1)
            return launch_step_k<MODELS, CTRL, INTEG, AERO, true, false>(ks, a, tiles, n_tiles, counter, wq_blocks, s);
    }
    // A single step is bound by its loads, so what counts is waves in flight: without the
    // loop, its sums' lost parts and what is held across steps the kernel takes 91 to 98
    // registers instead of 119 to 161 (32768 worlds of 14 drones, with a masked reset:
    // rotor interface 22.8 -> 20.6 us, torque 25.9 -> 21.8)
    if constexpr (INTEG == RK4 && !AERO) {
        if (a.K == 1 && ks.mode != LM_WQ)
            return launch_step_k<MODELS, CTRL, INTEG, AERO, false, true>(ks, a, tiles, n_tiles, counter, wq_blocks, s);
    }
    return launch_step_k<MODELS, CTRL, INTEG, AERO, false, false>(ks, a, tiles, n_tiles, counter, wq_blocks, s);
}

template <int MODELS, int CTRL, int INTEG, bool AERO>
static int wq_blocks_t(int tile) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_step_wq<MODELS, CTRL, INTEG, AERO, false>, tile, 0) !=
        hipSuccess)
        return 1;
    return nb > 0 ? nb : 1;
}

// the launches and occupancies of the variants compiled in part P (cf_dispatch.hpp)
template <int P>
hipError_t launch_step_part(const KernelSel& ks, const StepArgs& a, const int4* tiles, int n_tiles, unsigned* counter,
                            int wq_blocks, hipStream_t s);
template <int P>
int step_wq_part(const KernelSel& ks);

template <>
hipError_t launch_step_part<CF_PART>(const KernelSel& ks, const StepArgs& a, const int4* tiles, int n_tiles,
                                     unsigned* counter, int wq_blocks, hipStream_t s) {
    return dispatch<STEP_PARTS>(ks, [&](auto m, auto c, auto i, auto e) {
        return launch_step_t<m(), c(), i(), e() != 0>(ks, a, tiles, n_tiles, counter, wq_blocks, s);
    });
}

template <>
int step_wq_part<CF_PART>(const KernelSel& ks) {
    int n = 1;
    (void)dispatch<STEP_PARTS>(ks, [&](auto m, auto c, auto i, auto e) {
        n = wq_blocks_t<m(), c(), i(), e() != 0>(ks.tile);
        return hipSuccess;
    });
    return n;
}

#if CF_PART == 0
template <> hipError_t launch_step_part<1>(const KernelSel&, const StepArgs&, const int4*, int, unsigned*, int, hipStream_t);
template <> hipError_t launch_step_part<2>(const KernelSel&, const StepArgs&, const int4*, int, unsigned*, int, hipStream_t);
template <> int step_wq_part<1>(const KernelSel&);
template <> int step_wq_part<2>(const KernelSel&);

hipError_t launch_step(const KernelSel& ks, const StepArgs& a, const int4* tiles, int n_tiles, unsigned* counter,
                       int wq_blocks, hipStream_t s) {
    if (ks.mode == LM_QUAD) return launch_step_quad(ks, a, s);
    return in_part<STEP_PARTS>(ks, [&](auto p) { return launch_step_part<p()>(ks, a, tiles, n_tiles, counter, wq_blocks, s); });
}

int step_wq_blocks_per_cu(const KernelSel& ks) {
    return in_part<STEP_PARTS>(ks, [&](auto p) { return step_wq_part<p()>(ks); });
}
#endif

}  // namespace cfk
