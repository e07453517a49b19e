// launch.hpp -- host-side launch of the step kernels.
//
// The kernel variants (lattice x storage x sensor kind x collision model x
// tile width x streaming scheme) are instantiated in one translation unit per storage
// family (step_f64.hip, step_f32.hip, step_f16.hip, step_bf16.hip) so that
// they compile in parallel; lbm.hip only sees the declaration.
#pragma once

#include <hip/hip_runtime.h>

#include "pair_kernel.hpp"
#include "step_kernel.hpp"

namespace lbm {

struct LaunchCfg {
    hipStream_t stream;
    int tile_x;        // 32, 64 or 128 cells x 8 rows; kRowTileX: one row, 3D ping-pong
                       // only (3D float64: 64)
    int scheme;        // kPingPong, kStream or kLocal
    bool sensor;       // evaluate sensor, block maxima and flags in this step
    int sensor_kind;   // kSensorL2 or kSensorKKn
    bool force;        // body force present
    bool smag;         // Smagorinsky subgrid model on
};

// Enqueues one step of lattice Q, storage policy T and arithmetic C.
template <int Q, typename T, typename C, bool SH>
void launch_step_kernel(const StepArgs<C> &a, const LaunchCfg &c);

// Enqueues nsteps (1 .. kMultiMaxSteps) sensor-free ping-pong steps of a 2D
// grid as one step_multi launch (a.src -> a.dst); a no-op for 3D lattices
// and stochastic rounding, which the host never sends here.
template <int Q, typename T, typename C, bool SH>
void launch_multi_kernel(const StepArgs<C> &a, int nsteps, const LaunchCfg &c);

// Enqueues two steps of a 3D grid as one step_pair launch (a.src -> a.dst;
// scheme kStream: both buffers in the slot order of the in-place scheme); a
// no-op where pair_supported is false, which the host never sends here.
// c.sensor: either step evaluates the sensor (p.sensor says which).
template <int Q, typename T, typename C, bool SH>
void launch_pair_kernel(const StepArgs<C> &a, const PairArgs &p, const LaunchCfg &c);

#ifdef LBM_LAUNCH_DEFINITIONS
template <int Q, typename T, typename C, bool SH, bool SENS, int SK, int MODEL, int BX, int SCH>
void launch_one(hipStream_t st, const StepArgs<C> &a) {
    constexpr int TY = (BX == kRowTileX) ? 1 : kTileY;
    const dim3 g(a.ntiles), b(BX, TY);
    hipLaunchKernelGGL((step_cells<Q, T, C, SH, SENS, SK, MODEL, BX, SCH, TY>), g, b, 0, st, a);
}

template <int Q, typename T, typename C, bool SH, bool SENS, int SK, int BX, int SCH>
void launch_model(const StepArgs<C> &a, const LaunchCfg &c) {
    switch ((c.force ? kModelForce : 0) | (c.smag ? kModelSmag : 0)) {
        case kModelForce: launch_one<Q, T, C, SH, SENS, SK, kModelForce, BX, SCH>(c.stream, a); break;
        case kModelSmag: launch_one<Q, T, C, SH, SENS, SK, kModelSmag, BX, SCH>(c.stream, a); break;
        case kModelForce | kModelSmag:
            launch_one<Q, T, C, SH, SENS, SK, kModelForce | kModelSmag, BX, SCH>(c.stream, a);
            break;
        default: launch_one<Q, T, C, SH, SENS, SK, 0, BX, SCH>(c.stream, a); break;
    }
}

template <int Q, typename T, typename C, bool SH, int BX, int SCH>
void launch_sk(const StepArgs<C> &a, const LaunchCfg &c) {
    if (!c.sensor) launch_model<Q, T, C, SH, false, kSensorL2, BX, SCH>(a, c);
    else if (c.sensor_kind == kSensorL2) launch_model<Q, T, C, SH, true, kSensorL2, BX, SCH>(a, c);
    else launch_model<Q, T, C, SH, true, kSensorKKn, BX, SCH>(a, c);
}

template <int Q, typename T, typename C, bool SH, int BX>
void launch_scheme(const StepArgs<C> &a, const LaunchCfg &c) {
    switch (c.scheme) {
        case kStream: launch_sk<Q, T, C, SH, BX, kStream>(a, c); break;
        case kLocal: launch_sk<Q, T, C, SH, BX, kLocal>(a, c); break;
        default: launch_sk<Q, T, C, SH, BX, kPingPong>(a, c); break;
    }
}

template <int Q, typename T, typename C, bool SH>
void launch_multi_kernel(const StepArgs<C> &a, int nsteps, const LaunchCfg &c) {
    if constexpr (Lattice<Q>::D == 2 && !Storage<T>::sr) {
        const int ntx = (a.nx + kMultiTile - 1) / kMultiTile, nty = (a.ny + kMultiTile - 1) / kMultiTile;
        const dim3 g(ntx * nty), b(kMultiEdge * kMultiEdge);
        switch ((c.force ? kModelForce : 0) | (c.smag ? kModelSmag : 0)) {
            case kModelForce:
                hipLaunchKernelGGL((step_multi<Q, T, C, SH, kModelForce>), g, b, 0, c.stream, a, nsteps);
                break;
            case kModelSmag:
                hipLaunchKernelGGL((step_multi<Q, T, C, SH, kModelSmag>), g, b, 0, c.stream, a, nsteps);
                break;
            case kModelForce | kModelSmag:
                hipLaunchKernelGGL((step_multi<Q, T, C, SH, kModelForce | kModelSmag>), g, b, 0, c.stream, a,
                                   nsteps);
                break;
            default: hipLaunchKernelGGL((step_multi<Q, T, C, SH, 0>), g, b, 0, c.stream, a, nsteps); break;
        }
    } else {
        (void)a, (void)nsteps, (void)c;
    }
}

template <int Q, typename T, typename C, bool SH, bool SENS, int SK, int MODEL>
void launch_pair_one(const StepArgs<C> &a, const PairArgs &p, const LaunchCfg &c) {
    if constexpr (pair_supported<Q, T, MODEL>()) {
        const dim3 g(p.ntiles), b(pair_threads<Q, T>());
        if constexpr (sizeof(T) == 4) {   // 3D float64 is never in place
            if (c.scheme == kStream) {
                hipLaunchKernelGGL((step_pair<Q, T, C, SH, SENS, SK, MODEL, true>), g, b, 0, c.stream, a, p);
                return;
            }
        }
        hipLaunchKernelGGL((step_pair<Q, T, C, SH, SENS, SK, MODEL, false>), g, b, 0, c.stream, a, p);
    } else {
        (void)a, (void)p, (void)c;
    }
}

template <int Q, typename T, typename C, bool SH, bool SENS, int SK>
void launch_pair_model(const StepArgs<C> &a, const PairArgs &p, const LaunchCfg &c) {
    if (c.force) launch_pair_one<Q, T, C, SH, SENS, SK, kModelForce>(a, p, c);
    else if (c.smag) launch_pair_one<Q, T, C, SH, SENS, SK, kModelSmag>(a, p, c);
    else launch_pair_one<Q, T, C, SH, SENS, SK, 0>(a, p, c);
}

template <int Q, typename T, typename C, bool SH>
void launch_pair_kernel(const StepArgs<C> &a, const PairArgs &p, const LaunchCfg &c) {
    if (!c.sensor) launch_pair_model<Q, T, C, SH, false, kSensorL2>(a, p, c);
    else if (c.sensor_kind == kSensorL2) launch_pair_model<Q, T, C, SH, true, kSensorL2>(a, p, c);
    else launch_pair_model<Q, T, C, SH, true, kSensorKKn>(a, p, c);
}

template <int Q, typename T, typename C, bool SH>
void launch_step_kernel(const StepArgs<C> &a, const LaunchCfg &c) {
    if constexpr (Lattice<Q>::D == 3 && sizeof(C) == 8) {   // one tile shape, ping-pong
        launch_sk<Q, T, C, SH, 64, kPingPong>(a, c);
    } else if (Lattice<Q>::D == 3 && c.tile_x == kRowTileX && c.scheme == kPingPong) {
        if constexpr (Lattice<Q>::D == 3) launch_sk<Q, T, C, SH, kRowTileX, kPingPong>(a, c);
    } else {
        switch (c.tile_x) {
            case 32: launch_scheme<Q, T, C, SH, 32>(a, c); break;
            case 64: launch_scheme<Q, T, C, SH, 64>(a, c); break;
            default: launch_scheme<Q, T, C, SH, 128>(a, c); break;
        }
    }
}
#endif

}  // namespace lbm
