// 2D constant-density time loop in launches of several steps (k_multi2d.hip).
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

#include "multi2d.h"
#include "plan.h"

namespace sw {

// Buffers of a run, single or double precision (meaning as in sw_fwd_io).
template <typename T>
struct Run2D {
    void *workspace;
    const T *wavelet;
    T *field[2];
    T *traces, *snaps, *ckpt;
    int saving_stride, ckpt_every, step0, nsteps_run;
};

// Tile and steps per launch of the plan (steps 0: the single-step kernels).
Multi2DChoice multi2d_choice(const sw_plan *p);

// Scratch bytes of a run of nsteps steps; levels: those between a launch's last
// two are wanted (snapshots, checkpoints; receivers want them by themselves).
// 0: the plan takes the single-step kernels.
int64_t multi2d_scratch_bytes(const sw_plan *p, int nsteps, bool levels);
// Whether a run of nsteps steps, with checkpoints or without, divides into
// launches of several.
bool multi2d_divides(const sw_plan *p, int nsteps, bool ckpt);

// Steps at the start of the run that the single-step kernels take (the rest
// divides into launches of several steps), or -1: all of them.
template <typename T>
int multi2d_singles(const sw_plan *p, const Run2D<T> &io, const void *scratch, int64_t bytes);

// The steps from step0 + singles on, after that many single steps from field[0].
template <typename T>
sw_status enqueue_multi2d(const sw_plan *p, const Run2D<T> &io, int singles, void *scratch, hipStream_t s);

extern template int multi2d_singles<float>(const sw_plan *, const Run2D<float> &, const void *, int64_t);
extern template int multi2d_singles<double>(const sw_plan *, const Run2D<double> &, const void *, int64_t);
extern template sw_status enqueue_multi2d<float>(const sw_plan *, const Run2D<float> &, int, void *, hipStream_t);
extern template sw_status enqueue_multi2d<double>(const sw_plan *, const Run2D<double> &, int, void *, hipStream_t);

}  // namespace sw
