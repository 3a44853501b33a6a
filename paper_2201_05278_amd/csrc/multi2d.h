// Several time steps of a 2D constant-density grid per launch: parameters and
// launchers shared by k_multi2d.hip and the time loops (forward2d.cpp).
#pragma once

#include "device.h"

namespace sw {

constexpr int kMulti2DMax = 8;      // steps per launch at most

// One launch: steps n .. n + nt - 1 from (cur = p^n, prv = p^{n-1}); level
// p^{n+s+1} goes to out[s] (NULL: not written).  Neither input is written.
template <typename T>
struct Multi2DParams {
    const T *cur, *prv;
    T *out[kMulti2DMax];
    const T *K;
    const typename Pair<T>::type *damp;     // (A, B) by squared layer distance
    Geom g;
    T c0, cz[11], cy[11];                   // as in StencilParamsT
    int bcz[2], bcy[2];                     // ghost conditions of the z and y sides
    int nt;                                 // steps of this launch
    int tz, ty, ntz, nty;                   // tile outputs and tile counts
    // injected values of the launch's steps, [nt][nuniq], added at the nodes
    // unode; box: inclusive (z, y) bounds of those nodes
    const int64_t *unode;
    const T *inj;
    int nuniq;
    int box[4];
    // recording of the previous launch's levels, by the blocks past the tiles:
    // rout[s][count] from rlev[s], s < rnt
    const T *rlev[kMulti2DMax];
    T *rout;
    int rnt;
    const int32_t *ptr;
    const int64_t *node;
    const T *wscaled;
    int count, group;
};

// Tile of a launch: rows and columns held on chip (the outputs plus nt R nodes
// around them).
struct Multi2DTile {
    int ez, ey;
};

// Steps per launch and tile for a grid of Z x Y nodes; steps 0: the radius or
// grid is left to the single-step kernels.
struct Multi2DChoice {
    int steps, tile;        // tile: index of the instantiated tiles
};
Multi2DChoice choose_multi2d(int r, int value_bytes, int Z, int Y, int cus);
Multi2DTile multi2d_tile(int tile, int value_bytes);
// Whether a tile is instantiated at a radius and holds any output after `steps` steps.
bool multi2d_tile_ok(int r, int value_bytes, int tile, int steps);
// Columns around a tile's outputs: nt R rounded up to whole 16-byte vectors.
constexpr int multi2d_pad_y(int halo, int value_bytes)
{
    return (halo + 16 / value_bytes - 1) / (16 / value_bytes) * (16 / value_bytes);
}

template <typename T>
hipError_t launch_multi2d(int r, int tile, Multi2DParams<T> &P, hipStream_t s);
extern template hipError_t launch_multi2d<float>(int, int, Multi2DParams<float> &, hipStream_t);
extern template hipError_t launch_multi2d<double>(int, int, Multi2DParams<double> &, hipStream_t);

// out[s][u] = the value the injection of step s adds at unique node u, for the
// amplitudes amp[s][nsrc], s < nsteps.
template <typename T>
struct InjectTable {
    const int32_t *uptr, *uent, *pid;
    const T *coef_a;
    int nuniq, nsrc, max_per_node;
};
template <typename T>
hipError_t launch_inject_all(const InjectTable<T> &t, const T *amp, int nsteps, T *out, hipStream_t s);
extern template hipError_t launch_inject_all<float>(const InjectTable<float> &, const float *, int, float *, hipStream_t);
extern template hipError_t launch_inject_all<double>(const InjectTable<double> &, const double *, int, double *,
                                                     hipStream_t);

}  // namespace sw
