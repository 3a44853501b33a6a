// Vector tiles of the 3D stencils (stencil_vec.h, stencil_vdvec.h): tiles,
// launchers and the choice of tile and z chunk.
#pragma once

#include "device.h"

struct sw_plan;

namespace sw {

// TX rows x lpr 16-byte vectors of columns, one thread per vector.
struct VecTile {
    int tx, lpr;
};
template <typename T> inline constexpr VecTile kVecTiles[8] = {{8, 16}, {12, 16}, {16, 16}, {24, 16},
                                                        {8, 32}, {12, 32}, {16, 32}, {24, 32}};
// doubles: the same columns with twice the threads per row
template <> inline constexpr VecTile kVecTiles<double>[8] = {{4, 32}, {8, 32}, {12, 32}, {16, 32},
                                                      {24, 32}, {4, 64}, {8, 64}, {12, 64}};
constexpr int kVecTileCount = 8;

constexpr int kVecMirror = 8;   // MODE_FWD of a plan with mirror sides: kernels of their own

struct VecChoice {
    int tile = -1, zc = 0;      // tile -1: the scalar tiles
    bool mirror = false;        // the plan has mirror sides
};

// Tile and chunk of a 3D plan in a mode that the library picks for.
VecChoice choose_vec(const sw_plan *p, int mode);

// Whether the plan's launches in a mode have vector tile `tile`, and the longest z chunk of its 32-bit windows.
bool vec_instance(const sw_plan *p, int mode, int tile);
int vec_zmax(const sw_plan *p);
// Rows and columns of a vector tile of the plan.
void vec_extents(const sw_plan *p, int tile, int &rows, int &cols);

// Threads and mode of a kernel for which a block's registers suffice (768
// threads: 168 each; 1024: 128).
constexpr bool vec_fits(int threads, int r, int mode)
{
    const int need = 76 + 9 * r + (mode == MODE_IMAGE ? 16 : mode == MODE_IMAGE2 ? 26 : 0);
    return threads <= 512 || (threads <= 768 && need <= 160);
}

// Launch with a choice: sets the tile counts of P.
template <typename T>
hipError_t launch_vec(int r, const VecChoice &c, int mode, StencilParamsT<T> &P, hipStream_t s);

template <typename T, int R>
hipError_t launch_vec_radius(int tile, int mode, StencilParamsT<T> &P, hipStream_t s);
template <typename T, int R>
int vec_resident_radius(int tile, int mode);

// The batch launch on 16-row, 64-column vector tiles (arguments as launch_const_batch).
hipError_t launch_vec_batch(int r, const StencilParams *shots, const int *tile_start, int nshots, int parity, int nblocks,
                            hipStream_t s);
template <int R>
hipError_t launch_vec_batch_radius(const StencilParams *shots, const int *tile_start, int nshots, int parity, int nblocks,
                                   hipStream_t s);

// Variable density (stencil_vdvec.h): rows x columns, as many threads as the
// columns per thread of the scheme and radius leave.
struct VdTile {
    int tx, ty;
};
inline constexpr VdTile kVdTiles[5] = {{8, 64}, {16, 64}, {16, 128}, {32, 32}, {32, 64}};
constexpr int kVdTileCount = 5;
inline constexpr int kStagRadii[2] = {2, 8};    // staggered: smallest and largest radius
constexpr int kVdThreads = 512;     // at most, in a block: two waves per SIMD leave a thread 256 registers
// Columns per thread (scheme as in launch_vd).
constexpr int vd_columns(int scheme, int r)
{
    return r <= (scheme == 1 ? 4 : 6) ? 4 : 2;
}

hipError_t launch_vdvec(int scheme, int r, const VecChoice &c, int mode, StencilParams &P, hipStream_t s);
template <int R>
hipError_t launch_vdvec_radius(int scheme, int tile, int mode, StencilParams &P, hipStream_t s);
// Resident blocks per CU of the centred kernel (scheme 2).
template <int R>
int vdvec_resident_radius(int scheme, int tile);

}  // namespace sw
