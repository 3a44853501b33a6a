// Choice and dispatch of the vector tiles.
#include "vec.h"

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "runtime.h"

namespace sw {

#define SW_X(T, R)                                                                             \
    extern template hipError_t launch_vec_radius<T, R>(int, int, StencilParamsT<T> &, hipStream_t); \
    extern template int vec_resident_radius<T, R>(int, int);
#define SW_XR(R)                     \
    SW_X(float, R) SW_X(double, R)   \
    extern template hipError_t launch_vec_batch_radius<R>(const StencilParams *, const int *, int, int, int, hipStream_t);
SW_XR(1) SW_XR(2) SW_XR(3) SW_XR(4) SW_XR(5) SW_XR(6) SW_XR(7) SW_XR(8) SW_XR(9) SW_XR(10)
#undef SW_XR
#undef SW_X

template <typename T>
hipError_t launch_vec(int r, const VecChoice &c, int mode, StencilParamsT<T> &P, hipStream_t s)
{
    const VecTile t = kVecTiles<T>[c.tile];
    const int cols = t.lpr * int(16 / sizeof(T));
    P.ntx = (P.g.X + t.tx - 1) / t.tx;
    P.nty = (P.g.Y + cols - 1) / cols;
    P.zc = c.zc;
    P.nzc = (P.g.Z + c.zc - 1) / c.zc;
    P.xfast = 0;
    if (c.mirror) mode = kVecMirror;
    switch (r) {
    case 1: return launch_vec_radius<T, 1>(c.tile, mode, P, s);
    case 2: return launch_vec_radius<T, 2>(c.tile, mode, P, s);
    case 3: return launch_vec_radius<T, 3>(c.tile, mode, P, s);
    case 4: return launch_vec_radius<T, 4>(c.tile, mode, P, s);
    case 5: return launch_vec_radius<T, 5>(c.tile, mode, P, s);
    case 6: return launch_vec_radius<T, 6>(c.tile, mode, P, s);
    case 7: return launch_vec_radius<T, 7>(c.tile, mode, P, s);
    case 8: return launch_vec_radius<T, 8>(c.tile, mode, P, s);
    case 9: return launch_vec_radius<T, 9>(c.tile, mode, P, s);
    case 10: return launch_vec_radius<T, 10>(c.tile, mode, P, s);
    default: return hipErrorInvalidValue;
    }
}
template hipError_t launch_vec<float>(int, const VecChoice &, int, StencilParamsT<float> &, hipStream_t);
template hipError_t launch_vec<double>(int, const VecChoice &, int, StencilParamsT<double> &, hipStream_t);

namespace {

template <typename T>
int resident(int r, int tile, int mode)
{
    switch (r) {
    case 1: return vec_resident_radius<T, 1>(tile, mode);
    case 2: return vec_resident_radius<T, 2>(tile, mode);
    case 3: return vec_resident_radius<T, 3>(tile, mode);
    case 4: return vec_resident_radius<T, 4>(tile, mode);
    case 5: return vec_resident_radius<T, 5>(tile, mode);
    case 6: return vec_resident_radius<T, 6>(tile, mode);
    case 7: return vec_resident_radius<T, 7>(tile, mode);
    case 8: return vec_resident_radius<T, 8>(tile, mode);
    case 9: return vec_resident_radius<T, 9>(tile, mode);
    case 10: return vec_resident_radius<T, 10>(tile, mode);
    default: return 0;
    }
}

}  // namespace

hipError_t launch_vec_batch(int r, const StencilParams *shots, const int *tile_start, int nshots, int parity, int nblocks,
                            hipStream_t s)
{
    switch (r) {
    case 1: return launch_vec_batch_radius<1>(shots, tile_start, nshots, parity, nblocks, s);
    case 2: return launch_vec_batch_radius<2>(shots, tile_start, nshots, parity, nblocks, s);
    case 3: return launch_vec_batch_radius<3>(shots, tile_start, nshots, parity, nblocks, s);
    case 4: return launch_vec_batch_radius<4>(shots, tile_start, nshots, parity, nblocks, s);
    case 5: return launch_vec_batch_radius<5>(shots, tile_start, nshots, parity, nblocks, s);
    case 6: return launch_vec_batch_radius<6>(shots, tile_start, nshots, parity, nblocks, s);
    case 7: return launch_vec_batch_radius<7>(shots, tile_start, nshots, parity, nblocks, s);
    case 8: return launch_vec_batch_radius<8>(shots, tile_start, nshots, parity, nblocks, s);
    case 9: return launch_vec_batch_radius<9>(shots, tile_start, nshots, parity, nblocks, s);
    case 10: return launch_vec_batch_radius<10>(shots, tile_start, nshots, parity, nblocks, s);
    default: return hipErrorInvalidValue;
    }
}

namespace {

// Cost model of a launch, in microseconds, fitted to forward launches of every
// tile and chunk count on eleven grids of 2.4 M .. 207 M nodes at SO2 .. SO20
// (its choices ran within 1.6% of the sweep's best on average, 12% at worst):
//   planes = zc + a 2R + c            what a block marches over, warm-up included
//   plane  = nodes of the tile k (1 + hx 2R / TX + hy 64 / TY), its halo included
//   launch = max(load planes plane, latency planes rounds)
// load is the blocks of the busiest CU where all blocks are resident at once
// (w: how far it counts beyond the mean), else the mean plus a tail, times pm.
// Chunks that make one round of just under a whole number of blocks per CU win
// wherever they exist: the blocks then march through z together, a few long
// streams that HBM serves at 5.4 TB/s (592^3 SO8: 250 blocks of 24 x 128
// columns and 296 planes, 0.611 ms; 2960 blocks of 74 planes 0.683 ms).
// Mirror sides along x or y end that: the blocks at those sides make ghosts on
// every plane and fall behind, so one round costs edge times its load (592^3
// SO8, every side mirrored: one round 0.730 ms, 8 chunks of 74 planes 0.677),
// and a tile that has the CU to itself waits at their second barrier with
// nothing else to run.  So tiles are taken there of which two fit and whose
// waves spread evenly over the SIMDs (207 x 801 x 801, SO8: 24 x 64 columns
// 0.566 ms, 16 x 64 0.429; in doubles 24 x 64 0.957, 16 x 64 0.861).
struct CostModel {
    double k, k1, a, c, hx, hy, w, tail, pm, latency, idle, edge;
};
constexpr CostModel kCost32{4.07e-4, 6.3e-7, 0.061, 1.3, 0.17, 0.25, 1.8, 0.075, 1.21, 1.35, 1.55, 1.5};
constexpr CostModel kCost64{5.08e-4, 0.0, 0.084, 1.8, 0.24, 0.11, 1.0, 0.26, 1.03, 1.54, 0.21, 1.15};

template <typename T>
VecChoice choose(const sw_plan *p, int mode)
{
    constexpr int kCUs = 256;
    constexpr int kFourWaves = sizeof(T) == 4 ? 2 : 1;      // the tile of 4 waves, one per SIMD
    constexpr CostModel m = sizeof(T) == 4 ? kCost32 : kCost64;
    VecChoice best;
    const int slots = resident<T>(p->r, kFourWaves, mode);  // waves per SIMD
    if (slots <= 0) return best;
    const int Z = p->dims[0], X = p->dims[1], Y = p->dims[2], R = p->r;
    const int64_t pbytes = int64_t(p->pad[1]) * p->pad[2] * int64_t(sizeof(T));
    const bool edges = p->prob.bc[1][0] || p->prob.bc[1][1] || p->prob.bc[2][0] || p->prob.bc[2][1];
    const int zmax = int(std::max<int64_t>(1, (int64_t(1) << 31) / pbytes - 4 * R - 2));
    double cost = 0.0;
    for (int i = 0; i < kVecTileCount; ++i) {
        const VecTile t = kVecTiles<T>[i];
        const int cols = t.lpr * int(16 / sizeof(T)), waves = t.tx * t.lpr / 64;
        // resident blocks, with a block's waves spread over the four SIMDs (6
        // waves take two slots of each of two SIMDs)
        const int res = std::min(resident<T>(R, i, mode), waves >= 4 ? slots / ((waves + 3) / 4) : slots * 4 / waves);
        if (res <= 0 || (edges && slots >= 4 && (res < 2 || (waves > 2 && waves % 4)))) continue;
        const double tiles = double((X + t.tx - 1) / t.tx) * ((Y + cols - 1) / cols);
        const double used = double(X) * Y / (tiles * t.tx * cols);
        const double nodes = t.tx * cols * (sizeof(T) / 4.0) * (used + (1.0 - used) * m.idle);
        const double plane = nodes * (m.k + m.k1 * R * R) * (1.0 + m.hx * 2 * R / t.tx + m.hy * 64.0 / cols);
        for (int n = 1; n <= Z; ++n) {
            const int zc = (Z + n - 1) / n;
            if (zc > zmax) continue;
            if (zc < 4 && n > 1) break;
            const double per_cu = tiles * ((Z + zc - 1) / zc) / kCUs;
            const bool once = per_cu <= res;
            const double load = once ? (m.w * std::ceil(per_cu) + (1.0 - m.w) * per_cu) * (edges ? m.edge : 1.0)
                                     : (per_cu + m.tail * res) * m.pm;
            const double planes = zc + m.a * 2 * R + m.c;
            const double wait = m.latency * (1.0 + 0.02 * R) * planes * (once ? 1.0 : std::ceil(per_cu / res));
            const double us = std::max(load * planes * plane, wait);
            if (best.tile < 0 || us < cost) {
                cost = us;
                best.tile = i;
                best.zc = zc;
            }
        }
    }
    return best;
}

}  // namespace

VecChoice choose_vec(const sw_plan *p, int mode)
{
    if (p->ndim != 3 || p->prob.scheme != SW_CONST || !default_tiling(p) || (p->mirror && mode != MODE_FWD)) return {};
    if (p->mirror) mode = kVecMirror;
    VecChoice c = p->prob.dtype == SW_F64 ? choose<double>(p, mode) : choose<float>(p, mode);
    c.mirror = p->mirror;
    return c;
}

}  // namespace sw
