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
    extern template hipError_t launch_vec_batch_radius<R>(const StencilParams *, const int *, int, int, int, hipStream_t); \
    extern template hipError_t launch_vdvec_radius<R>(int, int, int, StencilParams &, hipStream_t); \
    extern template int vdvec_resident_radius<R>(int, int);
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

hipError_t launch_vdvec(int scheme, int r, const VecChoice &c, int mode, StencilParams &P, hipStream_t s)
{
    const VdTile t = kVdTiles[c.tile];
    P.ntx = (P.g.X + t.tx - 1) / t.tx;
    P.nty = (P.g.Y + t.ty - 1) / t.ty;
    P.zc = c.zc;
    P.nzc = (P.g.Z + c.zc - 1) / c.zc;
    P.xfast = 0;
    switch (r) {
    case 1: return launch_vdvec_radius<1>(scheme, c.tile, mode, P, s);
    case 2: return launch_vdvec_radius<2>(scheme, c.tile, mode, P, s);
    case 3: return launch_vdvec_radius<3>(scheme, c.tile, mode, P, s);
    case 4: return launch_vdvec_radius<4>(scheme, c.tile, mode, P, s);
    case 5: return launch_vdvec_radius<5>(scheme, c.tile, mode, P, s);
    case 6: return launch_vdvec_radius<6>(scheme, c.tile, mode, P, s);
    case 7: return launch_vdvec_radius<7>(scheme, c.tile, mode, P, s);
    case 8: return launch_vdvec_radius<8>(scheme, c.tile, mode, P, s);
    case 9: return launch_vdvec_radius<9>(scheme, c.tile, mode, P, s);
    case 10: return launch_vdvec_radius<10>(scheme, c.tile, mode, P, s);
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
// and the other waves of a SIMD must fill the wait at their second barrier.  So
// their own constants (fitted to 350 grids of 0.3 M .. 250 M nodes in single
// precision up to SO18 and 300 in double at SO2 and SO4, every tile and 14 chunk
// counts each) charge a plane by the waves it leaves per SIMD (qw), more where
// those differ between SIMDs (uneven), and favour at equal waits a tile that has
// the CU to itself (ql).  Choices ran 3.0% behind the sweep's best on average,
// 17% at worst (with the constants above 17% and 130%).  Of 1300 other grids six
// ran more than 1.5% behind the scalar tiles, 8% at worst (67 of 366 with the
// constants above, 25%: 768 x 532 x 507 SO18, 1373 us against 1041, now 958).
// In doubles 3.6% on average, 16% at worst (9.5% and 54%), no grid behind the
// scalar tiles.
// In doubles from SO6 on the general constants hold, with tiles of which two
// fit and whose waves spread evenly over the SIMDs (207 x 801 x 801 SO8: 24 x 64
// 0.957 ms, 16 x 64 0.861).  Imaging launches, with up to seven streams, want the
// even spread too.
struct CostModel {
    double k, k1, a, c, hx, hy, w, tail, pm, latency, lr, idle, edge, qw, uneven, ql;
};
constexpr CostModel kCost32{4.07e-4, 6.3e-7, 0.061, 1.3, 0.17, 0.25, 1.8, 0.075, 1.21, 1.35, 0.02, 1.55, 1.5, 0.0, 1.0, 1.0};
constexpr CostModel kCost64{5.08e-4, 0.0, 0.084, 1.8, 0.24, 0.11, 1.0, 0.26, 1.03, 1.54, 0.02, 0.21, 1.15, 0.0, 1.0, 1.0};
constexpr CostModel kMirror32{4.07e-4, 3.1e-7, 0.0088, 1.19, 0.366, 0.128, 1.68, 0.145, 1.205, 2.06, 0.052, 0.656, 1.254, 0.163, 1.276, 0.978};
constexpr CostModel kMirror64{3.51e-4, 0.0, 0.0604, 0.112, 0.151, 0.207, 1.016, 0.281, 1.09, 1.445, 0.0646, 0.55, 1.099, 1.016, 1.461, 0.98};

template <typename T>
VecChoice choose(const sw_plan *p, int mode)
{
    const int cus = compute_units(p);
    constexpr int kFourWaves = sizeof(T) == 4 ? 2 : 1;      // the tile of 4 waves, one per SIMD
    VecChoice best;
    const int slots = resident<T>(p->r, kFourWaves, mode);  // waves per SIMD
    if (slots <= 0) return best;
    const int Z = p->dims[0], X = p->dims[1], Y = p->dims[2], R = p->r;
    const bool edges = p->prob.bc[1][0] || p->prob.bc[1][1] || p->prob.bc[2][0] || p->prob.bc[2][1];
    const bool image = mode == MODE_IMAGE || mode == MODE_IMAGE2;
    const bool own = edges && (sizeof(T) == 4 || R <= 2);           // constants of mirrored sides
    const CostModel m = sizeof(T) == 4 ? (own ? kMirror32 : kCost32) : own ? kMirror64 : kCost64;
    const int zmax = vec_zmax(p);
    double cost = 0.0;
    for (int i = 0; i < kVecTileCount; ++i) {
        const VecTile t = kVecTiles<T>[i];
        const int cols = t.lpr * int(16 / sizeof(T)), waves = t.tx * t.lpr / 64;
        // resident blocks, with a block's waves spread over the four SIMDs (6
        // waves take two slots of each of two SIMDs)
        // (a block of more waves than that is compiled for its own registers)
        const int fit = resident<T>(R, i, mode);
        if (fit <= 0 || (sizeof(T) == 4 && edges && R == 10 && i != kFourWaves)) continue;     // (the others spill)
        const int res = std::max(1, std::min(fit, waves >= 4 ? slots / ((waves + 3) / 4) : slots * 4 / waves));
        const bool uneven = waves > 2 && waves % 4;
        if (!own && slots >= 4 && (((edges || image) && uneven) || (edges && res < 2))) continue;
        const double tiles = double((X + t.tx - 1) / t.tx) * ((Y + cols - 1) / cols);
        const double used = double(X) * Y / (tiles * t.tx * cols);
        const double nodes = t.tx * cols * (sizeof(T) / 4.0) * (used + (1.0 - used) * m.idle);
        const double plane = nodes * (m.k + m.k1 * R * R) * (1.0 + m.hx * 2 * R / t.tx + m.hy * 64.0 / cols) *
                             std::pow(4.0 / std::min(4.0, res * waves / 4.0), m.qw) * (uneven ? m.uneven : 1.0);
        for (int n = 1, last = 0; n <= Z; ++n) {
            const int zc = (Z + n - 1) / n;
            if (zc > zmax || zc == last) continue;
            if (zc < 4 && n > 1) break;
            last = zc;
            const double per_cu = tiles * ((Z + zc - 1) / zc) / cus;
            const bool once = per_cu <= res;
            const double load = once ? (m.w * std::ceil(per_cu) + (1.0 - m.w) * per_cu) * (edges ? m.edge : 1.0)
                                     : (per_cu + m.tail * res) * m.pm;
            const double planes = zc + m.a * 2 * R + m.c;
            const double wait = m.latency * (1.0 + m.lr * R) * planes * (once ? 1.0 : std::ceil(per_cu / res)) *
                                (res < 2 ? m.ql : 1.0);
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

// The same for variable density, whose kernels leave two waves per SIMD: blocks
// that fill a round march together and each further round costs as much again,
// a last partial one a little less where its blocks have a SIMD to themselves
// (fitted to sweeps on six grids of 2.7 M .. 207 M nodes at SO4, SO8 and SO16:
// its choices ran within 1% of the sweep's best on average, staggered, and 3%,
// centred).  Sweeps of 609 staggered and 795 centred grids of 0.5 M .. 250 M nodes
// showed other orders to be further off (staggered SO16 9% on average, 64% at
// worst; centred SO14 19%, 43%), so these have constants of their own: staggered
// forward launches but SO8 (1% on average, 12% at worst), centred ones at SO2,
// SO4, SO6 and SO14, whose kernels leave three waves per SIMD or four (waves: how
// much a plane gains by them) and, but for SO2, want 8 x 64 columns (5%, 28%).
struct VdCost {
    double hx, hy, warm, plane, tail, alone, last, waves;
};
constexpr VdCost kStagCost{0.147, 1.2, 0.176, 1.78, 0.26, 1.0, 1.0, 0.0};
constexpr VdCost kStagForward{0.142, 0.035, 0.32, 0.68, 0.146, 0.71, 0.54, 0.0};
constexpr VdCost kCentCost{0.3, 1.235, 0.239, 0.0, 0.0, 0.25, 0.6, 0.0};
constexpr VdCost kCentNarrow{0.0, 0.56, 0.0365, 0.05, 0.0, 0.25, 0.08, 0.27};

int vd_resident(const sw_plan *p, int tile)
{
    switch (p->r) {
    case 1: return vdvec_resident_radius<1>(p->prob.scheme, tile);
    case 2: return vdvec_resident_radius<2>(p->prob.scheme, tile);
    case 3: return vdvec_resident_radius<3>(p->prob.scheme, tile);
    case 7: return vdvec_resident_radius<7>(p->prob.scheme, tile);
    default: return 0;
    }
}

// cost: that of the choice, for the comparison with the scalar tiles.
VecChoice choose_vd(const sw_plan *p, int mode, double &cost)
{
    const int cus = compute_units(p);
    VecChoice best;
    const bool stag = p->prob.scheme == SW_VD_STAGGERED;
    const bool narrow = !stag && (p->r <= 3 || p->r == 7);
    const VdCost m = stag ? (mode == MODE_FWD && p->r != 4 ? kStagForward : kStagCost) : narrow ? kCentNarrow : kCentCost;
    const int Z = p->dims[0], X = p->dims[1], Y = p->dims[2], R = p->r;
    const int warm = stag ? 2 * R - 1 : 2 * R;
    const int zmax = vec_zmax(p);
    cost = 0.0;
    for (int i = 0; i < kVdTileCount; ++i) {
        const VdTile t = kVdTiles[i];
        const int threads = t.tx * t.ty / vd_columns(p->prob.scheme, R);
        if (threads > kVdThreads || (narrow ? R > 1 && i > 0 : !stag && t.tx > 16 && t.ty > 32)) continue;
        const int res = narrow ? vd_resident(p, i) : 512 / threads;     // two waves per SIMD
        if (res <= 0) continue;
        const double waves = res * threads / 256.0;
        const double tiles = double((X + t.tx - 1) / t.tx) * ((Y + t.ty - 1) / t.ty);
        const double plane = t.tx * t.ty * (1.0 + m.hx * 2 * R / t.tx + m.hy * 2 * R / t.ty) *
                             (1.0 + m.waves * (waves - 2.0)) * 2.0 / waves;
        for (int n = 1, last = 0; n <= Z; ++n) {
            const int zc = (Z + n - 1) / n;
            if (zc > zmax || zc == last) continue;
            if (zc < 4 && n > 1) break;
            last = zc;
            const double per_cu = tiles * ((Z + zc - 1) / zc) / cus;
            const double full = std::floor(per_cu / res), rest = per_cu - full * res;
            const double half = full > 0.0 ? m.last : m.alone;      // of a round with every other slot empty
            const double part = rest > 1e-9 ? std::min(1.0, half + (1.0 - half) * std::ceil(rest) / res) : 0.0;
            const double rounds = per_cu <= res ? std::max(full, part) : full + (1.0 - m.tail) * part + m.tail * rest / res;
            const double us = rounds * res * (zc + m.warm * warm + m.plane) * plane;
            if (best.tile < 0 || us < cost) {
                cost = us;
                best.tile = i;
                best.zc = zc;
            }
        }
    }
    return best;
}

// Cost of a scalar variable-density launch in the units of choose_vd: whole
// rounds of resident blocks, a last one half by its share (less than one round:
// as the root of its share, since a lone block has more of the machine).
double vd_scalar_cost(const sw_plan *p)
{
    const int cus = compute_units(p);
    const Tiling t = choose_tiling(p);
    const int res = resident_blocks(p, t);
    if (res <= 0) return 0.0;
    const double tiles = double((p->dims[1] + t.tx - 1) / t.tx) * ((p->dims[2] + 63) / 64);
    const double per = tiles * ((p->dims[0] + t.zc - 1) / t.zc) / (double(cus) * res);
    const double rest = per - std::floor(per);
    const double rounds = per <= 1.0 ? std::max(std::sqrt(per), 0.3) : std::floor(per) + (rest < 1e-9 ? 0.0 : 0.5 + 0.5 * rest);
    return rounds * res * t.zc * t.tx * 64.0;
}

// Where the variable-density vector tiles are the faster ones.  Recording and
// imaging launches gain at every size (staggered gradients of 160^3 .. 400^3, SO4
// .. SO16: 2% .. 56%).  Staggered R = 1 has little to share between neighbours
// (280^3 97 against 120 us), and from R = 9 on three queues leave no registers
// (280^3 SO20 561 against 1182 us).
// Forward launches of both kinds gain or lose with how their blocks fill the
// last round, by more than the kernels differ at some orders (staggered SO12,
// 340^3 503 against 425 us but 440^3 887 against 957).  So the two costs decide:
// vector tiles run where the scalar cost is above the mean (geometric) of the
// vector cost and the ideal by the order's factor, centred SO2 up to 40 M nodes
// only (above, five of seven grids where the costs chose vector tiles lost 2 to 5%
// by them).  Of 489 other grids this left 2 more than 1.5% slower than the scalar
// tiles, 2% at worst (a rule by size alone 59 of 1229, 9%).  At the other orders
// vector tiles run throughout: staggered SO8 (11 of 214 slower, 7% at worst; 592^3
// 1287 against 1349 us) and SO16 (1 of 55, 3%; 1.5 times as fast on average),
// centred SO6 .. SO14, SO18 and SO20 (3 of 418, 4%; 1.2 times as fast and more on
// average).
bool vd_vectors(const sw_plan *p, int mode, double cost)
{
    const bool stag = p->prob.scheme == SW_VD_STAGGERED;
    if (stag && (p->r < kStagRadii[0] || p->r > kStagRadii[1])) return false;
    if (mode != MODE_FWD) return true;
    constexpr double kStag[9] = {0, 0, 1.07, 0.99, 0, 1.02, 1.0, 0.967, 0};
    constexpr double kCent[11] = {0, 1.21, 1.12, 0, 0, 0, 0, 0, 0.896, 0, 0};
    const double factor = stag ? kStag[p->r] : kCent[p->r];
    const double scalar = factor > 0.0 ? vd_scalar_cost(p) : 0.0;
    if (scalar <= 0.0) return true;
    const double nodes = double(p->dims[0]) * p->dims[1] * p->dims[2], ideal = nodes / compute_units(p);
    if (!stag && p->r == 1 && nodes > 40e6) return false;
    return scalar > factor * std::sqrt(cost * ideal);
}

// Constant density: vector tiles, but where the scalar ones are as fast or
// faster.  SO2 above 130 M nodes (nine grids: 0.95 .. 1.05 of the scalar tiles'
// time); SO20 with sides mirrored along x or y above 10 M nodes, whose kernel has
// registers for two waves per SIMD only (466 x 495 x 397: 557 us against 666 on vector tiles).
bool const_vectors(const sw_plan *p, int mode)
{
    const double nodes = double(p->dims[0]) * p->dims[1] * p->dims[2];
    const bool edges = p->prob.bc[1][0] || p->prob.bc[1][1] || p->prob.bc[2][0] || p->prob.bc[2][1];
    if (p->prob.dtype == SW_F64) return true;
    if (edges) return p->r < 10 || nodes < 10e6;
    return p->r > 1 || p->mirror || mode != MODE_FWD || nodes < 130e6;
}

}  // namespace

int vec_zmax(const sw_plan *p)
{
    const int64_t pbytes = int64_t(p->pad[1]) * p->pad[2] * (p->prob.dtype == SW_F64 ? 8 : 4);
    return int(std::max<int64_t>(1, (int64_t(1) << 31) / pbytes - 4 * p->r - 2));
}

bool vec_instance(const sw_plan *p, int mode, int tile)
{
    const bool f64 = p->prob.dtype == SW_F64, vd = p->prob.scheme != SW_CONST;
    if (p->ndim != 3 || tile < 0 || tile >= (vd ? kVdTileCount : kVecTileCount)) return false;
    if (mode != MODE_FWD && (p->mirror || f64 || p->prob.scheme == SW_VD_CENTRED)) return false;
    if (vd) {
        if (p->prob.scheme == SW_VD_STAGGERED && (p->r < kStagRadii[0] || p->r > kStagRadii[1])) return false;
        return kVdTiles[tile].tx * kVdTiles[tile].ty / vd_columns(p->prob.scheme, p->r) <= kVdThreads;
    }
    const VecTile t = f64 ? kVecTiles<double>[tile] : kVecTiles<float>[tile];
    return vec_fits(t.tx * t.lpr, p->r, mode);
}

void vec_extents(const sw_plan *p, int tile, int &rows, int &cols)
{
    const bool f64 = p->prob.dtype == SW_F64;
    if (p->prob.scheme != SW_CONST) {
        rows = kVdTiles[tile].tx;
        cols = kVdTiles[tile].ty;
    } else {
        rows = f64 ? kVecTiles<double>[tile].tx : kVecTiles<float>[tile].tx;
        cols = f64 ? kVecTiles<double>[tile].lpr * 2 : kVecTiles<float>[tile].lpr * 4;
    }
}

// The library's choice in a mode; searched: whether the search had what it needs
// (a device that reports its occupancy).
static VecChoice search_vec(const sw_plan *p, int mode, bool &searched)
{
    searched = true;
    if (p->prob.scheme != SW_CONST) {
        double cost;
        const VecChoice c = choose_vd(p, mode, cost);
        searched = c.tile >= 0 && p->ncu > 0;
        return vd_vectors(p, mode, cost) ? c : VecChoice{};
    }
    if (!const_vectors(p, mode)) return {};
    if (p->mirror) mode = kVecMirror;
    const VecChoice c = p->prob.dtype == SW_F64 ? choose<double>(p, mode) : choose<float>(p, mode);
    searched = c.tile >= 0;
    return c;
}

VecChoice choose_vec(const sw_plan *p, int mode)
{
    const bool forward_only = p->mirror || p->prob.dtype == SW_F64 || p->prob.scheme == SW_VD_CENTRED;   // (no adjoint)
    if (p->ndim != 3 || !library_picks(p, mode) || (forward_only && mode != MODE_FWD)) return {};
    const bool mirror = p->prob.scheme == SW_CONST && p->mirror;
    if (const sw_plan::Pin &pin = p->pin[mode]; pin.tile >= 0) return {pin.tile, std::min(pin.extent, p->dims[0]), mirror};
    uint64_t v = p->choice[mode].load(std::memory_order_relaxed);
    if (!v) {
        bool searched = false;
        const VecChoice c = search_vec(p, mode, searched);
        v = Choice::pack(c.tile, c.zc);
        if (searched) p->choice[mode].store(v, std::memory_order_relaxed);
    }
    return {Choice::first(v), Choice::second(v), mirror};
}

}  // namespace sw
