// Several time steps of a 2D constant-density grid in one launch.
//
// A 2D grid of the sizes in use (0.08 .. 1 M nodes) is bound by launches and
// by the latency of a march through memory, not by bytes: everything it needs
// fits the caches.  So a block holds a whole tile on chip, EZ x EY nodes around
// its tz x ty outputs with nt R nodes on each side, and advances it nt steps:
// the nodes that turn stale from the tile's edge inwards (R per step) are the
// ones around the outputs.  p^n of the tile is staged in LDS, double buffered,
// one barrier per step; each thread owns 2 rows of one 16-byte vector of
// columns, keeps its p^{n-1}, K and damping pair in registers, reads the z
// neighbours as whole vectors (2R + 2 of them for two rows) and the y
// neighbours as the vectors beside its own.
// The mirror ghosts of an edge tile are written in LDS after every step, the
// sources of the launch's steps are added in LDS where they lie, and the
// receivers of the previous launch's levels are recorded by extra blocks, so
// that a launch is all there is per nt steps.
//
// What bounds it now: about 3.6 us of launch per nt steps, the loads of a tile
// (halos included), and the vector units, at 20 .. 24 instructions per node and
// step with the halo nodes counted.  Per step, single-step kernels (stencil
// marching along z, ghost fill, injection, recording) before, this after:
//   281^2 SO8 FP32                        13.7 -> 1.97 us
//   421 x 1841 SO8 FP32, mirror sides     19.3 -> 4.1 us
//   421 x 1841 SO4 FP64, mirror sides     18.3 -> 4.3 us
//   4040^2 SO8 FP32                       76.9 -> 43.5 us
//
// Every value is computed by the operations of the single-step kernels in their
// order (const_tile, k_inject, k_record), so the results are bitwise theirs.
#include <algorithm>
#include <cmath>

#include "multi2d.h"
#include "stencil_const.h"

namespace sw {

namespace {

template <typename T>
struct alignas(16) Vec {
    T v[16 / sizeof(T)];
};

template <typename T, int R, int EZ, int LPR>
struct TileOf {
    static constexpr int CW = 16 / int(sizeof(T));      // columns per thread
    static constexpr int RZ = 2;                        // rows per thread
    static constexpr int EY = LPR * CW;
    static constexpr int NTH = LPR * EZ / RZ;
    static constexpr int NV = (R + CW - 1) / CW;        // vectors read on each side along y
    static constexpr int PC = NV * CW;                  // pad columns
    static constexpr int LYP = EY + 2 * PC;
    static constexpr int ROWS = EZ + 2 * R;             // pad rows above and below
    static constexpr size_t lds = 2 * sizeof(T) * ROWS * LYP;
};

template <typename T, int R, int EZ, int LPR, bool INNER>
__device__ __forceinline__ void multi_tile(const Multi2DParams<T> &P, int z0, int y0, bool src, bool mirror, T *S,
                                           T *sval, int *sloc)
{
    using G_ = TileOf<T, R, EZ, LPR>;
    using T2 = typename Pair<T>::type;
    using V = Vec<T>;
    constexpr int CW = G_::CW, RZ = G_::RZ, PC = G_::PC, NV = G_::NV, LYP = G_::LYP;
    constexpr int BUF = G_::ROWS * LYP;
    const Geom &g = P.g;
    const int tid = threadIdx.x;
    const int col = (tid % LPR) * CW, row = (tid / LPR) * RZ;      // first node owned, tile coordinates
    const int halo = R * P.nt, pady = multi2d_pad_y(halo, int(sizeof(T)));
    const int zt = z0 - halo, yt = y0 - pady;                      // grid coordinates of the tile's first node
    const int z = zt + row, y = yt + col;

    // own nodes: in the grid, not held at zero (bit i * CW + c), and written out
    unsigned live = 0;
    bool out_row[RZ];
    const bool out_col = col >= pady && col < pady + P.ty && y < g.Y;
    const bool whole = y + CW <= g.Y;
    T prev[RZ][CW], k[RZ][CW], a[INNER ? 1 : RZ][CW], b[INNER ? 1 : RZ][CW];
    V first[RZ], vp[RZ], vk[RZ];
    bool in[RZ];
#pragma unroll
    for (int i = 0; i < RZ; ++i) {
        const int zi = z + i;
        out_row[i] = out_col && row + i >= halo && row + i < halo + P.tz && zi < g.Z;
        in[i] = INNER || (zi >= 0 && zi < g.Z && y >= 0 && y < g.Y);
        first[i] = vp[i] = vk[i] = V{};
        if (in[i]) {
            const int o = int(g.origin) + zi * g.py + y;
            first[i] = *reinterpret_cast<const V *>(P.cur + o);
            vp[i] = *reinterpret_cast<const V *>(P.prv + o);
            vk[i] = *reinterpret_cast<const V *>(P.K + o);
        }
    }
    if constexpr (!INNER) {
        // (A, B) by squared layer distance, entry 0 = (1, 1): loaded without
        // branches, in flight together with the fields
        T2 ab[RZ][CW];
#pragma unroll
        for (int i = 0; i < RZ; ++i)
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                const int zi = z + i;
                const int ez = max(0, max(g.lo[0] - zi, zi - (g.lo[0] + g.np[0] - 1)));
                const int ey = max(0, max(g.lo[2] - (y + c), y + c - (g.lo[2] + g.np[2] - 1)));
                const bool ok = in[i] && y + c < g.Y;
                ab[i][c] = P.damp[ok ? ez * ez + ey * ey : 0];
                const bool held = axis_dirichlet(zi, g.Z, P.bcz[0], P.bcz[1]) ||
                                  axis_dirichlet(y + c, g.Y, P.bcy[0], P.bcy[1]);
                if (ok && !held) live |= 1u << (i * CW + c);
            }
#pragma unroll
        for (int i = 0; i < RZ; ++i)
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                a[i][c] = ab[i][c].x;
                b[i][c] = ab[i][c].y;
            }
    }
#pragma unroll
    for (int i = 0; i < RZ; ++i)
#pragma unroll
        for (int c = 0; c < CW; ++c) {
            const bool ok = INNER || (in[i] && y + c < g.Y);
            first[i].v[c] = ok ? first[i].v[c] : T(0);
            prev[i][c] = ok ? vp[i].v[c] : T(0);
            k[i][c] = ok ? vk[i].v[c] : T(0);
        }
    const int own = (R + row) * LYP + PC + col;
#pragma unroll
    for (int i = 0; i < RZ; ++i) *reinterpret_cast<V *>(S + own + i * LYP) = first[i];

    // injected values and their places (both buffers share them)
    if (src)
        for (int u = tid; u < P.nuniq; u += G_::NTH) {
            const int rel = int(P.unode[u] - g.origin);
            const int uz = rel / g.py - zt, uy = rel % g.py - yt;
            const bool in = uz >= 0 && uz < EZ && uy >= 0 && uy < G_::EY;
            sloc[u] = in ? (R + uz) * LYP + PC + uy : -1;
            for (int s = 0; s < P.nt; ++s) sval[s * P.nuniq + u] = P.inj[size_t(s) * P.nuniq + u];
        }
    __syncthreads();

    // mirror ghosts of a buffer: ghost layer k takes +-the node k inside the boundary node
    auto ghosts = [&](T *B) {
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            if (P.bcz[side])
                for (int e = tid; e < R * G_::EY; e += G_::NTH) {
                    const int kk = 1 + e / G_::EY, c = e % G_::EY;
                    const int d = (side ? g.Z - 1 + kk : -kk) - zt, q = (side ? g.Z - 1 - kk : kk) - zt;
                    if (d >= 0 && d < EZ && q >= 0 && q < EZ) {
                        const T v = B[(R + q) * LYP + PC + c];
                        B[(R + d) * LYP + PC + c] = P.bcz[side] == 1 ? -v : v;
                    }
                }
            if (P.bcy[side])
                for (int e = tid; e < R * EZ; e += G_::NTH) {
                    const int kk = 1 + e % R, r = e / R;
                    const int d = (side ? g.Y - 1 + kk : -kk) - yt, q = (side ? g.Y - 1 - kk : kk) - yt;
                    if (d >= 0 && d < G_::EY && q >= 0 && q < G_::EY) {
                        const T v = B[(R + r) * LYP + PC + q];
                        B[(R + r) * LYP + PC + d] = P.bcy[side] == 1 ? -v : v;
                    }
                }
        }
    };
    if (mirror) {
        ghosts(S);
        __syncthreads();
    }

    for (int s = 0; s < P.nt; ++s) {
        const T *A = S + (s & 1) * BUF;
        T *N = S + ((s + 1) & 1) * BUF;
        // rows that still matter: the outputs and what later steps read around them
        const int need = R * (P.nt - 1 - s);
        const bool active = row + RZ > halo - need && row < halo + P.tz + need;
        V nw[RZ];
        if (active) {
            V q[2 * R + RZ];
#pragma unroll
            for (int j = 0; j < 2 * R + RZ; ++j) q[j] = *reinterpret_cast<const V *>(A + own + (j - R) * LYP);
#pragma unroll
            for (int i = 0; i < RZ; ++i) {
                T w[(2 * NV + 1) * CW];
#pragma unroll
                for (int j = 0; j < 2 * NV + 1; ++j) {
                    const V t = j == NV ? q[R + i] : *reinterpret_cast<const V *>(A + own + i * LYP + (j - NV) * CW);
#pragma unroll
                    for (int c = 0; c < CW; ++c) w[j * CW + c] = t.v[c];
                }
#pragma unroll
                for (int c = 0; c < CW; ++c) {
                    const T cc = q[R + i].v[c];
                    T lap = P.c0 * cc;
#pragma unroll
                    for (int j = 1; j <= R; ++j) lap = fmat(P.cz[j], q[R + i + j].v[c] + q[R + i - j].v[c], lap);
#pragma unroll
                    for (int j = 1; j <= R; ++j) lap = fmat(P.cy[j], w[PC + c + j] + w[PC + c - j], lap);
                    T o;
                    if constexpr (INNER) {
                        o = leapfrog(T(1), T(1), k[i][c], lap, cc, prev[i][c]);
                    } else {
                        o = leapfrog(a[i][c], b[i][c], k[i][c], lap, cc, prev[i][c]);
                        o = (live >> (i * CW + c)) & 1 ? o : T(0);
                    }
                    nw[i].v[c] = o;
                    prev[i][c] = cc;
                }
                *reinterpret_cast<V *>(N + own + i * LYP) = nw[i];
            }
        }
        __syncthreads();
        if (src) {
            for (int u = tid; u < P.nuniq; u += G_::NTH)
                if (sloc[u] >= 0) N[sloc[u]] += sval[s * P.nuniq + u];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < RZ; ++i) nw[i] = *reinterpret_cast<const V *>(N + own + i * LYP);
        }
        if (mirror) {
            ghosts(N);
            __syncthreads();
        }
        T *out = P.out[s];
        if (out) {
#pragma unroll
            for (int i = 0; i < RZ; ++i) {
                if (!out_row[i]) continue;
                T *d = out + (int(g.origin) + (z + i) * g.py + y);
                if (whole) {
                    *reinterpret_cast<V *>(d) = nw[i];
                } else {
#pragma unroll
                    for (int c = 0; c < CW; ++c)
                        if (y + c < g.Y) d[c] = nw[i].v[c];
                }
            }
        }
    }
}

template <typename T>
__device__ inline T record_sum(T v, int group)
{
    for (int off = group / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Receivers of the previous launch's levels: a group of lanes per (level,
// receiver), as k_record.
template <typename T>
__device__ __forceinline__ void record_levels(const Multi2DParams<T> &P, int64_t first)
{
    const int64_t item = (first + threadIdx.x) / P.group;
    const int sub = threadIdx.x % P.group;
    const bool in = item < int64_t(P.rnt) * P.count;
    const int lev = in ? int(item / P.count) : 0, pt = in ? int(item % P.count) : 0;
    T acc = T(0);
    if (in) {
        const T *field = P.rlev[lev];
        for (int e = P.ptr[pt] + sub; e < P.ptr[pt + 1]; e += P.group) acc += P.wscaled[e] * field[P.node[e]];
    }
    acc = record_sum(acc, P.group);
    if (in && sub == 0) P.rout[item] = acc;
}

template <typename T, int R, int EZ, int LPR>
__global__ void __launch_bounds__((TileOf<T, R, EZ, LPR>::NTH)) k_multi2d(Multi2DParams<T> P)
{
    using G_ = TileOf<T, R, EZ, LPR>;
    __shared__ __align__(16) T S[2 * G_::ROWS * G_::LYP];
    extern __shared__ __align__(16) unsigned char dyn[];
    const int tiles = P.ntz * P.nty;
    if (int(blockIdx.x) >= tiles) {
        record_levels(P, int64_t(blockIdx.x - tiles) * G_::NTH);
        return;
    }
    const int bid = xcd_remap(blockIdx.x, tiles);
    const int z0 = (bid / P.nty) * P.tz, y0 = (bid % P.nty) * P.ty;
    const int halo = R * P.nt, pady = multi2d_pad_y(halo, int(sizeof(T)));
    const int zt = z0 - halo, yt = y0 - pady;
    const Geom &g = P.g;
    T *sval = reinterpret_cast<T *>(dyn);
    int *sloc = reinterpret_cast<int *>(sval + size_t(P.nt) * P.nuniq);
    const bool src = P.nuniq > 0 && P.box[0] < zt + EZ && P.box[1] >= zt && P.box[2] < yt + G_::EY && P.box[3] >= yt;
    // every node of the tile undamped and off the boundary: no pair, no mask
    const bool inner = zt >= max(1, g.lo[0]) && zt + EZ <= min(g.Z - 1, g.lo[0] + g.np[0]) &&
                       yt >= max(1, g.lo[2]) && yt + G_::EY <= min(g.Y - 1, g.lo[2] + g.np[2]);
    if (inner) {
        multi_tile<T, R, EZ, LPR, true>(P, z0, y0, src, false, S, sval, sloc);
        return;
    }
    const bool mirror = (P.bcz[0] && zt < 0) || (P.bcz[1] && zt + EZ > g.Z) || (P.bcy[0] && yt < 0) ||
                        (P.bcy[1] && yt + G_::EY > g.Y);
    multi_tile<T, R, EZ, LPR, false>(P, z0, y0, src, mirror, S, sval, sloc);
}

template <typename T, int G>
__global__ void __launch_bounds__(256) k_inject_all(InjectTable<T> t, const T *__restrict__ amp, T *__restrict__ out)
{
    const int gid = blockIdx.x * blockDim.x + threadIdx.x;
    const int u = gid / G, sub = gid % G;
    amp += size_t(blockIdx.y) * t.nsrc;
    T sa = T(0);
    if (u < t.nuniq)
        for (int k = t.uptr[u] + sub; k < t.uptr[u + 1]; k += G) {
            const int e = t.uent[k];
            sa = fmat(t.coef_a[e], amp[t.pid[e]], sa);
        }
#pragma unroll
    for (int off = G / 2; off > 0; off >>= 1) sa += __shfl_xor(sa, off, G);
    if (u < t.nuniq && sub == 0) out[size_t(blockIdx.y) * t.nuniq + u] = sa;
}

template <typename T, int R, int EZ, int LPR>
hipError_t launch_tile(Multi2DParams<T> &P, hipStream_t s)
{
    using G_ = TileOf<T, R, EZ, LPR>;
    const int64_t rec = P.rnt > 0 ? (int64_t(P.rnt) * P.count * P.group + G_::NTH - 1) / G_::NTH : 0;
    const size_t dyn = size_t(P.nuniq) * (P.nt * sizeof(T) + sizeof(int));
    hipLaunchKernelGGL((k_multi2d<T, R, EZ, LPR>), dim3(unsigned(int64_t(P.ntz) * P.nty + rec)), dim3(G_::NTH),
                       unsigned(dyn), s, P);
    return hipGetLastError();
}

constexpr Multi2DTile kTiles[] = {{64, 32}, {32, 32}, {64, 16}, {48, 16}, {32, 16}};    // ey: vectors

// Radii whose neighbour vectors fit the 128 registers of a 1024-thread block.
template <typename T>
constexpr int kWideMax = sizeof(T) == 4 ? 6 : 5;

template <typename T, int R>
hipError_t launch_radius(int tile, Multi2DParams<T> &P, hipStream_t s)
{
    switch (tile) {
    case 0:
        if constexpr (R <= kWideMax<T>) return launch_tile<T, R, 64, 32>(P, s);
        else return hipErrorInvalidValue;
    case 1: return launch_tile<T, R, 32, 32>(P, s);
    case 2: return launch_tile<T, R, 64, 16>(P, s);
    case 3: return launch_tile<T, R, 48, 16>(P, s);
    case 4: return launch_tile<T, R, 32, 16>(P, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

// Steps per launch and tile by a model of a launch of nt steps, fitted to a
// sweep of every tile and step count over 136^2 .. 1180 x 1980 nodes, SO2 .. SO20
// and both precisions (rms error 12%; its choices ran within 1% of the sweep's
// best on average, 18% at worst):
//   launch = 3.56 us + max(0.98 us nt, busy (1.26e-4 + 2.6e-5 R) us) + loads,
// busy = node updates of the tiles of one CU over the nt steps (the rows that
// still matter), loads = 1.13e-4 us per byte of one array they read.  Few steps
// leave the launch and the loads to be paid often, many leave the tile little
// but halo.  A single-step sweep (stencil, injection, recording, mirror ghosts)
// measured 8.5 us + 1.75 us R, plus about 4e-6 us per node and 4 bytes; where
// the model with a quarter on top is not below that, the plan keeps it (SO20
// at 1180 x 1980: 41 against 32 us per step).
// The model knows neither the caches nor rounds past its grids: 4200 random
// grids up to 200 M nodes gave, per radius and precision, the number of nodes
// above which single steps are the faster ones.  Tiles that are mostly halo
// (SO18, SO20; SO12 and SO14 in doubles) lose first, the others once the
// levels of a launch outgrow the caches.  Rate of several steps over that of
// single ones: SO20 1.05 at 1.52 M nodes and 0.93 at 1.94 M, SO10 1.14 at
// 20.8 M and 0.91 at 28.8 M, SO12 1.09 at 21.7 M and 0.86 at 29.4 M (between 34
// and 82 M some grids gain up to 1.2 again, as many lose); in doubles SO6
// 1.09 at 13.1 M and 0.95 at 18.6 M, SO8 1.14 at 11.9 M and 0.96 at 16.7 M,
// SO10 1.07 at 9.7 M and 0.87 at 12.5 M, SO12 1.08 at 1.0 M and 0.88 at
// 1.24 M, SO14 1.13 at 0.27 M and 0.88 at 0.41 M.  Of 3000 grids
// that still take several steps none is more than 1% slower than with single
// steps.
Multi2DChoice choose_multi2d(int r, int value_bytes, int Z, int Y, int cus)
{
    Multi2DChoice best{};
    constexpr double kNone = 1e18;
    constexpr double kNodes32[11] = {0, kNone, kNone, kNone, kNone, 23e6, 23e6, kNone, kNone, 1.45e6, 1.45e6};
    constexpr double kNodes64[11] = {0, kNone, kNone, 15.5e6, 14e6, 10e6, 1.1e6, 0.3e6, kNone, kNone, kNone};
    if (double(Z) * Y > (value_bytes == 4 ? kNodes32 : kNodes64)[r]) return best;
    double cost = (8.5 + 1.75 * r + 1e-6 * value_bytes * double(Z) * Y) / 1.25;
    for (int tile = 0; tile < int(sizeof(kTiles) / sizeof(kTiles[0])); ++tile) {
        const Multi2DTile t = multi2d_tile(tile, value_bytes);
        for (int nt = 2; nt <= kMulti2DMax; ++nt) {
            const int tz = t.ez - 2 * r * nt, ty = t.ey - 2 * multi2d_pad_y(r * nt, value_bytes);
            if (!multi2d_tile_ok(r, value_bytes, tile, nt)) break;
            const double tiles = double((Z + tz - 1) / tz) * ((Y + ty - 1) / ty);
            const double per_cu = std::ceil(tiles / cus);
            int rows = 0;
            for (int s = 0; s < nt; ++s) rows += std::min(t.ez, tz + 2 * r * s);
            const double busy = per_cu * rows * t.ey * (1.26e-4 + 2.6e-5 * r);
            const double loads = 1.13e-4 * per_cu * t.ez * t.ey * value_bytes;
            const double c = (3.56 + std::max(0.98 * nt, busy) + loads) / nt;
            if (c < cost) {
                cost = c;
                best = {nt, tile};
            }
        }
    }
    return best;
}

bool multi2d_tile_ok(int r, int value_bytes, int tile, int steps)
{
    if (tile < 0 || tile >= int(sizeof(kTiles) / sizeof(kTiles[0])) || steps < 2 || steps > kMulti2DMax ||
        (tile == 0 && r > (value_bytes == 4 ? kWideMax<float> : kWideMax<double>)))
        return false;
    const Multi2DTile t = multi2d_tile(tile, value_bytes);
    return t.ez > 2 * r * steps && t.ey > 2 * multi2d_pad_y(r * steps, value_bytes);
}

Multi2DTile multi2d_tile(int tile, int value_bytes)
{
    Multi2DTile t = kTiles[tile];
    t.ey *= 16 / value_bytes;
    return t;
}

template <typename T>
hipError_t launch_multi2d(int r, int tile, Multi2DParams<T> &P, hipStream_t s)
{
    switch (r) {
    case 1: return launch_radius<T, 1>(tile, P, s);
    case 2: return launch_radius<T, 2>(tile, P, s);
    case 3: return launch_radius<T, 3>(tile, P, s);
    case 4: return launch_radius<T, 4>(tile, P, s);
    case 5: return launch_radius<T, 5>(tile, P, s);
    case 6: return launch_radius<T, 6>(tile, P, s);
    case 7: return launch_radius<T, 7>(tile, P, s);
    case 8: return launch_radius<T, 8>(tile, P, s);
    case 9: return launch_radius<T, 9>(tile, P, s);
    case 10: return launch_radius<T, 10>(tile, P, s);
    default: return hipErrorInvalidValue;
    }
}
template hipError_t launch_multi2d<float>(int, int, Multi2DParams<float> &, hipStream_t);
template hipError_t launch_multi2d<double>(int, int, Multi2DParams<double> &, hipStream_t);

template <typename T>
hipError_t launch_inject_all(const InjectTable<T> &t, const T *amp, int nsteps, T *out, hipStream_t s)
{
    if (t.nuniq <= 0 || nsteps <= 0) return hipSuccess;
    int G = 1;
    while (G < t.max_per_node && G < 64) G <<= 1;
    for (int n = 0; n < nsteps; n += 65535) {
        const dim3 grid(unsigned((int64_t(t.nuniq) * G + 255) / 256), unsigned(std::min(nsteps - n, 65535)));
        const T *a = amp + size_t(n) * t.nsrc;
        T *o = out + size_t(n) * t.nuniq;
        switch (G) {
        case 1: hipLaunchKernelGGL((k_inject_all<T, 1>), grid, dim3(256), 0, s, t, a, o); break;
        case 2: hipLaunchKernelGGL((k_inject_all<T, 2>), grid, dim3(256), 0, s, t, a, o); break;
        case 4: hipLaunchKernelGGL((k_inject_all<T, 4>), grid, dim3(256), 0, s, t, a, o); break;
        case 8: hipLaunchKernelGGL((k_inject_all<T, 8>), grid, dim3(256), 0, s, t, a, o); break;
        case 16: hipLaunchKernelGGL((k_inject_all<T, 16>), grid, dim3(256), 0, s, t, a, o); break;
        case 32: hipLaunchKernelGGL((k_inject_all<T, 32>), grid, dim3(256), 0, s, t, a, o); break;
        default: hipLaunchKernelGGL((k_inject_all<T, 64>), grid, dim3(256), 0, s, t, a, o); break;
        }
    }
    return hipGetLastError();
}
template hipError_t launch_inject_all<float>(const InjectTable<float> &, const float *, int, float *, hipStream_t);
template hipError_t launch_inject_all<double>(const InjectTable<double> &, const double *, int, double *, hipStream_t);

}  // namespace sw
