// Constant-density stencil on vector tiles (3D): the update, modes, blocking
// along z and addressing of const_tile (stencil_const.h), with a 16-byte vector
// of columns per thread in place of several rows of one column.
//
// A block owns TX rows x TY = LPR * CW columns (CW = 4 floats or 2 doubles) and
// one thread per vector.  So a plane takes one 16-byte load per array and
// thread, the x neighbours are read from LDS as whole vectors and the y
// neighbours as the NV vectors on either side: per node a quarter of the loads,
// of the LDS instructions and of the addressing of the scalar tiles.  The halo
// of a plane (2R rows, 2 NV vectors of every row) is one more load for the
// threads it needs.  The column's planes z - R .. z + R + 1 rotate through
// registers, the last of them the load in flight.
// What bounds it: HBM at the larger sizes (592^3 SO8, 3 reads and 1 write per
// node: 0.614 ms, 5.4 TB/s, where the scalar tiles take 0.69), the chain of
// loads, barrier and LDS reads per plane where a launch is one round (128^3 with
// its layer 14 against 20 us).  High orders at sizes between have no one limit:
// 336^3 SO16 (149 us, scalar tiles 222) moves 5.15 TB/s with the halo re-reads
// (reads 1.35 of the algorithmic bytes), its SIMDs issue vector instructions in
// 54% of the cycles and LDS is busy in 21%.
// Mirror ghosts are made in LDS (x, y) and by the plane that is loaded (z), so
// that no ghost fill runs before the sweep (53 us of 960 us per step at
// 207 x 801 x 801 in double precision).
// The damping pairs of a thread's nodes change along z only inside the layer, so
// they stay in registers and are looked up again where the plane's distance to
// the physical box changes.
#pragma once

#include <atomic>

#include "stencil_const.h"
#include "vec.h"

namespace sw {

template <typename T>
struct VecOf {
    static constexpr int CW = 16 / int(sizeof(T));
    typedef T type __attribute__((ext_vector_type(16 / sizeof(T))));
};

template <typename T, int NT>
__device__ __forceinline__ typename VecOf<T>::type buf_ldv(__amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    return __builtin_bit_cast(typename VecOf<T>::type, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, NT ? 2 : 0));
}

// A 16-byte buffer store reads its data a little after it issues: an instruction
// right behind it that overwrites the first data register changes what the last
// four lanes store (seen with a plane offset in an SGPR, a form for which the
// compiler inserts no wait: the imaging kernels stored the gradient in place of
// the wavefield in a few nodes).  So two wait states follow every such store,
// and nothing is scheduled between.
template <typename T, int NT>
__device__ __forceinline__ void buf_stv(typename VecOf<T>::type v, __amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    using V = decltype(__builtin_amdgcn_raw_buffer_load_b128(r, 0, 0, 0));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(V, v), r, voff, soff, NT ? 2 : 0);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 1");
    __builtin_amdgcn_sched_barrier(0);
}

// Values of the two LDS planes of a tile.
template <typename T, int R, int TX, int LPR>
constexpr int vec_lds()
{
    constexpr int CW = VecOf<T>::CW, PC = (R + CW - 1) / CW * CW;
    return 2 * (TX + 2 * R) * (LPR * CW + 2 * PC);
}

// MIRROR: 0 no mirror sides; 1 mirror sides, none along x or y within the tile's
// halo (z alone: the queue's planes); 2 any.
template <typename T, int R, int TX, int LPR, int MODE, int NT, int MIRROR>
__device__ __forceinline__ void vec_tile(const StencilParamsT<T> &P, int bid, T *lds)
{
    using T2 = typename Pair<T>::type;
    using V = typename VecOf<T>::type;
    constexpr int CW = VecOf<T>::CW;
    constexpr int ES = int(sizeof(T));
    constexpr int TY = LPR * CW;
    constexpr int NTH = TX * LPR;
    constexpr int NV = (R + CW - 1) / CW;        // vectors of y halo on each side
    constexpr int PC = NV * CW;
    constexpr int LYP = TY + 2 * PC;
    constexpr int PLANE = vec_lds<T, R, TX, LPR>() / 2;
    constexpr int NXH = 2 * R * LPR;             // halo vectors: rows above and below
    constexpr int NH = NXH + TX * 2 * NV;        // and beside the tile's rows
    constexpr int NHT = (NH + NTH - 1) / NTH;
    constexpr int Q = 2 * R + 2;
    constexpr int kOut = 0x7ffffe00;
    constexpr bool kImage = (MODE == MODE_IMAGE || MODE == MODE_IMAGE2);
    constexpr bool XY = MIRROR == 2;

    const Geom &g = P.g;
    const int tid = threadIdx.x;
    const int row = tid / LPR, col = (tid % LPR) * CW;
    int tx, ty, zc;
    tile_of(bid, P.ntx, P.nty, P.xfast, tx, ty, zc);
    const int x0 = tx * TX, y0 = ty * TY;
    const int x = x0 + row, y = y0 + col;
    const int zb = zc * P.zc;
    const int ze = min(zb + P.zc, g.Z);
    const int64_t sz = int64_t(g.px) * g.py;
    const int zw = zb - R, zt = ze + R;
    const int pb = int(sz) * ES;
    const uint32_t wbytes = uint32_t(zt - zw) * uint32_t(pb);
    const int64_t w0 = g.base + int64_t(zw) * sz;
    const auto rc = buf_res(P.cur + w0, wbytes);
    const auto rn = buf_res(P.nxt + w0, wbytes);
    const auto rk = buf_res(P.K + w0, wbytes);
    const auto rd = buf_res(P.damp, uint32_t(P.ndamp) * uint32_t(sizeof(T2)));
    __amdgpu_buffer_rsrc_t rs = rk, rg = rk, rs2 = rk;
    if constexpr (MODE != MODE_FWD) rs = buf_res(P.store + w0, wbytes);
    if constexpr (kImage) rg = buf_res(P.grad + w0, wbytes);
    if constexpr (MODE == MODE_IMAGE2) rs2 = buf_res(P.store2 + w0, wbytes);
    auto soff = [&](int z) -> int { return (z - zw) * pb; };
    // vector at (x, y .. y + CW - 1): its offset if the grid holds any node of it,
    // else past every window (reads zero)
    auto rd_off = [&](int xx, int yy) -> int {
        return xx >= 0 && xx < g.X && yy >= 0 && yy < g.Y ? (g.xy0 + xx * g.py + yy) * ES : kOut;
    };
    const int ro = rd_off(x, y);
    const bool in = ro != kOut;
    // the grid ends inside a vector that this tile reads: its nodes past the end
    // read zero and are written as zero
    const bool ragged = g.Y % CW != 0 && g.Y < y0 + TY + PC;
    auto clip = [&](V v, int yy) -> V {
#pragma unroll
        for (int c = 0; c < CW; ++c) v[c] = yy + c < g.Y ? v[c] : T(0);
        return v;
    };
    // mirrored sides this tile's halo reaches: their ghosts are made in LDS from
    // the nodes beside them (the tile or its halo holds all R of them)
    const int mxl = XY && x0 < R ? P.bcm[1][0] : 0, mxh = XY && x0 + TX + R > g.X ? P.bcm[1][1] : 0;
    const int myl = XY && y0 < R ? P.bcm[2][0] : 0, myh = XY && y0 + TY + R > g.Y ? P.bcm[2][1] : 0;
    const bool mirror = mxl | mxh | myl | myh;
    // nodes of this thread on a side that a Dirichlet condition holds at zero (bit per node)
    unsigned held = 0;
#pragma unroll
    for (int c = 0; c < CW; ++c)
        if (XY && axis_dirichlet(x, g.X, P.bcm[1][0], P.bcm[1][1])) held |= 1u << c;
        else if (XY && axis_dirichlet(y + c, g.Y, P.bcm[2][0], P.bcm[2][1]))
            held |= 1u << c;
    const bool holds = mxl == 1 || mxh == 1 || myl == 1 || myh == 1;

    const int ex = max(0, max(g.lo[1] - x, x - (g.lo[1] + g.np[1] - 1)));
    int e2[CW];
#pragma unroll
    for (int c = 0; c < CW; ++c) {
        const int ey = max(0, max(g.lo[2] - (y + c), y + c - (g.lo[2] + g.np[2] - 1)));
        e2[c] = in && y + c < g.Y ? ex * ex + ey * ey : 0;      // keeps table reads in range
    }
    const bool inner_xy = x0 >= g.lo[1] && x0 + TX <= g.lo[1] + g.np[1] && y0 >= g.lo[2] && y0 + TY <= g.lo[2] + g.np[2];

    int ho[NHT], hl[NHT], hyy[NHT];
#pragma unroll
    for (int s = 0; s < NHT; ++s) {
        const int e = tid + s * NTH;
        int hr, hc;
        if (e < NXH) {                           // rows above and below
            const int k = e / LPR;
            hr = k < R ? k : TX + k;
            hc = PC + (e % LPR) * CW;
        } else {                                 // vectors left and right of the tile's rows
            const int e3 = e - NXH, k = e3 % (2 * NV);
            hr = R + e3 / (2 * NV);
            hc = k < NV ? k * CW : TY + k * CW;
        }
        const bool ok = e < NH;
        hyy[s] = y0 - PC + hc;
        ho[s] = ok ? rd_off(x0 - R + hr, hyy[s]) : kOut;
        hl[s] = hr * LYP + hc;
    }

    V q[Q];                                      // q[(u + k) % Q] = p^n at plane z - R + k in unrolled step u
    // (off the grid: zero, or the plane across a mirrored side, negated for Dirichlet)
    auto ld_cur = [&](int z) -> V {
        const int bc = !MIRROR ? 0 : z < 0 ? P.bcm[0][0] : z >= g.Z ? P.bcm[0][1] : 0;
        const int m = bc == 0 ? z : z < 0 ? -z : 2 * (g.Z - 1) - z;
        V v{};
        if (m >= 0 && m < g.Z) v = buf_ldv<T, 0>(rc, ro, soff(m));
        if (bc == 1) v = -v;
        return v;
    };
#pragma unroll
    for (int k = 0; k <= 2 * R; ++k) q[k] = ld_cur(zb - R + k);
    struct Slot {
        V p, k, h[NHT], d, g, d2;                // (unused ones take no registers)
    };
    Slot S[2];
    auto load = [&](int z, Slot &L) {
        const int so = soff(z);
#pragma unroll
        for (int s = 0; s < NHT; ++s) L.h[s] = buf_ldv<T, 0>(rc, ho[s], so);
        L.p = buf_ldv<T, NT>(rn, ro, so);
        L.k = buf_ldv<T, NT>(rk, ro, so);
        if constexpr (kImage) {
            L.d = buf_ldv<T, NT>(rs, ro, so);
            L.g = buf_ldv<T, NT>(rg, ro, so);
        }
        if constexpr (MODE == MODE_IMAGE2) L.d2 = buf_ldv<T, NT>(rs2, ro, so);
    };
    load(zb, S[0]);
    V a, b;
#pragma unroll
    for (int c = 0; c < CW; ++c) a[c] = b[c] = T(1);
    int ez0 = inner_xy ? 0 : -1;                 // layer distance along z that (a, b) hold for
    const int own = (R + row) * LYP + PC + col;
    for (int zz = zb; zz < ze; zz += Q) {
#pragma unroll
        for (int u = 0; u < Q; ++u) {
            const int z = zz + u;
            if (z < ze) {
                Slot &W = S[u % 2];
                const int ez = max(0, max(g.lo[0] - z, z - (g.lo[0] + g.np[0] - 1)));
                if (ez != ez0) {
                    ez0 = ez;
#pragma unroll
                    for (int c = 0; c < CW; ++c) {
                        const T2 ab = buf_ld2t<T>(rd, (ez * ez + e2[c]) * int(sizeof(T2)));
                        a[c] = ab.x;
                        b[c] = ab.y;
                    }
                }
                if (z + 1 < ze) {
                    q[(u + 2 * R + 1) % Q] = ld_cur(z + 1 + R);
                    load(z + 1, S[(u + 1) % 2]);
                }
                T *L = lds + (u % 2) * PLANE;
                V cc = q[(u + R) % Q];
                if (ragged) cc = clip(cc, y);
                *reinterpret_cast<V *>(L + own) = cc;
#pragma unroll
                for (int s = 0; s < NHT; ++s) {
                    if (s * NTH + tid >= NH) continue;
                    V h = W.h[s];
                    if (ragged) h = clip(h, hyy[s]);
                    *reinterpret_cast<V *>(L + hl[s]) = h;
                }
                __syncthreads();
                if (XY && mirror) {
                    // ghost k of a side takes +-the node k inside its boundary node: rows, then columns
                    int first = tid;
                    asm volatile("" : "+v"(first));      // (keeps these addresses out of the march's registers)
                    for (int e = first; e < 2 * R * TY; e += NTH) {
                        const int side = e / (R * TY), k = 1 + e / TY % R, c = PC + e % TY;
                        const int bc = side ? mxh : mxl;
                        const int d = (side ? g.X - 1 + k : -k) - x0, q = (side ? g.X - 1 - k : k) - x0;
                        if (bc && d >= -R && d < TX + R && q >= -R && q < TX + R) {
                            const T v = L[(R + q) * LYP + c];
                            L[(R + d) * LYP + c] = bc == 1 ? -v : v;
                        }
                    }
                    for (int e = first; e < 2 * R * TX; e += NTH) {
                        const int side = e / (R * TX), k = 1 + e % R, r = R + e / R % TX;
                        const int bc = side ? myh : myl;
                        const int d = (side ? g.Y - 1 + k : -k) - y0, q = (side ? g.Y - 1 - k : k) - y0;
                        if (bc && d >= -PC && d < TY + PC && q >= -PC && q < TY + PC) {
                            const T v = L[r * LYP + PC + q];
                            L[r * LYP + PC + d] = bc == 1 ? -v : v;
                        }
                    }
                    __syncthreads();
                    cc = *reinterpret_cast<const V *>(L + own);      // a vector the grid ends in holds ghosts now
                }

                const int so = soff(z);
                V lap = P.c0 * cc;
#pragma unroll
                for (int j = 1; j <= R; ++j) {
                    const V t = q[(u + R + j) % Q] + q[(u + R - j) % Q];
#pragma unroll
                    for (int c = 0; c < CW; ++c) lap[c] = fmat(P.cz[j], t[c], lap[c]);
                }
#pragma unroll
                for (int j = 1; j <= R; ++j) {
                    const V t = *reinterpret_cast<const V *>(L + own + j * LYP) +
                                *reinterpret_cast<const V *>(L + own - j * LYP);
#pragma unroll
                    for (int c = 0; c < CW; ++c) lap[c] = fmat(P.cx[j], t[c], lap[c]);
                }
                T w[(2 * NV + 1) * CW];
#pragma unroll
                for (int k = 0; k < 2 * NV + 1; ++k) {
                    const V t = k == NV ? cc : *reinterpret_cast<const V *>(L + own + (k - NV) * CW);
#pragma unroll
                    for (int c = 0; c < CW; ++c) w[k * CW + c] = t[c];
                }
#pragma unroll
                for (int j = 1; j <= R; ++j)
#pragma unroll
                    for (int c = 0; c < CW; ++c) lap[c] = fmat(P.cy[j], w[PC + c + j] + w[PC + c - j], lap[c]);
                V out;
#pragma unroll
                for (int c = 0; c < CW; ++c) out[c] = leapfrog(a[c], b[c], W.k[c], lap[c], cc[c], W.p[c]);
                const bool plane = MIRROR && axis_dirichlet(z, g.Z, P.bcm[0][0], P.bcm[0][1]);
                if (holds || plane) {
#pragma unroll
                    for (int c = 0; c < CW; ++c) out[c] = plane || (held >> c & 1) ? T(0) : out[c];
                }
                auto put = [&](V v, __amdgpu_buffer_rsrc_t r) {
                    if (ragged) {
#pragma unroll
                        for (int c = 0; c < CW; ++c) v[c] = y + c < g.Y ? v[c] : T(0);
                    }
                    buf_stv<T, NT>(v, r, ro, so);
                };
                put(out, rn);
                if constexpr (MODE == MODE_STORE) put(W.k * lap, rs);
                if constexpr (kImage) {
                    V s;
#pragma unroll
                    for (int c = 0; c < CW; ++c) {
                        const T k2 = W.k[c] * W.k[c];
                        if constexpr (MODE == MODE_IMAGE) s[c] = fmat(cc[c], W.d[c] / k2, W.g[c]);
                        else s[c] = fmat(cc[c], W.d[c] / k2, fmat(W.p[c], W.d2[c] / k2, W.g[c]));
                    }
                    put(s, rg);
                }
            }
        }
    }
}

// Waves per SIMD that the kernels of mirror plans are held to (the number that
// the others reach; the ghost code alone would cost them one).
template <int R>
constexpr int vec_mirror_waves()
{
    return R <= 4 ? 4 : R <= 8 ? 3 : 2;
}

template <typename T, int R, int TX, int LPR, int MODE, int NT>
__global__ void __launch_bounds__((TX * LPR)) k_vec(StencilParamsT<T> P)
{
    __shared__ __align__(16) T lds[vec_lds<T, R, TX, LPR>()];
    vec_tile<T, R, TX, LPR, MODE, NT, 0>(P, xcd_remap(blockIdx.x, gridDim.x), lds);
}

// Forward of a plan with mirror sides.  The tiles away from its x and y sides
// run the code without ghosts: sharing it costs every plane of every tile (the
// ghost code stands between the barrier and the reads), 15% at 592^3 SO8.
template <typename T, int R, int TX, int LPR, int NT>
__global__ void __launch_bounds__((TX * LPR), (vec_mirror_waves<R>())) k_vec_mirror(StencilParamsT<T> P)
{
    constexpr int TY = LPR * VecOf<T>::CW;
    __shared__ __align__(16) T lds[vec_lds<T, R, TX, LPR>()];
    const int bid = xcd_remap(blockIdx.x, gridDim.x);
    int tx, ty, zc;
    tile_of(bid, P.ntx, P.nty, P.xfast, tx, ty, zc);
    const bool edge = (P.bcm[1][0] && tx * TX < R) || (P.bcm[1][1] && tx * TX + TX + R > P.g.X) ||
                      (P.bcm[2][0] && ty * TY < R) || (P.bcm[2][1] && ty * TY + TY + R > P.g.Y);
    if (edge) vec_tile<T, R, TX, LPR, MODE_FWD, NT, 2>(P, bid, lds);
    else vec_tile<T, R, TX, LPR, MODE_FWD, NT, 1>(P, bid, lds);
}

// Many grids in one launch, as k_const_batch: tiles of 16 rows x 64 columns.
template <int R>
__global__ void __launch_bounds__(256) k_vec_batch(const StencilParams *__restrict__ shots, const int *__restrict__ tile_start,
                                                   int nshots, int parity)
{
    __shared__ __align__(16) float lds[vec_lds<float, R, 16, 16>()];
    const int total = tile_start[nshots];
    const int first = xcd_remap(blockIdx.x, gridDim.x);
    for (int t = first; t < total; t += gridDim.x) {
        int lo = 0, hi = nshots - 1;          // last shot with tile_start <= t
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (tile_start[mid] <= t) lo = mid; else hi = mid - 1;
        }
        StencilParams P = shots[lo];
        if (parity) {
            float *c = const_cast<float *>(P.cur);
            P.cur = P.nxt;
            P.nxt = c;
        }
        vec_tile<float, R, 16, 16, MODE_FWD, 1, 0>(P, t - tile_start[lo], lds);
        __syncthreads();                      // LDS is reused by the next tile
    }
}

template <int R>
hipError_t launch_vec_batch_radius(const StencilParams *shots, const int *tile_start, int nshots, int parity, int nblocks,
                                   hipStream_t s)
{
    hipLaunchKernelGGL((k_vec_batch<R>), dim3(nblocks), dim3(256), 0, s, shots, tile_start, nshots, parity);
    return hipGetLastError();
}

// Resident blocks per CU of a kernel, asked once per kernel (0, and asked again,
// where the query fails).
template <auto KERN>
int blocks_per_cu(int threads)
{
    static std::atomic<int> known{0};
    int n = known.load(std::memory_order_relaxed);
    if (n > 0) return n;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, KERN, threads, 0) != hipSuccess) return 0;
    known.store(n, std::memory_order_relaxed);
    return n;
}

template <typename T, int R, int TX, int LPR, int MODE>
constexpr auto vec_kernel()
{
    if constexpr (MODE == kVecMirror) return k_vec_mirror<T, R, TX, LPR, 1>;
    else return k_vec<T, R, TX, LPR, MODE, 1>;
}

// Tiles of a value type and mode: index I of kVecTiles.
template <typename T, int R, int MODE, int I>
constexpr bool vec_has()
{
    return vec_fits(kVecTiles<T>[I].tx * kVecTiles<T>[I].lpr, R, MODE);
}

template <typename T, int R, int MODE, int I>
hipError_t launch_vec_tile(StencilParamsT<T> &P, hipStream_t s)
{
    if constexpr (vec_has<T, R, MODE, I>()) {
        constexpr VecTile t = kVecTiles<T>[I];
        hipLaunchKernelGGL((vec_kernel<T, R, t.tx, t.lpr, MODE>()), dim3(P.ntx * P.nty * P.nzc), dim3(t.tx * t.lpr), 0, s, P);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

template <typename T, int R, int MODE, int I>
int vec_resident_tile()
{
    if constexpr (vec_has<T, R, MODE, I>()) {
        constexpr VecTile t = kVecTiles<T>[I];
        return blocks_per_cu<vec_kernel<T, R, t.tx, t.lpr, MODE>()>(t.tx * t.lpr);
    }
    return 0;
}

template <typename T, int R, int MODE>
hipError_t launch_vec_mode(int tile, StencilParamsT<T> &P, hipStream_t s)
{
    switch (tile) {
    case 0: return launch_vec_tile<T, R, MODE, 0>(P, s);
    case 1: return launch_vec_tile<T, R, MODE, 1>(P, s);
    case 2: return launch_vec_tile<T, R, MODE, 2>(P, s);
    case 3: return launch_vec_tile<T, R, MODE, 3>(P, s);
    case 4: return launch_vec_tile<T, R, MODE, 4>(P, s);
    case 5: return launch_vec_tile<T, R, MODE, 5>(P, s);
    case 6: return launch_vec_tile<T, R, MODE, 6>(P, s);
    case 7: return launch_vec_tile<T, R, MODE, 7>(P, s);
    default: return hipErrorInvalidValue;
    }
}

template <typename T, int R, int MODE>
int vec_resident_mode(int tile)
{
    switch (tile) {
    case 0: return vec_resident_tile<T, R, MODE, 0>();
    case 1: return vec_resident_tile<T, R, MODE, 1>();
    case 2: return vec_resident_tile<T, R, MODE, 2>();
    case 3: return vec_resident_tile<T, R, MODE, 3>();
    case 4: return vec_resident_tile<T, R, MODE, 4>();
    case 5: return vec_resident_tile<T, R, MODE, 5>();
    case 6: return vec_resident_tile<T, R, MODE, 6>();
    case 7: return vec_resident_tile<T, R, MODE, 7>();
    default: return 0;
    }
}

template <typename T, int R>
hipError_t launch_vec_radius(int tile, int mode, StencilParamsT<T> &P, hipStream_t s)
{
    if (mode == MODE_FWD) return launch_vec_mode<T, R, MODE_FWD>(tile, P, s);
    if (mode == kVecMirror) return launch_vec_mode<T, R, kVecMirror>(tile, P, s);
    if constexpr (sizeof(T) == 4) {
        if (mode == MODE_STORE) return launch_vec_mode<T, R, MODE_STORE>(tile, P, s);
        if (mode == MODE_IMAGE) return launch_vec_mode<T, R, MODE_IMAGE>(tile, P, s);
        if (mode == MODE_IMAGE2) return launch_vec_mode<T, R, MODE_IMAGE2>(tile, P, s);
    }
    return hipErrorInvalidValue;
}

template <typename T, int R>
int vec_resident_radius(int tile, int mode)
{
    if (mode == MODE_FWD) return vec_resident_mode<T, R, MODE_FWD>(tile);
    if (mode == kVecMirror) return vec_resident_mode<T, R, kVecMirror>(tile);
    if constexpr (sizeof(T) == 4) {
        if (mode == MODE_STORE) return vec_resident_mode<T, R, MODE_STORE>(tile);
        if (mode == MODE_IMAGE) return vec_resident_mode<T, R, MODE_IMAGE>(tile);
        if (mode == MODE_IMAGE2) return vec_resident_mode<T, R, MODE_IMAGE2>(tile);
    }
    return 0;
}

#define SW_VEC_BATCH(R) template hipError_t launch_vec_batch_radius<R>(const StencilParams *, const int *, int, int, int, hipStream_t);
#define SW_VEC_RADIUS(T, R)                                                              \
    template hipError_t launch_vec_radius<T, R>(int, int, StencilParamsT<T> &, hipStream_t); \
    template int vec_resident_radius<T, R>(int, int);

}  // namespace sw
