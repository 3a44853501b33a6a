// Variable-density stencils on vector tiles (3D, single precision): the
// operators, modes, chunking and halo rules of k_stag and k_cent
// (stencil_vd.h), with a vector of CW columns per thread in place of rows of
// one column, as vec_tile (stencil_vec.h).
//
// A block owns TX rows x TY = LPR * CW columns, one thread per vector.  The
// scalar tiles issue a load, an LDS access and its address for every value, and
// the instruction stream, not memory, sets their pace.  With vectors the loads
// and LDS instructions per node drop to a quarter, and queue entries rotate
// through registers without moves.
// What bounds them: instructions.  Staggered, 592^3 SO8: 113 vector instructions
// per node keep the SIMDs 45% busy and LDS 31%, in phases that a block's barriers
// keep apart, 1.318 ms per step (scalar tiles 1.361; 20 bytes per node at the
// card's rate take 0.74); 240^3 104 against 122 us.  Centred, 280^3 SO8: 103 per
// node, in half of the cycles of SIMDs that hold two waves, LDS 34% (three fifths
// of that bank conflicts of the 32-column tile's rows), 4.4 TB/s with the halo
// re-reads; 132 against 156 us.
// CW is 4 up to R = 4 (staggered) and R = 6 (centred), else 2: three (two)
// queues of 2R vectors of 4 would not leave two waves per SIMD their registers
// (two columns per thread at R = 4, held to four waves, ran no faster: centred
// 136 us, staggered spilled, 288).
//
// The wavefield's mirror ghosts and the model's ghosts are read from the stored
// halo.  A vector that the grid ends in is cut where nothing lies beyond (no
// mirror side), and stored node by node, so that what lies past the grid's end
// stays as it was.
#pragma once

#include "stencil_vec.h"

namespace sw {

template <int CW>
struct VecF {
    typedef float type __attribute__((ext_vector_type(CW)));
};

template <int CW, int NT>
__device__ __forceinline__ typename VecF<CW>::type buf_ldw(__amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    if constexpr (CW == 4) return buf_ldv<float, NT>(r, voff, soff);
    else return __builtin_bit_cast(typename VecF<CW>::type, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, NT ? 2 : 0));
}

template <int CW, int NT>
__device__ __forceinline__ void buf_stw(typename VecF<CW>::type v, __amdgpu_buffer_rsrc_t r, int voff, int soff)
{
    if constexpr (CW == 4) {
        buf_stv<float, NT>(v, r, voff, soff);
    } else {
        using V = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V, v), r, voff, soff, NT ? 2 : 0);
    }
}

// What a thread of a vector tile knows of its place: the tile, its vector, the
// damping distances, which nodes a Dirichlet side holds, the offsets of plane
// reads and the cut of vectors that the grid ends in.
template <int CW, int TX, int LPR, int H>
struct VdPlace {
    static constexpr int kOut = 0x7ffffe00;
    static constexpr int TY = LPR * CW;
    static constexpr int NV = (H + CW - 1) / CW;            // vectors of y halo on each side
    using V = typename VecF<CW>::type;

    int x0, y0, x, y, zb, ze, ylim, ro, rr, e2[CW];
    unsigned held;
    bool ragged, holds, inner_xy;

    __device__ __forceinline__ VdPlace(const StencilParams &P)
    {
        const Geom &g = P.g;
        const int tid = threadIdx.x;
        int tx, ty, zc;
        tile_of(xcd_remap(blockIdx.x, gridDim.x), P.ntx, P.nty, P.xfast, tx, ty, zc);
        x0 = tx * TX;
        y0 = ty * TY;
        x = x0 + tid / LPR;
        y = y0 + (tid % LPR) * CW;
        zb = zc * P.zc;
        ze = min(zb + P.zc, g.Z);
        ylim = P.bcm[2][1] ? 0x7fffffff : g.Y;
        ragged = g.Y % CW != 0 && g.Y < y0 + TY + NV * CW;
        ro = x < g.X && y < g.Y ? (g.xy0 + x * g.py + y) * 4 : kOut;
        rr = wave_off(P, x, y);
        const int ex = max(0, max(g.lo[1] - x, x - (g.lo[1] + g.np[1] - 1)));
        held = 0;
#pragma unroll
        for (int c = 0; c < CW; ++c) {
            const int ey = max(0, max(g.lo[2] - (y + c), y + c - (g.lo[2] + g.np[2] - 1)));
            e2[c] = x < g.X && y + c < g.Y ? ex * ex + ey * ey : 0;      // keeps table reads in range
            if (axis_dirichlet(x, g.X, P.bcm[1][0], P.bcm[1][1]) || axis_dirichlet(y + c, g.Y, P.bcm[2][0], P.bcm[2][1]))
                held |= 1u << c;
        }
        holds = P.bcm[1][0] == 1 || P.bcm[1][1] == 1 || P.bcm[2][0] == 1 || P.bcm[2][1] == 1;
        inner_xy = x0 >= g.lo[1] && x0 + TX <= g.lo[1] + g.np[1] && y0 >= g.lo[2] && y0 + TY <= g.lo[2] + g.np[2];
    }
    // byte offset in a plane of the vector at (xx, yy), yy a multiple of CW:
    // wavefield reads (nothing off the grid but mirror ghosts) ...
    __device__ __forceinline__ static int wave_off(const StencilParams &P, int xx, int yy)
    {
        const Geom &g = P.g;
        const bool xok = axis_read(xx, g.X, P.bcm[1][0], P.bcm[1][1], P.gh);
        const bool yok = (yy >= 0 && yy < g.Y) || (yy < 0 && P.bcm[2][0] && yy + CW > -P.gh) ||
                         (yy >= g.Y && P.bcm[2][1] && yy < g.Y + P.gh);
        return xok && yok ? (g.xy0 + xx * g.py + yy) * 4 : kOut;
    }
    // ... and model reads (the whole stored halo of hs nodes; what lies beyond
    // only feeds nodes off the grid)
    __device__ __forceinline__ static int model_off(const StencilParams &P, int xx, int yy, int hs)
    {
        const Geom &g = P.g;
        const bool ok = xx >= -hs && xx < g.X + hs && yy + CW > -hs && yy < g.Y + hs;
        return ok ? (g.xy0 + xx * g.py + yy) * 4 : kOut;
    }
    __device__ __forceinline__ V clip(V v, int yy) const
    {
#pragma unroll
        for (int c = 0; c < CW; ++c) v[c] = yy + c < ylim ? v[c] : 0.0f;
        return v;
    }
    template <int NT>
    __device__ __forceinline__ void put(const Geom &g, V v, __amdgpu_buffer_rsrc_t r, int so) const
    {
        if (ragged && y < g.Y && y + CW > g.Y) {
#pragma unroll
            for (int c = 0; c < CW; ++c)
                if (y + c < g.Y) buf_st<NT>(v[c], r, ro + 4 * c, so);
        } else {
            buf_stw<CW, NT>(v, r, ro, so);
        }
    }
};

template <int R, int TX, int TY, int MODE>
__global__ void __launch_bounds__((TX * TY / vd_columns(1, R)), 2) k_stag_vec(StencilParams P)
{
#pragma clang fp contract(off)
    constexpr int CW = vd_columns(1, R), LPR = TY / CW, NT = 1;
    constexpr int H = 2 * R - 1;                       // node halo of the face fluxes
    using PL = VdPlace<CW, TX, LPR, H>;
    using V = typename VecF<CW>::type;
    using V2 = typename VecF<2>::type;
    using V4 = typename VecF<4>::type;
    constexpr int NTH = TX * LPR;
    constexpr int NV = PL::NV;
    constexpr int Q = 2 * R + 2;
    constexpr int R4 = (R + 3) / 4 * 4;
    constexpr int M = R4 + (R + 2) / 4 * 4;            // LDS columns left of the tile
    static_assert(M >= NV * CW && M % 4 == 0, "the margin holds the halo");
    // y faces: face m lies between LDS columns m and m + 1; runs of 4 from M - R4
    constexpr int F0 = M - R4;
    constexpr int NRY = (TY + R4 + R - 1 + 3) / 4;
    constexpr int L0 = (R + 2) / 4 * 4;                // a run reads columns m - L0 .. (NVY of them)
    constexpr int NVY = (L0 + 4 + R + 3) / 4 * 4;
    constexpr int LYP0 = F0 + 4 * (NRY - 1) - L0 + NVY;
    constexpr int LYP = LYP0 > M + TY + NV * CW ? LYP0 : M + TY + NV * CW;
    static_assert(LYP % 2 == 0, "rows keep the alignment of vectors");
    constexpr int FYP = NRY * 4;
    // x faces: face t lies between rows t + R - 1 and t + R (row H + i is row i
    // of the tile); runs of MX faces of two columns
    constexpr int FX = TX + 2 * R - 1;
    constexpr int PAIRS = TY / 2;
    constexpr int NRX0 = NTH / PAIRS, NRX1 = (FX + 2) / 3;
    constexpr int NRX = NRX0 < NRX1 ? NRX0 : NRX1;
    constexpr int MX = (FX + NRX - 1) / NRX;
    constexpr int NIX = NRX * PAIRS, NI = NIX + TX * NRY;
    constexpr int NIT = (NI + NTH - 1) / NTH;
    constexpr int LX = TX + 2 * H;
    constexpr int ROWS = NRX * MX + 2 * R - 1 > LX ? NRX * MX + 2 * R - 1 : LX;
    constexpr int LYA = (LYP + 3) / 4 * 4;
    __shared__ __align__(16) float sp[ROWS][LYA];
    __shared__ __align__(16) float sb[ROWS][LYA];
    __shared__ __align__(16) float sfx[NRX * MX][TY];
    __shared__ __align__(16) float sfy[TX][FYP];
    constexpr int NXH = 2 * H * LPR;                   // halo vectors: rows above and below
    constexpr int NH = NXH + TX * 2 * NV;              // and beside the tile's rows
    constexpr int NHT = (NH + NTH - 1) / NTH;
    constexpr bool kImage = (MODE == MODE_IMAGE || MODE == MODE_IMAGE2);

    const Geom &g = P.g;
    const PL at(P);
    const int tid = threadIdx.x, row = tid / LPR, col = (tid % LPR) * CW;
    const int zb = at.zb, ze = at.ze;
    const int64_t sz = int64_t(g.px) * g.py;
    const int zw = zb - H, zt = ze + H;
    const int pb = int(sz) * 4;
    const uint32_t wbytes = uint32_t(zt - zw) * uint32_t(pb);
    const int64_t w0 = g.base + int64_t(zw) * sz;
    const auto rc = buf_res(P.cur + w0, wbytes);
    const auto rn = buf_res(P.nxt + w0, wbytes);
    const auto rb = buf_res(P.aux + w0, wbytes);
    const auto rk = buf_res(P.K + w0, wbytes);
    const auto rd = buf_res(P.damp, uint32_t(P.ndamp) * 8u);
    __amdgpu_buffer_rsrc_t rs = rk, ru = rk, rg = rk, rs2 = rk;
    if constexpr (MODE != MODE_FWD) rs = buf_res(P.store + w0, wbytes);
    if constexpr (MODE == MODE_STORE) ru = buf_res(P.ustore + w0, wbytes);
    if constexpr (kImage) rg = buf_res(P.grad + w0, wbytes);
    if constexpr (MODE == MODE_IMAGE2) rs2 = buf_res(P.store2 + w0, wbytes);
    auto soff = [&](int z) -> int { return (z - zw) * pb; };
    const int rm = PL::model_off(P, at.x, at.y, 2 * R);

    int hp[NHT], hm[NHT], hl[NHT], hyy[NHT];
#pragma unroll
    for (int s = 0; s < NHT; ++s) {
        const int e = tid + s * NTH;
        int hr, hc;
        if (e < NXH) {
            const int k = e / LPR;
            hr = k < H ? k : TX + k;
            hc = M + (e % LPR) * CW;
        } else {
            const int e3 = e - NXH, k = e3 % (2 * NV);
            hr = H + e3 / (2 * NV);
            hc = M + (k < NV ? (k - NV) * CW : TY + (k - NV) * CW);
        }
        const bool ok = e < NH;
        hyy[s] = at.y0 - M + hc;
        hp[s] = ok ? PL::wave_off(P, at.x0 - H + hr, hyy[s]) : PL::kOut;
        hm[s] = ok ? PL::model_off(P, at.x0 - H + hr, hyy[s], 2 * R) : PL::kOut;
        hl[s] = ok ? hr * LYA + hc : 0;
    }

    // queues (unrolled step u): pq[(u + k) % Q] = p(z + k) and bq[..] = b(z + k), the last of
    // them (k = 2R) in flight; fq[(u + k) % Q] = z flux at face (z - R + k) + 1/2
    V pq[Q], bq[Q], fq[Q];
    auto ld_p = [&](int z) -> V {
        if (!axis_read(z, g.Z, P.bcm[0][0], P.bcm[0][1], P.gh)) return V{};
        return buf_ldw<CW, 0>(rc, at.rr, soff(z));
    };
    const int zs = zb - H;
#pragma unroll
    for (int k = 0; k < 2 * R; ++k) {
        pq[k] = ld_p(zs + k);
        bq[k] = buf_ldw<CW, 0>(rb, rm, soff(zs + k));
    }
#pragma unroll
    for (int k = 0; k < Q; ++k) fq[k] = V{};

    struct Slot {
        V p, k, d, gr, d2;                             // (unused ones take no registers)
    };
    V hvp[NHT], hvb[NHT];
    auto load_halo = [&](int z) {
        const int so = soff(z);
#pragma unroll
        for (int s = 0; s < NHT; ++s) {
            hvp[s] = buf_ldw<CW, 0>(rc, hp[s], so);
            hvb[s] = buf_ldw<CW, 0>(rb, hm[s], so);
        }
    };
    auto load = [&](int z, Slot &L) {
        const int so = soff(z);
        L.p = buf_ldw<CW, NT>(rn, at.ro, so);
        L.k = buf_ldw<CW, NT>(rk, at.ro, so);
        if constexpr (kImage) {
            L.d = buf_ldw<CW, NT>(rs, at.ro, so);
            L.gr = buf_ldw<CW, NT>(rg, at.ro, so);
        }
        if constexpr (MODE == MODE_IMAGE2) L.d2 = buf_ldw<CW, NT>(rs2, at.ro, so);
    };
    V a, b;
#pragma unroll
    for (int c = 0; c < CW; ++c) a[c] = b[c] = 1.0f;
    int ez0 = at.inner_xy ? 0 : -1;                    // layer distance along z that (a, b) hold for
    for (int zz = zs; zz < ze; zz += Q) {
#pragma unroll
        for (int u = 0; u < Q; ++u) {
            const int z = zz + u;
            if (z < ze) {
                Slot W;
                if (z >= zb) load(z, W);
                if (z + 1 < ze) {
                    pq[(u + 2 * R) % Q] = ld_p(z + 2 * R);
                    bq[(u + 2 * R) % Q] = buf_ldw<CW, 0>(rb, rm, soff(z + 2 * R));
                }
                // z flux at face (z + R - 1) + 1/2
                V dp{}, bf{};
#pragma unroll
                for (int l = 1; l <= R; ++l) {
                    const V dd = pq[(u + R - 1 + l) % Q] - pq[(u + R - l) % Q], bb = bq[(u + R - 1 + l) % Q] + bq[(u + R - l) % Q];
#pragma unroll
                    for (int c = 0; c < CW; ++c) {
                        dp[c] = fmaf(P.sz[l], dd[c], dp[c]);
                        bf[c] = fmaf(P.mj[l], bb[c], bf[c]);
                    }
                }
                fq[(u + 2 * R - 1) % Q] = bf * dp;

                if (z >= zb) {
                    // phase one: stage p and b of plane z with an H-node halo
                    const int ez = max(0, max(g.lo[0] - z, z - (g.lo[0] + g.np[0] - 1)));
                    if (ez != ez0) {
                        ez0 = ez;
#pragma unroll
                        for (int c = 0; c < CW; ++c) {
                            const float2 ab = buf_ld2(rd, (ez * ez + at.e2[c]) * 8);
                            a[c] = ab.x;
                            b[c] = ab.y;
                        }
                    }
                    V cc = pq[u % Q];
                    if (at.ragged) cc = at.clip(cc, at.y);
                    *reinterpret_cast<V *>(&sp[H + row][M + col]) = cc;
                    *reinterpret_cast<V *>(&sb[H + row][M + col]) = bq[u % Q];
#pragma unroll
                    for (int s = 0; s < NHT; ++s) {
                        if (s * NTH + tid >= NH) continue;
                        V h = hvp[s];
                        if (at.ragged) h = at.clip(h, hyy[s]);
                        *reinterpret_cast<V *>(&sp[0][0] + hl[s]) = h;
                        *reinterpret_cast<V *>(&sb[0][0] + hl[s]) = hvb[s];
                    }
                    if (z + 1 < ze) load_halo(z + 1);
                    __syncthreads();

                    // phase two: every x and y face flux of the tile, once, by runs
#pragma unroll
                    for (int s = 0; s < NIT; ++s) {
                        const int e = tid + s * NTH;
                        if (e < NIX) {
                            const int c = e % PAIRS * 2, t0 = e / PAIRS * MX;
                            V2 vp[MX + 2 * R - 1], vb[MX + 2 * R - 1];
#pragma unroll
                            for (int j = 0; j < MX + 2 * R - 1; ++j) {
                                vp[j] = *reinterpret_cast<const V2 *>(&sp[t0 + j][M + c]);
                                vb[j] = *reinterpret_cast<const V2 *>(&sb[t0 + j][M + c]);
                            }
#pragma unroll
                            for (int f = 0; f < MX; ++f) {
                                V2 dx{}, bx{};
#pragma unroll
                                for (int l = 1; l <= R; ++l) {
                                    const V2 dd = vp[f + R - 1 + l] - vp[f + R - l], bb = vb[f + R - 1 + l] + vb[f + R - l];
#pragma unroll
                                    for (int k = 0; k < 2; ++k) {
                                        dx[k] = fmaf(P.sx[l], dd[k], dx[k]);
                                        bx[k] = fmaf(P.mj[l], bb[k], bx[k]);
                                    }
                                }
                                *reinterpret_cast<V2 *>(&sfx[t0 + f][c]) = bx * dx;
                            }
                        } else if (e < NI) {
                            const int q = e - NIX, r = q / NRY, c0 = q % NRY * 4;
                            float vp[NVY], vb[NVY];
#pragma unroll
                            for (int j = 0; j < NVY / 4; ++j) {
                                const V4 p4 = *reinterpret_cast<const V4 *>(&sp[H + r][F0 - L0 + c0 + 4 * j]);
                                const V4 b4 = *reinterpret_cast<const V4 *>(&sb[H + r][F0 - L0 + c0 + 4 * j]);
#pragma unroll
                                for (int k = 0; k < 4; ++k) {
                                    vp[4 * j + k] = p4[k];
                                    vb[4 * j + k] = b4[k];
                                }
                            }
                            V4 out;
#pragma unroll
                            for (int f = 0; f < 4; ++f) {
                                float dy = 0.0f, by = 0.0f;
#pragma unroll
                                for (int l = 1; l <= R; ++l) {
                                    dy = fmaf(P.sy[l], vp[L0 + f + l] - vp[L0 + f + 1 - l], dy);
                                    by = fmaf(P.mj[l], vb[L0 + f + l] + vb[L0 + f + 1 - l], by);
                                }
                                out[f] = by * dy;
                            }
                            *reinterpret_cast<V4 *>(&sfy[r][c0]) = out;
                        }
                    }
                    __syncthreads();

                    // phase three: divergence and update
                    const int so = soff(z);
                    V dzs{}, dxs{}, dys{};
#pragma unroll
                    for (int j = 1; j <= R; ++j) {
                        const V dz = fq[(u + R + j - 1) % Q] - fq[(u + R - j) % Q];
                        const V dx = *reinterpret_cast<const V *>(&sfx[row + R + j - 1][col]) -
                                     *reinterpret_cast<const V *>(&sfx[row + R - j][col]);
#pragma unroll
                        for (int c = 0; c < CW; ++c) {
                            dzs[c] = fmaf(P.sz[j], dz[c], dzs[c]);
                            dxs[c] = fmaf(P.sx[j], dx[c], dxs[c]);
                        }
                    }
                    // face m of node column n (LDS): n - R .. n + R - 1; sfy column m - F0
                    constexpr int W0 = (R4 - R) / CW * CW;            // first of the aligned vectors
                    constexpr int NW = ((R4 + R - 1 + CW - 1) - W0 + CW) / CW;
                    float w[NW * CW];
#pragma unroll
                    for (int k = 0; k < NW; ++k) {
                        const V t = *reinterpret_cast<const V *>(&sfy[row][col + W0 + k * CW]);
#pragma unroll
                        for (int c = 0; c < CW; ++c) w[k * CW + c] = t[c];
                    }
#pragma unroll
                    for (int j = 1; j <= R; ++j)
#pragma unroll
                        for (int c = 0; c < CW; ++c)
                            dys[c] = fmaf(P.sy[j], w[R4 - W0 + c + j - 1] - w[R4 - W0 + c - j], dys[c]);
                    const V lap = dzs + dxs + dys;
                    V out;
#pragma unroll
                    for (int c = 0; c < CW; ++c) out[c] = leapfrog(a[c], b[c], W.k[c], lap[c], cc[c], W.p[c]);
                    const bool plane = axis_dirichlet(z, g.Z, P.bcm[0][0], P.bcm[0][1]);
                    if (at.holds || plane) {
#pragma unroll
                        for (int c = 0; c < CW; ++c) out[c] = plane || (at.held >> c & 1) ? 0.0f : out[c];
                    }
                    at.template put<NT>(g, out, rn, so);
                    if constexpr (MODE == MODE_STORE) {
                        at.template put<NT>(g, W.k * lap, rs, so);
                        at.template put<NT>(g, cc, ru, so);
                    }
                    if constexpr (kImage) {
                        V s;
#pragma unroll
                        for (int c = 0; c < CW; ++c) {
                            const float k2 = W.k[c] * W.k[c];
                            if constexpr (MODE == MODE_IMAGE) s[c] = fmaf(cc[c], W.d[c] / k2, W.gr[c]);
                            else s[c] = fmaf(cc[c], W.d[c] / k2, fmaf(W.p[c], W.d2[c] / k2, W.gr[c]));
                        }
                        at.template put<NT>(g, s, rg, so);
                    }
                } else if (z + 1 == zb) {
                    load_halo(zb);
                }
            }
        }
    }
}

template <int R, int TX, int TY>
__global__ void __launch_bounds__((TX * TY / vd_columns(2, R)), 2) k_cent_vec(StencilParams P)
{
#pragma clang fp contract(off)
    constexpr int CW = vd_columns(2, R), LPR = TY / CW, NT = 1;
    using PL = VdPlace<CW, TX, LPR, R>;
    using V = typename VecF<CW>::type;
    constexpr int NTH = TX * LPR;
    constexpr int NV = PL::NV, PC = NV * CW, LYP = TY + 2 * PC, LXR = TX + 2 * R;
    constexpr int Q = 2 * R + 2;
    constexpr int NXH = 2 * R * LPR, NH = NXH + TX * 2 * NV, NHT = (NH + NTH - 1) / NTH;
    __shared__ __align__(16) float lds[2][2][LXR * LYP];       // [plane parity][p, rho]

    const Geom &g = P.g;
    const PL at(P);
    const int tid = threadIdx.x, row = tid / LPR, col = (tid % LPR) * CW;
    const int zb = at.zb, ze = at.ze;
    const int64_t sz = int64_t(g.px) * g.py;
    const int zw = zb - R, zt = ze + R;
    const int pb = int(sz) * 4;
    const uint32_t wbytes = uint32_t(zt - zw) * uint32_t(pb);
    const int64_t w0 = g.base + int64_t(zw) * sz;
    const auto rc = buf_res(P.cur + w0, wbytes);
    const auto rn = buf_res(P.nxt + w0, wbytes);
    const auto rb = buf_res(P.aux + w0, wbytes);
    const auto rk = buf_res(P.K + w0, wbytes);
    const auto rd = buf_res(P.damp, uint32_t(P.ndamp) * 8u);
    auto soff = [&](int z) -> int { return (z - zw) * pb; };
    const int rm = PL::model_off(P, at.x, at.y, R);

    int hp[NHT], hm[NHT], hl[NHT], hyy[NHT];
#pragma unroll
    for (int s = 0; s < NHT; ++s) {
        const int e = tid + s * NTH;
        int hr, hc;
        if (e < NXH) {
            const int k = e / LPR;
            hr = k < R ? k : TX + k;
            hc = PC + (e % LPR) * CW;
        } else {
            const int e3 = e - NXH, k = e3 % (2 * NV);
            hr = R + e3 / (2 * NV);
            hc = k < NV ? k * CW : TY + k * CW;
        }
        const bool ok = e < NH;
        hyy[s] = at.y0 - PC + hc;
        hp[s] = ok ? PL::wave_off(P, at.x0 - R + hr, hyy[s]) : PL::kOut;
        hm[s] = ok ? PL::model_off(P, at.x0 - R + hr, hyy[s], R) : PL::kOut;
        hl[s] = ok ? hr * LYP + hc : 0;
    }

    V q[Q], qr[Q];                                     // [(u + k) % Q] = p, rho at plane z - R + k in unrolled step u
    auto ld_p = [&](int z) -> V {
        if (!axis_read(z, g.Z, P.bcm[0][0], P.bcm[0][1], P.gh)) return V{};
        return buf_ldw<CW, 0>(rc, at.rr, soff(z));
    };
#pragma unroll
    for (int k = 0; k <= 2 * R; ++k) {
        q[k] = ld_p(zb - R + k);
        qr[k] = buf_ldw<CW, 0>(rb, rm, soff(zb - R + k));
    }
    struct Slot {
        V p, k;
    };
    Slot S[2];
    V hvp[NHT], hvr[NHT];
    auto load_halo = [&](int z) {
        const int so = soff(z);
#pragma unroll
        for (int s = 0; s < NHT; ++s) {
            hvp[s] = buf_ldw<CW, 0>(rc, hp[s], so);
            hvr[s] = buf_ldw<CW, 0>(rb, hm[s], so);
        }
    };
    auto load = [&](int z, Slot &L) {
        L.p = buf_ldw<CW, NT>(rn, at.ro, soff(z));
        L.k = buf_ldw<CW, NT>(rk, at.ro, soff(z));
    };
    load_halo(zb);
    load(zb, S[0]);
    V a, b;
#pragma unroll
    for (int c = 0; c < CW; ++c) a[c] = b[c] = 1.0f;
    int ez0 = at.inner_xy ? 0 : -1;
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
                        const float2 ab = buf_ld2(rd, (ez * ez + at.e2[c]) * 8);
                        a[c] = ab.x;
                        b[c] = ab.y;
                    }
                }
                float *L = lds[u % 2][0], *U = lds[u % 2][1];
                V cc = q[(u + R) % Q];
                if (at.ragged) cc = at.clip(cc, at.y);
                *reinterpret_cast<V *>(L + own) = cc;
                *reinterpret_cast<V *>(U + own) = qr[(u + R) % Q];
#pragma unroll
                for (int s = 0; s < NHT; ++s) {
                    if (s * NTH + tid >= NH) continue;
                    V h = hvp[s];
                    if (at.ragged) h = at.clip(h, hyy[s]);
                    *reinterpret_cast<V *>(L + hl[s]) = h;
                    *reinterpret_cast<V *>(U + hl[s]) = hvr[s];
                }
                if (z + 1 < ze) {
                    load_halo(z + 1);
                    q[(u + 2 * R + 1) % Q] = ld_p(z + 1 + R);
                    qr[(u + 2 * R + 1) % Q] = buf_ldw<CW, 0>(rb, rm, soff(z + 1 + R));
                    load(z + 1, S[(u + 1) % 2]);
                }
                __syncthreads();

                V lap = P.c0 * cc, dpz{}, drz{}, dpx{}, drx{}, dpy{}, dry{};
#pragma unroll
                for (int j = 1; j <= R; ++j) {
                    const V hi = q[(u + R + j) % Q], lo = q[(u + R - j) % Q];
                    const V t = hi + lo, d = hi - lo, dr = qr[(u + R + j) % Q] - qr[(u + R - j) % Q];
#pragma unroll
                    for (int c = 0; c < CW; ++c) {
                        lap[c] = fmaf(P.cz[j], t[c], lap[c]);
                        dpz[c] = fmaf(P.sz[j], d[c], dpz[c]);
                        drz[c] = fmaf(P.sz[j], dr[c], drz[c]);
                    }
                }
#pragma unroll
                for (int j = 1; j <= R; ++j) {
                    const V hi = *reinterpret_cast<const V *>(L + own + j * LYP);
                    const V lo = *reinterpret_cast<const V *>(L + own - j * LYP);
                    const V t = hi + lo, d = hi - lo;
                    const V dr = *reinterpret_cast<const V *>(U + own + j * LYP) -
                                 *reinterpret_cast<const V *>(U + own - j * LYP);
#pragma unroll
                    for (int c = 0; c < CW; ++c) {
                        lap[c] = fmaf(P.cx[j], t[c], lap[c]);
                        dpx[c] = fmaf(P.sx[j], d[c], dpx[c]);
                        drx[c] = fmaf(P.sx[j], dr[c], drx[c]);
                    }
                }
                float w[(2 * NV + 1) * CW], v[(2 * NV + 1) * CW];
#pragma unroll
                for (int k = 0; k < 2 * NV + 1; ++k) {
                    const V t = k == NV ? cc : *reinterpret_cast<const V *>(L + own + (k - NV) * CW);
                    const V r = k == NV ? qr[(u + R) % Q] : *reinterpret_cast<const V *>(U + own + (k - NV) * CW);
#pragma unroll
                    for (int c = 0; c < CW; ++c) {
                        w[k * CW + c] = t[c];
                        v[k * CW + c] = r[c];
                    }
                }
#pragma unroll
                for (int j = 1; j <= R; ++j)
#pragma unroll
                    for (int c = 0; c < CW; ++c) {
                        lap[c] = fmaf(P.cy[j], w[PC + c + j] + w[PC + c - j], lap[c]);
                        dpy[c] = fmaf(P.sy[j], w[PC + c + j] - w[PC + c - j], dpy[c]);
                        dry[c] = fmaf(P.sy[j], v[PC + c + j] - v[PC + c - j], dry[c]);
                    }
                V out;
#pragma unroll
                for (int c = 0; c < CW; ++c) {
                    const float grad = fmaf(drz[c], dpz[c], fmaf(drx[c], dpx[c], dry[c] * dpy[c]));
                    const float Lp = lap[c] - grad / qr[(u + R) % Q][c];
                    out[c] = leapfrog(a[c], b[c], W.k[c], Lp, cc[c], W.p[c]);
                }
                const bool plane = axis_dirichlet(z, g.Z, P.bcm[0][0], P.bcm[0][1]);
                if (at.holds || plane) {
#pragma unroll
                    for (int c = 0; c < CW; ++c) out[c] = plane || (at.held >> c & 1) ? 0.0f : out[c];
                }
                at.template put<NT>(g, out, rn, soff(z));
            }
        }
    }
}

template <int SCHEME, int R, int MODE, int I>
hipError_t launch_vd_tile(StencilParams &P, hipStream_t s)
{
    constexpr VdTile t = kVdTiles[I];
    constexpr int threads = t.tx * t.ty / vd_columns(SCHEME, R);
    if constexpr (threads <= kVdThreads) {
        const dim3 grid(P.ntx * P.nty * P.nzc), block(threads);
        if constexpr (SCHEME == 1) hipLaunchKernelGGL((k_stag_vec<R, t.tx, t.ty, MODE>), grid, block, 0, s, P);
        else hipLaunchKernelGGL((k_cent_vec<R, t.tx, t.ty>), grid, block, 0, s, P);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

template <int SCHEME, int R, int MODE>
hipError_t launch_vd_mode(int tile, StencilParams &P, hipStream_t s)
{
    switch (tile) {
    case 0: return launch_vd_tile<SCHEME, R, MODE, 0>(P, s);
    case 1: return launch_vd_tile<SCHEME, R, MODE, 1>(P, s);
    case 2: return launch_vd_tile<SCHEME, R, MODE, 2>(P, s);
    case 3: return launch_vd_tile<SCHEME, R, MODE, 3>(P, s);
    case 4: return launch_vd_tile<SCHEME, R, MODE, 4>(P, s);
    default: return hipErrorInvalidValue;
    }
}

template <int R>
hipError_t launch_vdvec_radius(int scheme, int tile, int mode, StencilParams &P, hipStream_t s)
{
    if (scheme != 1) return mode == MODE_FWD ? launch_vd_mode<2, R, MODE_FWD>(tile, P, s) : hipErrorInvalidValue;
    if constexpr (R >= kStagRadii[0] && R <= kStagRadii[1]) {
        if (mode == MODE_STORE) return launch_vd_mode<1, R, MODE_STORE>(tile, P, s);
        if (mode == MODE_IMAGE) return launch_vd_mode<1, R, MODE_IMAGE>(tile, P, s);
        if (mode == MODE_IMAGE2) return launch_vd_mode<1, R, MODE_IMAGE2>(tile, P, s);
        return launch_vd_mode<1, R, MODE_FWD>(tile, P, s);
    }
    return hipErrorInvalidValue;
}

template <int R, int I>
int vdvec_resident_tile()
{
    constexpr VdTile t = kVdTiles[I];
    constexpr int threads = t.tx * t.ty / vd_columns(2, R);
    if constexpr (threads <= kVdThreads) return blocks_per_cu<k_cent_vec<R, t.tx, t.ty>>(threads);
    return 0;
}

template <int R>
int vdvec_resident_radius(int scheme, int tile)
{
    if (scheme != 2) return 0;
    switch (tile) {
    case 0: return vdvec_resident_tile<R, 0>();
    case 1: return vdvec_resident_tile<R, 1>();
    case 2: return vdvec_resident_tile<R, 2>();
    case 3: return vdvec_resident_tile<R, 3>();
    case 4: return vdvec_resident_tile<R, 4>();
    default: return 0;
    }
}

#define SW_VDVEC_RADIUS(R)                                                                  \
    template hipError_t launch_vdvec_radius<R>(int, int, int, StencilParams &, hipStream_t); \
    template int vdvec_resident_radius<R>(int, int);

}  // namespace sw
