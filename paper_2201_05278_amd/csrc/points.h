// Source injection of one step and recording of the step before in one launch.
// A step's level is final once its sources are in, and the next stencil launch
// only reads it, so its receivers need not be recorded before that launch: they
// go with the next step's injection, which writes the other buffer.  On small
// grids the two point launches were half of a step (83 x 97 x 101 and its layer,
// SO4: 4.3 and 4.9 us of 19.2 us per step; 16.8 with one); what bounds them is their own chain of
// loads (entry, node, value) and the gap between dependent launches, so that
// one launch for both costs what the longer one did.
#pragma once

#include "device.h"

namespace sw {

// Sum over groups of G consecutive lanes (a power of two), as the butterfly of
// the single kernels.
template <typename T>
__device__ __forceinline__ T group_total(T v, int G)
{
    for (int off = G / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, G);
    return v;
}

template <typename T, typename Table>
__device__ __forceinline__ void inject_group(const Table &t, int gid, int G, const T *amp, T *field)
{
    const int u = gid / G, sub = gid % G;
    T sa = T(0);
    if (u < t.nuniq)
        for (int k = t.uptr[u] + sub; k < t.uptr[u + 1]; k += G) {
            const int e = t.uent[k];
            if constexpr (sizeof(T) == 4) sa = fmaf(t.coef_a[e], amp[t.pid[e]], sa);
            else sa = fma(t.coef_a[e], amp[t.pid[e]], sa);
        }
    sa = group_total(sa, G);
    if (u < t.nuniq && sub == 0) field[t.unode[u]] += sa;
}

template <typename T, typename Table>
__device__ __forceinline__ void record_group(const Table &t, int gid, int G, const T *field, T *out)
{
    const int pt = gid / G, sub = gid % G;
    T acc = T(0);
    if (pt < t.count)
        for (int e = t.ptr[pt] + sub; e < t.ptr[pt + 1]; e += G) acc += t.wscaled[e] * field[t.node[e]];
    acc = group_total(acc, G);
    if (pt < t.count && sub == 0) out[pt] = acc;
}

// Blocks 0 .. nsb - 1: injection into `nxt`; the others: recording of `cur`.
template <typename T, typename Table>
__global__ void __launch_bounds__(256) k_points(Table src, int nsb, int gs, const T *amp, T *nxt, Table rec, int gr,
                                                const T *cur, T *out)
{
    const int b = blockIdx.x;
    if (b < nsb) inject_group<T>(src, b * 256 + threadIdx.x, gs, amp, nxt);
    else record_group<T>(rec, (b - nsb) * 256 + threadIdx.x, gr, cur, out);
}

inline int point_group(int max_entries)
{
    int g = 1;
    while (g < max_entries && g < 64) g <<= 1;
    return g;
}

inline int point_blocks(int n, int G) { return int((int64_t(n) * G + 255) / 256); }

template <typename T, typename Table>
hipError_t launch_points_t(const Table &src, const T *amp, T *nxt, const Table &rec, const T *cur, T *out, hipStream_t s)
{
    const int gs = point_group(src.max_per_node), gr = point_group(rec.max_per_point);
    const int nsb = point_blocks(src.nuniq, gs), nrb = cur ? point_blocks(rec.count, gr) : 0;
    if (nsb + nrb == 0) return hipSuccess;
    hipLaunchKernelGGL((k_points<T, Table>), dim3(nsb + nrb), dim3(256), 0, s, src, nsb, gs, amp, nxt, rec, gr, cur, out);
    return hipGetLastError();
}

}  // namespace sw
