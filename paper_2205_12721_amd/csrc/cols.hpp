// What the column forms of the quad and the hex kernels share.
#pragma once
#include "tmop_dev.hpp"

namespace tmop {

// The last axis' table rows of one point of the column (uniform over the lanes,
// so in scalar registers).  A loop over the column's points takes each row
// from the load it issued one point earlier: with the load at the point
// itself, every point began by waiting for the scalar cache.
template <int NI, typename CT>
struct ColRow {
    CT b[NI], g[NI];
    double w;
    __device__ __forceinline__ void load(const Tab &tb, int q3)
    {
#pragma unroll
        for (int k = 0; k < NI; ++k) {
            b[k] = tabB<CT>(tb, q3 * NI + k);
            g[k] = tabG<CT>(tb, q3 * NI + k);
        }
        w = tb.t->w[q3];
    }
};

// Sum over the workgroup of NW waves (thread 0).
template <int NW>
__device__ __forceinline__ void col_reduce3(double &s, double &m, double &b, double *red)
{
    s = wave_sum(s);
    m = wave_min(m);
    b = wave_sum(b);
    if constexpr (NW > 1) {
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        if (lane == 0) {
            red[w] = s;
            red[NW + w] = m;
            red[2 * NW + w] = b;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int k = 1; k < NW; ++k) {
                s += red[k];
                m = fmin(m, red[NW + k]);
                b += red[2 * NW + k];
            }
        }
    }
}

}  // namespace tmop
