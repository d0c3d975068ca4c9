// Scalar recurrences of preconditioned MINRES on the device.
#pragma once
#include "tmop_dev.hpp"
#include "vec.hpp"

namespace tmop {

// Sum of part[0..nb) by one wave (lane l adds l, l+64, ... in that order,
// 16 loads in flight, then a butterfly): the same bits in every workgroup.
__device__ inline double wave_sum_partials(const double *__restrict__ part, int nb)
{
    constexpr int RU = 16;
    const int l = threadIdx.x & 63;
    double s = 0.0;
    for (int k0 = 0; k0 < nb; k0 += 64 * RU) {
        double t[RU];
#pragma unroll
        for (int r = 0; r < RU; ++r) {
            const int k = k0 + r * 64 + l;
            t[r] = k < nb ? part[k] : 0.0;
        }
#pragma unroll
        for (int r = 0; r < RU; ++r) s += t[r];
    }
    return wave_sum(s);
}

// Sums of pa[0..na) (wave 0) and, when pb is given, pb[0..nb) (wave 1), to
// every thread of the workgroup after one barrier.  Called at most once per
// kernel, by every thread.
__device__ inline void sum_partials(const double *__restrict__ pa, int na,
                                    const double *__restrict__ pb, int nb, double &a, double &b)
{
    __shared__ double sh[2];
    const int w = threadIdx.x >> 6;
    if (w == 0) {
        const double t = wave_sum_partials(pa, na);
        if (threadIdx.x == 0) sh[0] = t;
    } else if (w == 1 && pb) {
        const double t = wave_sum_partials(pb, nb);
        if (threadIdx.x == 64) sh[1] = t;
    }
    __syncthreads();
    a = sh[0];
    b = pb ? sh[1] : 0.0;
}

// The state before the first iteration, from <b, M^{-1} b>.
__device__ inline MinresState mr_state0(double bb, double rtol)
{
    MinresState o;
    const double b1 = sqrt(fmax(bb, 0.0));
    o.tmp = bb;
    o.beta1 = b1;
    o.beta = b1;
    o.oldb = 0.0;
    o.alpha = 0.0;
    o.dbar = 0.0;
    o.eps = 0.0;
    o.oldeps = 0.0;
    o.phibar = b1;
    o.phi = 0.0;
    o.cs = -1.0;
    o.sn = 0.0;
    o.gamma = 1.0;
    o.delta = 0.0;
    o.rtol = rtol;
    o.its = 0;
    o.stop = (b1 > 0.0 && bb >= 0.0) ? 0x7fffffff : -1;
    o.indefinite_precond = bb < 0.0 ? 1 : 0;
    o.pad = 0;
    return o;
}

// Scalars of the update of iteration jm (Givens rotation of the Lanczos
// tridiagonal matrix) from the state before it, alpha_jm and beta_{jm+1}^2.
struct MrUpd {
    MinresState o;  // state after the update
    double ig, oldeps, delta, phi;
};

__device__ inline MrUpd mr_scalars(const MinresState &sin, int jm, double alpha, double bb)
{
    MrUpd u;
    const double beta = sqrt(fmax(bb, 0.0));
    u.oldeps = sin.eps;
    u.delta = sin.cs * sin.dbar + sin.sn * alpha;
    const double gbar = sin.sn * sin.dbar - sin.cs * alpha;
    const double eps = sin.sn * beta;
    const double dbar = -sin.cs * beta;
    const double gamma = fmax(hypot(gbar, beta), 2.2250738585072014e-308);
    const double cs = gbar / gamma, sn = beta / gamma;
    u.phi = cs * sin.phibar;
    const double phibar = sn * sin.phibar;
    u.ig = 1.0 / gamma;
    MinresState o = sin;
    o.tmp = bb;
    o.alpha = alpha;
    o.oldb = sin.beta;
    o.beta = beta;
    o.oldeps = u.oldeps;
    o.eps = eps;
    o.dbar = dbar;
    o.delta = u.delta;
    o.gamma = gamma;
    o.cs = cs;
    o.sn = sn;
    o.phi = u.phi;
    o.phibar = phibar;
    o.its = jm + 1;
    if (bb < 0.0) o.indefinite_precond = 1;
    if (phibar <= sin.rtol * sin.beta1 || beta == 0.0) o.stop = jm;
    u.o = o;
    return u;
}


// MrL2 at one node: loads first, then (after the sum of alpha) the new values,
// which every element of the node works out alike and its owner writes.
template <int D>
struct MrL2Node {
    double h[D], q[D], m[D];
    size_t at;
    __device__ __forceinline__ void load(const MrL2 &a, int nx, int node)
    {
        at = node;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            h[c] = a.hv[at + (size_t)c * nx];
            q[c] = a.r2[at + (size_t)c * nx];
            m[c] = a.minv ? a.minv[at + (size_t)c * nx] : 1.0;
        }
    }
    __device__ __forceinline__ void update(const MrL2 &a, int nx, double ab, bool own, double *z,
                                           double &s) const
    {
#pragma unroll
        for (int c = 0; c < D; ++c) {
            const double t = h[c] - ab * q[c];
            z[c] = a.minv ? m[c] * t : t;
            if (own) {
                a.hvo[at + (size_t)c * nx] = t;
                a.z[at + (size_t)c * nx] = z[c];
                s += t * z[c];
            }
        }
    }
};

// alpha / beta to every lane; false when the solve stopped before iteration j
__device__ __forceinline__ bool mr_l2_ratio(const MrL2 &a, double &ab)
{
    const int stop = a.st->stop;
    const double beta = a.st->beta;
    double alpha, unused;
    sum_partials(a.part1, a.nb1, nullptr, 0, alpha, unused);
    ab = alpha / beta;
    return a.j <= stop;
}

}  // namespace tmop
