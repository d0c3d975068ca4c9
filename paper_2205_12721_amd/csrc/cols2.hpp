// Quad energy and gradient in column form: a lane keeps one column of points
// (q1 fixed, q2 = 0 .. n_q-1).
//
// In the pencil form (kernels2d.hpp) every value passes through LDS between
// the sweeps and a point's four J entries come from it and go back to it.
// Here a lane applies axis 1 to its element's nodes, read from LDS, with its
// own row of the tables, and then has all that its n_q points need: 4 n_i
// values in registers.  Each point is one step of a loop whose table rows are
// scalars; its share of the gradient goes to 4 n_i sums in registers, which
// pass through LDS once for the transposed axis 1.
#pragma once
#include "cols.hpp"
#include "kernels2d.hpp"

namespace tmop {

template <int P_, int NQ_, int WL_>
struct C2 {
    static constexpr int P = P_, NQ = NQ_, WL = WL_;
    static constexpr int NI = P + 1, NP = NI * NI, NW = WL / 64;
    static constexpr int EPB = WL / NQ;  // elements per workgroup
    static constexpr int LN = EPB * NQ;  // lanes with a column
    static constexpr int ES = 2 * NP + 1;  // an element's nodes in LDS (odd: no bank conflicts)
    static constexpr int PL = (EPB * NP + WL - 1) / WL;  // nodes per lane in the gather
};

// GRAD: the gradient's E-vector; EN: the energy partials (as b2_gradient).
template <class C, bool GRAD, bool EN>
__device__ __forceinline__ void c2_energy(const Geom &g, const Tab &tb, const Target &tg,
                                          const double *__restrict__ x, double *__restrict__ gE,
                                          double *__restrict__ part, int e0, int nel)
{
    constexpr int P = C::P, NQ = C::NQ, NI = C::NI, NP = C::NP;
    __shared__ union {
        double X[C::EPB * C::ES];
        double U[GRAD ? 4 * NI * C::LN : 1];
    } L;
    __shared__ double red[3 * C::NW];
    const int tid = threadIdx.x;
    // lanes without a column (past the last element) work on the first one's
    const int el = tid / NQ, q1 = tid % NQ;
    const bool act = tid < C::LN && el < nel;
    double b1[NI], g1[NI];
#pragma unroll
    for (int k = 0; k < NI; ++k) {
        b1[k] = tb.t->B[q1 * NI + k];
        g1[k] = tb.t->G[q1 * NI + k];
    }
    const double w1 = tb.t->w[q1];
    {
        double v[C::PL][2];
#pragma unroll
        for (int k = 0; k < C::PL; ++k) {
            const int idx = tid + k * C::WL;
            v[k][0] = v[k][1] = 0.0;
            if (idx < nel * NP) {
                const int i = idx % NP;
                int gx, gy;
                const int node = node2<P>(g, e0 + idx / NP, i % NI, i / NI, gx, gy);
                v[k][0] = x[node];
                v[k][1] = x[(size_t)g.nx + node];
            }
        }
#pragma unroll
        for (int k = 0; k < C::PL; ++k) {
            const int idx = tid + k * C::WL;
            if (idx < nel * NP) {
                double *o = L.X + (idx / NP) * C::ES + idx % NP;
                o[0] = v[k][0];
                o[NP] = v[k][1];
            }
        }
    }
    __syncthreads();
    // axis 1: B and G of the column's q1
    double xb[2][NI], xg[2][NI];
    const double *X = L.X + (act ? el : 0) * C::ES;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int k = 0; k < NI; ++k) {
            double sb = 0.0, sg = 0.0;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const double v = X[c * NP + k * NI + i];
                sb += b1[i] * v;
                sg += g1[i] * v;
            }
            xb[c][k] = sb;
            xg[c][k] = sg;
        }
    double esum = 0.0, dmin = 1.0e300, bad = 0.0;
    double ug[GRAD ? 2 : 1][NI], ub[GRAD ? 2 : 1][NI];  // axis 1 still to apply: G, B
    if (GRAD) {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int k = 0; k < NI; ++k) ug[GRAD ? c : 0][k] = ub[GRAD ? c : 0][k] = 0.0;
    }
    if (act) {
        const Tab tp = tb.again();
        ColRow<NI, double> row, next;
        next.load(tp, 0);
#pragma unroll 1
        for (int q2 = 0; q2 < NQ; ++q2) {
            row = next;
            next.load(tp, q2 + 1 < NQ ? q2 + 1 : 0);
            double J[4] = {0.0, 0.0, 0.0, 0.0}, Pm[4], mu, detA;
#pragma unroll
            for (int k = 0; k < NI; ++k)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    J[c * 2] += row.b[k] * xg[c][k];
                    J[c * 2 + 1] += row.g[k] * xb[c][k];
                }
            const double z = w1 * row.w * tg.detW;
            const bool ok = metric_first<2>(tg, J, z, &mu, Pm, &detA);
            if (EN) dmin = fmin(dmin, detA);
            if (!ok) {
                if (EN) bad += 1.0;
#pragma unroll
                for (int k = 0; k < 4; ++k) Pm[k] = 0.0;
            } else if (EN) {
                esum += z * mu;
            }
            if (GRAD) {
#pragma unroll
                for (int k = 0; k < NI; ++k)
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        ug[GRAD ? c : 0][k] += row.b[k] * Pm[c * 2];
                        ub[GRAD ? c : 0][k] += row.g[k] * Pm[c * 2 + 1];
                    }
            }
        }
    }
    if constexpr (GRAD) {
        __syncthreads();  // X has been read
        if (act) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int k = 0; k < NI; ++k) {
                    L.U[(c * NI + k) * C::LN + tid] = ug[c][k];
                    L.U[((2 + c) * NI + k) * C::LN + tid] = ub[c][k];
                }
        }
        __syncthreads();
        // axis 1: lines (c, i2, element), n_i consecutive outputs each
        const Tab tp = tb.again();
        for (int pen = tid; pen < 2 * NI * C::EPB; pen += C::WL) {
            const int e = pen % C::EPB, s = pen / C::EPB;
            if (e >= nel) continue;
            const double *u = L.U + s * C::LN + e * NQ;
            double y[NI];
#pragma unroll
            for (int k = 0; k < NI; ++k) y[k] = 0.0;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const double a = u[q], b = u[2 * NI * C::LN + q];
#pragma unroll
                for (int k = 0; k < NI; ++k)
                    y[k] += tp.t->G[q * NI + k] * a + tp.t->B[q * NI + k] * b;
            }
            double *o = gE + ev_index2<P>(g, e0 + e, s / NI, 0, s % NI);
#pragma unroll
            for (int k = 0; k < NI; ++k) o[k] = y[k];
        }
    }
    if constexpr (EN) {
        col_reduce3<C::NW>(esum, dmin, bad, red);
        if (tid == 0) {
            part[blockIdx.x] = esum;
            part[gridDim.x + blockIdx.x] = dmin;
            part[2 * gridDim.x + blockIdx.x] = bad;
        }
    }
}

template <class C, bool GRAD, bool EN>
__global__ __launch_bounds__(C::WL) void k2c_energy(Geom g, BasisTables tba, Target tg, const double *__restrict__ x, double *__restrict__ gE, double *__restrict__ part)
{
    const Tab tb = kernel_tables<sizeof(Geom)>();
    const int e0 = xcd_block(blockIdx.x, gridDim.x) * C::EPB;
    c2_energy<C, GRAD, EN>(g, tb, tg, x, gE, part, e0, min(C::EPB, g.ne - e0));
}

// One wave per workgroup needs no barriers between waves; 256 lanes measured
// the same to 3% slower.  (At n_q <= 3 two waves: one would hold fewer elements
// than a workgroup of the pencil form, so that the no-allocation energy would
// accept smaller meshes than it did.)  From 640 workgroups of the pencil form
// on; a column's points follow one another, so below that the pencil form's
// shorter workgroups win.  Gradient / energy + gradient, whole calls, us,
// pencil -> column: p2 n_q4 64^2 8.2 / 23.9 -> 8.0 / 24.2, 128^2 9.4 / 27.1 ->
// 8.4 / 25.5, 256^2 22.9 / 45.6 -> 13.6 / 31.8; p3 n_q5 64^2 8.0 / 24.9 -> 8.5 /
// 25.1, 96^2 9.1 / 26.7 -> 8.9 / 25.8, 256^2 30.2 / 53.8 -> 21.6 / 44.5; p4 n_q5
// 48^2 8.0 / 25.5 -> 8.8 / 25.6, 96^2 10.8 / 28.3 -> 10.4 / 26.9; p4 n_q7 256^2
// 55.3 / 87.3 -> 37.1 / 56.5.
template <int P, int NQ>
struct ColForm2 {
    static constexpr int WL = NQ <= 3 ? 128 : 64;
    static constexpr int energy_min = 640 * S2<P, NQ>::EPB;
};

}  // namespace tmop
