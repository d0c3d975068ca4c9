// Hex kernels in column form: a lane keeps one column (q1, q2) of an
// element's quadrature points.  After the contractions along axes 1 and 2 the
// lane reads the 9 n_i values of its column from LDS once, walks the n_q
// points of the column with everything in registers (axis-3 contraction,
// point work, axis-3 transposed contraction into accumulators) and writes the
// 9 n_i results back in place.  Against the pencil form (kernels3d.hpp), which
// stores the 9 n_q^3 point values in LDS between those three stages, this
// halves the LDS traffic, takes five barriers instead of eight (none for a
// workgroup of one wave), and needs less LDS per element, so that more
// elements are in flight: these kernels are bound by LDS issue and by the
// serial chain of a workgroup's stages, not by arithmetic.
//
// The element nodes are read straight into registers, one 1D line of n_i
// consecutive nodes per lane (neighbouring lanes take neighbouring elements
// along x), which also saves the staging of the nodes in LDS.
//
//   lines   (c, i3, i2, el)  -> R1 [(c, v)][i3, i2][el, q1]   v = B, G
//   pencils (c, i3, el, q1)  -> R2 [(c, w)][i3][el, q2, q1]   w = GB, BG, BB
//   columns (el, q2, q1)     -> point work -> R2 in place
//   and back the same way.
//
// R1 and R2 share storage: a stage reads all of its input into registers
// before any lane writes its output.  Every sum runs in the order of the
// pencil form, so both give the same bits.
#pragma once
#include <climits>

#include "cols.hpp"
#include "kernels3d.hpp"

namespace tmop {
// Column form of class (P, NQ) with WL lanes per workgroup: EPB = WL / n_q^2
// elements.
template <int P_, int NQ_, int WL_>
struct C3 {
    static constexpr int P = P_, NQ = NQ_, WL = WL_;
    static constexpr int NI = P + 1;
    static constexpr int NP = NI * NI * NI;
    static constexpr int NQ2 = NQ * NQ;
    static constexpr int NQ3 = NQ * NQ * NQ;
    static constexpr int NW = WL / 64;
    static constexpr int EPB = WL / NQ2;
    // row lengths in LDS: R1 rows odd, R2 columns of one element spaced so
    // that the rows of consecutive i3 follow each other in the banks
    static constexpr int RS = (EPB * NQ) % 2 ? EPB * NQ : EPB * NQ + 1;
    static constexpr int N2 = NQ2 % 16 == 0 ? NQ2 + 4 : NQ2;
    static constexpr int CS = EPB * N2;
    // passes of the workgroup over the lines and over the pencils
    static constexpr int NL = EPB * 3 * NI * NI;
    static constexpr int NPEN = EPB * 3 * NI * NQ;
    static constexpr int PL = (NL + WL - 1) / WL;
    static constexpr int PP = (NPEN + WL - 1) / WL;
    static_assert(EPB >= 1, "a column per lane");
};

template <class C, typename CT>
union ColLds {
    CT R1[6 * C::NI * C::NI * C::RS];
    CT R2[9 * C::NI * C::CS];
};

// Line `it` of this lane: element of the block, component and (i2, i3).
template <class C>
struct ColLine {
    int el, c, i2, i3;
    bool in;
    __device__ __forceinline__ ColLine(int it, int nel)
    {
        const int pen = (int)threadIdx.x + it * C::WL;
        el = pen % C::EPB;
        const int r = pen / C::EPB;
        i2 = r % C::NI;
        i3 = (r / C::NI) % C::NI;
        c = r / (C::NI * C::NI);
        in = pen < C::NL && el < nel;
        if (!in) {
            el = 0;
            c = 0;
        }
    }
};

// Pencil `it` of this lane, and where its rows start in R1 and R2.
template <class C>
struct ColPencil {
    static constexpr int NQ = C::NQ;
    int r1, r2;
    bool in;
    __device__ __forceinline__ ColPencil(int it)
    {
        int pen = (int)threadIdx.x + it * C::WL;
        in = C::NPEN % C::WL == 0 || pen < C::NPEN;
        if (!in) pen = 0;
        const int q1 = pen % NQ, el = (pen / NQ) % C::EPB;
        const int r = pen / (NQ * C::EPB);  // c * NI + i3
        const int i3 = r % C::NI, c = r / C::NI;
        r1 = (c * 2 * C::NI * C::NI + i3 * C::NI) * C::RS + el * NQ + q1;
        r2 = (c * 3 * C::NI + i3) * C::CS + el * C::N2 + q1;
    }
};

// The lane's lines of `vec` for the block's elements, fixed DoFs as zero when
// masked.  Lanes without a line read node 0 of element e0.
template <class C, typename CT>
__device__ __forceinline__ void col_load(const Geom &g, const double *__restrict__ vec, int e0,
                                         int nel, bool masked, CT (&xv)[C::PL][C::NI])
{
    constexpr int P = C::P, NQ = C::NQ, NI = C::NI;
    const bool box = !g.e2n && !(masked && g.ess_mode == 2);
    if (box) {
        const bool bmask = masked && g.ess_mode == 0;
        double v[C::PL][NI];
        bool row[C::PL], lo[C::PL], hi[C::PL];
#pragma unroll
        for (int it = 0; it < C::PL; ++it) {
            const ColLine<C> l(it, nel);
            int ex, ey, ez;
            box_elem<3>(g, e0 + l.el, ex, ey, ez);
            const int gx = ex * P, gy = ey * P + l.i2, gz = ez * P + l.i3;
            const double *a = vec + (uint32_t)(l.c * g.nx + gx + g.M[0] * (gy + g.M[1] * gz));
#pragma unroll
            for (int k = 0; k < NI; ++k) v[it][k] = a[k];
            row[it] = bmask && (gy == 0 || gy == g.M[1] - 1 || gz == 0 || gz == g.M[2] - 1);
            lo[it] = bmask && ex == 0;
            hi[it] = bmask && ex == g.nel[0] - 1;
        }
#pragma unroll
        for (int it = 0; it < C::PL; ++it)
#pragma unroll
            for (int k = 0; k < NI; ++k) {
                const bool fix = row[it] || (k == 0 && lo[it]) || (k == P && hi[it]);
                xv[it][k] = fix ? (CT)0 : (CT)v[it][k];
            }
        return;
    }
#pragma unroll
    for (int it = 0; it < C::PL; ++it) {
        const ColLine<C> l(it, nel);
#pragma unroll
        for (int k = 0; k < NI; ++k) {
            int gx, gy, gz;
            const int node = node3<P>(g, e0 + l.el, k, l.i2, l.i3, gx, gy, gz);
            const double v = vec[(size_t)l.c * g.nx + node];
            xv[it][k] = masked && is_fixed(g, l.c, node, gx, gy, gz) ? (CT)0 : (CT)v;
        }
    }
}

// Axes 1 and 2: the lane's lines -> R1 -> R2, ending with a barrier.
template <class C, typename CT>
__device__ __forceinline__ void col_forward(const Tab &tables, int nel,
                                            const CT (&xv)[C::PL][C::NI],
                                            ColLds<C, CT> &L)
{
    constexpr int P = C::P, NQ = C::NQ, NI = C::NI;
    Tab tb = tables.again();
#pragma unroll
    for (int it = 0; it < C::PL; ++it) {
        const ColLine<C> l(it, nel);
        if (l.in) {
            CT *o = L.R1 + (l.c * 2 * NI * NI + l.i3 * NI + l.i2) * C::RS + l.el * NQ;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                CT b = 0, d = 0;
#pragma unroll
                for (int k = 0; k < NI; ++k) {
                    b += tabB<CT>(tb, q * NI + k) * xv[it][k];
                    d += tabG<CT>(tb, q * NI + k) * xv[it][k];
                }
                o[q] = b;
                o[NI * NI * C::RS + q] = d;
            }
        }
    }
    __syncthreads();
    tb = tables.again();
    CT xb[C::PP][NI], xg[C::PP][NI];
#pragma unroll
    for (int it = 0; it < C::PP; ++it) {
        const ColPencil<C> p(it);
        const CT *t = L.R1 + p.r1;
#pragma unroll
        for (int k = 0; k < NI; ++k) {
            xb[it][k] = t[k * C::RS];
            xg[it][k] = t[(NI * NI + k) * C::RS];
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < C::PP; ++it) {
        const ColPencil<C> p(it);
        if (p.in) {
            CT *o = L.R2 + p.r2;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                CT gb = 0, bg = 0, bb = 0;
#pragma unroll
                for (int k = 0; k < NI; ++k) {
                    const CT b2 = tabB<CT>(tb, q * NI + k), g2 = tabG<CT>(tb, q * NI + k);
                    gb += b2 * xg[it][k];
                    bg += g2 * xb[it][k];
                    bb += b2 * xb[it][k];
                }
                o[q * NQ] = gb;
                o[NI * C::CS + q * NQ] = bg;
                o[2 * NI * C::CS + q * NQ] = bb;
            }
        }
    }
    __syncthreads();
}

// The lane's column: t[c*3+w][i3].
template <class C, typename CT>
__device__ __forceinline__ void col_read(const ColLds<C, CT> &L, int at, CT (&t)[9][C::NI])
{
    constexpr int NI = C::NI;
#pragma unroll
    for (int w = 0; w < 9; ++w)
#pragma unroll
        for (int k = 0; k < C::NI; ++k) t[w][k] = L.R2[(w * C::NI + k) * C::CS + at];
}

// Axis 3 at one point of the column: J[c*3+b].
template <int NI, typename CT>
__device__ __forceinline__ void col_point(const ColRow<NI, CT> &r, const CT (&t)[9][NI], CT *J)
{
#pragma unroll
    for (int w = 0; w < 9; ++w) J[w] = 0;
#pragma unroll
    for (int k = 0; k < NI; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            J[c * 3] += r.b[k] * t[c * 3][k];
            J[c * 3 + 1] += r.b[k] * t[c * 3 + 1][k];
            J[c * 3 + 2] += r.g[k] * t[c * 3 + 2][k];
        }
}

// The same with the column read from LDS at every point (fewer registers).
template <class C, typename CT>
__device__ __forceinline__ void col_point_lds(const ColRow<C::NI, CT> &r,
                                              const ColLds<C, CT> &L, int at, CT *J)
{
    constexpr int NI = C::NI;
    asm volatile("" : "+v"(at));  // keep the reads inside the loop over the points
#pragma unroll
    for (int w = 0; w < 9; ++w) J[w] = 0;
#pragma unroll
    for (int k = 0; k < NI; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            J[c * 3] += r.b[k] * L.R2[(c * 3 * NI + k) * C::CS + at];
            J[c * 3 + 1] += r.b[k] * L.R2[((c * 3 + 1) * NI + k) * C::CS + at];
            J[c * 3 + 2] += r.g[k] * L.R2[((c * 3 + 2) * NI + k) * C::CS + at];
        }
}

// Its transpose: the point's values Y[c*3+b] into the accumulators.
template <int NI, typename CT>
__device__ __forceinline__ void col_accumulate(const ColRow<NI, CT> &r, const CT *Y,
                                               CT (&acc)[9][NI])
{
#pragma unroll
    for (int k = 0; k < NI; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            acc[c * 3][k] += r.b[k] * Y[c * 3];
            acc[c * 3 + 1][k] += r.b[k] * Y[c * 3 + 1];
            acc[c * 3 + 2][k] += r.g[k] * Y[c * 3 + 2];
        }
}

// s + (a b + c d) as the pencil form rounds it: c d rounded, a b + c d fused.
template <typename CT>
__device__ __forceinline__ CT add_two(CT s, CT a, CT b, CT c, CT d)
{
#pragma clang fp contract(on)
    const CT m = a * b + c * d;
    return s + m;
}

// Accumulators back to R2 and the transposed contractions of axes 2 and 1 ->
// E-vector.
template <class C, typename CT, typename OT>
__device__ __forceinline__ void col_backward(const Tab &tables, const Geom &g, int e0, int nel,
                                             int at, bool act, const CT (&acc)[9][C::NI],
                                             ColLds<C, CT> &L, OT *__restrict__ out)
{
    constexpr int P = C::P, NQ = C::NQ, NI = C::NI;
    if (act) {
#pragma unroll
        for (int w = 0; w < 9; ++w)
#pragma unroll
            for (int k = 0; k < NI; ++k) L.R2[(w * NI + k) * C::CS + at] = acc[w][k];
    }
    __syncthreads();
    Tab tb = tables.again();
    CT t0[C::PP][NQ], t1[C::PP][NQ], t2[C::PP][NQ];
#pragma unroll
    for (int it = 0; it < C::PP; ++it) {
        const ColPencil<C> p(it);
        const CT *t = L.R2 + p.r2;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            t0[it][q] = t[q * NQ];
            t1[it][q] = t[NI * C::CS + q * NQ];
            t2[it][q] = t[2 * NI * C::CS + q * NQ];
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < C::PP; ++it) {
        const ColPencil<C> p(it);
        if (p.in) {
            CT *o = L.R1 + p.r1;
#pragma unroll
            for (int k = 0; k < NI; ++k) {
                CT u0 = 0, u1 = 0;
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const CT b2 = tabB<CT>(tb, q * NI + k), g2 = tabG<CT>(tb, q * NI + k);
                    u0 += b2 * t0[it][q];
                    u1 = add_two(u1, g2, t1[it][q], b2, t2[it][q]);
                }
                o[k * C::RS] = u0;              // G along axis 1 still to apply
                o[(NI * NI + k) * C::RS] = u1;  // B along axis 1 still to apply
            }
        }
    }
    __syncthreads();
    tb = tables.again();
#pragma unroll
    for (int it = 0; it < C::PL; ++it) {
        const ColLine<C> l(it, nel);
        if (l.in) {
            const CT *t = L.R1 + (l.c * 2 * NI * NI + l.i3 * NI + l.i2) * C::RS + l.el * NQ;
            CT u0[NQ], u1[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                u0[q] = t[q];
                u1[q] = t[NI * NI * C::RS + q];
            }
            OT *o = out + ev_index3<P>(g, e0 + l.el, l.c, 0, l.i2, l.i3);
#pragma unroll
            for (int k = 0; k < NI; ++k) {
                CT s = 0;
#pragma unroll
                for (int q = 0; q < NQ; ++q)
                    s = add_two(s, tabG<CT>(tb, q * NI + k), u0[q], tabB<CT>(tb, q * NI + k), u1[q]);
                o[k] = (OT)s;
            }
        }
    }
}

// Product of the 1D weights of column q12 = q1 + n_q q2.
template <int NQ>
__device__ __forceinline__ double col_weight(const Tab &tables, int q12)
{
    const Tab tb = tables.again();
    double w1 = 0.0, w2 = 0.0;
#pragma unroll
    for (int k = 0; k < NQ; ++k) {
        const double w = tb.t->w[k];
        if (q12 % NQ == k) w1 = w;
        if (q12 / NQ == k) w2 = w;
    }
    return w1 * w2;
}

// Energy partials (as b3_energy), and with GRAD the gradient E-vector (as
// b3_gradient); EN: the energy partials are wanted.  The same point code
// serves both, so their values agree bitwise.
template <class C, bool GRAD, bool EN>
__device__ __forceinline__ void c3_energy(const Geom &g, const Tab &tb, const Target &tg,
                                          const double *__restrict__ x, double *__restrict__ gE,
                                          double *__restrict__ part, int e0, int nel)
{
    constexpr int P = C::P, NQ = C::NQ, NI = C::NI;
    __shared__ ColLds<C, double> L;
    __shared__ double red[3 * C::NW];
    double xv[C::PL][NI];
    col_load<C, double>(g, x, e0, nel, false, xv);
    col_forward<C, double>(tb, nel, xv, L);
    const int el = (int)threadIdx.x / C::NQ2, q12 = (int)threadIdx.x % C::NQ2;
    const bool act = el < nel && (C::EPB * C::NQ2 == C::WL || (int)threadIdx.x < C::EPB * C::NQ2);
    const int at = act ? el * C::N2 + q12 : 0;
    double esum = 0.0, dmin = 1.0e300, bad = 0.0;
    double acc[GRAD ? 9 : 1][NI];
    if (GRAD) {
#pragma unroll
        for (int w = 0; w < 9; ++w)
#pragma unroll
            for (int k = 0; k < NI; ++k) acc[GRAD ? w : 0][k] = 0.0;
    }
    if (act) {
        double t[9][NI];
        col_read<C, double>(L, at, t);
        const double w12 = col_weight<NQ>(tb, q12);
        const Tab tp = tb.again();
        ColRow<NI, double> row, next;
        next.load(tp, 0);
#pragma unroll 1
        for (int q3 = 0; q3 < NQ; ++q3) {
            row = next;
            next.load(tp, q3 + 1 < NQ ? q3 + 1 : 0);
            double J[9], Pm[9], mu, detA;
            col_point<NI, double>(row, t, J);
            const double z = w12 * row.w * tg.detW;
            const bool ok = metric_first<3>(tg, J, z, &mu, Pm, &detA);
            if (EN) dmin = fmin(dmin, detA);
            if (!ok) {
                if (EN) bad += 1.0;
#pragma unroll
                for (int k = 0; k < 9; ++k) Pm[k] = 0.0;
            } else if (EN) {
                esum += z * mu;
            }
            if constexpr (GRAD) col_accumulate<NI, double>(row, Pm, acc);
        }
    }
    if constexpr (GRAD)
        col_backward<C, double, double>(tb, g, e0, nel, at, act, acc, L, gE);
    if constexpr (EN) {
        col_reduce3<C::NW>(esum, dmin, bad, red);
        if (threadIdx.x == 0) {
            part[blockIdx.x] = esum;
            part[gridDim.x + blockIdx.x] = dmin;
            part[2 * gridDim.x + blockIdx.x] = bad;
        }
    }
}

// Hessian setup, compact storage (as b3_setupc).
template <class C, typename TT>
__device__ __forceinline__ void c3_setupc(const Geom &g, const Tab &tb, const Target &tg,
                                          const double *__restrict__ x, TT *__restrict__ Q, int e0,
                                          int nel)
{
    constexpr int P = C::P, NQ = C::NQ, NI = C::NI;
    __shared__ ColLds<C, double> L;
    double xv[C::PL][NI];
    col_load<C, double>(g, x, e0, nel, false, xv);
    col_forward<C, double>(tb, nel, xv, L);
    const int el = (int)threadIdx.x / C::NQ2, q12 = (int)threadIdx.x % C::NQ2;
    if (el >= nel || (int)threadIdx.x >= C::EPB * C::NQ2) return;
    double t[9][NI];
    col_read<C, double>(L, el * C::N2 + q12, t);
    const double w12 = col_weight<NQ>(tb, q12);
    TT *qe = Q + (size_t)(e0 + el) * QLay<TT, NC3, C::NQ3>::STRIDE;
    const Tab tp = tb.again();
    ColRow<NI, double> row, next;
    next.load(tp, 0);
#pragma unroll 1
    for (int q3 = 0; q3 < NQ; ++q3) {
        row = next;
        next.load(tp, q3 + 1 < NQ ? q3 + 1 : 0);
        double J[9];
        col_point<NI, double>(row, t, J);
        TT hs[NC3];
        compact_point3<TT>(tg, J, w12 * row.w * tg.detW, hs);
        qdata_store<TT, NC3, C::NQ3>(qe, q3 * C::NQ2 + q12, hs);
    }
}

// Hessian action on compact data (as b3_applyc).  The data of the column's
// next point is loaded while the current point computes.
// RD: the column is read from LDS at every point instead of kept.
template <class C, typename TT, typename CT, bool RD>
__device__ __forceinline__ void c3_applyc(const Geom &g, const Tab &tb, const Target &tg,
                                          const TT *__restrict__ Q, const double *__restrict__ v,
                                          CT *__restrict__ yE, int e0, int nel)
{
    constexpr int P = C::P, NQ = C::NQ, NI = C::NI;
    using QL = QLay<TT, NC3, C::NQ3>;
    __shared__ ColLds<C, CT> L;
    const int el = (int)threadIdx.x / C::NQ2, q12 = (int)threadIdx.x % C::NQ2;
    const bool act = el < nel && (C::EPB * C::NQ2 == C::WL || (int)threadIdx.x < C::EPB * C::NQ2);
    const int at = act ? el * C::N2 + q12 : 0;
    const TT *qe = Q + (size_t)(e0 + (act ? el : 0)) * QL::STRIDE;
    const int q0 = act ? q12 : 0;
    CT xv[C::PL][NI];
    col_load<C, CT>(g, v, e0, nel, true, xv);
    TT nx[NC3];
    qdata_load<TT, NC3, C::NQ3>(qe, q0, nx);
    col_forward<C, CT>(tb, nel, xv, L);
    CT t[9][NI], acc[9][NI];
    if (!RD) col_read<C, CT>(L, at, t);
#pragma unroll
    for (int w = 0; w < 9; ++w)
#pragma unroll
        for (int k = 0; k < NI; ++k) acc[w][k] = 0;
    const Tab tp = tb.again();
    ColRow<NI, CT> row, next;
    next.load(tp, 0);
#pragma unroll 1
    for (int q3 = 0; q3 < NQ; ++q3) {
        row = next;
        next.load(tp, q3 + 1 < NQ ? q3 + 1 : 0);
        CT d[NC3];
#pragma unroll
        for (int m = 0; m < NC3; ++m) d[m] = (CT)nx[m];
        if (q3 + 1 < NQ) qdata_load<TT, NC3, C::NQ3>(qe, (q3 + 1) * C::NQ2 + q0, nx);
        CT J[9], Y[9];
        if (RD)
            col_point_lds<C, CT>(row, L, at, J);
        else
            col_point<NI, CT>(row, t, J);
        if (tg.ideal) {
            compact_action3<CT>(d, d[9], d[10], d[11], d[12], J, Y);
        } else {
            CT M[9], Yt[9];
            mul_winv<3, CT>(tg, J, M, false);
            compact_action3<CT>(d, d[9], d[10], d[11], d[12], M, Yt);
            mul_winv<3, CT>(tg, Yt, Y, true);
        }
        col_accumulate<NI, CT>(row, Y, acc);
    }
    col_backward<C, CT, CT>(tb, g, e0, nel, at, act, acc, L, yE);
}

// ------------------------------------------------------------------------
// Which kernels run in column form, with how many lanes per workgroup (0: the
// pencil form only) and from how many elements on.
//
// Lanes: one wave per workgroup needs no barriers but leaves lanes idle where
// 64 is not near a multiple of n_q^2, and the LDS limits large workgroups.
// Each entry is the fastest of 64, 128 and 256 lanes on meshes of n = 16 to 48
// elements per side, us, pencil -> column:
//   energy, gradient with energy: p1 n_q3 40^3 31 / 49 -> 17 / 28; p2 n_q4 40^3
//   78 / 119 -> 41 / 75; p3 n_q5 24^3 37 / 57 -> 23 / 43; p4 n_q6 24^3 65 /
//   108 -> 45 / 91; p4 n_q7 20^3 62 / 103 -> 36 / 70; p2 n_q9 20^3 85 / 133 ->
//   36 / 70.  At n_q = 3 one wave would hold 7 elements (8% faster at p = 2),
//   fewer than the 9 of the pencil form, so that the no-allocation energy
//   would accept smaller meshes than it did.
//   Compact setup: p2 n_q4 105 -> 84, p3 n_q5 39 -> 33, p4 n_q6 88 -> 72; slower
//   where its stores end runs inside 128-byte lines (p1 n_q9 118 -> 143, p2
//   n_q5 100 -> 117, p4 n_q9 140 -> 152; see also the largest meshes below).
//   Compact action in FP64: p1 n_q3 41 -> 36, p2 n_q3 63 -> 49, p2 n_q4 111 ->
//   103, p3 n_q4 34 -> 28 with the column re-read from LDS (kept in registers
//   it takes more than the 256 of two waves per SIMD, 36); from n_q = 5 at p >=
//   3 on equal or slower, and with 9 points the layer-chunked form is faster.
//   In FP32, where a column takes half the registers: p2 n_q4 55 -> 49, p2
//   n_q9 71 -> 63, p3 n_q6 50 -> 39, p4 n_q6 58 -> 52 (re-read).
//
// Elements: a column's points are walked one after the other, so a workgroup
// takes longer, and on a mesh of few workgroups per CU that is the kernel's
// time (9^3 elements p3 n_q5: gradient 7.9 us pencil, 9.1 column; FP32 action
// 5.3 / 8.4).  The lines lie where the two meet, counted in workgroups of the
// pencil form (256 CUs): energy and gradient about 1024 (16^3 p2 n_q4, 1024:
// 10.6 -> 9.2; 12^3, 432: 7.2 -> 8.2), at p = 4 with n_q <= 6 4096; compact
// setup 4096, n_q = 6 8192 (FP64: only p = 4, from 16384 on: 20^3 35.5 -> 38.2,
// 25^3 91.4 -> 86.6; p3 25^3 81.8 -> 85.7), n_q >= 7 1024; FP64 action 1024, n_q = 5 2048; FP32 action 1536 for n_q <= 4 and n_q =
// 9 at p = 1, n_q = 5 and p = 4 n_q <= 7 8192 (p2 n_q5 20^3, 4000: 15.6 -> 17.1;
// 32^3: 54 -> 47), else 4096 (p2 n_q9 13^3, 2366: 24.2 -> 27.6; 16^3: 35.6 -> 33.5).
//
// Largest meshes: the setup stores a column layer by layer, n_q^2 points of 16
// bytes at a time, so the 128-byte lines at both ends of a layer are written in
// two parts, some time apart.  The 256 MB last-level cache puts them together;
// beyond it they reach memory as parts.  Where a layer is a few lines long
// that costs more than the form saves, in FP64 above all (41.4 against 42.5 us
// at 42^3 p1 n_q3, 200 MB, but 345 against 632 at 84^3; p2 n_q3 53^3 112 / 168;
// p1 n_q2 81^3 103 / 150): such classes keep the pencil form, or take the
// column form up to 256 MB of data (p1 n_q4 FP64 32^3 38.2 -> 35.7, 64^3 288 ->
// 322; p3 n_q5 FP64 25^3 40.0 -> 38.2, 51^3 411 -> 439), in FP32 320 MB (p1 n_q2
// 81^3 87 -> 72, 90^3 111 -> 113, 128^3 313 -> 345).  The action reads the data
// so; beyond 256 MB n_q = 3, p1 n_q4 and p2 n_q5 in FP64 and p1 n_q3 in FP32 keep
// the pencil form (p1 n_q3 FP64 42^3 49.2 -> 46.9, 84^3 433 -> 462, FP32 53^3 52.6
// -> 48.5, 84^3 232 -> 254; p2 n_q5 25^3 47.8 -> 47.2, 51^3 408 -> 421).
// ------------------------------------------------------------------------
template <int P, int NQ>
struct ColForm {
    static constexpr int energy = NQ <= 3 ? 128
                                  : NQ == 6 ? (P == 3 ? 256 : 128)
                                  : NQ == 9 ? (P <= 3 ? 256 : 128)
                                            : 64;
    template <typename TT>
    static constexpr int setupc()
    {
        if (sizeof(TT) == 8 && (NQ <= 3 || (P == 3 && NQ == 6))) return 0;
        return NQ <= 4   ? 64
               : NQ == 5 ? (P == 3 ? 64 : 0)
               : NQ == 9 ? (P == 3 ? 256 : 0)
                         : 128;
    }
    template <typename TT>
    static constexpr int applyc()
    {
        if (sizeof(TT) == 8)
            return NQ <= 4 ? 64 : P == 2 && NQ == 5 ? 128 : 0;
        if ((P == 2 && NQ == 3) || (P == 4 && NQ == 5)) return 0;
        return NQ <= 4 ? (P == 3 ? 128 : 64) : NQ == 5 ? 128 : 256;
    }
    template <typename TT>
    static constexpr bool reread()
    {
        return sizeof(TT) == 8 ? P == 3 : P == 4 || (P == 3 && NQ == 4);
    }
    // smallest element counts
    static constexpr int EPB0 = S3<P, NQ>::EPB;
    static constexpr int energy_min = EPB0 * (P == 4 && NQ <= 6 ? 4096 : 1024);
    template <typename TT>
    static constexpr int setupc_min()
    {
        return EPB0 * (NQ >= 7 ? 1024 : NQ == 6 ? (sizeof(TT) == 8 ? 16384 : 8192) : 4096);
    }
    template <typename TT>
    static constexpr int applyc_min()
    {
        if (sizeof(TT) == 8) return EPB0 * (NQ == 5 ? 2048 : 1024);
        return EPB0 * (NQ <= 4 || (NQ == 9 && P == 1) ? 1536
                       : NQ == 5 || (P == 4 && NQ <= 7) ? 8192
                                                        : 4096);
    }
    // largest element counts: no limit, or so many MB of quadrature data (whole
    // lines of the runs and planes, without what pads them further)
    template <typename TT, long MB>
    static constexpr int within()
    {
        using L = QLay<TT, NC3, NQ * NQ * NQ>;
        constexpr long NQ3 = NQ * NQ * NQ, RUN = (NQ3 * 16 + 127) / 128 * 128;
        constexpr long PLANE = (NQ3 * (long)sizeof(TT) + 127) / 128 * 128;
        return (int)((MB << 20) / (L::NV * RUN + (NC3 - L::TAIL) * PLANE));
    }
    template <typename TT>
    static constexpr int setupc_max()
    {
        if (sizeof(TT) == 8 && (NQ == 5 || (P == 1 && NQ == 4))) return within<TT, 256>();
        return NQ == 2 ? within<TT, 320>() : INT_MAX;
    }
    template <typename TT>
    static constexpr int applyc_max()
    {
        const bool part = sizeof(TT) == 8 ? NQ == 3 || (P == 1 && NQ == 4) || (P == 2 && NQ == 5)
                                          : P == 1 && NQ == 3;
        return part ? within<TT, 256>() : INT_MAX;
    }
};

// ------------------------------------------------------------------------
// Kernel entry points, as in kernels3d.hpp.
// ------------------------------------------------------------------------

template <class C, bool GRAD, bool EN>
__global__ __launch_bounds__(C::WL) __attribute__((amdgpu_waves_per_eu(2))) void k3c_energy(Geom g, BasisTables tba, Target tg, const double *__restrict__ x, double *__restrict__ gE, double *__restrict__ part)
{
    const Tab tb = kernel_tables<sizeof(Geom)>();
    const int e0 = xcd_block(blockIdx.x, gridDim.x) * C::EPB;
    c3_energy<C, GRAD, EN>(g, tb, tg, x, gE, part, e0, min(C::EPB, g.ne - e0));
}

template <class C, typename TT>
__global__ __launch_bounds__(C::WL) void k3c_setupc(Geom g, BasisTables tba, Target tg, const double *__restrict__ x, TT *__restrict__ Q)
{
    const Tab tb = kernel_tables<sizeof(Geom)>();
    const int e0 = xcd_block(blockIdx.x, gridDim.x) * C::EPB;
    c3_setupc<C, TT>(g, tb, tg, x, Q, e0, min(C::EPB, g.ne - e0));
}

template <class C, typename TT, typename CT, bool RD>
__global__ __launch_bounds__(C::WL) __attribute__((amdgpu_waves_per_eu(2))) void k3c_applyc(Geom g, BasisTables tba, Target tg, const TT *__restrict__ Q, const double *__restrict__ v, CT *__restrict__ yE)
{
    const Tab tb = kernel_tables<sizeof(Geom)>();
    const int e0 = xcd_block(blockIdx.x, gridDim.x) * C::EPB;
    c3_applyc<C, TT, CT, RD>(g, tb, tg, Q, v, yE, e0, min(C::EPB, g.ne - e0));
}

template <class C, typename TT>
__global__ __launch_bounds__(C::WL) void kb3c_setupc(BasisTables tba, const Tile *__restrict__ tiles, const SlotDev *__restrict__ slots, const int *__restrict__ gate, int vin)
{
    const Tab tb = kernel_tables<0>();
    const Tile t = tiles[blockIdx.x];
    if (gate && !gate[t.slot]) return;
    const SlotDev &s = slots[t.slot];
    c3_setupc<C, TT>(s.g, tb, s.tg, s.vec[vin], (TT *)s.H, t.e0, min(C::EPB, s.g.ne - t.e0));
}

template <class C, typename TT, typename CT, bool RD>
__global__ __launch_bounds__(C::WL) __attribute__((amdgpu_waves_per_eu(2))) void kb3c_applyc(BasisTables tba, const Tile *__restrict__ tiles, const SlotDev *__restrict__ slots, const int *__restrict__ gate, int vin)
{
    const Tab tb = kernel_tables<0>();
    const Tile t = tiles[blockIdx.x];
    if (gate && !gate[t.slot]) return;
    const SlotDev &s = slots[t.slot];
    c3_applyc<C, TT, CT, RD>(s.g, tb, s.tg, (const TT *)s.H, s.vec[vin], (CT *)s.eV, t.e0, min(C::EPB, s.g.ne - t.e0));
}

}  // namespace tmop
