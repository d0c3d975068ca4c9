// Quad kernel instantiations for p = 1..4, n_q = p+1 .. p+3.
#include "cols2.hpp"
#include "kernels2d.hpp"
#include "minres_one.hpp"
#include "ops.hpp"

namespace tmop {

// The kernels without the limiting term; energy and gradient in the form that
// ColForm2 gives for the mesh.
template <int P, int NQ>
struct plain_k2 {
    static constexpr int EPB = S2<P, NQ>::EPB;
    using CE = C2<P, NQ, ColForm2<P, NQ>::WL>;
    static_assert(CE::EPB >= EPB, "the no-allocation energy takes the meshes it took");
    static bool col(int ne) { return ne >= ColForm2<P, NQ>::energy_min; }
    static int energy_epb(int ne) { return col(ne) ? CE::EPB : EPB; }
    static dim3 grid(const Geom &g, int epb = EPB) { return dim3((g.ne + epb - 1) / epb); }
    static void energy(hipStream_t s, const Geom &g, const Tables &t, const Target &w,
                       const double *x, double *part)
    {
        if (col(g.ne))
            hipLaunchKernelGGL((k2c_energy<CE, false, true>), grid(g, CE::EPB), dim3(CE::WL), 0, s, g,
                               t, w, x, (double *)nullptr, part);
        else
            hipLaunchKernelGGL((k2_energy<P, NQ, false>), grid(g), dim3(BLOCK), 0, s, g, t, w, x,
                               part);
    }
    template <bool EN>
    static void gradient(hipStream_t s, const Geom &g, const Tables &t, const Target &w,
                         const double *x, double *gE, double *part)
    {
        if (col(g.ne))
            hipLaunchKernelGGL((k2c_energy<CE, true, EN>), grid(g, CE::EPB), dim3(CE::WL), 0, s, g, t,
                               w, x, gE, part);
        else
            hipLaunchKernelGGL((k2_gradient<P, NQ, false, EN>), grid(g), dim3(BLOCK), 0, s, g, t, w, x,
                               gE, part);
    }
    template <typename TT>
    static void setupc(hipStream_t s, const Geom &g, const Tables &t, const Target &w,
                       const double *x, TT *Q)
    {
        hipLaunchKernelGGL((k2_setupc<P, NQ, TT>), grid(g), dim3(BLOCK), 0, s, g, t, w, x, Q);
    }
    template <typename TT>
    static void applyc(hipStream_t s, const Geom &g, const Tables &t, const Target &w, const TT *Q,
                       const double *v, TT *yE)
    {
        hipLaunchKernelGGL((k2_applyc<P, NQ, TT, TT, false>), grid(g), dim3(BLOCK), 0, s, g, t, w,
                           Q, v, yE);
    }
};

static bool ops2_elem(int p, int nq, Ops *out)
{
#define TMOP_CASE(P, NQ) \
    if (p == P && nq == NQ) TMOP_OPS_BODY(k2, S2, P, NQ)
    TMOP_CASE(1, 2) TMOP_CASE(1, 3) TMOP_CASE(1, 4)
    TMOP_CASE(2, 3) TMOP_CASE(2, 4) TMOP_CASE(2, 5)
    TMOP_CASE(3, 4) TMOP_CASE(3, 5) TMOP_CASE(3, 6)
    TMOP_CASE(4, 5) TMOP_CASE(4, 6) TMOP_CASE(4, 7)
#undef TMOP_CASE
    return false;
}

template <int P, int NQ, typename TT, bool COMPACT>
static void apply_l2_2(hipStream_t s, const Geom &g, const Tables &t, const Target &w, const void *H,
                       const MrL2 &a, void *yE)
{
    constexpr int EPB = S2<P, NQ>::EPB;
    hipLaunchKernelGGL((k2_apply_l2<P, NQ, TT, COMPACT>), dim3((g.ne + EPB - 1) / EPB), dim3(BLOCK), 0,
                       s, g, t, w, (const TT *)H, a, (TT *)yE);
}

template <int P, int NQ>
static bool fill_minres2(Ops *o)
{
    o->apply_l2[0][0] = apply_l2_2<P, NQ, double, false>;
    o->apply_l2[0][1] = apply_l2_2<P, NQ, float, false>;
    o->apply_l2[1][0] = apply_l2_2<P, NQ, double, true>;
    o->apply_l2[1][1] = apply_l2_2<P, NQ, float, true>;
    o->minres_one[0][0] = minres_one2<P, NQ, double, false>;
    o->minres_one[0][1] = minres_one2<P, NQ, float, false>;
    o->minres_one[1][0] = minres_one2<P, NQ, double, true>;
    o->minres_one[1][1] = minres_one2<P, NQ, float, true>;
    return true;
}

bool ops2(int p, int nq, Ops *out)
{
    if (!ops2_elem(p, nq, out)) return false;
#define TMOP_CASE(P, NQ) \
    if (p == P && nq == NQ) return fill_minres2<P, NQ>(out);
    TMOP_CASE(1, 2) TMOP_CASE(1, 3) TMOP_CASE(1, 4)
    TMOP_CASE(2, 3) TMOP_CASE(2, 4) TMOP_CASE(2, 5)
    TMOP_CASE(3, 4) TMOP_CASE(3, 5) TMOP_CASE(3, 6)
    TMOP_CASE(4, 5) TMOP_CASE(4, 6) TMOP_CASE(4, 7)
#undef TMOP_CASE
    return true;
}

bool bops2(int p, int nq, BOps *out)
{
#define TMOP_CASE(P, NQ) \
    if (p == P && nq == NQ) TMOP_BOPS_BODY(kb2, S2, P, NQ)
    TMOP_CASE(1, 2) TMOP_CASE(1, 3) TMOP_CASE(1, 4)
    TMOP_CASE(2, 3) TMOP_CASE(2, 4) TMOP_CASE(2, 5)
    TMOP_CASE(3, 4) TMOP_CASE(3, 5) TMOP_CASE(3, 6)
    TMOP_CASE(4, 5) TMOP_CASE(4, 6) TMOP_CASE(4, 7)
#undef TMOP_CASE
    return false;
}

bool find_bops(int dim, int p, int nq, BOps *out)
{
    if (dim == 2) return bops2(p, nq, out);
    if (dim != 3) return false;
    switch (p) {
    case 1: return bops3_p1(nq, out);
    case 2: return bops3_p2(nq, out);
    case 3: return bops3_p3(nq, out);
    case 4: return bops3_p4(nq, out);
    default: return false;
    }
}

bool find_ops(int dim, int p, int nq, Ops *out)
{
    if (dim == 2) return ops2(p, nq, out);
    if (dim != 3) return false;
    switch (p) {
    case 1: return ops3_p1(nq, out);
    case 2: return ops3_p2(nq, out);
    case 3: return ops3_p3(nq, out);
    case 4: return ops3_p4(nq, out);
    default: return false;
    }
}

}  // namespace tmop
