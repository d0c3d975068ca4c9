// Hessian-action launchers of the hex kernels for every tile shape of a
// class (elements per workgroup: half, base, double), filled into the launch
// tables; shapes that do not exist for a class (tile_ok3) are never
// instantiated.
#pragma once
#include "cols3.hpp"
#include "kernels3d.hpp"
#include "ops.hpp"

namespace tmop {

// The kernels without the limiting term that have a column form, in the form
// and with the workgroup that ColForm gives for the mesh.
template <int P, int NQ>
struct plain_k3 {
    using F = ColForm<P, NQ>;
    using CE = C3<P, NQ, F::energy>;
    static constexpr int EPB0 = S3<P, NQ>::EPB;
    static dim3 grid(const Geom &g, int epb) { return dim3((g.ne + epb - 1) / epb); }
    static int energy_epb(int ne) { return ne >= F::energy_min ? CE::EPB : EPB0; }
    static void energy(hipStream_t s, const Geom &g, const Tables &t, const Target &w,
                       const double *x, double *part)
    {
        if (g.ne >= F::energy_min)
            hipLaunchKernelGGL((k3c_energy<CE, false, true>), grid(g, CE::EPB), dim3(CE::WL), 0, s,
                               g, t, w, x, (double *)nullptr, part);
        else
            hipLaunchKernelGGL((k3_energy<P, NQ, false>), grid(g, EPB0), dim3(BLOCK), 0, s, g, t, w,
                               x, part);
    }
    template <bool EN>
    static void gradient(hipStream_t s, const Geom &g, const Tables &t, const Target &w,
                         const double *x, double *gE, double *part)
    {
        if (g.ne >= F::energy_min)
            hipLaunchKernelGGL((k3c_energy<CE, true, EN>), grid(g, CE::EPB), dim3(CE::WL), 0, s, g,
                               t, w, x, gE, part);
        else
            hipLaunchKernelGGL((k3_gradient<P, NQ, false, EN>), grid(g, EPB0), dim3(BLOCK), 0, s, g,
                               t, w, x, gE, part);
    }
    template <typename TT>
    static void setupc(hipStream_t s, const Geom &g, const Tables &t, const Target &w,
                       const double *x, TT *Q)
    {
        constexpr int WL = F::template setupc<TT>();
        if constexpr (WL > 0) {
            using C = C3<P, NQ, WL>;
            if (g.ne >= F::template setupc_min<TT>() && g.ne <= F::template setupc_max<TT>()) {
                hipLaunchKernelGGL((k3c_setupc<C, TT>), grid(g, C::EPB), dim3(C::WL), 0, s, g, t, w,
                                   x, Q);
                return;
            }
        }
        hipLaunchKernelGGL((k3_setupc<P, NQ, TT>), grid(g, EPB0), dim3(BLOCK), 0, s, g, t, w, x, Q);
    }
    template <typename TT>
    static void applyc(hipStream_t s, const Geom &g, const Tables &t, const Target &w, const TT *Q,
                       const double *v, TT *yE)
    {
        constexpr int WL = F::template applyc<TT>();
        if constexpr (WL > 0) {
            using C = C3<P, NQ, WL>;
            if (g.ne >= F::template applyc_min<TT>() && g.ne <= F::template applyc_max<TT>()) {
                hipLaunchKernelGGL((k3c_applyc<C, TT, TT, F::template reread<TT>()>),
                                   grid(g, C::EPB), dim3(C::WL), 0, s, g, t, w, Q, v, yE);
                return;
            }
        }
        hipLaunchKernelGGL((k3_applyc<P, NQ, TT, TT, false>), grid(g, EPB0), dim3(BLOCK), 0, s, g, t,
                           w, Q, v, yE);
    }
};

// Column form of the batched compact setup and action, by precision; taken
// for a class whose resident meshes have so many elements together.
// (Energy and gradient keep the pencil form there: a solve's energy is summed
// by tiles, and is to have the same bits alone and with others.)
template <int P, int NQ, typename TT, int IDX>
inline void fill_bcol3(BOps &o)
{
    using F = ColForm<P, NQ>;
    constexpr int WS = F::template setupc<TT>(), WA = F::template applyc<TT>();
    if constexpr (WS > 0) {
        using C = C3<P, NQ, WS>;
        o.setupc_col[IDX] = BCol{C::EPB, F::template setupc_min<TT>(), F::template setupc_max<TT>(),
                                 [](int n, hipStream_t s, const Tables &t, const Tile *tl,
                                    const SlotDev *sl, const int *gt, int vin, double *) {
                                     hipLaunchKernelGGL((kb3c_setupc<C, TT>), dim3(n), dim3(C::WL),
                                                        0, s, t, tl, sl, gt, vin);
                                 }};
    }
    if constexpr (WA > 0) {
        using C = C3<P, NQ, WA>;
        o.applyc_col[IDX] =
            BCol{C::EPB, F::template applyc_min<TT>(), F::template applyc_max<TT>(),
                 [](int n, hipStream_t s, const Tables &t, const Tile *tl, const SlotDev *sl,
                    const int *gt, int vin, double *) {
                     hipLaunchKernelGGL((kb3c_applyc<C, TT, TT, F::template reread<TT>()>), dim3(n),
                                        dim3(C::WL), 0, s, t, tl, sl, gt, vin);
                 }};
    }
}

template <int P, int NQ, int T2, int IDX>
inline void fill_tile3(Ops &o)
{
    if constexpr (tile_ok3<P, NQ, T2>()) {
        o.epb_t[IDX] = S3<P, NQ, T2>::EPB;
        o.apply64_t[IDX] = [](int grid, hipStream_t s, const Geom &g, const Tables &t,
                              const double *H, const double *v, double *yE) {
            hipLaunchKernelGGL((k3_apply<P, NQ, double, double, false, T2>), dim3(grid),
                               dim3(BLOCK), 0, s, g, t, H, v, yE);
        };
        o.apply32_t[IDX] = [](int grid, hipStream_t s, const Geom &g, const Tables &t,
                              const float *H, const double *v, float *yE) {
            hipLaunchKernelGGL((k3_apply<P, NQ, float, float, false, T2>), dim3(grid),
                               dim3(BLOCK), 0, s, g, t, H, v, yE);
        };
        if constexpr (T2 == 2) {
            // the base shape: plain_k3, which chooses the column form
            o.applyc64_t[IDX] = o.applyc64;
            o.applyc32_t[IDX] = o.applyc32;
            if constexpr (flat_apply3<P, NQ, double>()) {
                o.apply64 = [](int grid, hipStream_t s, const Geom &g, const Tables &t,
                               const double *H, const double *v, double *yE) {
                    if (g.lim != 0.0)
                        hipLaunchKernelGGL((k3_apply<P, NQ, double, double, true>), dim3(grid),
                                           dim3(BLOCK), 0, s, g, t, H, v, yE);
                    else if (grid >= FLAT_MIN)
                        hipLaunchKernelGGL((k3_apply<P, NQ, double, double, false, 2, true>),
                                           dim3(grid), dim3(BLOCK), 0, s, g, t, H, v, yE);
                    else
                        hipLaunchKernelGGL((k3_apply<P, NQ, double, double, false>), dim3(grid),
                                           dim3(BLOCK), 0, s, g, t, H, v, yE);
                };
                o.apply64_t[IDX] = o.apply64;
            }
            if constexpr (flat_apply3<P, NQ, float>()) {
                o.apply32 = [](int grid, hipStream_t s, const Geom &g, const Tables &t,
                               const float *H, const double *v, float *yE) {
                    if (g.lim != 0.0)
                        hipLaunchKernelGGL((k3_apply<P, NQ, float, float, true>), dim3(grid),
                                           dim3(BLOCK), 0, s, g, t, H, v, yE);
                    else if (grid >= FLAT_MIN)
                        hipLaunchKernelGGL((k3_apply<P, NQ, float, float, false, 2, true>),
                                           dim3(grid), dim3(BLOCK), 0, s, g, t, H, v, yE);
                    else
                        hipLaunchKernelGGL((k3_apply<P, NQ, float, float, false>), dim3(grid),
                                           dim3(BLOCK), 0, s, g, t, H, v, yE);
                };
                o.apply32_t[IDX] = o.apply32;
            }
        } else {
            o.applyc64_t[IDX] = [](int grid, hipStream_t s, const Geom &g, const Tables &t,
                                   const Target &w, const double *Q, const double *v, double *yE) {
                hipLaunchKernelGGL((k3_applyc<P, NQ, double, double, false, T2>), dim3(grid),
                                   dim3(BLOCK), 0, s, g, t, w, Q, v, yE);
            };
            o.applyc32_t[IDX] = [](int grid, hipStream_t s, const Geom &g, const Tables &t,
                                   const Target &w, const float *Q, const double *v, float *yE) {
                hipLaunchKernelGGL((k3_applyc<P, NQ, float, float, false, T2>), dim3(grid),
                                   dim3(BLOCK), 0, s, g, t, w, Q, v, yE);
            };
        }
    } else {
        o.epb_t[IDX] = 0;
        o.apply64_t[IDX] = nullptr;
        o.apply32_t[IDX] = nullptr;
        o.applyc64_t[IDX] = nullptr;
        o.applyc32_t[IDX] = nullptr;
    }
}

// Matrix-core forward sweeps (forward3_mfma) where the class has them.
template <int P, int NQ>
inline void fill_mfma3(Ops &o)
{
    if constexpr (3 * NQ <= 16) {
        o.energyM = [](int grid, hipStream_t s, const Geom &g, const Tables &t, const Target &w,
                       const double *x, double *part) {
            hipLaunchKernelGGL((k3_energy<P, NQ, false, true>), dim3(grid), dim3(BLOCK), 0, s, g,
                               t, w, x, part);
        };
        o.gradientM = [](int grid, hipStream_t s, const Geom &g, const Tables &t,
                         const Target &w, const double *x, double *gE, double *part) {
            hipLaunchKernelGGL((k3_gradient<P, NQ, false, false, true>), dim3(grid), dim3(BLOCK),
                               0, s, g, t, w, x, gE, part);
        };
        o.gradientEM = [](int grid, hipStream_t s, const Geom &g, const Tables &t,
                          const Target &w, const double *x, double *gE, double *part) {
            hipLaunchKernelGGL((k3_gradient<P, NQ, false, true, true>), dim3(grid), dim3(BLOCK),
                               0, s, g, t, w, x, gE, part);
        };
        o.setupM64 = [](int grid, hipStream_t s, const Geom &g, const Tables &t,
                        const Target &w, const double *x, double *H) {
            hipLaunchKernelGGL((k3_setup<P, NQ, double, true>), dim3(grid), dim3(BLOCK), 0, s, g,
                               t, w, x, H);
        };
        o.setupcM64 = [](int grid, hipStream_t s, const Geom &g, const Tables &t,
                         const Target &w, const double *x, double *Q) {
            hipLaunchKernelGGL((k3_setupc<P, NQ, double, true>), dim3(grid), dim3(BLOCK), 0, s,
                               g, t, w, x, Q);
        };
    } else {
        o.energyM = nullptr;
        o.gradientM = nullptr;
        o.gradientEM = nullptr;
        o.setupM64 = nullptr;
        o.setupcM64 = nullptr;
    }
}

// Setup with the element diagonal (b3_setupd, b3_setupcd) where the class's
// points fit one pass of the workgroup.
template <int P, int NQ>
inline void fill_setupd3(Ops &o)
{
    if constexpr (S3<P, NQ>::EPB * S3<P, NQ>::NQ3 <= BLOCK) {
        o.setupd64 = [](int grid, hipStream_t s, const Geom &g, const Tables &t, const Target &w,
                        const double *x, double *H, double *dE) {
            if (g.lim != 0.0)
                hipLaunchKernelGGL((k3_setupd<P, NQ, double, true>), dim3(grid), dim3(BLOCK), 0, s,
                                   g, t, w, x, H, dE);
            else if (hold_setup3<P, NQ, true>() && g.ne >= hold_setup3_min<NQ>())
                hipLaunchKernelGGL((k3_setupd<P, NQ, double, false, hold_setup3<P, NQ, true>()>),
                                   dim3(grid), dim3(BLOCK), 0, s, g, t, w, x, H, dE);
            else
                hipLaunchKernelGGL((k3_setupd<P, NQ, double, false>), dim3(grid), dim3(BLOCK), 0, s,
                                   g, t, w, x, H, dE);
        };
        o.setupd32 = [](int grid, hipStream_t s, const Geom &g, const Tables &t, const Target &w,
                        const double *x, float *H, double *dE) {
            if (g.lim != 0.0)
                hipLaunchKernelGGL((k3_setupd<P, NQ, float, true>), dim3(grid), dim3(BLOCK), 0, s,
                                   g, t, w, x, H, dE);
            else
                hipLaunchKernelGGL((k3_setupd<P, NQ, float, false>), dim3(grid), dim3(BLOCK), 0, s,
                                   g, t, w, x, H, dE);
        };
        o.setupcd64 = [](int grid, hipStream_t s, const Geom &g, const Tables &t, const Target &w,
                         const double *x, double *Q, double *dE) {
            if (g.lim != 0.0)
                hipLaunchKernelGGL((k3_setupcd<P, NQ, double, true>), dim3(grid), dim3(BLOCK), 0, s,
                                   g, t, w, x, Q, dE);
            else
                hipLaunchKernelGGL((k3_setupcd<P, NQ, double, false>), dim3(grid), dim3(BLOCK), 0,
                                   s, g, t, w, x, Q, dE);
        };
        o.setupcd32 = [](int grid, hipStream_t s, const Geom &g, const Tables &t, const Target &w,
                         const double *x, float *Q, double *dE) {
            if (g.lim != 0.0)
                hipLaunchKernelGGL((k3_setupcd<P, NQ, float, true>), dim3(grid), dim3(BLOCK), 0, s,
                                   g, t, w, x, Q, dE);
            else
                hipLaunchKernelGGL((k3_setupcd<P, NQ, float, false>), dim3(grid), dim3(BLOCK), 0, s,
                                   g, t, w, x, Q, dE);
        };
    } else {
        o.setupd64 = nullptr;
        o.setupd32 = nullptr;
        o.setupcd64 = nullptr;
        o.setupcd32 = nullptr;
    }
}

template <int P, int NQ, typename TT, bool COMPACT>
inline void apply_l2_3(hipStream_t s, const Geom &g, const Tables &t, const Target &w, const void *H,
                       const MrL2 &a, void *yE)
{
    constexpr int EPB = S3<P, NQ>::EPB;
    hipLaunchKernelGGL((k3_apply_l2<P, NQ, TT, COMPACT>), dim3((g.ne + EPB - 1) / EPB), dim3(BLOCK), 0,
                       s, g, t, w, (const TT *)H, a, (TT *)yE);
}

template <int P, int NQ>
inline void fill_tiles_k3(Ops &o)
{
    if constexpr (S3<P, NQ>::NQ3 <= BLOCK) {
        o.apply_l2[0][0] = apply_l2_3<P, NQ, double, false>;
        o.apply_l2[0][1] = apply_l2_3<P, NQ, float, false>;
        o.apply_l2[1][0] = apply_l2_3<P, NQ, double, true>;
        o.apply_l2[1][1] = apply_l2_3<P, NQ, float, true>;
    }
    if constexpr (hold_setup3<P, NQ, false>())
        o.setup64 = [](int grid, hipStream_t s, const Geom &g, const Tables &t, const Target &w,
                       const double *x, double *H) {
            if (g.ne >= hold_setup3_min<NQ>())
                hipLaunchKernelGGL((k3_setup<P, NQ, double, false, true>), dim3(grid), dim3(BLOCK),
                                   0, s, g, t, w, x, H);
            else
                hipLaunchKernelGGL((k3_setup<P, NQ, double>), dim3(grid), dim3(BLOCK), 0, s, g, t, w,
                                   x, H);
        };
    fill_tile3<P, NQ, 1, 0>(o);
    fill_tile3<P, NQ, 2, 1>(o);
    fill_tile3<P, NQ, 4, 2>(o);
    fill_mfma3<P, NQ>(o);
    fill_setupd3<P, NQ>(o);
}

template <int P, int NQ, int T2, int IDX>
inline void fill_btile3(BOps &o)
{
    if constexpr (tile_ok3<P, NQ, T2>()) {
        o.epb_t[IDX] = S3<P, NQ, T2>::EPB;
        o.apply_t[0][0][IDX] = [](int grid, hipStream_t s, const Tables &t, const Tile *tl,
                                  const SlotDev *sl, const int *gt, int vin, double *) {
            hipLaunchKernelGGL((kb3_apply<P, NQ, double, double, false, T2>), dim3(grid), dim3(BLOCK),
                               0, s, t, tl, sl, gt, vin);
        };
        o.apply_t[0][1][IDX] = [](int grid, hipStream_t s, const Tables &t, const Tile *tl,
                                  const SlotDev *sl, const int *gt, int vin, double *) {
            hipLaunchKernelGGL((kb3_apply<P, NQ, float, float, false, T2>), dim3(grid), dim3(BLOCK), 0,
                               s, t, tl, sl, gt, vin);
        };
        o.apply_t[1][0][IDX] = [](int grid, hipStream_t s, const Tables &t, const Tile *tl,
                                  const SlotDev *sl, const int *gt, int vin, double *) {
            hipLaunchKernelGGL((kb3_applyc<P, NQ, double, double, false, T2>), dim3(grid), dim3(BLOCK),
                               0, s, t, tl, sl, gt, vin);
        };
        o.apply_t[1][1][IDX] = [](int grid, hipStream_t s, const Tables &t, const Tile *tl,
                                  const SlotDev *sl, const int *gt, int vin, double *) {
            hipLaunchKernelGGL((kb3_applyc<P, NQ, float, float, false, T2>), dim3(grid), dim3(BLOCK), 0,
                               s, t, tl, sl, gt, vin);
        };
    } else {
        o.epb_t[IDX] = 0;
        for (int a = 0; a < 2; ++a)
            for (int b = 0; b < 2; ++b) o.apply_t[a][b][IDX] = nullptr;
    }
}

template <int P, int NQ>
inline void fill_tiles_kb3(BOps &o)
{
    fill_bcol3<P, NQ, double, 0>(o);
    fill_bcol3<P, NQ, float, 1>(o);
    fill_btile3<P, NQ, 1, 0>(o);
    fill_btile3<P, NQ, 2, 1>(o);
    fill_btile3<P, NQ, 4, 2>(o);
}

}  // namespace tmop
