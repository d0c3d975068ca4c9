// Host launchers of the node-level kernels (vec.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tmop_dev.hpp"

namespace tmop {

// Device-resident scalar state of one MINRES solve.
struct MinresState {
    double tmp;
    double beta1, beta, oldb, alpha, dbar, eps, oldeps, phibar, phi, cs, sn, gamma, delta, rtol;
    int its;
    int stop;  // last iteration index that runs; INT_MAX while running
    int indefinite_precond;
    int pad;
};

// Scalars of one MINRES update, kept when the Lanczos vectors stay resident
// and the solution is formed once after the loop: the update m takes
// w_m = (v_m - oldeps w_{m-2} - delta w_{m-1}) ig and x += phi w_m, with
// v_m = sv z_m (z_m the unscaled preconditioned Lanczos vector).
struct MrHist {
    double ig, oldeps, delta, phi, sv;
    double pad[3];
};
// Most updates one combination can take (one lane per coefficient).
constexpr int MR_MAX_BASIS = 256;
// The second Lanczos update of iteration j (k_mr_l2), done by the next
// iteration's element kernel as it gathers its input: z = M^{-1}(hv - alpha /
// beta r2), alpha the sum of part1[0..nb1).  The new hv goes to hvo, another
// buffer, since elements share nodes; part2 gets a partial of beta^2 per
// workgroup.
struct MrL2 {
    const double *hv, *r2, *minv;
    double *hvo, *z, *part2;
    const double *part1;
    int nb1, j;
    const MinresState *st;
};
// Most workgroups of an element kernel that does so (each of the next
// kernel's sums their partials).  Below it the solve waits for launches, some
// 4 us each: hex 8^3 p3 n_q5 (256 workgroups) 16.2 -> 13.5 us per iteration.
constexpr int MR_L2_GRID = 1024;
// A MINRES solve in one launch (minres_one.hpp): dx = H_c^{-1} b with the Lanczos vectors z_j in
// bank (as in minres_resident), at most max_its iterations.  mst[0] and
// mst[1] get the final state.
struct MrOne {
    const int32_t *ptr, *ent;
    const void *H;
    void *eV;
    const double *b, *minv;
    double *r1, *r2, *bank;
    long stride;
    double *dx;
    MinresState *mst;
    double rtol;
    int max_its;
};

// DoFs per vector tile (workgroup of VTILE_LANES lanes) of a pool slot: three per
// lane, and on large slots so many that the slot has at most VTILE_MAX tiles.
// Every workgroup of the two MINRES vector kernels sums the partials of all of
// its slot's tiles, so their reads grow with the square of the tile count: with
// three per lane throughout, a lockstep position of one 48^3 p = 4 slot (28000
// tiles) took 1818 us, of one 64^3 p = 2 slot 465, of one 32^3 p = 4 slot 357;
// so limited they take 941, 396 and 287.
constexpr int VTILE_LANES = 256;
constexpr int VTILE_MAX = 1024;
inline int vtile_dofs(int ndof)
{
    const long per = (long)VTILE_LANES * VTILE_MAX;
    const int k = (int)((ndof + per - 1) / per);
    return VTILE_LANES * (k > 3 ? k : 3);
}

void launch_gather(const Geom &g, const int32_t *csr_ptr, const int32_t *csr_ent, const void *eV,
                   bool fp32, double *out, int fix_mode, const double *src, hipStream_t s);
// Energy partials are reduced in slices of ESLICE, or of a multiple of it so
// that there are at most NSLICE slices (vec.hip).  Scratch of
// launch_energy_reduce: 3 NSLICE doubles; of launch_gather_norm:
// ENERGY_SCRATCH.
constexpr int ESLICE = 1024;
constexpr int NSLICE = 2048;
constexpr int ENERGY_SCRATCH = 3 * NSLICE + NSLICE;
inline __host__ __device__ int energy_slice_len(int nb)
{
    const int n = (nb + ESLICE - 1) / ESLICE;
    return ESLICE * ((n + NSLICE - 1) / NSLICE);
}
inline int energy_slices(int nb) { return (nb + energy_slice_len(nb) - 1) / energy_slice_len(nb); }
// Most nodes of a mesh whose gradient is gathered by one workgroup of 1024
// lanes that also sums everything up.  Against one launch more (3 to 4 us) a
// lane's nodes follow one another, each a chain of dependent loads, on quads of
// up to 4, on hexes 8 copies, on general meshes through the element lists.
// Energy + gradient, us, one workgroup / several: box quads p1 1640 nodes 21.8 /
// 23.1, 2254 (p3) 22.9 / 23.6, 2970 23.5 / 23.1; box hexes p2 729 23.3 / 25.0, p1
// 1320 25.1 / 24.7, 3360 32.8 / 25.6; element lists: quads p1 650 22.4 / 24.2,
// 1122 24.5 / 24.5, 4032 32.4 / 24.1; hexes p1 720 26.4 / 28.1, 1320 35.1 / 27.7,
// 3360 59.4 / 28.8.
inline int gn_one_nodes(const Geom &g) { return g.dim == 2 && !g.e2n ? 2048 : 1024; }
// F, min det, count of points with det T <= 0 from nb energy partials: to out[0..2].
void launch_energy_reduce(const double *part, int nb, double *sl, double *out, hipStream_t s);
// The gradient G^T eV (fixed DoFs 0) to grad, the reduced energy partials to
// out[0..2] and |grad|^2 to out[8].
void launch_gather_norm(const Geom &g, const int32_t *csr_ptr, const int32_t *csr_ent,
                        const double *eV, double *grad, const double *part, int nb, double *sl,
                        double *out, hipStream_t s);
void launch_reduce_sum(const double *part, int nb, double *out, hipStream_t s);
int reduce_blocks(long n);
void launch_dot(long n, const double *a, const double *b, double *part, double *out,
                hipStream_t s);
void launch_absmax(long n, const double *a, double *part, double *out, hipStream_t s);
void launch_step(long n, const double *x, const double *dx, double alpha, double *xt,
                 hipStream_t s);
void launch_jacobi(long n, const double *d, const double *dmax, double *minv, hipStream_t s);

void mr_init(long n, const double *b, const double *minv, double *r1, double *r2, double *y,
             double *v, double *x, double *w, double *w1, double *w2, double *part,
             MinresState *st, double rtol, hipStream_t s);
void mr_gather_upd(const Geom &g, const int32_t *csr_ptr, const int32_t *csr_ent, const void *eV,
                   bool fp32, int j, const MinresState *sin, MinresState *sout,
                   const double *p1prev, const double *p2prev, const double *zp, const double *zc,
                   const double *w1, const double *w2, double *wout, double *x, double *r1hv,
                   double *part, MrHist *hist, unsigned long long *progress, int nb2, hipStream_t s);
// What mr_gather_upd writes to progress: gathers begun, and in the upper half
// whether the solve has stopped.
inline __host__ __device__ unsigned long long mr_progress(int begun, bool stopped)
{
    return (unsigned long long)begun | ((unsigned long long)stopped << 32);
}
// Workgroups of mr_gather_upd, i.e. the count of its partials (nb1 below);
// at most MR_MAX_PARTIALS.
int mr_gather_grid(const Geom &g);
constexpr int MR_MAX_PARTIALS = 2048;
void mr_lanczos2(long n, int nb1, int j, const MinresState *st, const double *part1, double *hv,
                 const double *r2, const double *minv, double *z, double *part2, hipStream_t s);
void mr_finish(long n, int nb1, int jm, const MinresState *sin, MinresState *sout,
               const double *p1, const double *p2, const double *zp, const double *w1,
               const double *w2, double *wout, double *x, hipStream_t s);
void mr_combine(long n, int nb1, int jm, const MinresState *sin, MinresState *sout,
                const double *p1, const double *p2, MrHist *hist, const double *bank, long stride,
                double *x, hipStream_t s);

}  // namespace tmop
