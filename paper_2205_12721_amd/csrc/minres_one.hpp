// All of preconditioned MINRES in one workgroup, for the smallest meshes.
#pragma once
#include "gather.hpp"
#include "kernels2d.hpp"
#include "minres_dev.hpp"

namespace tmop {

constexpr int MR1_V = 4, MR1_LANES = MR1_V * BLOCK;  // blocks of elements at once
constexpr int MR1_NODES = 2;                         // nodes per lane

// Sum over the workgroup, to every lane; one barrier.  red: MR1_LANES / 64
// doubles that no lane still reads.
__device__ __forceinline__ double mr1_sum(double v, double *red, int tid)
{
    constexpr int NW = MR1_LANES / 64;
    v = wave_sum(v);
    if ((tid & 63) == 0) red[tid >> 6] = v;
    __syncthreads();
    double s = red[tid & (NW - 1)];
#pragma unroll
    for (int k = 1; k < NW; k *= 2) s += __shfl_xor(s, k);
    return s;
}

// One iteration needs the whole of <v, H v> before the new z, and the whole of
// beta^2 before the next v: over several workgroups those are three launches
// of 3 to 4 us each (quads 8 x 8, p = 2), nearly all of it latency.  Here
// they are barriers of one workgroup, and nothing leaves the compute unit but
// through its L1 and L2.  Vectors stay in global memory, where the element
// kernel's code reads and writes them; a lane keeps its nodes' entries in
// registers from the gather to the new z.  The scalar recurrence is done by
// the last wave, which has the least to do in the next element stage.
template <int P, int NQ, typename TT, bool COMPACT>
__global__ __launch_bounds__(MR1_LANES) void k2_minres_one(Geom g, BasisTables tba, Target tg, MrOne a)
{
    const Tab tb = kernel_tables<sizeof(Geom)>();
    constexpr int DIM = 2, EPB = S2<P, NQ>::EPB;
    __shared__ double red[2][MR1_LANES / 64];
    __shared__ MrHist hist[MR_MAX_BASIS];
    __shared__ double coef[MR_MAX_BASIS];
    __shared__ MinresState S;
    const int tid = threadIdx.x + BLOCK * threadIdx.y;
    TT *eV = (TT *)a.eV;
    double s = 0.0;
    for (int node = tid; node < g.nx; node += MR1_LANES)
#pragma unroll
        for (int c = 0; c < DIM; ++c) {
            const size_t idx = (size_t)c * g.nx + node;
            const double bi = a.b[idx], yi = a.minv ? a.minv[idx] * bi : bi;
            a.r1[idx] = bi;
            a.r2[idx] = bi;
            a.bank[idx] = yi;
            s += bi * yi;
        }
    s = mr1_sum(s, red[0], tid);
    if (tid == 0) S = mr_state0(s, a.rtol);
    double *R1 = a.r1, *R2 = a.r2;
    __syncthreads();
    for (int j = 0; j < a.max_its; ++j) {
        const double *z = a.bank + (size_t)j * a.stride;
        double *zn = a.bank + (size_t)(j + 1) * a.stride;
        for (int b0 = 0; b0 < g.ne; b0 += MR1_V * EPB) {
            const int e0 = b0 + (int)threadIdx.y * EPB;
            const int nel = min(max(g.ne - e0, 0), EPB);
            if constexpr (COMPACT)
                b2_applyc<P, NQ, TT, TT, false, MR1_V>(g, tb, tg, (const TT *)a.H, z, eV, e0, nel);
            else
                b2_apply<P, NQ, TT, TT, false, MR1_V>(g, tb, (const TT *)a.H, z, eV, e0, nel);
            __syncthreads();
        }
        // S: the state after the update of iteration j - 1
        if (j > S.stop) break;
        const double beta = S.beta, sc = beta > 0.0 ? 1.0 / beta : 0.0;
        const double cr = j >= 1 ? beta / S.oldb : 0.0;
        // (the lane's node numbers are opaque here: what follows from them,
        // kept from one iteration to the next, would not fit the registers)
        int node0 = tid;
        asm volatile("" : "+v"(node0));
        double h[MR1_NODES][DIM], q2[MR1_NODES][DIM], mi[MR1_NODES][DIM];
        s = 0.0;
#pragma unroll
        for (int k = 0; k < MR1_NODES; ++k) {
            const int node = node0 + k * MR1_LANES;
            if (node >= g.nx) continue;
            double y[DIM], zv[DIM], q1[DIM];
            bool fixed[DIM];
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                const size_t idx = (size_t)c * g.nx + node;
                zv[c] = z[idx];
                q1[c] = R1[idx];
                q2[k][c] = R2[idx];
                mi[k][c] = a.minv ? a.minv[idx] : 1.0;
            }
            gather_node<DIM, TT>(g, a.ptr, a.ent, eV, node, y, fixed);
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                const double vi = sc * zv[c];
                double t = fixed[c] ? vi : sc * y[c];
                if (j >= 1) t -= cr * q1[c];
                h[k][c] = t;
                s += vi * t;
            }
        }
        const double alpha = mr1_sum(s, red[1], tid), ab = alpha / beta;
        s = 0.0;
#pragma unroll
        for (int k = 0; k < MR1_NODES; ++k) {
            const int node = node0 + k * MR1_LANES;
            if (node >= g.nx) continue;
#pragma unroll
            for (int c = 0; c < DIM; ++c) {
                const size_t idx = (size_t)c * g.nx + node;
                const double t = h[k][c] - ab * q2[k][c];
                const double zi = a.minv ? mi[k][c] * t : t;
                R1[idx] = t;
                zn[idx] = zi;
                s += t * zi;
            }
        }
        const double bb = mr1_sum(s, red[0], tid);
        if (tid >= MR1_LANES - 64) {
            const MrUpd u = mr_scalars(S, j, alpha, bb);
            if (tid == MR1_LANES - 1) {
                S = u.o;
                hist[j] = MrHist{u.ig, u.oldeps, u.delta, u.phi, sc, {}};
            }
        }
        double *t = R1;  // r1 <- r2, r2 <- hv
        R1 = R2;
        R2 = t;
    }
    __syncthreads();
    // dx = sum_i c_i v_i, the coefficients as in k_mr_combine
    const int K = S.its;
    if (tid < K) {
        double a2 = 0.0, a1 = 0.0, c = 0.0;
        for (int m = tid; m < K; ++m) {
            const double wn = ((m == tid ? 1.0 : 0.0) - hist[m].oldeps * a2 - hist[m].delta * a1) * hist[m].ig;
            c += hist[m].phi * wn;
            a2 = a1;
            a1 = wn;
        }
        coef[tid] = c * hist[tid].sv;
    }
    __syncthreads();
    for (int i = tid; i < DIM * g.nx; i += MR1_LANES) {
        double acc = 0.0;
#pragma unroll 4
        for (int m = 0; m < K; ++m) acc += coef[m] * a.bank[(size_t)m * a.stride + i];
        a.dx[i] = acc;
    }
    if (tid < 2) a.mst[tid] = S;
}

// Used up to two passes over MR1_V blocks of elements, one at p = 4, and two
// nodes per lane.  us per iteration, three launches -> one: p1 n_q2 8x8 16.6 ->
// 4.9, 20x20 16.9 -> 10.8, 32x32 (4 passes) 17.1 -> 22.9; p2 n_q4 4x4 16.0 ->
// 5.1, 8x8 16.8 -> 7.5, 10x10 17.0 -> 10.3, 16x16 (4 passes) 16.8 -> 20.8; p3
// n_q5 6x6 16.7 -> 8.8, 8x8 17.0 -> 13.2, 10x10 (3 passes) 17.2 -> 18.2; p4 n_q5
// 6x6 17.9 -> 10.8, 8x8 (2 passes) 18.3 -> 16.9; p4 n_q7 4x4 18.6 -> 14.7, 6x6
// (2 passes) 19.3 -> 26.3: one compute unit is busy with the point work there.
template <int P, int NQ, typename TT, bool COMPACT>
inline bool minres_one2(hipStream_t s, const Geom &g, const Tables &t, const Target &w, const MrOne &a)
{
    constexpr int ELEMS = (P <= 3 ? 2 : 1) * MR1_V * S2<P, NQ>::EPB;
    if (g.nx > MR1_NODES * MR1_LANES || g.ne > ELEMS || a.max_its >= MR_MAX_BASIS) return false;
    hipLaunchKernelGGL((k2_minres_one<P, NQ, TT, COMPACT>), dim3(1), dim3(BLOCK, MR1_V), 0, s, g, t, w,
                       a);
    return true;
}

}  // namespace tmop
