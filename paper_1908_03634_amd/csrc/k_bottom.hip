// k_bottom.hip -- Krylov solve of the coarsest grid in one workgroup.
//
// Runs where the grid that ends the hierarchy is not solved directly (more
// than kDirectBottomCells cells, or cells that are not all coupled) and does
// not end the single-workgroup coarse cycle: extents that stop halving early
// (25 x 15 x 11 below 200 x 120 x 88) and one-level grids.
//
// BiCGStab in FP64 to ||r|| <= rtol ||r0||.  An iteration is a serial chain of
// stencil passes and global sums over a few thousand cells, so latency and the
// LDS of one CU bound it, not memory: vectors stay on chip (the search direction,
// the residual and the shadow residual in LDS, where the stencil reads its
// neighbours; the rest, the coefficients and the neighbour indices in
// registers), sums are vector-pipeline wavefront sums and one LDS exchange with
// one barrier each, and sums of the same data share that exchange: five
// barriers an iteration.  An iteration takes 2.6 us at 891 cells, 4.1 us at 3003
// and 7.1 us at 25 x 15 x 11 (FP32 coefficients; 13.5 us with FP64 ones), 30 us at
// 25 x 15 x 11 with every vector in global memory and the cells labelled on every
// call; beyond 5120 cells, vectors in global memory, 47 us at 15625 (91 us before).
//
// A solve that ends without the tolerance returns the iterate of the smallest
// residual.  Each step copies that iterate to global memory as it leaves it, a
// store that nothing waits for: 2% of an iteration where vectors are in global
// memory and 6% where FP64 coefficients already spill (3073 to 5120 cells).
// (25^3 cells capped at 40 iterations, nine solves: 22.8 ms; 44.3 ms when the
// solve was run again up to that iterate, 46.7 ms by the form before that.)
#include "mp_device.h"
#include "mp_kernels.h"
#include "mp_krylov.h"
#include <type_traits>

namespace mp {

namespace {

__device__ __forceinline__ double block_min(double v, double* sh)
{
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, kWave));
    const int w = (int)threadIdx.x / kWave, nw = (int)blockDim.x / kWave;
    __syncthreads();
    if ((threadIdx.x & (kWave - 1)) == 0) sh[w] = v;
    __syncthreads();
    double s = sh[0];
    for (int q = 1; q < nw; q++) s = fmin(s, sh[q]);
    return s;
}

// Neighbour indices of a cell, 14 bits each (grids of at most 16384 cells), and
// whether its high faces lie inside the domain.
struct PackedNb {
    unsigned x, y, z;
    __device__ __forceinline__ PackedNb() : x(0), y(0), z(0) {}
    __device__ __forceinline__ explicit PackedNb(const Nb32& b)
        : x((unsigned)b.xm | ((unsigned)b.xp << 14) | ((unsigned)b.hx << 28)),
          y((unsigned)b.ym | ((unsigned)b.yp << 14) | ((unsigned)b.hy << 28)),
          z((unsigned)b.zm | ((unsigned)b.zp << 14) | ((unsigned)b.hz << 28))
    {
    }
    static __device__ __forceinline__ int lo(unsigned v) { return (int)(v & 0x3fffu); }
    static __device__ __forceinline__ int hi(unsigned v) { return (int)((v >> 14) & 0x3fffu); }
    static __device__ __forceinline__ bool in(unsigned v) { return (v >> 28) != 0u; }
};

// The six face coefficients of cell q (x low, x high, y low, ...; 0 on walls).
template <typename T>
__device__ __forceinline__ void face6(const T* __restrict__ cx, const T* __restrict__ cy, const T* __restrict__ cz,
                                      int q, const PackedNb& nb, T (&c)[6])
{
    const T xh = cx[PackedNb::hi(nb.x)], yh = cy[PackedNb::hi(nb.y)], zh = cz[PackedNb::hi(nb.z)];
    c[0] = cx[q];
    c[1] = PackedNb::in(nb.x) ? xh : T(0);
    c[2] = cy[q];
    c[3] = PackedNb::in(nb.y) ? yh : T(0);
    c[4] = cz[q];
    c[5] = PackedNb::in(nb.z) ? zh : T(0);
}

}  // namespace

// 1024 / VJ threads, cell q = tid + threads * m.  Fewer wavefronts with more
// cells each: the exchanges cost less and a thread has the registers for its
// cells' coefficients; too few cannot hide the LDS reads' latency.  M > 0: at
// most M cells per thread, on chip.  M = 0: any number of cells, vectors and
// neighbour indices in `work` (kBottomWork doubles per cell; labels there in
// every form).  Sums run as in 1024 threads (or, below 1024 cells, one per
// cell): cell m of a thread belongs to partial sum m % VJ.
template <typename T, int VJ, int M>
__global__ __launch_bounds__(1024 / VJ) void k_bottom(Dims d, const T* __restrict__ bin, T* __restrict__ xout,
                                                 const T* __restrict__ cx, const T* __restrict__ cy,
                                                 const T* __restrict__ cz, double h2, double rtol, int maxit,
                                                 int use_x0, double* __restrict__ work, double* __restrict__ iters,
                                                 const double* __restrict__ skip_if_direct)
{
    constexpr int N = M > 0 ? M : 1;
    constexpr int TH = 1024 / VJ;
    constexpr bool HOLD = M > 0 && VJ > 1;
    using HT = std::conditional_t<(M > 6), T, double>;  // (six cells' FP64 coefficients fit, ten cells' do not)
    // what the stencil is applied to: M > 0 the search direction and the
    // residual each in its own buffer, M = 0 both in one in turn
    __shared__ double bufA[M > 0 ? TH * M : 16384];
    __shared__ double bufB[M > 0 ? TH * M : 1];
    __shared__ double bufH[M > 0 ? TH * M : 1];
    __shared__ double red[2][2][kWaves];
    __shared__ double shm[kWaves];
    if (skip_if_direct && skip_if_direct[0] == 1.0) return;
    const int n = (int)d.n();
    const int tid = (int)threadIdx.x, nt = TH;
    double* lab = work;
    double* const xb = work + 9 * (long long)n;  // the iterate of the smallest residual
    double* const vb = M > 0 ? bufB : bufA;
    const double inv_h2 = 1.0 / h2;
    int half = 0;

    PackedNb rnb[N];
    HT rc[HOLD ? N : 1][6];
    double rx[N], rv[N], rt[N];
    auto cell = [&](int u) { return tid + nt * u; };
    auto live = [&](int u) { return M == 0 || cell(u) < n; };
    // f(u, u % VJ) for every cell of this thread.  M > 0: the M slots without a
    // branch (their LDS reads issue together); a slot past the last cell has
    // coefficients and vectors of 0, and its own place in LDS
    auto each = [&](auto f) {
        if constexpr (M > 0) {
#pragma unroll
            for (int u = 0; u < M; u++) {
                f(u, u % VJ);
                if (M > 4 && u % 2 == 1) __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll 1
            for (int u = 0; cell(u) < n; u += VJ) {
#pragma unroll
                for (int j = 0; j < VJ; j++)
                    if (cell(u + j) < n) f(u + j, j);
            }
        }
    };
    auto X = [&](int u) -> double& {
        if constexpr (M > 0) return rx[u];
        else return work[n + cell(u)];
    };
    auto R = [&](int u) -> double& {  // residual r, then s = r - alpha v
        if constexpr (M > 0) return bufB[cell(u)];
        else return work[2 * n + cell(u)];
    };
    auto H = [&](int u) -> double& {  // shadow residual
        if constexpr (M > 0) return bufH[cell(u)];
        else return work[3 * n + cell(u)];
    };
    auto P = [&](int u) -> double& {
        if constexpr (M > 0) return bufA[cell(u)];
        else return work[4 * n + cell(u)];
    };
    auto V = [&](int u) -> double& {
        if constexpr (M > 0) return rv[u];
        else return work[5 * n + cell(u)];
    };
    auto TV = [&](int u) -> double& {
        if constexpr (M > 0) return rt[u];
        else return work[6 * n + cell(u)];
    };
    auto NB = [&](int u) -> PackedNb& {
        if constexpr (M > 0) return rnb[u];
        else return reinterpret_cast<PackedNb*>(work + 7 * n)[cell(u)];
    };
    // the vector the stencil reads next (M > 0: it is where R and P live)
    auto publish = [&](int u, double v) {
        if constexpr (M == 0) bufA[cell(u)] = v;
    };

    // every face inside the domain nonzero: one connected part (the usual
    // case; a grid that fails this may still be one)
    double cut[1][VJ] = {}, s1[1], s2[2];
    each([&](int u, int g) {
        const int q = cell(u);
        const int t = q / d.nx, k = t / d.ny, j = t - k * d.ny, i = q - t * d.nx;
        PackedNb nb;
        T k6[6] = {};
        if (live(u)) {
            nb = PackedNb(nb32(d, q, i, j, k));
            face6<T>(cx, cy, cz, q, nb, k6);
        } else {
            nb.x = nb.y = nb.z = (unsigned)q | ((unsigned)q << 14);
        }
        NB(u) = nb;
        if constexpr (HOLD) {
#pragma unroll
            for (int f = 0; f < 6; f++) rc[u][f] = (HT)k6[f];
        }
        if (!live(u)) return;
        if (((i > 0 || d.px) && k6[0] == T(0)) || ((j > 0 || d.py) && k6[2] == T(0)) ||
            ((k > 0 || d.pz) && k6[4] == T(0)))
            cut[0][g] = 1.0;
    });
    totals<VJ, 1>(cut, s1, red, half);
    const bool parts = s1[0] != 0.0;
    if (parts) {
        // labels by minimum-label propagation (in place: the fixed point, each
        // part's smallest index, does not depend on the order of the updates)
        for (int q = tid; q < n; q += nt) lab[q] = (double)q;
        for (;;) {
            __syncthreads();
            double changed[1][VJ] = {};
#pragma unroll 1
            for (int q = tid; q < n; q += nt) {
                const int t = q / d.nx, k = t / d.ny, j = t - k * d.ny, i = q - t * d.nx;
                const PackedNb pn(nb32(d, q, i, j, k));
                T k6[6];
                face6<T>(cx, cy, cz, q, pn, k6);
                const int nq[6] = {PackedNb::lo(pn.x), PackedNb::hi(pn.x), PackedNb::lo(pn.y),
                                   PackedNb::hi(pn.y), PackedNb::lo(pn.z), PackedNb::hi(pn.z)};
                double m = lab[q];
                for (int f = 0; f < 6; f++)
                    if (k6[f] != T(0)) m = fmin(m, lab[nq[f]]);
                if (m < lab[q]) {
                    lab[q] = m;
                    changed[0][0] = 1.0;
                }
            }
            totals<VJ, 1>(changed, s1, red, half);
            if (s1[0] == 0.0) break;
        }
    }
    // TV(u) = mean of get(u) over the connected part of cell u (the constants
    // on the parts span the operator's null space)
    auto part_means = [&](auto get) {
        if (!parts) {
            double p[1][VJ] = {};
            each([&](int u, int g) { p[0][g] += live(u) ? get(u) : 0.0; });
            totals<VJ, 1>(p, s1, red, half);
            const double m = s1[0] / (double)n;
            each([&](int u, int) { TV(u) = m; });
            return;
        }
        double lo = (double)n;
        each([&](int u, int) {
            if (live(u)) lo = fmin(lo, lab[cell(u)]);
        });
        double cur = block_min(lo, shm);
        while (cur < (double)n) {
            double p[2][VJ] = {}, nxt = (double)n;
            each([&](int u, int g) {
                const double l = live(u) ? lab[cell(u)] : -1.0;
                if (l == cur) {
                    p[0][g] += get(u);
                    p[1][g] += 1.0;
                } else if (l > cur) {
                    nxt = fmin(nxt, l);
                }
            });
            totals<VJ, 2>(p, s2, red, half);
            const double m = s2[0] / s2[1];
            each([&](int u, int) {
                if (live(u) && lab[cell(u)] == cur) TV(u) = m;
            });
            cur = block_min(nxt, shm);
        }
    };
    // (A y)_q of the published vector y: the arithmetic of stencil_sums
    auto apply = [&](int u, const double* y) {
        const int q = cell(u);
        PackedNb nb = NB(u);
        double c[6];
        if constexpr (HOLD) {
#pragma unroll
            for (int f = 0; f < 6; f++) {
                HT k = rc[u][f];
                if constexpr (sizeof(HT) == 4) asm("" : "+v"(k));
                c[f] = (double)k;
            }
        } else {
            PackedNb nc = nb;
            if (!live(u)) nc.x = nc.y = nc.z = 0u;
            T k6[6];
            face6<T>(cx, cy, cz, live(u) ? q : 0, nc, k6);
#pragma unroll
            for (int f = 0; f < 6; f++) c[f] = live(u) ? (double)k6[f] : 0.0;
        }
        // (opaque to the compiler, which would else keep the unpacked indices
        // across iterations: more registers than there are)
        asm("" : "+v"(nb.x), "+v"(nb.y), "+v"(nb.z));
        const double cs = coef_sum<double>(c[0], c[1], c[2], c[3], c[4], c[5]);
        double s = c[0] * y[PackedNb::lo(nb.x)];
        s = fma(c[1], y[PackedNb::hi(nb.x)], s);
        s = fma(c[2], y[PackedNb::lo(nb.y)], s);
        s = fma(c[3], y[PackedNb::hi(nb.y)], s);
        s = fma(c[4], y[PackedNb::lo(nb.z)], s);
        s = fma(c[5], y[PackedNb::hi(nb.z)], s);
        return (cs * y[q] - s) * inv_h2;
    };

    part_means([&](int u) { return (double)bin[cell(u)]; });
    each([&](int u, int) {
        const double x0 = use_x0 && live(u) ? (double)xout[cell(u)] : 0.0;
        X(u) = x0;
        if constexpr (M > 0) P(u) = x0;
        publish(u, x0);
    });
    if (use_x0) __syncthreads();
    double p0[1][VJ] = {};
    each([&](int u, int g) {
        const double rq = live(u) ? ((double)bin[cell(u)] - TV(u)) - (use_x0 ? apply(u, bufA) : 0.0) : 0.0;
        R(u) = rq;
        H(u) = rq;
        V(u) = 0.0;
        p0[0][g] = fma(rq, rq, p0[0][g]);
    });
    totals<VJ, 1>(p0, s1, red, half);  // (all reads of the published x are done)
    each([&](int u, int) { P(u) = 0.0; });
    const double bnorm2 = s1[0], tol2 = rtol * rtol * bnorm2;
    double rho = 1.0, alpha = 1.0, omega = 1.0;
    // squared residual of the current iterate and of the best one, which is the
    // current one (`best`) or lies in xb: a step copies it there as it leaves it
    double rr_cur = bnorm2, rr_best = bnorm2, rho1 = bnorm2;
    bool best = true;
    int it = 0;  // iterations begun (each ends in a break or a full step)
    if (bnorm2 > 0.0) {
#pragma unroll 1
        for (; it < maxit; it++) {
            if (rho1 == 0.0) break;
            const double beta = (rho1 / rho) * (alpha / omega);
            each([&](int u, int) {
                const double p = R(u) + beta * (P(u) - omega * V(u));
                P(u) = p;
                publish(u, p);
            });
            __syncthreads();
            double a1[1][VJ] = {};
            each([&](int u, int g) {
                const double v = apply(u, bufA);
                V(u) = v;
                a1[0][g] = fma(H(u), v, a1[0][g]);
            });
            totals<VJ, 1>(a1, s1, red, half);
            if (s1[0] == 0.0) break;
            alpha = rho1 / s1[0];
            double a2[1][VJ] = {};
            each([&](int u, int g) {
                const double s = R(u) - alpha * V(u);
                R(u) = s;
                publish(u, s);
                a2[0][g] = fma(s, s, a2[0][g]);
            });
            totals<VJ, 1>(a2, s1, red, half);
            const double ss = s1[0];
            if (ss <= tol2) {
                each([&](int u, int) { X(u) += alpha * P(u); });
                rr_cur = ss;
                break;
            }
            double a3[2][VJ] = {};
            each([&](int u, int g) {
                const double t = apply(u, vb);
                TV(u) = t;
                a3[0][g] = fma(t, R(u), a3[0][g]);
                a3[1][g] = fma(t, t, a3[1][g]);
            });
            totals<VJ, 2>(a3, s2, red, half);
            if (s2[1] == 0.0) {
                rr_cur = ss;
                break;
            }
            omega = s2[0] / s2[1];
            // the residual's norm and the next iteration's rho1 share an exchange
            double a4[2][VJ] = {};
            each([&](int u, int g) {
                const double s = R(u), x = X(u);
                if (best && live(u)) xb[cell(u)] = x;
                X(u) = x + (alpha * P(u) + omega * s);
                const double r = s - omega * TV(u);
                R(u) = r;
                a4[0][g] = fma(r, r, a4[0][g]);
                a4[1][g] = fma(H(u), r, a4[1][g]);
            });
            totals<VJ, 2>(a4, s2, red, half);
            rho = rho1;
            rr_cur = s2[0];
            rho1 = s2[1];
            const bool better = rr_cur < rr_best;
            best = false;
            if (rr_cur <= tol2 || omega == 0.0) break;
            if (better) rr_best = rr_cur;
            best = better;
        }
    }
    // the iterate when converged, else the best one (a thread reads what it wrote)
    if (!(rr_cur <= tol2) && !best)
        each([&](int u, int) {
            if (live(u)) X(u) = xb[cell(u)];
        });
    if (iters && tid == 0) iters[0] += (double)(it < maxit ? it + (bnorm2 > 0.0 ? 1 : 0) : it);
    part_means([&](int u) { return X(u); });
    each([&](int u, int) {
        if (live(u)) xout[cell(u)] = (T)(X(u) - TV(u));
    });
}

template <typename T>
void launch_bottom(const Dims& d, const T* rhs, T* phi, const T* cx, const T* cy, const T* cz, double h2, double rtol,
                   int maxit, int use_x0, double* work, double* iters, const double* skip_if_direct, hipStream_t s)
{
    const int n = (int)d.n();
    auto go = [&](auto kernel, int vj) {
        hipLaunchKernelGGL(kernel, dim3(1), dim3(1024 / vj), 0, s, d, rhs, phi, cx, cy, cz, h2, rtol, maxit, use_x0, work,
                           iters, skip_if_direct);
    };
    // three vectors of 5120 cells fill 120 of the 160 KB of LDS.  Threads by
    // measurement before the best iterate was copied out (us per iteration at 280,
    // 891, 3003 and 4125 cells): 256 gave 2.2, 2.2, 7.6 and 13, 512 gave 2.6, 2.1,
    // 3.8 and 8.0, 1024 gave 3.6, 2.9, 5.0 and 25 (coefficients spilt); the forms
    // taken run at 2.3, 2.6, 4.1 and 7.1 now
    if (n <= 256) go(k_bottom<T, 4, 1>, 4);
    else if (n <= 512) go(k_bottom<T, 4, 2>, 4);
    else if (n <= 1024) go(k_bottom<T, 2, 2>, 2);
    else if (n <= 2048) go(k_bottom<T, 2, 4>, 2);
    else if (n <= 3072) go(k_bottom<T, 2, 6>, 2);
    else if (n <= 5120) go(k_bottom<T, 2, 10>, 2);
    else go(k_bottom<T, 1, 0>, 1);
}

template void launch_bottom<float>(const Dims&, const float*, float*, const float*, const float*, const float*, double,
                                   double, int, int, double*, double*, const double*, hipStream_t);
template void launch_bottom<double>(const Dims&, const double*, double*, const double*, const double*, const double*,
                                    double, double, int, int, double*, double*, const double*, hipStream_t);

}  // namespace mp
