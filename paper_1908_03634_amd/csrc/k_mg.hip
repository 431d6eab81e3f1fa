// k_mg.hip -- gfx950 multigrid kernels launched one per operation: one colour
// of red-black Gauss-Seidel (the reference the fused sweep is checked
// against, and the fallback for odd periodic extents), residual + 8-cell
// restriction, piecewise-constant prolongation, and the FP64 finest-level
// operator, residual and update of the iterative refinement.
//
// The stencils are bandwidth-bound (about 20 flops per 24-48 bytes), so no
// matrix cores are involved.  Launches are 3D (x fastest, 64 lanes along x)
// so no thread divides a 64-bit index; the FP64 residual marches along z
// keeping the z-neighbours of its column in registers.
#include "mp_device.h"
#include "mp_kernels.h"
#include "mp_launch.h"

#include <math.h>

namespace mp {

// ------------------------------------------------------------------ smoother

template <typename T, bool CELL>
__global__ __launch_bounds__(256) void k_rbgs(Dims d, T* __restrict__ x, const T* __restrict__ b, Coef<T> C, T h2,
                                              int colour, int zero_init)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const int k = blockIdx.z * blockDim.z + threadIdx.z;
    if (p >= (d.nx + 1) / 2 || j >= d.ny || k >= d.nz) return;
    rbgs_cell<T, CELL>(d, x, b, C, h2, colour, zero_init, p, j, k);
}

template <typename T>
void launch_rbgs(const Dims& d, T* phi, const T* rhs, const Coef<T>& c, T h2, int colour, int zero_init,
                 hipStream_t s)
{
    const Shape3 sh = cells3((d.nx + 1) / 2, d.ny, d.nz);
    if (c.cell)
        hipLaunchKernelGGL((k_rbgs<T, true>), sh.grid, sh.block, 0, s, d, phi, rhs, c, h2, colour, zero_init);
    else
        hipLaunchKernelGGL((k_rbgs<T, false>), sh.grid, sh.block, 0, s, d, phi, rhs, c, h2, colour, zero_init);
}

// The two colour passes that follow a prolongation, with the prolongation
// folded in (ec: coarse correction; piecewise constant, parent of (i,j,k) is
// (i/2, j/2, k/2)).  ALL (first colour): every value read, neighbours and
// own, is x + e of its parent, the values the separate prolongation would
// have stored; the other colour is left as stored.  Otherwise (second
// colour): the neighbours, just updated, are read as stored and the cell's
// own value as x + e.  Together they equal launch_prolong followed by two
// plain passes, bit for bit.
__device__ __forceinline__ long long parent_of(const Dims& d, int i, int j, int k)
{
    return ((long long)(k >> 1) * (d.ny >> 1) + (j >> 1)) * (d.nx >> 1) + (i >> 1);
}

template <typename T, bool CELL, bool ALL>
__global__ __launch_bounds__(256) void k_rbgs_e(Dims d, T* __restrict__ x, const T* __restrict__ b, Coef<T> C, T h2,
                                                int colour, const T* __restrict__ ec)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const int k = blockIdx.z * blockDim.z + threadIdx.z;
    if (p >= (d.nx + 1) / 2 || j >= d.ny || k >= d.nz) return;
    const int i = 2 * p + ((j + k + colour) & 1);
    if (i >= d.nx) return;
    const long long q = ((long long)k * d.ny + j) * d.nx + i;
    const Nbr nb = neighbours(d, q, i, j, k);
    T c0, c1, c2, c3, c4, c5;
    coef6<T, CELL>(C, d, q, nb, i, j, k, c0, c1, c2, c3, c4, c5);
    const T own = x[q] + ec[parent_of(d, i, j, k)];
    if constexpr (ALL) {
        // neighbour coordinates (a wall neighbour is the cell itself)
        const int im = i > 0 ? i - 1 : (d.px ? d.nx - 1 : i), ip = i < d.nx - 1 ? i + 1 : (d.px ? 0 : i);
        const int jm = j > 0 ? j - 1 : (d.py ? d.ny - 1 : j), jp = j < d.ny - 1 ? j + 1 : (d.py ? 0 : j);
        const int km = k > 0 ? k - 1 : (d.pz ? d.nz - 1 : k), kp = k < d.nz - 1 ? k + 1 : (d.pz ? 0 : k);
        const T xm = x[nb.xm] + ec[parent_of(d, im, j, k)], xp = x[nb.xp] + ec[parent_of(d, ip, j, k)];
        const T ym = x[nb.ym] + ec[parent_of(d, i, jm, k)], yp = x[nb.yp] + ec[parent_of(d, i, jp, k)];
        const T zm = x[nb.zm] + ec[parent_of(d, i, j, km)], zp = x[nb.zp] + ec[parent_of(d, i, j, kp)];
        x[q] = gs_value<T>(c0, c1, c2, c3, c4, c5, xm, xp, ym, yp, zm, zp, b[q], h2, own);
    } else {
        x[q] = gs_value<T>(c0, c1, c2, c3, c4, c5, x[nb.xm], x[nb.xp], x[nb.ym], x[nb.yp], x[nb.zm], x[nb.zp], b[q],
                           h2, own);
    }
}

template <typename T>
void launch_rbgs_e(const Dims& d, T* phi, const T* rhs, const Coef<T>& c, T h2, int colour, int first,
                   const T* ec, hipStream_t s)
{
    const Shape3 sh = cells3((d.nx + 1) / 2, d.ny, d.nz);
    if (c.cell) {
        if (first)
            hipLaunchKernelGGL((k_rbgs_e<T, true, true>), sh.grid, sh.block, 0, s, d, phi, rhs, c, h2, colour, ec);
        else
            hipLaunchKernelGGL((k_rbgs_e<T, true, false>), sh.grid, sh.block, 0, s, d, phi, rhs, c, h2, colour, ec);
    } else {
        if (first)
            hipLaunchKernelGGL((k_rbgs_e<T, false, true>), sh.grid, sh.block, 0, s, d, phi, rhs, c, h2, colour, ec);
        else
            hipLaunchKernelGGL((k_rbgs_e<T, false, false>), sh.grid, sh.block, 0, s, d, phi, rhs, c, h2, colour, ec);
    }
}

// Both colours of a sweep in one launch, out of place, for levels of even
// extents where a launch costs more than its cells.  A workgroup owns a box of
// cell pairs (2p, 2p + 1) of rows, one red and one black cell each, one pair per
// thread, and the red cells of the pairs around the box, one per further thread:
// a black cell's six neighbours are the red cells of its own pair and of the
// pairs beside it along x, y and z.  Every thread updates its red cell from old
// values and publishes it in LDS; after one barrier the owners update their black
// cells.  A red value depends on old values only, so the red cells evaluated
// again by a neighbouring workgroup have the bits of the colour pass.  What
// bounds it is the latency of one chain (load, red, barrier, black): the loads of
// the black update are issued before the barrier, and no thread evaluates more
// than one red cell (128^3 FP64 solve, 64^3 to 16^3 levels: 4.9 us a sweep
// against 7.6 us for two colour passes; 256^3 mixed, 64^3 and 32^3 levels: 5.2 us,
// 5.6 with the outer red cells evaluated after the barrier by the threads that
// need them).  Old values (MODE): FS_ZERO 0 (first
// sweep from a zero iterate), FS_PLAIN x as stored, FS_PROLONG x + e of the
// parent cell (first sweep after prolongation).  Every cell takes the operands of
// rbgs_cell / k_rbgs_e: a black cell's neighbour behind a wall is its value as
// the colour pass finds it stored (x, without e).
template <typename T, int MODE, bool CELL>
struct RbPair {
    Dims d;
    const T* __restrict__ xo;
    const T* __restrict__ b;
    Coef<T> C;
    const T* __restrict__ ec;
    T h2;

    __device__ __forceinline__ int parent(int i, int j, int k) const
    {
        return ((k >> 1) * (d.ny >> 1) + (j >> 1)) * (d.nx >> 1) + (i >> 1);
    }
    __device__ __forceinline__ T old_at(int q, int i, int j, int k) const
    {
        if constexpr (MODE == FS_ZERO) return T(0);
        else if constexpr (MODE == FS_PLAIN) return xo[q];
        else return xo[q] + ec[parent(i, j, k)];
    }
    // face coefficients of cell q = (i, j, k) in stencil order (coef6)
    __device__ __forceinline__ void coefs(int q, const Nb32& nb, int i, int j, int k, T (&c)[6]) const
    {
        if constexpr (CELL) {
            const T* cc = C.cell;
            const T cq = cc[q], xl = cc[nb.xm], xh = cc[nb.xp], yl = cc[nb.ym], yh = cc[nb.yp], zl = cc[nb.zm],
                    zh = cc[nb.zp];
            c[0] = (i > 0 || d.px) ? harm(xl, cq) : T(0);
            c[1] = nb.hx ? harm(cq, xh) : T(0);
            c[2] = (j > 0 || d.py) ? harm(yl, cq) : T(0);
            c[3] = nb.hy ? harm(cq, yh) : T(0);
            c[4] = (k > 0 || d.pz) ? harm(zl, cq) : T(0);
            c[5] = nb.hz ? harm(cq, zh) : T(0);
        } else {
            const T xh = C.x[nb.xp], yh = C.y[nb.yp], zh = C.z[nb.zp];
            c[0] = C.x[q];
            c[1] = nb.hx ? xh : T(0);
            c[2] = C.y[q];
            c[3] = nb.hy ? yh : T(0);
            c[4] = C.z[q];
            c[5] = nb.hz ? zh : T(0);
        }
    }
    // new value of red cell (i, j, k) (coordinates inside the grid)
    __device__ __forceinline__ T red(int i, int j, int k) const
    {
        const int q = (k * d.ny + j) * d.nx + i;
        const Nb32 nb = nb32(d, q, i, j, k);
        T c[6];
        coefs(q, nb, i, j, k, c);
        T v[6], own;
        if constexpr (MODE == FS_ZERO) {
            own = v[0] = v[1] = v[2] = v[3] = v[4] = v[5] = T(0);
        } else {
            // neighbour coordinates (a wall neighbour is the cell itself)
            const int im = i > 0 ? i - 1 : (d.px ? d.nx - 1 : i), ip = i < d.nx - 1 ? i + 1 : (d.px ? 0 : i);
            const int jm = j > 0 ? j - 1 : (d.py ? d.ny - 1 : j), jp = j < d.ny - 1 ? j + 1 : (d.py ? 0 : j);
            const int km = k > 0 ? k - 1 : (d.pz ? d.nz - 1 : k), kp = k < d.nz - 1 ? k + 1 : (d.pz ? 0 : k);
            own = old_at(q, i, j, k);
            v[0] = old_at(nb.xm, im, j, k);
            v[1] = old_at(nb.xp, ip, j, k);
            v[2] = old_at(nb.ym, i, jm, k);
            v[3] = old_at(nb.yp, i, jp, k);
            v[4] = old_at(nb.zm, i, j, km);
            v[5] = old_at(nb.zp, i, j, kp);
        }
        return gs_value<T>(c[0], c[1], c[2], c[3], c[4], c[5], v[0], v[1], v[2], v[3], v[4], v[5], b[q], h2, own);
    }
};

template <typename T, int MODE, bool CELL>
__global__ __launch_bounds__(1024) void k_rb_pair(Dims d, RbBox s, const T* __restrict__ xo, T* __restrict__ xn,
                                                  const T* __restrict__ b, Coef<T> C, T h2, const T* __restrict__ ec)
{
    __shared__ T sred[kRbShared];
    const int np = d.nx / 2;
    const int p0 = (int)blockIdx.x * s.bx, j0 = (int)blockIdx.y * s.by, k0 = (int)blockIdx.z * s.bz;
    // the box's extents inside the grid
    const int ex = min(s.bx, np - p0), ey = min(s.by, d.ny - j0), ez = min(s.bz, d.nz - k0);
    const RbPair<T, MODE, CELL> o{d, xo, b, C, ec, h2};
    auto slot = [&](int u, int v, int w) { return ((w + 1) * (s.by + 2) + v + 1) * (s.bx + 2) + u + 1; };
    // pair (u, v, w) of the box, or of its surroundings
    int t = (int)threadIdx.x, u, v, w;
    const int nown = s.bx * s.by * s.bz;
    bool own = t < nown, need;
    if (own) {
        u = t & (s.bx - 1);
        v = (t >> s.lx) & (s.by - 1);
        w = t >> (s.lx + s.ly);
        need = own = u < ex && v < ey && w < ez;
    } else {
        t -= nown;
        if (t < s.hx) {
            u = t & 1 ? ex : -1;
            v = (t >> 1) & (s.by - 1);
            w = t >> (1 + s.ly);
            need = v < ey && w < ez;
        } else if (t < s.hx + s.hy) {
            t -= s.hx;
            u = t & (s.bx - 1);
            v = (t >> s.lx) & 1 ? ey : -1;
            w = t >> (1 + s.lx);
            need = u < ex && w < ez;
        } else if (t < s.hx + s.hy + s.hz) {
            t -= s.hx + s.hy;
            u = t & (s.bx - 1);
            v = (t >> s.lx) & (s.by - 1);
            w = t >> (s.lx + s.ly) ? ez : -1;
            need = u < ex && v < ey;
        } else {
            u = v = w = 0;
            need = false;
        }
    }
    // its place in the grid: around the box across a wrap, or nowhere
    int p = p0 + u, j = j0 + v, k = k0 + w;
    if (need && !own) {
        if (p < 0 || p >= np) {
            need = d.px;
            p = p < 0 ? np - 1 : 0;
        }
        if (j < 0 || j >= d.ny) {
            need = need && d.py;
            j = j < 0 ? d.ny - 1 : 0;
        }
        if (k < 0 || k >= d.nz) {
            need = need && d.pz;
            k = k < 0 ? d.nz - 1 : 0;
        }
    }
    const int par = (j + k) & 1;  // the red cell is 2p + par
    const int ir = 2 * p + par, ib = 2 * p + 1 - par;
    const int row = (k * d.ny + j) * d.nx, q = row + ib;
    // the black update's operands that do not wait for red values
    T c[6], bq = T(0), stored = T(0), old = T(0);
    if (own) {
        const Nb32 nb = nb32(d, q, ib, j, k);
        o.coefs(q, nb, ib, j, k, c);
        bq = b[q];
        if constexpr (MODE != FS_ZERO) stored = xo[q];  // as the second colour pass finds it
        old = o.old_at(q, ib, j, k);
    }
    T rv = T(0);
    if (need) {
        rv = o.red(ir, j, k);
        sred[slot(u, v, w)] = rv;
    }
    __syncthreads();
    if (!own) return;
    // the red cell of the pair beside this one along axis a: across a wrap inside
    // the box where it spans the axis; the stored black value behind a wall
    const bool sx = s.hx == 0, sy = s.hy == 0, sz = s.hz == 0;
    auto red_at = [&](int a, int du, int dv, int dw) -> T {
        int un = u + du, vn = v + dv, wn = w + dw;
        bool wall = false;
        if (a == 0) {
            const int g = p + du;
            if (g < 0 || g >= np) {
                wall = !d.px;
                if (sx) un = g < 0 ? np - 1 : 0;
            }
        } else if (a == 1) {
            const int g = j + dv;
            if (g < 0 || g >= d.ny) {
                wall = !d.py;
                if (sy) vn = g < 0 ? d.ny - 1 : 0;
            }
        } else {
            const int g = k + dw;
            if (g < 0 || g >= d.nz) {
                wall = !d.pz;
                if (sz) wn = g < 0 ? d.nz - 1 : 0;
            }
        }
        return wall ? stored : sred[slot(un, vn, wn)];
    };
    // one x neighbour is the pair's red cell, the other that of the pair beside it
    const T vo = red_at(0, par ? -1 : 1, 0, 0);
    const T ym = red_at(1, 0, -1, 0), yp = red_at(1, 0, 1, 0);
    const T zm = red_at(2, 0, 0, -1), zp = red_at(2, 0, 0, 1);
    const T xm = par ? vo : rv, xp = par ? rv : vo;
    xn[row + ir] = rv;
    xn[q] = gs_value<T>(c[0], c[1], c[2], c[3], c[4], c[5], xm, xp, ym, yp, zm, zp, bq, h2, old);
}

bool rb_pair_supported(const Dims& d)
{
    return rb_extents(d.nx, d.ny, d.nz) && d.n() < (1LL << 31);
}

template <typename T, int MODE>
static void rb_pair_launch(const Dims& d, const T* xo, T* xn, const T* b, const Coef<T>& c, T h2, const T* ec,
                           hipStream_t s)
{
    const RbBox x = rb_box(d.nx, d.ny, d.nz);
    const dim3 grid((d.nx / 2 + x.bx - 1) / x.bx, (d.ny + x.by - 1) / x.by, (d.nz + x.bz - 1) / x.bz);
    if (c.cell)
        hipLaunchKernelGGL((k_rb_pair<T, MODE, true>), grid, dim3(x.threads()), 0, s, d, x, xo, xn, b, c, h2, ec);
    else
        hipLaunchKernelGGL((k_rb_pair<T, MODE, false>), grid, dim3(x.threads()), 0, s, d, x, xo, xn, b, c, h2, ec);
}

template <typename T>
void launch_rb_pair(const Dims& d, const T* xo, T* xn, const T* b, const Coef<T>& c, T h2, int mode, const T* ec,
                    hipStream_t s)
{
    if (mode == FS_ZERO) rb_pair_launch<T, FS_ZERO>(d, xo, xn, b, c, h2, ec, s);
    else if (mode == FS_PROLONG) rb_pair_launch<T, FS_PROLONG>(d, xo, xn, b, c, h2, ec, s);
    else rb_pair_launch<T, FS_PLAIN>(d, xo, xn, b, c, h2, ec, s);
}

// --------------------------------------------------------- transfer operators

// Coarse right-hand side = mean of the 8 fine residuals, one fine cell per
// thread (a thread with the eight children of a coarse cell leaves small grids
// without wavefronts: 32^3 FP64 cell coefficients 12.8 us, 4.1 here), the
// children then summed through LDS by z, then y, then x child.  Blocks are
// boxes of even extents, powers of two.
template <typename T, bool CELL>
__global__ __launch_bounds__(256) void k_resid_restrict(Dims d, const T* __restrict__ x, const T* __restrict__ b,
                                                        Coef<T> C, T inv_h2, T* __restrict__ bc)
{
    __shared__ T r[256];
    const int bx = (int)blockDim.x, by = (int)blockDim.y, bz = (int)blockDim.z;
    const int i0 = (int)blockIdx.x * bx, j0 = (int)blockIdx.y * by, k0 = (int)blockIdx.z * bz;
    const int i = i0 + (int)threadIdx.x, j = j0 + (int)threadIdx.y, k = k0 + (int)threadIdx.z;
    const int t = ((int)threadIdx.z * by + (int)threadIdx.y) * bx + (int)threadIdx.x;
    if (i < d.nx && j < d.ny && k < d.nz) r[t] = resid_cell<T, CELL>(d, x, b, C, inv_h2, i, j, k);
    __syncthreads();
    // thread t < coarse cells of the block: coarse cell (I, J, K) of it
    const int cx = bx / 2, cy = by / 2;
    if (t >= cx * cy * (bz / 2)) return;
    const int I = t % cx, J = t / cx % cy, K = t / (cx * cy);
    if (i0 + 2 * I >= d.nx || j0 + 2 * J >= d.ny || k0 + 2 * K >= d.nz) return;
    T acc = T(0);
#pragma unroll
    for (int c = 0; c < 2; c++)
#pragma unroll
        for (int bb = 0; bb < 2; bb++)
#pragma unroll
            for (int a = 0; a < 2; a++) acc += r[((2 * K + c) * by + 2 * J + bb) * bx + 2 * I + a];
    bc[((long long)(k0 / 2 + K) * (d.ny / 2) + j0 / 2 + J) * (d.nx / 2) + i0 / 2 + I] = T(0.125) * acc;
}

template <typename T>
void launch_resid_restrict(const Dims& fine, const T* phi, const T* rhs, const Coef<T>& c, T inv_h2, T* coarse_rhs,
                           hipStream_t s)
{
    const int bx = pow2_at_least(fine.nx, 64), by = pow2_at_least(fine.ny, 128 / bx);
    const int bz = pow2_at_least(fine.nz, 256 / (bx * by));
    const dim3 block(bx, by, bz);
    const dim3 grid((fine.nx + bx - 1) / bx, (fine.ny + by - 1) / by, (fine.nz + bz - 1) / bz);
    if (c.cell)
        hipLaunchKernelGGL((k_resid_restrict<T, true>), grid, block, 0, s, fine, phi, rhs, c, inv_h2, coarse_rhs);
    else
        hipLaunchKernelGGL((k_resid_restrict<T, false>), grid, block, 0, s, fine, phi, rhs, c, inv_h2, coarse_rhs);
}

// Fine x += coarse e of the parent cell.
template <typename T>
__global__ __launch_bounds__(256) void k_prolong(Dims d, T* __restrict__ x, const T* __restrict__ e)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const int k = blockIdx.z * blockDim.z + threadIdx.z;
    if (i >= d.nx || j >= d.ny || k >= d.nz) return;
    const int nxc = d.nx / 2, nyc = d.ny / 2;
    x[((long long)k * d.ny + j) * d.nx + i] += e[((long long)(k >> 1) * nyc + (j >> 1)) * nxc + (i >> 1)];
}

template <typename T>
void launch_prolong(const Dims& fine, T* phi, const T* coarse_phi, hipStream_t s)
{
    const Shape3 sh = cells3(fine.nx, fine.ny, fine.nz);
    hipLaunchKernelGGL((k_prolong<T>), sh.grid, sh.block, 0, s, fine, phi, coarse_phi);
}

// --------------------------------------------------------- FP64 level 0

template <bool CELL>
__global__ __launch_bounds__(256) void k_apply64(Dims d, const double* __restrict__ x, Coef<double> C, double inv_h2,
                                                 double* __restrict__ y)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const int k = blockIdx.z * blockDim.z + threadIdx.z;
    if (i >= d.nx || j >= d.ny || k >= d.nz) return;
    const long long q = ((long long)k * d.ny + j) * d.nx + i;
    const Nbr nb = neighbours(d, q, i, j, k);
    double c0, c1, c2, c3, c4, c5;
    coef6<double, CELL>(C, d, q, nb, i, j, k, c0, c1, c2, c3, c4, c5);
    // M x = -(A x) = the residual of a zero right-hand side
    y[q] = resid_value<double>(c0, c1, c2, c3, c4, c5, x[nb.xm], x[nb.xp], x[nb.ym], x[nb.yp], x[nb.zm], x[nb.zp],
                                x[q], 0.0, inv_h2);
}

void launch_apply64(const Dims& d, const double* x, const Coef<double>& c, double inv_h2, double* y, hipStream_t s)
{
    const Shape3 sh = cells3(d.nx, d.ny, d.nz);
    if (c.cell)
        hipLaunchKernelGGL(k_apply64<true>, sh.grid, sh.block, 0, s, d, x, c, inv_h2, y);
    else
        hipLaunchKernelGGL(k_apply64<false>, sh.grid, sh.block, 0, s, d, x, c, inv_h2, y);
}

// r = b - A x for a column of lz cells per thread; the column's z-neighbours
// and z-face coefficients stay in registers (in cell mode the z-face value
// formed for the high face of one plane is the low face of the next).  Same
// arithmetic, in the same order, as resid_cell.
template <bool CELL>
__global__ __launch_bounds__(256) void k_resid64(Dims d, int lz, const double* __restrict__ x,
                                                 const double* __restrict__ b, Coef<double> C, double inv_h2,
                                                 float* __restrict__ r32, const double* __restrict__ inv_s,
                                                 double* part)
{
    __shared__ double sh[4];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int j = blockIdx.y * blockDim.y + threadIdx.y;
    const int z0 = blockIdx.z * lz;
    const int z1 = min(z0 + lz, d.nz);
    double acc = 0.0;
    if (i < d.nx && j < d.ny) {
        const double is = r32 ? inv_s[0] : 0.0;
        const long long sy = d.nx, sz = (long long)d.nx * d.ny;
        const long long oxm = i > 0 ? -1 : (d.px ? d.nx - 1 : 0);
        const long long oxp = i < d.nx - 1 ? 1 : (d.px ? -(long long)(d.nx - 1) : 0);
        const bool hxm = i > 0 || d.px, hxp = i < d.nx - 1 || d.px;
        const long long oym = j > 0 ? -sy : (d.py ? (long long)(d.ny - 1) * sy : 0);
        const long long oyp = j < d.ny - 1 ? sy : (d.py ? -(long long)(d.ny - 1) * sy : 0);
        const bool hym = j > 0 || d.py, hyp = j < d.ny - 1 || d.py;
        long long q = (long long)z0 * sz + (long long)j * d.nx + i;
        const long long qm = z0 > 0 ? q - sz : (d.pz ? q + (long long)(d.nz - 1) * sz : q);
        double xzm = x[qm];
        double x0 = x[q];
        double cc0 = 0.0, czl;
        if constexpr (CELL) {
            cc0 = C.cell[q];
            czl = (z0 > 0 || d.pz) ? harm(C.cell[qm], cc0) : 0.0;
        } else {
            czl = C.z[q];
        }
        for (int k = z0; k < z1; k++) {
            const bool last = k == d.nz - 1;
            const bool hzp = !last || d.pz;
            const long long qp = !last ? q + sz : (d.pz ? q - (long long)(d.nz - 1) * sz : q);
            const double xzp = x[qp];
            double c0, c1, c2, c3, czh, ccp = 0.0;
            if constexpr (CELL) {
                const double* cc = C.cell;
                ccp = cc[qp];
                czh = hzp ? harm(cc0, ccp) : 0.0;
                c0 = hxm ? harm(cc[q + oxm], cc0) : 0.0;
                c1 = hxp ? harm(cc0, cc[q + oxp]) : 0.0;
                c2 = hym ? harm(cc[q + oym], cc0) : 0.0;
                c3 = hyp ? harm(cc0, cc[q + oyp]) : 0.0;
            } else {
                czh = hzp ? C.z[qp] : 0.0;
                c0 = C.x[q];
                c1 = hxp ? C.x[q + oxp] : 0.0;
                c2 = C.y[q];
                c3 = hyp ? C.y[q + oyp] : 0.0;
            }
            const double r = resid_value<double>(c0, c1, c2, c3, czl, czh, x[q + oxm], x[q + oxp], x[q + oym],
                                                 x[q + oyp], xzm, xzp, x0, b[q], inv_h2);
            acc = fma(r, r, acc);
            if (r32) r32[q] = (float)(r * is);
            xzm = x0;
            x0 = xzp;
            czl = czh;
            cc0 = ccp;
            q += sz;
        }
    }
    const double s = block_sum(acc, sh);
    if (threadIdx.x == 0 && threadIdx.y == 0)
        part[((long long)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = s;
}

void launch_resid64(const Dims& d, const double* phi, const double* b, const Coef<double>& c, double inv_h2,
                    float* r32, const double* inv_s, double* partials, int* nb_out, hipStream_t s)
{
    const ShapeZ sh = zmarch(d.nx, d.ny, d.nz, kZBlocks);
    *nb_out = (int)sh.blocks();
    if (c.cell)
        hipLaunchKernelGGL(k_resid64<true>, sh.grid, sh.block, 0, s, d, sh.lz, phi, b, c, inv_h2, r32, inv_s,
                           partials);
    else
        hipLaunchKernelGGL(k_resid64<false>, sh.grid, sh.block, 0, s, d, sh.lz, phi, b, c, inv_h2, r32, inv_s,
                           partials);
}

// First refinement step from a zero iterate: the residual is b itself, so
// r32 = float(b * pair_in[1]) (the value the residual kernel would write) and
// the scale pair of the next step is the one of b.
__global__ __launch_bounds__(256) void k_scale32(long long n, const double* __restrict__ b, float* __restrict__ r32,
                                                 const double* __restrict__ pair_in, double* __restrict__ pair_out)
{
    const double is = pair_in[1];
    const long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (q == 0) {
        pair_out[0] = pair_in[0];
        pair_out[1] = pair_in[1];
    }
    if (r32 && q < n) r32[q] = (float)(b[q] * is);
}

void launch_scale32(long long n, const double* b, float* r32, const double* pair_in, double* pair_out, hipStream_t st)
{
    const long long work = r32 ? n : 1;
    hipLaunchKernelGGL(k_scale32, dim3((unsigned)((work + 255) / 256)), dim3(256), 0, st, n, b, r32, pair_in,
                       pair_out);
}

__global__ __launch_bounds__(256) void k_ir_update(long long n, double* __restrict__ x, const float* __restrict__ e,
                                                   const double* __restrict__ s)
{
    const long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (q < n) x[q] = fma(s[0], (double)e[q], x[q]);
}

void launch_ir_update(long long n, double* phi, const float* e, const double* s, hipStream_t st)
{
    hipLaunchKernelGGL(k_ir_update, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, phi, e, s);
}

// ------------------------------------------------------------ instantiations

#define MP_INST(T)                                                                                                    \
    template void launch_rbgs<T>(const Dims&, T*, const T*, const Coef<T>&, T, int, int, hipStream_t);                \
    template void launch_rbgs_e<T>(const Dims&, T*, const T*, const Coef<T>&, T, int, int, const T*, hipStream_t);    \
    template void launch_rb_pair<T>(const Dims&, const T*, T*, const T*, const Coef<T>&, T, int, const T*,           \
                                    hipStream_t);                                                                     \
    template void launch_resid_restrict<T>(const Dims&, const T*, const T*, const Coef<T>&, T, T*, hipStream_t);      \
    template void launch_prolong<T>(const Dims&, T*, const T*, hipStream_t);
MP_INST(float)
MP_INST(double)

}  // namespace mp
