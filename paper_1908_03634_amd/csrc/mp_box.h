// mp_box.h -- boxes of cells that a workgroup owns (host arithmetic).
#pragma once

namespace mp {

constexpr int pow2_at_least(int n, int cap)
{
    int p = 1;
    while (p < n && p < cap) p <<= 1;
    return p;
}

// Pair sweep: pairs along x, rows and planes of a workgroup's box (powers of
// two), and the threads of the red cells around it along each axis (0 where the
// box spans the axis: a wrap then stays inside it).
struct RbBox {
    int bx, by, bz, lx, ly, lz, hx, hy, hz;  // lx = log2(bx), ...
    constexpr int threads() const { return bx * by * bz + (hx + hy + hz + 63) / 64 * 64; }
    // values held in LDS: the box and one pair, row and plane on each side
    constexpr int slots() const { return (bx + 2) * (by + 2) * (bz + 2); }
};

constexpr int kRbOwn = 256;      // pairs per box
constexpr int kRbShared = 1216;  // at least the slots of any box of extents that rb_extents allows

// Smoothed levels have even extents of at least 4.  (Thinner boxes would be
// longer: 2 x 128 x 2 cells have 1560 slots.)
constexpr bool rb_extents(int nx, int ny, int nz)
{
    return nx % 2 == 0 && ny % 2 == 0 && nz % 2 == 0 && nx >= 4 && ny >= 4 && nz >= 4;
}

constexpr RbBox rb_box(int nx, int ny, int nz)
{
    const int np = nx / 2;
    RbBox s{};
    s.bx = pow2_at_least(np, 64);
    const int rem = kRbOwn / s.bx;
    s.bz = pow2_at_least(nz, rem >= 16 ? 4 : rem >= 4 ? 2 : 1);
    s.by = pow2_at_least(ny, rem / s.bz);
    while (1 << s.lx < s.bx) s.lx++;
    while (1 << s.ly < s.by) s.ly++;
    while (1 << s.lz < s.bz) s.lz++;
    s.hx = s.bx < np ? 2 * s.by * s.bz : 0;
    s.hy = s.by < ny ? 2 * s.bx * s.bz : 0;
    s.hz = s.bz < nz ? 2 * s.bx * s.by : 0;
    return s;
}

}  // namespace mp
