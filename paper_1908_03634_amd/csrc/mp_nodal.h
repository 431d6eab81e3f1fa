// mp_nodal.h -- neighbours of a node along one axis (device and host).
#pragma once

namespace mp {

// Node neighbours along one axis (offsets -1, 0, +1) and the cells below and
// above the node (offsets -1, 0).  Missing ones (beyond a wall) are flagged
// and point at the node itself / cell 0 so every load stays in bounds.
struct Axis {
    int nd[3];
    bool nok[3];
    int ce[2];
    bool cok[2];
};

constexpr Axis axis_of(int i, int n, int per)
{
    Axis a{};
    for (int o = 0; o < 3; o++) {
        int t = i + o - 1;
        if (per) {
            t = t < 0 ? t + n : (t >= n ? t - n : t);
            a.nd[o] = t;
            a.nok[o] = true;
        } else {
            a.nok[o] = t >= 0 && t <= n;
            a.nd[o] = a.nok[o] ? t : i;
        }
    }
    for (int o = 0; o < 2; o++) {
        int t = i + o - 1;
        if (per) {
            t = t < 0 ? t + n : t;
            a.ce[o] = t;
            a.cok[o] = true;
        } else {
            a.cok[o] = t >= 0 && t < n;
            a.ce[o] = a.cok[o] ? t : 0;
        }
    }
    return a;
}

// The node beside the given one on side o (0 below, 1 above); beyond a wall the
// one on the other side, whose value meets sigma 0 there.  It has the other
// parity along the axis (even periodic extents), so a pass that updates the
// nodes of one parity never reads, beside a wall, what it writes.
constexpr int beside(const Axis& a, int o) { return a.nok[2 * o] ? a.nd[2 * o] : a.nd[2 - 2 * o]; }

// Two offsets of 16 bits in one word (low and high half, signed).
constexpr int pack16(int lo, int hi) { return (lo & 0xffff) | (int)((unsigned)hi << 16); }

// Offsets from node i to the nodes beside it, `stride` values apart.
constexpr int steps_beside(const Axis& a, int i, int stride)
{
    return pack16((beside(a, 0) - i) * stride, (beside(a, 1) - i) * stride);
}

}  // namespace mp
