// Host check of the nodes that a colour pass reads (mp_nodal.h): along an axis
// of n cells the node beside any node, walls included, lies in the grid and has
// the other parity, and away from walls it is the neighbour; the packed offsets
// lead to the same nodes.
#include "mp_nodal.h"

#include <cstdio>

int main()
{
    int bad = 0;
    for (int per = 0; per < 2; per++)
        for (int n = per ? 2 : 1; n <= 64; n += per ? 2 : 1) {
            const int m = n + (per ? 0 : 1);
            for (int i = 0; i < m; i++) {
                const mp::Axis a = mp::axis_of(i, n, per);
                for (int o = 0; o < 2; o++) {
                    const int q = mp::beside(a, o);
                    bool ok = q >= 0 && q < m && ((q ^ i) & 1) != 0;
                    if (a.nok[2 * o]) ok = ok && q == a.nd[2 * o];
                    // (rows of 3 to 129 values: the strides of a coarse level)
                    for (int stride = 1; stride <= 129; stride += 2) {
                        const int s = mp::steps_beside(a, i, stride);
                        ok = ok && (o ? s >> 16 : (int)(short)s) == (q - i) * stride;
                    }
                    if (!ok) {
                        printf("n %d periodic %d node %d side %d: reads %d\n", n, per, i, o, q);
                        bad++;
                    }
                }
            }
        }
    if (!bad) printf("ok\n");
    return bad != 0;
}
