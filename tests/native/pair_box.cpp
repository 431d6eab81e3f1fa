// Host check of the pair sweep's boxes (mp_box.h): for every extents that the
// sweep accepts, the LDS slots and the threads of a workgroup are within the
// kernel's array and launch bound, and the threads cover the box and its
// surroundings.
#include "mp_box.h"

#include <cstdio>

int main()
{
    int bad = 0, most = 0;
    for (int nx = 1; nx <= 160; nx++)
        for (int ny = 1; ny <= 300; ny++)
            for (int nz = 1; nz <= 20; nz++) {
                if (!mp::rb_extents(nx, ny, nz)) continue;
                const mp::RbBox s = mp::rb_box(nx, ny, nz);
                const bool ok = s.slots() <= mp::kRbShared && s.threads() <= 1024 &&
                                s.bx * s.by * s.bz <= mp::kRbOwn && 1 << s.lx == s.bx && 1 << s.ly == s.by &&
                                1 << s.lz == s.bz && s.threads() >= s.bx * s.by * s.bz + s.hx + s.hy + s.hz;
                if (s.slots() > most) most = s.slots();
                if (!ok && bad++ < 10)
                    printf("%d x %d x %d: box %d x %d x %d, %d slots, %d threads\n", nx, ny, nz, s.bx, s.by, s.bz,
                           s.slots(), s.threads());
            }
    printf("most slots %d of %d\n", most, mp::kRbShared);
    if (!bad) printf("ok\n");
    return bad != 0;
}
