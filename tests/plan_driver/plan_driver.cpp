// Prints the launch plan of each domain on standard input ("nx ny nz storage
// ncomp c_ns forcing" a line) for a device of 256 CUs: box, tile and chunk of
// the sweep, store policy, tile in a group, tile in a server, cells of a block.  Host code only.
#include <cstdio>

#include "lbm_internal.h"

int main()
{
    lbm_domain d{};
    lbm_params p{};
    p.tau[0] = p.tau[1] = 1.0;
    p.g_scale = 1.0;
    while (std::scanf("%d %d %d %d %d %d %d", &d.nx, &d.ny, &d.nz, &p.storage, &p.ncomp, &p.c_ns, &p.forcing) == 7) {
        if (hm_rt::validate(&d, &p)) return 1;
        const hm::Problem q = hm_rt::make_problem(&d, &p);
        const hm::Launch l = hm_rt::choose_launch(q, 256, false), s = hm_rt::choose_launch(q, 256, true);
        std::printf("%d %d %d %d %d %d %d %d %d %d %d %d\n", l.bx, l.by, l.bz, l.tile_x, l.tile_y, l.zchunk,
                    l.nt_stores ? 1 : 0, l.batch_x, l.batch_y, s.batch_x, s.batch_y, l.cells);
    }
    return 0;
}
