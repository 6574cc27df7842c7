// Host build of the int8 GEMM's launch plan, for tests/test_gemm_plan.py.
#define O2M_HD
#include "../paper_2609_05419_amd/csrc/tile_schedule.h"

extern "C" {
// deal, chunk, slots, fixed, grid
void t_plan(int mt, int nt, int kblocks, int batch, long stage_bytes, long *out) {
    const o2m::GemmSchedule s = o2m::gemm_plan(mt, nt, kblocks, batch, stage_bytes);
    out[0] = s.deal;
    out[1] = s.chunk;
    out[2] = s.slots;
    out[3] = s.fixed;
    out[4] = s.grid;
}
// tiles[4 * (x * slots + slot) + {valid, p, ti, tj}]
void t_plan_tiles(int mt, int nt, int chunk, int deal, int batch, long slots, int *tiles) {
    for (int x = 0; x < o2m::kXcds; ++x)
        for (long s = 0; s < slots; ++s) {
            const o2m::TileCoord c = o2m::tile_of(x, (int)s, mt, nt, chunk, deal, batch);
            int *o = tiles + 4 * (x * slots + s);
            o[0] = c.valid;
            o[1] = c.p;
            o[2] = c.ti;
            o[3] = c.tj;
        }
}
}
