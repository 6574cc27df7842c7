// Host build of the int8 GEMM's launch plan, for tests/test_gemm_plan.py.
#define O2M_HD
#include "../paper_2609_05419_amd/csrc/tile_schedule.h"

extern "C" {
// shape, tm, tn, mt, nt, deal, chunk, slots, fixed, grid, chain
void t_plan(int rows, int cols, int kblocks, int batch, long stage_bytes, long *out) {
    const o2m::GemmPlan p = o2m::gemm_plan(rows, cols, kblocks, batch, stage_bytes);
    const long v[11] = {p.shape, p.tm, p.tn, p.mt, p.nt, p.s.deal, p.s.chunk, p.s.slots, p.s.fixed, p.s.grid, p.chain};
    for (int i = 0; i < 11; ++i) out[i] = v[i];
}
double t_estimate(int shape, int rows, int cols, int kblocks, int batch, double sustained) {
    return o2m::gemm_estimate(o2m::gemm_shape_of(shape), rows, cols, kblocks, batch, sustained);
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
