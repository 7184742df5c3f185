// The dispatch rules of lc_launch.h as C functions, for tests/test_launch_rules.py.
#include "../../paper_1907_13415_amd/csrc/lc_launch.h"

using namespace lc;

extern "C" {
int rule_num_cu() { return NUM_CU; }
// out: blocks_x, blocks_y, xb, before of each launch
int rule_tile_launches(const lc_grid* g, int tx, int ty, int threads, int64_t* out) {
  int n = 0;
  tile_launches(*g, tx, ty, threads, [&](unsigned bx, unsigned by, int xb, int64_t before) {
    const int64_t v[4] = {bx, by, xb, before};
    for (int k = 0; k < 4; k++) out[4 * n + k] = v[k];
    n++;
  });
  return n;
}
int rule_auto_variant(const lc_grid* g, int isotropic) { return auto_variant(*g, isotropic != 0); }
int rule_form2d(const lc_grid* g, int isotropic, int timed) { return fused2d_form(*g, isotropic != 0, timed != 0); }
int rule_shape2d(const lc_grid* g) { return fused2d_shape(*g); }
int64_t rule_tiles2d(const lc_grid* g, int v) { return fused2d_tiles(*g, v); }
int rule_region_wraps_once(int n, int t) { return region_wraps_once(n, t); }
int rule_pick_chunk(int nz, int tiles, int most, int extra, int resident, double margin) {
  return pick_chunk(nz, tiles, most, extra, resident, margin);
}
int rule_even_chunk(int nz, int planes) { return even_chunk(nz, planes); }
int rule_rev_shape(const lc_grid* g) { return rev_shape(*g); }
int rule_march_takes(int n, const lc_grid* g) { return march_takes(n, g); }
int rule_march_beats_sweeps(int n, const lc_grid* g, int isotropic) {
  return march_beats_sweeps(n, g, isotropic != 0);
}
int rule_march_rows(int n, const lc_grid* g) { return march_rows(n, g); }
}
