// The library's rules on lattice sizes behind C names, for tests on the host.
#include "lbmhd_impl.h"

namespace lbk3 {
int diag3_chunk(long long tiles, int nz);
}

static lbk::Geom geom(int nx, int ny, int esize) {
  lbk::Geom g;
  g.nx = nx;
  g.ny = ny;
  g.pitch = (nx * esize + 255) / 256 * 256 / esize;
  g.plane = (long long)g.pitch * ny + 768 / esize;
  return g;
}

extern "C" int rule_stores_bypass(int nx, int ny, int esize, int kept) {
  return lbk::stores_bypass(geom(nx, ny, esize), size_t(esize), kept != 0);
}

// Rows of a strip for `tiles` tiles of columns.
extern "C" int rule_strip_rows(int tiles, int ny, int want, int lo, int hi, int big) {
  return lbk::split_rows(tiles, ny, want, lo, hi, big).rows;
}

// Strips of the diagnostics passes: their rows, or with `blocks` their count.
extern "C" int rule_diag(int nx, int ny, int storage, int blocks) {
  const lbk::Geom g = geom(nx, ny, storage == LBMHD_FP32 ? 4 : 2);
  return blocks ? lbk::diag_partials(storage, g) : lbk::diag_rows(storage, g);
}
extern "C" int rule_diag_by_row(int nx, int ny) { return lbk::diag_by_row(geom(nx, ny, 4)); }

extern "C" int rule_tile_wide(int nx, int ny, int storage, int k, int keep) {
  return lbk::tile_wide(storage, k, keep != 0, geom(nx, ny, storage == LBMHD_FP32 ? 4 : 2));
}

// Steps of a tile launch (0: by rows), whether k steps alone go to tiles, and
// whether kept states do.
extern "C" int rule_tile_steps(int nx, int ny, int storage, int les) {
  return lbk::tile_steps(storage, les & 4 ? 2 : les & 1, (les & 2) != 0, geom(nx, ny, storage == LBMHD_FP32 ? 4 : 2));
}
extern "C" int rule_tile_short(int nx, int ny, int storage, int nb, int k) {
  return lbk::tile_short_pays(storage, nb != 0, k, geom(nx, ny, storage == LBMHD_FP32 ? 4 : 2));
}
extern "C" int rule_tile_keep(int nx, int ny, int storage, int nb) {
  return lbk::tile_keep_pays(storage, nb != 0, geom(nx, ny, storage == LBMHD_FP32 ? 4 : 2));
}

// Whether the paired reverse step goes by tiles.
extern "C" int rule_adj_tile(int nx, int ny, int storage) {
  return lbk::adj_tile_pays(storage, geom(nx, ny, storage == LBMHD_FP32 ? 4 : 2));
}

// Planes of a block of the 3D diagnostics.
extern "C" int rule_diag3_chunk(int tiles, int nz) { return lbk3::diag3_chunk(tiles, nz); }
