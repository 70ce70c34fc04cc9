// First product with one list row: wide tiles and a rest by narrower ones (csrc/ffn_plan.h), as C functions.
#include "../paper_2510_15964_amd/csrc/ffn_plan.h"

using namespace lx;

extern "C" {

int may_mix(int Tt, int d, int cap, int blocks, int want) {
  return sdd_route(Tt, Tt, d, cap, blocks, want).mix;
}
int mix_grid(int Tt, int cap) { return sdd_mix_grid(Tt, cap); }
// -2: a list of n entries does not run so, otherwise the tile of the rest (-1: none).
int mix_tail(int Tt, int n) {
  const SddMix m = sdd_mix(Tt, n);
  return sdd_mixes(m) ? m.tail : -2;
}
// Token tiles and list entries of workgroup w: first tile, tiles, first entry, entries; 0: none.
int mix_item(int Tt, int n, int w, int* out) {
  int id;
  GridItem it;
  if (!sdd_mix_item(sdd_mix(Tt, n), Tt, n, w, id, it)) return 0;
  const TileInfo& t = kTileInfo[id];
  out[0] = it.m * t.tm;
  out[1] = t.tm;
  out[2] = it.n * t.tn;
  out[3] = t.tn;
  return 1;
}
// Second product: -2: by the plan's own tile, otherwise the tile of the rest.
int down_tail(int Tt, int d, int cap, int want) {
  return dsd_route(Tt, Tt, d, 64ll * (cap + 3), cap, ~(size_t)0, want).by == kByMix ? sdd_mix(Tt, d / 64).tail : -2;
}
int keeps_own(int cap, int n) { return sdd_keeps_own(cap, n); }

}  // extern "C"
