// How the launches with lists per group of token tiles deal their work (csrc/ffn_plan.h), as C functions.
#include "../paper_2510_15964_amd/csrc/ffn_plan.h"

using namespace lx;

extern "C" {

// The unit of workgroup w of the second product as chunk * GM + rank; -1: none.
int unit_of(int order, int GM, int GN, int w) {
  int chunk, rank;
  return dsd_unit(order, GM, GN, w, chunk, rank) ? chunk * GM + rank : -1;
}
int order_of(int Tt, int gt, int d, int Fb, int nnz_cap) {
  const int id = choose_dsd(Tt, gt, d, nnz_cap, 0, 0).id, GM = Tt / kTileInfo[id].tm, GN = ceil_div(d, 64 * kTileInfo[id].tn);
  return dsd_order(GM, GN, kTileInfo[id].tn, dsd_lean(id, Tt, gt, GM, GN, nnz_cap, 64ll * Fb), 128ll * Fb * d);
}
// bit 0: the first product by tiles of one stage, bit 1: the second.
int lean_of(int Tt, int gt, int d, int Fb, int nnz_cap) {
  const int up = choose_sdd(Tt, gt, d, nnz_cap, 0), down = choose_dsd(Tt, gt, d, nnz_cap, 0, 0).id;
  const TileInfo& t = kTileInfo[down];
  return (sdd_lean(up, Tt, gt, nnz_cap) ? 1 : 0) | (dsd_lean(down, Tt, gt, Tt / t.tm, ceil_div(d, 64 * t.tn), nnz_cap, 64ll * Fb) ? 2 : 0);
}
// 1: an XCD takes half of every list in the first product, 0: whole lists.
int halves_of(int Tt, int gt, int nnz_cap) { return sdd_halves(Tt, gt, nnz_cap); }
int quick(int a, int b) { return quick_div(a, b); }

}  // extern "C"
