// How the launches with lists per group of token tiles deal their work (csrc/ffn_plan.h), as C functions.
#include "../paper_2510_15964_amd/csrc/ffn_plan.h"

using namespace lx;

extern "C" {

// The unit of workgroup w of the second product as chunk * GM + rank; -1: none.
int unit_of(int order, int GM, int GN, int w) {
  int chunk, rank;
  return dsd_unit(order, GM, GN, w, chunk, rank) ? chunk * GM + rank : -1;
}
int order_of(int Tt, int gt, int d, int Fb, int nnz_cap) { return dsd_route(Tt, gt, d, 64ll * Fb, nnz_cap, 0, 0).order; }
// bit 0: the first product by tiles of one stage, bit 1: the second.
int lean_of(int Tt, int gt, int d, int Fb, int nnz_cap) {
  return (sdd_route(Tt, gt, d, nnz_cap, Tt / gt * Fb, 0).by == kByLean ? 1 : 0) |
         (dsd_route(Tt, gt, d, 64ll * Fb, nnz_cap, 0, 0).by == kByLean ? 2 : 0);
}
// 1: an XCD takes half of every list in the first product, 0: whole lists.
int halves_of(int Tt, int gt, int d, int Fb, int nnz_cap) { return sdd_route(Tt, gt, d, nnz_cap, Tt / gt * Fb, 0).halves; }
int quick(int a, int b) { return quick_div(a, b); }

}  // extern "C"
