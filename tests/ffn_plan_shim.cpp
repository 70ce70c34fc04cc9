// The tile rules of csrc/ffn_plan.h as C functions (compiled by ffn_plan.py with the host compiler).
#include "../paper_2510_15964_amd/csrc/ffn_plan.h"

using namespace lx;

extern "C" {

// The first product's tile for a list of n entries handed over with the capacity nnz_cap.
int sdd_tile(int Tt, int gt, int d, int nnz_cap, int blocks, int want, int n) {
  const SddPlan p = plan_sdd(Tt, gt, d, nnz_cap, blocks, want);
  if (!p.allowed || sdd_keeps_own(nnz_cap, n)) return p.id;
  if (kTileInfo[p.id].resident == 1)
    return sdd_pick<1>(p.id, p.allowed, sdd_limit<1>(p.id, p.grid, Tt, gt, n), Tt, gt, d, n);
  return sdd_pick<2>(p.id, p.allowed, sdd_limit<2>(p.id, p.grid, Tt, gt, n), Tt, gt, d, n);
}
// 1: the kernel of that tile alone is launched, 0: one that chooses among its set.
int sdd_alone(int Tt, int gt, int d, int nnz_cap, int blocks, int want) {
  return plan_sdd(Tt, gt, d, nnz_cap, blocks, want).allowed == 0;
}
// Workgroups launched, and those that the tile of sdd_tile needs.
int sdd_launched(int Tt, int gt, int d, int nnz_cap, int blocks, int want) {
  return plan_sdd(Tt, gt, d, nnz_cap, blocks, want).grid;
}
int sdd_needed(int id, int Tt, int gt, int n) { return sdd_grid(kTileInfo[id], Tt, gt, n); }
// The tile that the rule took before the list's length played a part, and the model's time for a tile.
int sdd_tile_of_capacity(int Tt, int gt, int d, int nnz_cap, int want) { return choose_sdd(Tt, gt, d, nnz_cap, want); }
float sdd_us(int id, int Tt, int gt, int d, int n) { return sdd_cost(kTileInfo[id], kTileInfo[id].resident, Tt, gt, d, n); }
// The second product's tile; *pieces: 1, or what the lists of its last units are cut into.
int dsd_tile(int Tt, int gt, int d, int nnz_cap, long long part_bytes, int want, int* pieces) {
  const DsdPlan p = choose_dsd(Tt, gt, d, nnz_cap, (size_t)part_bytes, want);
  *pieces = p.pieces;
  return p.id;
}
// The kernel that the first product of a list with that capacity is launched by (Route), and the tile that it runs with for
// a list of n entries (-1: quarters, or 4 x 4 tiles and narrower ones).
int sdd_by(int Tt, int gt, int d, int nnz_cap, int blocks, int want, int n, int* tile) {
  const SddRoute r = sdd_route(Tt, gt, d, nnz_cap, blocks, want);
  const bool mixes = r.mix && sdd_keeps_own(nnz_cap, n) && sdd_mixes(sdd_mix(Tt, n));
  *tile = r.by == kNothing || r.by == kByQuarters || mixes ? -1 : sdd_tile(Tt, gt, d, nnz_cap, blocks, want, n);
  return r.by;
}
// Likewise the second; *pieces as in dsd_tile.
int dsd_by(int Tt, int gt, int d, int F, int nnz_cap, long long part_bytes, int want, int* tile, int* pieces) {
  const DsdRoute r = dsd_route(Tt, gt, d, F, nnz_cap, (size_t)part_bytes, want);
  *tile = r.by == kByQuarters || r.by == kByMix ? -1 : r.plan.id;
  *pieces = r.by == kByQuarters || r.by == kByMix ? 1 : r.plan.pieces;
  return r.by;
}
// The first product by pieces, as ffn_sdd_even's workgroups find theirs: workgroups launched for a list with that capacity, and per
// workgroup tile, first entry, entries in out (room for cap of them; tile -1: none); *per: the most entries of a piece.
int even_items(const int* row_ptr, int Tt, int cap, int room, int* out, int* per) {
  auto clip = [&](int v) { return v < cap ? v : cap; };
  auto entries = [&](int i) { return i < Tt ? clip(row_ptr[i + 1]) - clip(row_ptr[i]) : 0; };
  const bool two = Tt > 64;
  EvenLane lane[64];
  for (int l = 0; l < 64; ++l) lane[l] = {two ? entries(2 * l) : entries(l), two ? entries(2 * l + 1) : 0, 0, 0};
  auto pieces = [&](int p) {
    int k = 0;
    for (const EvenLane& l : lane) k += l.pieces(p);
    return k;
  };
  *per = even_per(pieces, [&] { return pieces(kEvenShort); });
  int firsts = 0, total = 0;
  for (EvenLane& l : lane) l.cut(*per), firsts += l.firsts(), total += l.k0 + l.k1;
  const int grid = sdd_even_grid(Tt, cap), found = sdd_even_grid(Tt, clip(row_ptr[Tt]));
  for (int w = 0; w < grid && w < room; ++w) {
    int* o = out + 3 * w;
    o[0] = -1;
    int work = w < found ? even_place(w, total) : -1;
    if (work < 0) continue;
    const bool second = work >= firsts;
    if (second) work -= firsts;
    for (int l = 0; l < 64; ++l) {
      const int mine = second ? lane[l].k0 + lane[l].k1 - lane[l].firsts() : lane[l].firsts();
      if (work >= mine) {
        work -= mine;
        continue;
      }
      const EvenPiece p = lane[l].piece(second, work);
      o[0] = (two ? 2 * l : l) + p.odd, o[1] = p.first, o[2] = p.count;
      break;
    }
  }
  return grid;
}
// The predictor by quarters of its tiles (where d is no multiple of 128).
int predict_quarters(int items, int d) { return quarters_pay(items, d, 0); }
// 1: the gradients of the LoRA matrices by quadrants, 0: by parts.
int grads_by_quads(int Tt, int d, int F) { return lora_grads_by_quads(Tt, d, F); }

}  // extern "C"
