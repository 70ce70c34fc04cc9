// Which attention backward calls run in one launch and which rows a workgroup takes (csrc/attn_plan.h), as C functions.
#include "../paper_2510_15964_amd/csrc/attn_plan.h"

using namespace lx;

extern "C" {

int meet(const long long* n, const long long* stride, long long row, long long delta) {
  return tensors_meet({{n[0], n[1], n[2]}, {stride[0], stride[1], stride[2]}, row}, delta);
}
int pays(int D, long long rows, int nblk, int causal, double mean) { return bwd_one_launch_pays(D, rows, nblk, causal, mean); }
// at: byte addresses of Q, K, V, O, dO; dQ, dK, dV; LSE, row_ptr, col_idx, Delta, the rescaled LSE
int sides_apart(const long long* n, const long long* stride, long long row, const long long* at, long long stats, long long ptrs,
                long long entries) {
  auto p = [&](int i) { return (const void*)at[i]; };
  return bwd_sides_apart({{{n[0], n[1], n[2]}, {stride[0], stride[1], stride[2]}, row},
                          {p(0), p(1), p(2), p(3), p(4)},
                          {p(5), p(6), p(7)},
                          {p(8), stats},
                          {{p(9), ptrs}, {p(10), entries}},
                          {{p(11), stats}, {p(12), stats}}});
}

// turns, places, cohorts, pairs, grid
void turns(int pairs, int nblk, int slots, int rows_per_wg, int* out) {
  const AttnTurns t = attn_turns(pairs, nblk, slots, rows_per_wg);
  const int v[5] = {t.turns, t.places, t.cohorts, t.pairs, t.grid};
  for (int i = 0; i < 5; ++i) out[i] = v[i];
}
int rank_in_turn(int r, int k, int n, int turns) { return turn_rank(r, k, n, turns); }

}  // extern "C"
