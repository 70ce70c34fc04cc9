// Which attention backward calls run in one launch and which rows a workgroup takes (csrc/attn_plan.h), as C functions.
#include <chrono>

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
// How a launch is laid out: rows per workgroup, heads of a group, workgroups of a group, spread, grid, turns
void shape(int B, int Hh, int nblk, int slots, int may_turn, int forced, int* out) {
  const AttnShape s = attn_shape(B, Hh, nblk, slots, may_turn, forced);
  const int v[6] = {s.rows_per_wg, s.vheads, s.gz, s.spread, s.grid, s.by_turns.turns};
  for (int i = 0; i < 6; ++i) out[i] = v[i];
}
// Nanoseconds of a call, over 2000 of them
}  // extern "C"
template <class F>
static double ns_of(F f) {
  volatile int sink = 0;
  const auto start = std::chrono::steady_clock::now();
  for (int i = 0; i < 2000; ++i) sink = sink + f();
  return std::chrono::duration<double, std::nano>(std::chrono::steady_clock::now() - start).count() / 2000;
}
extern "C" {
double turns_ns(int pairs, int nblk, int slots, int rows) {
  volatile int p = pairs, n = nblk, s = slots, r = rows;
  return ns_of([&] { return attn_turns(p, n, s, r).turns; });
}
double rows_ns(int pairs, int nblk, int slots, int) {
  volatile int p = pairs, n = nblk, s = slots;
  return ns_of([&] { return attn_rows_per_wg(n, p, s, 0); });
}
int rank_in_turn(int r, int k, int n, int turns) { return turn_rank(r, k, n, turns); }

}  // extern "C"
