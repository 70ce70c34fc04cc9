// Which attention backward calls run their two sides in one launch, and which rows of the mask a workgroup of any
// attention kernel takes.  Plain C++, without the device's headers.
#pragma once
#include "lx_chip.h"

namespace lx {

// Where the elements of a call's tensors [B, Hh, S, D] lie, in bytes: rows of `row`, n[i] of them stride[i] apart.
struct TensorShape {
  long long n[3], stride[3], row;
  long long extent() const {
    long long e = row;
    for (int i = 0; i < 3; ++i) e += (n[i] - 1) * stride[i];
    return e;
  }
};
struct Range {
  const void* p;
  long long bytes;
};
inline long long byte_distance(const void* a, const void* b) { return (const char*)b - (const char*)a; }
inline bool ranges_meet(const Range& a, const Range& b) {
  const long long d = byte_distance(a.p, b.p);
  return d < a.bytes && -d < b.bytes;
}
// Whether two tensors of that shape, the second `delta` bytes behind the first, have a byte in common: some difference of
// two of their rows' places is less than a row from delta.  The places are sums over the dimensions, so this goes down
// from the longest stride, with the differences that the shorter ones can still make up for: two at most where the
// dimensions are nested, which tensors interleaved in one buffer are too.  Where they are not, and there are many, the
// tensors count as meeting.
inline bool tensors_meet(const TensorShape& t, long long delta) {
  struct {
    long long n, stride;
  } dim[3];
  int dims = 0;
  for (int i = 0; i < 3; ++i) {
    if (t.n[i] <= 1 || t.stride[i] == 0) continue;
    int at = dims++;
    for (; at > 0 && dim[at - 1].stride < t.stride[i]; --at) dim[at] = dim[at - 1];
    dim[at] = {t.n[i], t.stride[i]};
  }
  struct Walk {
    decltype(dim)& d;
    int dims;
    long long row;
    bool operator()(long long delta, int level) const {
      if (level == dims) return delta < row && -delta < row;
      const long long s = d[level].stride, most = d[level].n - 1;
      long long reach = row - 1;       // of the dimensions below
      for (int i = level + 1; i < dims; ++i) reach += (d[i].n - 1) * d[i].stride;
      auto floor_div = [&](long long a) { return a >= 0 ? a / s : -((-a + s - 1) / s); };
      long long lo = -floor_div(reach - delta), hi = floor_div(delta + reach);
      lo = lo < -most ? -most : lo;
      hi = hi > most ? most : hi;
      if (hi - lo >= 8) return true;
      for (long long k = lo; k <= hi; ++k)
        if ((*this)(delta - k * s, level + 1)) return true;
      return false;
    }
  };
  return Walk{dim, dims, t.row}(delta, 0);
}

// The buffers of a backward call: tensors of one shape, and what lies in one piece.
struct BwdBuffers {
  TensorShape shape;
  const void *in[5], *out[3];          // Q, K, V, O, dO; dQ, dK, dV
  Range lse, list[2];                  // list: what the query side walks
  Range scratch[2];                    // Delta, the rescaled LSE
};
// Whether the two sides may run side by side.  One after the other, an output may lie over whatever the query side alone
// reads (O, LSE, its list) or over the rows that a workgroup alone reads (dK on K, dV on V, dQ on O), an output that is not
// wanted on another one's place, and the rescaled LSE on LSE.
inline bool bwd_sides_apart(const BwdBuffers& b) {
  const long long extent = b.shape.extent();
  for (int o = 0; o < 3; ++o) {
    for (const void* in : b.in)
      if (tensors_meet(b.shape, byte_distance(in, b.out[o]))) return false;
    for (int p = 0; p < o; ++p)
      if (tensors_meet(b.shape, byte_distance(b.out[p], b.out[o]))) return false;
    const Range out = {b.out[o], extent};
    if (ranges_meet(out, b.lse) || ranges_meet(out, b.list[0]) || ranges_meet(out, b.list[1])) return false;
  }
  return !ranges_meet(b.scratch[0], b.lse) && !ranges_meet(b.scratch[1], b.lse);
}

// Whether one launch pays.  The key side then makes Delta itself, for every block that it streams, from O tiles of which the
// other two launches need none; and a CU has room for three workgroups (head size 64) or one (128: three tiles a stage
// are 96 KB).  What it saves is the chain of loads that starts a launch, and a launch that lasts as long as its longest
// row.  While the rows of both sides are resident at once, it takes 0.56 - 0.85 of the time, whatever the lists: up to 384 rows
// of all heads and batch entries at head size 64, 128 at 128.  Up to twice that it pays where rows are of different
// lengths, as under a causal mask (one launch / two, us: 12 heads of 4096 tokens, all blocks 131 / 161, 10 % 25 / 37; D = 128, 4 of 4096
// 138 / 176), or lists short.  Without causality long lists take longer: head size 64, 768 rows, 10 / 30 / 60 / 100 % of 64 blocks 35 /
// 84 / 156 / 250 and 44 / 92 / 149 / 216, of 32 blocks 21 / 46 / 81 / 128 and 30 / 55 / 81 / 113, which is more won than lost while only the
// lists' capacity is known; 128, 256 rows of 64 38 / 89 / 163 / 260 and 46 / 89 / 136 / 176, of 16 18 / 30 / 49 / 72 and 24 / 37 / 50 / 54,
// so there the capacity has to say that they are short (`mean`: blocks per row).  With short rows up to 1728 (16 heads of 4096, all blocks 0.97, 24 of
// 4096 0.88 of the speed; causal, 1152 rows of 16 blocks, all of them 70 and 65 us, 10 % 18 and 23).
// Not at the token strides of the kernels with 64-bit addresses (kWideStride), where every row lies in pages of its own and
// reading O again costs more than a launch: head size 64, 2^26 elements, 128 heads of 512 tokens 114 us in one, 102 in two; 256
// of 256 76 and 72; 32 of 1024 96 and 86 (2^25: 62 and 59, 42 and 43, 55 and 53).
inline bool bwd_one_launch_pays(int D, long long rows, int nblk, bool causal, double mean) {
  if (D == 128) return rows <= 128 || (rows <= 256 && (causal || mean <= 2 || (mean <= 6 && 2 * mean <= nblk)));
  return rows <= 768 || (rows <= 1728 && rows * nblk <= 20000);
}

// ---- which rows of the mask a workgroup takes ----------------------------------------------------
// Estimate of a launch of `groups` workgroups with r rows each on average, `slots` of them at a time, in units of one row (see
// attn_rows_per_wg).
inline double attn_rows_cost(double r, long long groups, int slots, int nblk) {
  const double start = 0.38 * (1 + 16.0 / nblk);
  const long long full = groups / slots, left = groups % slots;
  if (groups <= slots) return (r + start) * (1 + 0.015 * r);
  const double f = (double)left / slots;
  const double part = 0.5 + (full > 1 && f <= 0.5 ? 0.35 : 1.1) * f, last = left == 0 ? 0.0 : part < 1.0 ? part : 1.0;
  return r * (full + last) + start * (full + (left > 0));
}
constexpr int kRMax = 8;   // rows of the mask per workgroup, at most
// Rows per workgroup, unless the caller fixed the number (`forced`): the smallest count with which all workgroups of the
// launch are resident at once on the chip's `slots` workgroup slots (a causal mask keeps the groups balanced for
// every count, because slots are filled in pairs k, 2G-1-k), or a smaller one with more workgroups than slots.
// Those pay a start per round, but the dispatcher hands them out as slots become free, which evens out pairs with
// long and short lists, and fewer pairs share an L2 at a time.  The estimate (attn_rows_cost), in units of one row: a round costs
// r rows plus its start, which weighs more where lists are short; a last round that is not full is faster,
// workgroups being alone on their CUs, and the more so when earlier rounds have spread the starts; a single round
// lasts 1.5 % longer per row, having nothing to even it out.  Over 173 launches of both head sizes
// (profiles/attn_rows_sweep.txt) the chosen count is 1.2 % slower than the best one on average, 14 % at worst (12 heads of
// 2048 tokens, D = 128, all blocks, dK and dV: 61 us with one row, 54 with two); against one round always, forward / dQ /
// dK and dV take 0.990 / 0.996 / 0.995 of the time with head size 128 and 0.994 / 0.990 / 0.994 with 64, at worst 1.03 /
// 1.05 / 1.06, the last at 2 x 40 heads of 2048 tokens, 25 % of the blocks, D = 128 (2 rows for 6; with all blocks
// the same choice takes 0.95 - 1.00).  What it is for: 4 x 32 heads of 2048 tokens, 25 %, D = 128, forward 82 -> 66 us
// (8 rows -> 4).
inline int attn_rows_per_wg(int nblk, long long pairs, int slots, int forced) {
  auto groups = [&](int r) { return (long long)((nblk + r - 1) / r) * pairs; };
  int r = 1;
  while (r < kRMax && groups(r) > slots) ++r;
  for (int q = r - 1; q >= 1; --q)
    if (attn_rows_cost(q, groups(q), slots, nblk) < attn_rows_cost(r, groups(r), slots, nblk)) r = q;
  if (forced > 0) r = forced;
  return r > nblk ? nblk : r;
}
// By turns: an XCD's (batch entry, head) pairs are x, x + 8, ..; the rows, at most 64, of several consecutive ones of those are
// a cohort, and a workgroup has one row of each of several cohorts, the same number of rows as every other one and about
// the same number of blocks, all workgroups being resident at once.  The rows of one pair (or four) that a workgroup has
// otherwise divide evenly only by chance: 8 x 33 heads of 256 tokens at head size 128 are two rows for each of 512 workgroups, otherwise
// 264 workgroups of four rows, CUs with two of them next to CUs with one.
// The rank of a list says less of its length where most lists have no more than a block, and a launch of several rounds evens
// out by itself, so it has to promise more than that:
// - where all workgroups are resident the other way too, a workgroup has fewer rows and the busiest CU a fifth fewer;
// - where they are several rounds, the estimate (with the rows that a workgroup has on average) says 12 % less, and there are
//   two workgroups to a CU: four or three (head size 64) even each other out unless they have a row each;
// - at most five rows: with six and seven the launches took 0.97 of the time, 26 of 152 more than 1.02, up to 1.12.
// 755 launches of 64 - 4096 tokens, 8 - 40 heads and 1 - 8 batch entries, 10 - 100 % of the blocks, for which it is taken, on the same
// buffers: forward 0.89, dQ 0.90, dK and dV 0.90 of the time on average, 0.72 - 1.11, 29 of them above 1.02, with a block or so per row
// (profiles/attn_turns_sweep.txt).  Of 695 more that were estimated 8 % faster, with workgroups of as many rows as the fullest one, 132 took more
// than 1.02 of the time, up to 1.16, 0.965 on average; of 810 with as many rows in a workgroup either way and a fifth fewer on the busiest CU
// 190, up to 1.17, 0.97 on average.  Forward / backward, us, that way / by turns: 2 x 40 of 2048, D = 128, all blocks 130.6 / 357.8 -> 124.3 /
// 351.0, 25 % 50.8 / 135.6 -> 46.2 / 128.2; 8 x 40 of 512, 40 % 32.6 / 88.9 -> 30.3 / 84.7.
constexpr int kTurnsMost = 5;
constexpr double kTurnsBusiest = 0.8, kTurnsRounds = 0.88;
struct AttnTurns {
  int turns, places, cohorts, pairs, grid;      // rows per workgroup (0: not by turns), cohorts at a time, of an XCD; pairs of a cohort
};
inline AttnTurns attn_turns(int pairs, int nblk, int slots, int rows_per_wg) {
  const AttnTurns none = {0, 0, 0, 0, 0};
  if (nblk > 64 || pairs < 8 || (long long)pairs * nblk <= slots) return none;      // (a row per workgroup is the least that there is)
  const int room = slots / 8, per = (pairs + 7) / 8, most = room / nblk;    // places of an XCD, its pairs, those at a time
  const int turns = (per + most - 1) / most;
  if (turns > kTurnsMost) return none;
  const int groups = (nblk + rows_per_wg - 1) / rows_per_wg, grid = 8 * most * nblk;
  const long long wgs = (long long)groups * pairs;
  const double rows = (double)nblk / groups;
  if (wgs <= slots) {
    const double busiest = (double)((wgs + kCUs - 1) / kCUs) * rows;
    if (turns >= rows_per_wg || (double)((grid + kCUs - 1) / kCUs) * pairs * nblk / grid > kTurnsBusiest * busiest) return none;
  } else if ((rows_per_wg > 1 && slots > 2 * kCUs) ||
             attn_rows_cost(turns, grid, slots, nblk) > kTurnsRounds * attn_rows_cost(rows, wgs, slots, nblk)) {
    return none;
  }
  // the largest cohorts that take no more turns (those of one pair take that many)
  for (int V = 64 / nblk;; --V) {
    const int G = V * nblk, Z = room / G, cohorts = (per + V - 1) / V;
    if (V == 1 || (cohorts + Z - 1) / Z == turns) return {turns, Z, cohorts, V, 8 * Z * G};
  }
}
// The rank by length, among the n rows of a cohort, of the row that a place's workgroup r takes in turn k of `turns`, so that
// the ranks of all turns add up to about the same for every r: up and down by turns, of an odd number the first three by
// r; n - 1 - 2 r in the first half, and 2 n - 1 - 2 r, for an even n 2 n - 2 - 2 r, in the second; r + n / 2 and r - (n + 1) / 2.
LX_HD int turn_rank(int r, int k, int n, int turns) {
  if (turns % 2 == 1 && turns >= 3) {
    const int low = (n + 1) / 2;         // r below: the first half
    if (k == 1) return r < low ? n - 1 - 2 * r : 2 * n - 1 - (n % 2 == 0 ? 1 : 0) - 2 * r;
    if (k == 2) return r < low ? r + n / 2 : r - low;
    if (k > 2) k -= 3;
  }
  return k % 2 == 0 ? r : n - 1 - r;
}

// How an attention launch of B * Hh pairs with nblk rows each is laid out, `slots` workgroups at a time.
struct AttnShape {
  int rows_per_wg, vheads, gz, spread, grid;      // (see AttnArgs)
  AttnTurns by_turns;
};
// Heads per group of workgroups: as many consecutive heads (4, 2 or 1) as divide the head count
// and whose rows one wavefront can rank (64 lanes).  The rows of the group are dealt to its
// workgroups together, so heads with long and with short lists even each other out.
inline int heads_per_group(int nblk, int heads) {
  for (int v = 4; v > 1; v /= 2)
    if (heads % v == 0 && v * nblk <= 64) return v;
  return 1;
}
// may_turn: the kernel can take its rows by turns; forced: rows per workgroup that the caller fixed, 0 otherwise.
inline AttnShape attn_shape(int B, int Hh, int nblk, int slots, bool may_turn, int forced) {
  AttnShape a = {};
  const long long pairs = (long long)B * Hh;
  a.rows_per_wg = attn_rows_per_wg(nblk, pairs, slots, forced);
  if (may_turn && forced == 0 && pairs < 1 << 20) a.by_turns = attn_turns((int)pairs, nblk, slots, a.rows_per_wg);
  a.vheads = heads_per_group(nblk, Hh);
  a.gz = (nblk + a.rows_per_wg - 1) / a.rows_per_wg * a.vheads;
  const int P = B * (Hh / a.vheads);
  const long long n = (long long)P * a.gz;
  a.spread = a.rows_per_wg <= 3 && n > kCUs && n <= slots;
  a.grid = a.by_turns.turns > 0 ? a.by_turns.grid : 8 * (P / 8 * a.gz + (P % 8 * a.gz + 7) / 8);
  return a;
}

}  // namespace lx
