// Which tile the 16-bit FFN products run with: a cost model over sizes.  Plain C++ for host and device: the host
// decides by the list's capacity, the first product's kernels decide again by its true length (see SddSet).
#pragma once
#include <stddef.h>

#include "lx_chip.h"

namespace lx {

// The tiles, widest first.  A wide tile moves fewer bytes and LDS reads per product (a workgroup step
// transfers TM + TN times 8 KiB for TM * TN products of 64 x 64 x 64), a narrow one gives the chip more
// workgroups and has the shorter step.  `resident` workgroups fit a CU; one workgroup per CU leaves room
// for a deeper ring, and eight wavefronts with a whole step of operands on the way hide its latency
// (2 x 2 tiles, 4096 tokens, 14 blocks, K = 2048, 224 workgroups: 25 -> 21 us).
enum TileId { kT44, kT24, kT22, kT22Deep, kT14, kT14Deep, kT12, kT11, kT11Many, kTiles };
// What a launch of a tile costs, in us: `round` per round of workgroups (finding the item, filling the
// ring, epilogue) and step[q - 1] per step with q workgroups on a CU.  Fitted to measured launches (64 - 8192 tokens,
// d 576 - 5120, 6 - 320 listed blocks, lists shared and per tile) of the kernels on the 32x32x16 matrix instruction, before
// the 16x16x32 one.  Checked with the present ones at 26 shapes, every tile of both products (profiles/ffn_tile_sweep.txt):
// model to measured 1.01 in the geometric mean, rms 19 %, and the tile that is taken is 1.4 % slower than the fastest one
// on average, 29 % at worst (first product, 8192 tokens, d = 2048, a list of 16 blocks per four token tiles: 52 us by 4 x 4
// tiles, 40 by 2 x 2; the next one 11 %).  On the same lists it took the kernels of the fit 2.0 % and 29 %.
struct TileInfo {
  int tm, tn, resident;
  float round, step[3];
};
constexpr TileInfo kTileInfo[kTiles] = {
    {4, 4, 1, 8.6f, {1.25f}},      {2, 4, 1, 7.4f, {0.69f}}, {2, 2, 2, 4.2f, {0.61f, 1.11f}},
    {2, 2, 1, 5.1f, {0.44f}},      {1, 4, 2, 4.8f, {0.69f, 1.28f}}, {1, 4, 1, 5.5f, {0.51f}},
    {1, 2, 2, 4.0f, {0.29f, 0.62f}}, {1, 1, 2, 3.8f, {0.17f, 0.39f}}, {1, 1, 3, 3.3f, {0.22f, 0.39f, 0.61f}},
};
LX_HD int ceil_div(int a, int b) { return (int)(((unsigned)a + (unsigned)b - 1) / (unsigned)b); }   // a >= 0
// `resident`: at most the tile's own
LX_HD float tile_cost(const TileInfo& t, int resident, int items, float steps) {
  const unsigned q = items <= kCUs ? 1 : ceil_div(items, kCUs), full = q / (unsigned)resident, rest = q % (unsigned)resident;
  const float all = t.step[resident - 1], last = rest == 0 ? 0.f : rest == 1 ? t.step[0] : t.step[1];
  return (float)(full + (rest ? 1 : 0)) * t.round + steps * ((float)full * all + last);
}
// Lists per group of tiles share few weight rows, so the bytes that the workgroups pull bound the launch:
// us for `wgs` workgroups of `steps` steps each at the rate that such launches reach (4096 - 8192 tokens,
// d 2048 - 4096: 9.3 - 13 TB/s through the L2s, of which some 6 TB/s miss).
LX_HD float pull_cost(const TileInfo& t, float wgs, float steps) {
  return wgs * steps * (float)((t.tm + t.tn) * 8192) / 11.5e6f;
}

// Whether a tile may run lists whose rows gt of the Tt token tiles share: tiles past the end are left
// out with one list row, otherwise the groups of TM tiles have to divide those of gt.  `want`: tiles per
// workgroup that the caller asked for (0: any).
inline bool tile_fits(const TileInfo& t, int Tt, int gt, int want) {
  if (want != 0) {
    int most = want;
    while (gt != Tt && gt % most != 0) most /= 2;
    if (t.tm != most) return false;
  }
  return gt == Tt || gt % t.tm == 0;
}

// ---- first product -------------------------------------------------------------------------
// Workgroups that hold all items of a list of n entries; the kernels find theirs in the first ones.  (Their numbers
// stay below 2^30: the launchers' callers see to that.)
LX_HD int sdd_grid(const TileInfo& t, int Tt, int gt, int n) {
  if (gt == Tt) return 8 * ceil_div(ceil_div(Tt, t.tm) * ceil_div(n, t.tn), 8);
  // items <= entries / tn + a ragged group per row; per XCD L = ceil(items / 8) of them in 4 * ceil(L / 4) slots at most
  const int items = ceil_div(n * (int)((unsigned)gt / t.tm), t.tn) + (t.tn > 1 ? (unsigned)Tt / t.tm : 0u);
  return 64 * ceil_div(ceil_div(items, 8), 8);
}
// us for a list of n entries; with lists per group of tiles half a ragged group per list row is added.
LX_HD int sdd_items_about(const TileInfo& t, int Tt, int gt, int n) {
  return (unsigned)n * ((unsigned)gt / t.tm) / t.tn + (unsigned)Tt / t.tm * (t.tn - 1) / (2 * t.tn);
}
LX_HD float sdd_cost(const TileInfo& t, int resident, int Tt, int gt, int d, int n) {
  const float steps = (float)((unsigned)d / 64);
  if (gt == Tt) return tile_cost(t, resident, ceil_div(Tt, t.tm) * ceil_div(n, t.tn), steps);
  const int items = sdd_items_about(t, Tt, gt, n);
  const float busy = tile_cost(t, resident, items, steps), pull = pull_cost(t, (float)items, steps);
  return (pull > busy ? pull : busy) + 0.25f * busy;
}
// With lists per group of tiles the deep 1 x 4 tile takes one round at most: a second one starts out of step with the
// first, and its L2 hits are gone.
LX_HD bool sdd_out_of_step(int id, int Tt, int gt, int n) {
  return id == kT14Deep && gt != Tt && sdd_items_about(kTileInfo[kT14Deep], Tt, gt, n) > kCUs;
}
// The tile for a list of at most nnz_cap entries.  With lists per group of tiles the number of entries varies
// between calls and a caller's capacity has slack: a seventh is taken off.
inline int choose_sdd(int Tt, int gt, int d, int nnz_cap, int want) {
  const int n = gt == Tt ? nnz_cap : (int)(6.f / 7.f * (float)nnz_cap);
  int best = -1;
  float least = 0.f;
  for (int id = 0; id < kTiles; ++id) {
    const TileInfo& t = kTileInfo[id];
    if (!tile_fits(t, Tt, gt, want) || sdd_out_of_step(id, Tt, gt, n)) continue;
    const float c = sdd_cost(t, t.resident, Tt, gt, d, n);
    if (best < 0 || c < least) best = id, least = c;
  }
  return best;
}

// A capacity may say little about a list, and only the device knows the length.  The tiles therefore come in sets,
// each compiled into one kernel, and the kernel takes the best of its set for the list that it finds: tiles of eight
// wavefronts, one workgroup per CU, and of four, two per CU (the narrow ones are in both; in the first, half of the
// wavefronts end at once).  The capacity decides the set and the grid: a tile is taken only if its items fit the
// workgroups that the capacity's own tile needs for this list, or that the CUs hold at once.
struct SddSet {
  int n, ids[6];
};
constexpr SddSet kSddWide = {6, {kT44, kT24, kT22Deep, kT14Deep, kT12, kT11}};
constexpr SddSet kSddNarrow = {4, {kT22, kT14, kT12, kT11}};
constexpr SddSet sdd_set(int resident) { return resident == 1 ? kSddWide : kSddNarrow; }
// The workgroups, out of the `grid` launched, that may have an item of a list of n entries.
template <int RESIDENT>
LX_HD int sdd_limit(int own, int grid, int Tt, int gt, int n) {
  const int need = sdd_grid(kTileInfo[own], Tt, gt, n), once = grid < RESIDENT * kCUs ? grid : RESIDENT * kCUs;
  return need > once ? need : once;
}
// The tile of a set for a list of n entries: `own`, the capacity's (its items always fit), or a better one of those
// in the bit mask `allowed` whose items fit `limit` workgroups.
template <int RESIDENT>
LX_HD int sdd_pick(int own, unsigned allowed, int limit, int Tt, int gt, int d, int n) {
  constexpr SddSet set = sdd_set(RESIDENT);
  int best = own;
  float least = 0.f;
  bool first = true;
#pragma unroll
  for (int k = 0; k < set.n; ++k) {
    const int id = set.ids[k];
    const TileInfo t = kTileInfo[id];
    if (id != own && (!(allowed >> id & 1u) || sdd_grid(t, Tt, gt, n) > limit || sdd_out_of_step(id, Tt, gt, n))) continue;
    const float c = sdd_cost(t, RESIDENT, Tt, gt, d, n);
    if (first || c < least) best = id, least = c, first = false;
  }
  return best;
}
// A list that fills three quarters of its capacity keeps the capacity's tile: the choice takes up to a microsecond.
LX_HD bool sdd_keeps_own(int nnz_cap, int n) { return n >= nnz_cap - nnz_cap / 4; }
struct SddPlan {
  int id, grid;          // the capacity's tile, whose `resident` names the set; workgroups
  unsigned allowed;      // tiles for sdd_pick, 0: `id` as it is
};
// `blocks`: every block that the list could hold.  The kernel chooses for one list row, whose length it reads anyway;
// with lists per group of tiles, where that is a load before the first, only if the capacity is every block, that is,
// if the caller knows nothing better, and with a list per tile only up to 64 tiles: from there on the 1 x 4 tile
// serves most lists, and the search costs every surplus workgroup more than it gains (64 tiles, d = 2048, 11 % of the
// blocks, every block as capacity: 42 us by the capacity's tile, 45 with the choice; 32 tiles 33.5 and 25.8).
inline SddPlan plan_sdd(int Tt, int gt, int d, int nnz_cap, int blocks, int want) {
  SddPlan p = {choose_sdd(Tt, gt, d, nnz_cap, want), 0, 0u};
  const int resident = kTileInfo[p.id].resident;
  p.grid = sdd_grid(kTileInfo[p.id], Tt, gt, nnz_cap);
  if (p.grid == 0 || p.id >= kT11) return p;      // (nothing is narrower than kT11)
  if (gt != Tt && (nnz_cap < blocks || (resident == 2 && Tt >= 64))) return p;
  if (p.grid < resident * kCUs) p.grid = resident * kCUs;
  for (int id = 0; id < kTiles; ++id)
    if (tile_fits(kTileInfo[id], Tt, gt, want)) p.allowed |= 1u << id;
  return p;
}

// ONE list row shared by all token tiles: items (group of TM tiles m, group of TN entries
// n), or for the dsd kernel (m, chunk of output columns n), in bands of `h` groups m that are walked
// along n, h items at a time; XCD x takes the x-th eighth of that order.  The workgroups that run
// together on an XCD then share h token groups and a few weight groups, and with at most h groups of
// tokens every weight row is fetched into one L2 only.
struct GridItem {
  int m, n;
};
LX_HD GridItem grid_item(int idx, int GM, int GN, int h) {
  const int per = h * GN, band = idx / per, left = GM - band * h;
  const int hb = left < h ? left : h, rem = idx - band * per;
  return {band * h + rem % hb, rem / hb};
}

// One list row: the items of 4 x 4 tiles that do not fill a round run by narrower tiles, halved or quartered, whose round
// is shorter.  Per XCD: L items, of which `whole` run as they are and each of the rest in `parts` of tile `tail` (-1:
// nothing is left, or more than half a round).  First product, plain and mixed, us: 8192 tokens, d = 4160, 36 blocks 167 ->
// 139; 4096, 4096, 72 164 -> 136; 2560, 3200, 110 132 -> 111; 8192, 1024, 40 57.5 -> 51.5; 3904, 5120, 96 224 -> 212; 6144, 4096,
// 190 510 -> 493; 31 sizes 0.999 - 1.21 times as fast, 1.12 in the geometric mean.  (2 x 4 tiles with a rest by 2 x 2 are
// slower than the 4 x 4 tiles that the plan takes there: ten sizes, 0.94 - 0.997.)
struct SddMix {
  int L, whole, tail, parts;
};
LX_HD SddMix sdd_mix(int Tt, int n) {
  constexpr int per = kCUs / 8;
  SddMix m = {ceil_div(ceil_div(Tt, 4) * ceil_div(n, 4), 8), 0, -1, 1};
  m.whole = m.L / per * per;
  const int rest = m.L - m.whole;
  if (rest > 0 && 4 * rest <= per)
    m.tail = kT22Deep, m.parts = 4;
  else if (rest > 0 && 2 * rest <= per)
    m.tail = kT24, m.parts = 2;
  return m;
}
// Whether lists of that length run so (with nothing left as well: whole rounds of the widest tile).
LX_HD bool sdd_mixes(const SddMix& m) { return m.whole > 0 && (m.tail >= 0 || m.whole == m.L); }
// Workgroup w: tile and item (along the tokens, along the list, in units of the tile); false past the end.
LX_HD bool sdd_mix_item(const SddMix& x, int Tt, int n, int w, int& id, GridItem& it) {
  const int GM = ceil_div(Tt, 4), GN = ceil_div(n, 4), slot = w / 8, over = slot - x.whole, rest = over > 0 ? over : 0;
  const int q = x.parts == 4 ? rest / 4 : x.parts == 2 ? rest / 2 : rest, part = rest - q * x.parts;
  const int at = over < 0 ? slot : x.whole + q, idx = w % 8 * x.L + at;
  if (at >= x.L || idx >= GM * GN) return false;
  it = grid_item(idx, GM, GN, 4);
  id = kT44;
  if (over < 0) return true;
  id = x.tail;
  it.m = 2 * it.m + part % 2;
  if (id == kT22Deep) it.n = 2 * it.n + part / 2;
  const int tn = id == kT22Deep ? 2 : 4;
  return 2 * it.m < Tt && tn * it.n < n;
}
// Whether a launch is laid out for that: for a list as long as its capacity it would be faster by the model.
inline bool sdd_may_mix(const SddPlan& p, int Tt, int gt, int d, int nnz_cap, int want) {
  if (want != 0 || gt != Tt || !p.allowed || kTileInfo[p.id].resident != 1) return false;
  const SddMix m = sdd_mix(Tt, nnz_cap);
  if (!sdd_mixes(m) || m.tail < 0) return false;
  const float steps = (float)(d / 64);
  const TileInfo &b = kTileInfo[kT44], &t = kTileInfo[m.tail];
  return (float)(m.whole / (kCUs / 8)) * (b.round + steps * b.step[0]) + t.round + steps * t.step[0] <
         0.98f * sdd_cost(kTileInfo[p.id], 1, Tt, gt, d, nnz_cap);
}
// Workgroups that hold any mix for lists up to n entries (the rest of an XCD takes a round at most).
inline int sdd_mix_grid(int Tt, int n) { return 8 * (sdd_mix(Tt, n).whole + kCUs / 8); }

// ---- second product ------------------------------------------------------------------------
// Its steps are the list entries.  With one list row and room for partial sums
// the units that do not fill a round may have their list cut into 2 - 4 pieces, each at least 8 entries
// long, which costs a second launch and the pieces' way through memory.
constexpr int kLastCut = kT22;     // the tiles whose lists may be cut: the wide ones up to this (a cut launch of narrow tiles never paid)
struct DsdPlan {
  int id, full, rest, pieces;
  size_t part_bytes() const {
    return pieces > 1 ? (size_t)rest * pieces * kTileInfo[id].tm * kTileInfo[id].tn * 4096 * sizeof(float) : 0;
  }
};
inline DsdPlan choose_dsd(int Tt, int gt, int d, int nnz_cap, size_t part_bytes, int want) {
  DsdPlan best = {-1, 0, 0, 1};
  float least = 0.f;
  for (int id = 0; id < kTiles; ++id) {
    const TileInfo& t = kTileInfo[id];
    if (!tile_fits(t, Tt, gt, want)) continue;
    const int items = ceil_div(Tt, t.tm) * ceil_div(d, 64 * t.tn);
    if (gt != Tt) {
      if (id == kT14Deep && items > kCUs) continue;
      // a launch of one round lasts as long as its longest list
      const float mean = 6.f / 7.f * (float)nnz_cap * gt / Tt;
      const float busy = tile_cost(t, t.resident, items, mean * (items <= kCUs * t.resident ? 1.35f : 1.1f));
      const float pull = pull_cost(t, (float)items, mean), c = (pull > busy ? pull : busy) + 0.25f * busy;
      if (best.id < 0 || c < least) best = {id, items, 0, 1}, least = c;
      continue;
    }
    const float c = tile_cost(t, t.resident, items, (float)nnz_cap);
    if (best.id < 0 || c < least) best = {id, items, 0, 1}, least = c;
    if (id > kLastCut) continue;
    for (int p = 2; p <= 4 && nnz_cap >= 8 * p; ++p) {
      const int full = items / (kCUs * t.resident) * (kCUs * t.resident);
      const DsdPlan plan = {id, full, items - full, p};
      if (plan.rest == 0 || plan.part_bytes() > part_bytes) continue;
      const float cc = (full > 0 ? tile_cost(t, t.resident, full, (float)nnz_cap) : 0.f) +
                       tile_cost(t, t.resident, plan.rest * p, (float)nnz_cap / p) + 5.f + (float)plan.part_bytes() / 2.5e6f;
      if (cc < least) best = plan, least = cc;
    }
  }
  return best;
}

// One list row: whether the launch runs by 4 x 4 tiles with a rest by narrower ones (SddMix, the 64-column chunks of the output
// in the place of the list's entries).  Second product, us, by the plan's own tile, that with cut lists, mixed: 4544 tokens, d = 4096,
// 48 blocks 122 / 109 / 102; 3968, 5120, 48 124 / 120 / 105; 5312, 3200, 30 82 / 75 / 68; 3904, 5120, 96 231 / 216 / 207; 8192, 5120, 96 429 / 411 / 402;
// 8192, 4608, 8 58 / - / 52; 66 sizes 1.00 - 1.21 times as fast as the first and 0.999 - 1.19 times as the second, which is left
// where more than half a round is.
inline bool dsd_may_mix(const DsdPlan& p, int Tt, int gt, int d, int nnz_cap, int want) {
  if (want != 0 || gt != Tt) return false;
  const SddMix m = sdd_mix(Tt, d / 64);
  if (!sdd_mixes(m) || m.tail < 0) return false;
  const TileInfo &own = kTileInfo[p.id], &b = kTileInfo[kT44], &t = kTileInfo[m.tail];
  const float n = (float)nnz_cap;
  const float plan = p.pieces == 1 ? tile_cost(own, own.resident, p.full, n)
                                   : (p.full > 0 ? tile_cost(own, own.resident, p.full, n) : 0.f) +
                                         tile_cost(own, own.resident, p.rest * p.pieces, n / p.pieces) + 5.f + (float)p.part_bytes() / 2.5e6f;
  return (float)(m.whole / (kCUs / 8)) * (b.round + n * b.step[0]) + t.round + n * t.step[0] < 0.98f * plan;
}

// Whether a launch of `items` 64 x 64 tiles, its weight rows ld elements apart, runs by quarters of them (Quarter): while all
// quarters are resident at once, with rings of eight pairs of steps one per CU, of four two.  Beyond, a quarter's 8 KB per
// 32 x 32 products is more than the L2s deliver (192 tokens, d = 5056, 68 blocks, 204 tiles 24 us, 33 by quarters; the
// second product, 237 tiles, 21 and 32).
constexpr int kQuarterTiles = kCUs / 2, kQuarterTilesAlone = kCUs / 4;
inline bool quarters_pay(int items, long long ld, int want) { return want == 0 && items <= kQuarterTiles && ld < 1 << 25; }

// Lists per group of token tiles: the units are (column chunk, of GN; token group, of GM).  The ways to deal them:
// - kByChunk: XCD w % 8 takes the w % 8th eighth of the units, chunk after chunk, and so fetches the weight rows of an
//   eighth of the columns only.  Where an eighth ends inside a chunk, its parts get long and short lists in
//   proportion: the groups by length (rank 0: the longest list) are dealt evenly over them.  Inside a part the longest go
//   first, except that every other 32 workgroups, one for each CU of the XCD, go the other way round: workgroups on a CU
//   then have long and short lists.
// - kByRank: the chunks of the longest list, then those of the next.  An XCD has an eighth of the columns here too if the
//   number of chunks divides eight or is divided by it, and the workgroups that run together have lists of similar
//   length: they walk along the columns at the same pace, and what one fetches the others find in the L2 (4096 tokens,
//   d = 4096, 10 % of the blocks: 84.5 us, 89.4 by kByChunk).  With other numbers every XCD fetches all columns: 8192 tokens,
//   d = 4160, 8 % 207 us, 137 by kByChunk; 7424 tokens, d = 2624, 25 % 238 and 142; 2048 tokens, d = 3200, 50 % 214 and 133.
//   By 64 columns (tiles of one weight group) the workgroups of a tile that run together are many, and by rank is the better
//   one also with a multiple of four chunks: d = 768, 96 tiles, 20 % 23.6 us, 26.5 by kByChunk; d = 1280, 64 tiles, 10 % 21.3
//   and 23.4.
// - kUnranked: kByChunk by the number of the token group instead of its rank, up to one workgroup per CU: nothing to even
//   out, and the ranking costs a load and three barriers.
// With every block listed all lists are one, the tiles keep in step without more ado, and by rank is faster with an even
// number of twelve chunks or more too: 64 tiles, d = 4608, 100 / 98 / 90 % of the blocks 913 / 858 / 936 us by rank and 980 / 833 / 718
// by chunk; d = 5120, 100 / 98 % 1018 / 943 and 1073 / 918; d = 3072 381 / 368 and 411 / 365.  Only the device knows, and a kernel
// that chose was slower elsewhere (48 tiles, d = 2048, 70 %, with the low-rank step 93 -> 105 us); one list row for all tiles
// is the way to run full lists (680 us for the 1073).
enum DsdOrder { kByChunk, kByRank, kUnranked };
constexpr int kBalTiles = 128;     // most token groups that are ranked; beyond, their numbers take the place of the ranks
// `weights`: bytes of the matrix.  One that fits an L2 (4 MB) may be in all of them: 5184 tokens, d = 704 11.7 us by rank, 12.0.
inline DsdOrder dsd_order(int GM, int GN, int tn, bool lean, long long weights) {
  if (GM * GN <= kCUs) return kUnranked;
  return !lean && (GN % 8 == 0 || 8 % GN == 0 || weights <= 4 << 20 || (tn == 1 && GN % 4 == 0)) ? kByRank : kByChunk;
}
// a / b for a >= 0, b > 0: a reciprocal and a correction (the compiler's division is some forty instructions, and
// they stand at the head of a workgroup's chain of loads)
LX_HD int quick_div(int a, int b) {
  if (a >= 1 << 22) return a / b;
#if defined(__HIP_DEVICE_COMPILE__)
  int q = (int)((float)a * __builtin_amdgcn_rcpf((float)b));
#else
  int q = (int)((float)a * (1.f / (float)b));
#endif
  const int r = a - q * b;
  q += r >= b ? 1 : 0;
  q -= r < 0 ? 1 : 0;
  return q;
}
// The unit of workgroup w; false past the end.
LX_HD bool dsd_unit(int order, int GM, int GN, int w, int& chunk, int& rank) {
  const int total = GM * GN;
  if (order == kByRank) {
    if (w >= total) return false;
    rank = quick_div(w, GN);
    chunk = w - rank * GN;
    // where all are resident, two per CU, the round robin of the dispatcher puts rows s and s + GM/2 on one CU: a long list
    // next to a short one
    const int half = (GM + 1) / 2;
    if (total <= 2 * kCUs && rank >= half) rank = GM - 1 - (rank - half);
    return true;
  }
  const int L = ceil_div(total, 8), x = w % 8, slot = w / 8;
  int unit = x * L + slot;
  if (order == kByChunk && slot / 32 % 2) {
    const int layer = slot / 32 * 32, width = L - layer < 32 ? L - layer : 32;
    unit = x * L + layer + width - 1 - (slot - layer);
  }
  if (slot >= L || unit >= total) return false;
  chunk = quick_div(unit, GM);
  rank = unit - chunk * GM;
  if (order == kUnranked || GM > kBalTiles) return true;
  // part s of the chunk begins at position 0, f, f + L, ...; the j-th of its n units out of the R that it and the
  // later ones share is rank ceil((j + 1) R / n) - 1 of those, the e-th of the later ones' b is rank e R / b
  const int over = chunk * GM - quick_div(chunk * GM, L) * L, f = L - over;
  const int s = rank < f ? 0 : quick_div(rank - f, L) + 1;
  const int begin = s == 0 ? 0 : f + (s - 1) * L, end = f + s * L < GM ? f + s * L : GM, n = end - begin;
  int e = quick_div((rank - begin + 1) * (GM - begin) + n - 1, n) - 1;
  for (int t = s - 1; t >= 0; --t) e = quick_div(e * (t == 0 ? GM : GM - f - (t - 1) * L), GM - f - t * L);
  rank = e;
  return true;
}
// First product, lists per group of token tiles: whether an XCD takes half of every list of a quarter of the tiles (see
// find_work) or the whole lists of an eighth of them.  The half saves weight rows that several tiles of the XCD list, and
// costs it the token rows of twice the tiles; with few entries in a list few are in common.  By halves / whole lists, us: 64
// tiles, d = 2048, lists of 6 entries in the mean 24.5 / 22.4; 96, 2048, 7 34.0 / 31.4; 64, 3200, 10 46.7 / 43.6; 96, 2048, 13
// 51.7 / 55.8; 128, 2048, 13 51.0 / 52.2; 128, 4096, 26 220 / 235.  980 launches of 2 - 10 % of the blocks take 0.982 of the
// time by halves always, at most 1.09; lines at 8, 10 and 13 entries 0.985, 0.983 and 0.981, the last at most 1.09 in twice
// as many launches.
inline bool sdd_halves(int Tt, int gt, int nnz_cap) { return 6.f / 7.f * (float)nnz_cap * gt >= 11.f * (float)Tt; }

// Lists per group of token tiles, 1 x 4 tiles: whether four workgroups per CU with one stage each (Tile14Lean) run the
// launch instead of two with two stages.  A workgroup is slower with the one, so it has to pay otherwise:
// - first product: up to one and a half rounds of two, where the second round is short (four: 0.8 - 1.0 of the time at
//   525 - 720 items: 8192 tokens, d = 768, 40 % of the blocks 41 -> 33 us, 4096 tokens, d = 1024, 55 % 45 -> 37; at 850
//   and more 1.0 - 1.15; asked after sdd_even);
// - second product: where an XCD's eighth is whole column chunks of more than 64 token groups, which two per CU would
//   walk through in more than one round, fetching the chunk's weight rows in each (8192 tokens, d = 2048, 10 / 30 % 50 / 101
//   -> 43 / 94 us; with parts of chunks or 64 groups 0.98 - 1.11 of the time).  A chunk's rows have to fit an L2 for that, and
//   the units must not fill whole rounds of two per CU (128 groups, d = 2048, 40 / 70 / 100 % 121 / 197 / 271 us by two, 121 / 202 / 280
//   by four), or the lists have to be short, a quarter of the groups' number, so that few of the rows are in use at a time:
//   d = 4096 by two / by four, 128 groups of 13 / 26 / 52 entries 118 / 174 / 277 and 105 / 168 / 304 us, 81 groups of 12 / 25 / 50
//   76 / 115 / 170 and 72 / 120 / 212.
inline bool sdd_lean(int id, int Tt, int gt, int nnz_cap) {
  if (id != kT14 || gt == Tt) return false;
  const int items = sdd_items_about(kTileInfo[kT14], Tt, gt, (int)(6.f / 7.f * (float)nnz_cap));
  return items > 2 * kCUs && items <= 3 * kCUs;
}
inline bool dsd_lean(int id, int Tt, int gt, int GM, int GN, int nnz_cap, long long ldw) {
  if (id != kT14 || gt == Tt || GN % 8 != 0 || GM <= 64 || GM * GN <= 2 * kCUs) return false;
  const float mean = 6.f / 7.f * (float)nnz_cap * gt / Tt;
  return 4.f * mean <= (float)GM || (256 * 2 * ldw <= 4 << 20 && GM * GN % (2 * kCUs) != 0);
}

// First product, a list per token tile: whether it runs by pieces of lists of about equal length, 2 to 8 entries each
// (find_piece), on a 1 x 8 tile of one stage, two workgroups to a CU.  By 1 x 4 tiles these launches are bound by what misses the L2s,
// some 6.3 TB/s (8192 tokens, d = 4096, 8 % of the blocks: 154 us, 156 without the matrix instructions, 72 without
// the transfers), and what one workgroup fetches its XCD's others find there only while they keep step along the contraction.
// They do if a round's workgroups have the same to do: 704 items of up to four entries are two or three to a CU, 1.4 rounds;
// 467 pieces of up to six, all resident, fetch 56 KB a step for at most 64 x 384 outputs each, 0.63 GB of misses in all where the items had 0.95, and
// take 134 us for 164 on one box, three fifths of their wavefronts' time in waits (12.5 TB/s from the L2s).  So the pieces are as short as lets them fill whole
// rounds of kEvenRound, and all of a launch transfer the same number of lines per step, the missing entries' from the first one
// (without: 1.02 times the time over 120 launches).  At least three entries (with four: 59 launches of 2 - 2.7 entries per workgroup of a
// round 0.95 of the time of the items before, now 0.88), two where those fit a round (of 15 launches 1.03 with four, now 0.90).
// Against the items before, which took their kernel by the model (1 x 4 tiles
// of one, two or four stages), for what the lines below take of calls drawn from 2 - 128 tiles, d = 512 - 5120, 3 - 100 % of the blocks,
// plain and with the low-rank step, up and gate product, on the same buffers (profiles/ffn_pieces_sweep.txt): with a capacity a tenth over
// the list 0.83 of the time where all columns are as likely (1116 launches, 10 of them above 1.02, 1.06 at most) and 0.89 where they
// differ as the support of trained layers does (548, 23 above 1.02, up to 1.13); 1.5 and 2 times the list 0.88 (756, 66, 1.09), beyond 0.84 (276, 4, 1.14).
// The lines:
// - more items than one round of 1 x 4 tiles holds (d = 2048, 3 entries per workgroup of a round 1.0 - 1.1, 16 tiles, d = 5120 0.96 - 1.05;
//   4 entries and more 0.77 - 0.95), which is also where the pieces have five entries;
// - where d is large and tiles are many (48 on, d >= 3200) also what pieces of three hold in one round (0.81 - 0.97 from 2.5
//   entries on).  Not what takes pieces of four: 1.02 and up to 1.14 where most tiles list the same columns, 0.96 elsewhere;
// - there from 90 tiles on not the longest pieces in one round: the waiting for nine lines a step outweighs what is saved where tiles have many
//   columns in common anyway (1.02 of the time, up to 1.19; with independent columns 0.85 - 0.97).  The two lines leave out 256 launches with
//   a tenth of room, 1.00 of the time where columns differ, 80 of 186 above 1.02, and 0.90 where they do not;
// - below d = 3200 not where the longest pieces just need a second round, which short ones then fill (7.5 entries:
//   0.95 - 1.15);
// - lists, or a loose capacity, of more than half of the blocks only from 97 tiles and d = 3200 on: with so many in common the 1 x 4
//   tiles keep step as they are (16 - 32 tiles, 60 - 80 %, 1.0 - 1.25), and a short list in a long capacity pays for the workgroups
//   that find nothing (7000 tokens, 4 %, d = 1792 30 -> 35 us).
constexpr int kEvenLeast = 3, kEvenMost = 8, kEvenRound = 2 * kCUs;
constexpr int kEvenShort = 2;      // of short lists
constexpr int kEvenTiles = 128;    // most token tiles: two per lane of the scan
// Workgroups that hold the pieces of any list of at most nnz_cap entries.
LX_HD int sdd_even_grid(int Tt, int nnz_cap) { return ceil_div(ceil_div(nnz_cap, kEvenMost) + Tt, kEvenRound) * kEvenRound; }
// The most entries of a piece: the fewest for which there are no more rounds than with the longest pieces.  pieces(p): pieces of
// all lists by at most p entries; short_pieces(): by kEvenShort, asked for only if the shortest others fit.
template <class Pieces, class Short>
LX_HD int even_per(Pieces pieces, Short short_pieces) {
  const int room = ceil_div(pieces(kEvenMost), kEvenRound) * kEvenRound;
  int per = kEvenMost;
#pragma unroll
  for (int p = kEvenMost - 1; p >= kEvenLeast; --p)
    if (pieces(p) <= room) per = p;
  // (n / 2 pieces or more are 3/2 of n / 3 less one per list, or more)
  if (per == kEvenLeast && 3 * pieces(kEvenLeast) <= 2 * (room + kEvenTiles) && short_pieces() <= room) per = kEvenShort;
  return per;
}
// The piece of workgroup w out of `total`, -1 past the end: XCD w % 8 takes the w % 8th eighth.
LX_HD int even_place(int w, int total) {
  const int L = ceil_div(total, 8), slot = w / 8, work = w % 8 * L + slot;
  return slot < L && work < total ? work : -1;
}
LX_HD int quick_div(int a, int b);
struct EvenPiece {
  int odd, first, count;      // 1: of the second of two tiles; entries of that tile's list
};
// The lists of one or two tiles, n0 and n1 entries, and the pieces that they fall into.  The pieces are numbered first halves
// before second ones; a first half is the larger one.
struct EvenLane {
  int n0, n1, k0, k1;
  static LX_HD int of(int n, int per) { return (int)((unsigned)(n + per - 1) / (unsigned)per); }
  LX_HD int pieces(int per) const { return of(n0, per) + of(n1, per); }
  LX_HD void cut(int per) { k0 = quick_div(n0 + per - 1, per), k1 = quick_div(n1 + per - 1, per); }
  LX_HD int firsts() const { return (k0 + 1) / 2 + (k1 + 1) / 2; }
  // number `work` of the lane's first halves, or of its second ones
  LX_HD EvenPiece piece(bool second, int work) const {
    const int held = second ? k0 / 2 : (k0 + 1) / 2;
    const bool b = work >= held;
    const int k = b ? k1 : k0, n = b ? n1 : n0, chunk = (b ? work - held : work) + (second ? (k + 1) / 2 : 0);
    const int first = quick_div(chunk * n, k);
    return {b ? 1 : 0, first, quick_div((chunk + 1) * n, k) - first};
  }
};
inline bool sdd_even(int Tt, int gt, int d, int nnz_cap, int blocks, int want) {
  if (want != 0 || gt != 1 || Tt < 2 || Tt > kEvenTiles || nnz_cap >= 1 << 16) return false;
  const float n = 6.f / 7.f * (float)nnz_cap;      // (a list that fills a capacity of a tenth over the mean has 1.06 n)
  auto pieces = [&](int per) { return n / (float)per + (float)Tt * (float)(per - 1) / (float)(2 * per); };
  if (n > 0.5f * (float)blocks && (Tt <= 96 || d < 3200)) return false;
  if (d >= 3200 && Tt >= 48) {
    if (n < 2.5f * kEvenRound || (pieces(3) > kEvenRound && pieces(4) <= 0.97f * kEvenRound)) return false;
    return Tt < 90 || pieces(kEvenMost - 1) <= 0.95f * kEvenRound || pieces(kEvenMost) > 0.99f * kEvenRound;
  }
  if (d < 3200 && n / kEvenMost + 0.44f * (float)Tt > 0.9f * kEvenRound && n < 4.3f * 2 * kEvenRound) return false;
  return sdd_items_about(kTileInfo[kT14], Tt, gt, (int)n) > kEvenRound;
}

// ---- which kernel a launch runs by -----------------------------------------------------------
// kByPieces: pieces of lists (find_piece); kBySet: a kernel that holds several tiles and takes the one that suits the list (SddSet,
// with `mix` its SddMix), kByMix: 4 x 4 tiles and narrower ones for a rest, kByLean: the 1 x 4 tile of one stage, kByTile: the plan's
// own tile.
enum Route { kNothing, kByQuarters, kBySet, kByMix, kByLean, kByTile, kByPieces };
struct SddRoute {
  Route by;
  SddPlan plan;
  bool mix, halves;
  int grid, items;         // workgroups; 64 x 64 tiles of the capacity (quarters)
};
inline SddRoute sdd_route(int Tt, int gt, int d, int nnz_cap, int blocks, int want) {
  SddRoute r = {kNothing, plan_sdd(Tt, gt, d, nnz_cap, blocks, want), false, sdd_halves(Tt, gt, nnz_cap), 0, 0};
  r.grid = r.plan.grid;
  if (r.grid == 0) return r;
  r.items = (long long)nnz_cap * gt < 1 << 20 ? nnz_cap * gt : 1 << 20;
  if (quarters_pay(r.items, d, want)) {
    r.by = kByQuarters;
    r.grid = 4 * sdd_grid(kTileInfo[kT11], Tt, gt, nnz_cap);
  } else if (sdd_even(Tt, gt, d, nnz_cap, blocks, want)) {
    r.by = kByPieces;
    r.grid = sdd_even_grid(Tt, nnz_cap);
  } else if (r.plan.allowed) {
    r.by = kBySet;
    r.mix = sdd_may_mix(r.plan, Tt, gt, d, nnz_cap, want);
    if (const int mixed = r.mix ? sdd_mix_grid(Tt, nnz_cap) : 0; mixed > r.grid) r.grid = mixed;
  } else {
    r.by = sdd_lean(r.plan.id, Tt, gt, nnz_cap) ? kByLean : kByTile;
  }
  return r;
}
struct DsdRoute {
  Route by;
  DsdPlan plan;
  int grid, items;
  int GM, GN;              // token groups and column chunks of the tile
  DsdOrder order;          // lists per group of token tiles
};
// part_bytes: room for partial sums.
inline DsdRoute dsd_route(int Tt, int gt, int d, long long ldw, int nnz_cap, size_t part_bytes, int want) {
  DsdRoute r = {kByQuarters, {}, 0, Tt < 4096 ? Tt * (d / 64) : 1 << 20, Tt, d / 64, kUnranked};
  if (quarters_pay(r.items, ldw, want)) {
    r.grid = 32 * ceil_div(r.items, 8);
    return r;
  }
  r.plan = choose_dsd(Tt, gt, d, nnz_cap, part_bytes, want);
  if (dsd_may_mix(r.plan, Tt, gt, d, nnz_cap, want)) {
    r.by = kByMix;
    r.grid = sdd_mix_grid(Tt, d / 64);
    return r;
  }
  const TileInfo& t = kTileInfo[r.plan.id];
  r.GM = Tt / t.tm;
  r.GN = ceil_div(d, 64 * t.tn);
  const bool lean = dsd_lean(r.plan.id, Tt, gt, r.GM, r.GN, nnz_cap, ldw);
  r.by = lean ? kByLean : kByTile;
  r.order = dsd_order(r.GM, r.GN, t.tn, lean, ldw * d * 2);
  r.grid = gt == Tt ? 8 * ceil_div(r.plan.full, 8) + 8 * ceil_div(r.plan.rest * r.plan.pieces, 8) : 8 * ceil_div(r.GM * r.GN, 8);
  return r;
}

// Gradients of the LoRA matrices: whether a workgroup per quadrant of a product adds all its token tiles (lora_tn_quad), or
// ranges of tiles are added apart, as parts in memory, and a second launch adds those.  By the shape only: the sums' order is
// not to change with a list's capacity.  Quadrants read both operands twice, so there must not be much to add, and a
// workgroup's start weighs as much as some ten tiles.  G, both gradients and the sums, us, by parts and by quadrants (F = 4 d, 5 / 20 / 70 % of
// the blocks): 8 tiles, d = 1024 23.8 / 23.4 / 26.5 and 13.7 / 16.0 / 20.1; 32, 768 25.9 / 26.8 / 31.3 and 15.2 / 17.7 / 22.2; 64, 2048 25.6 / 31.1 / 44.6
// and 23.0 / 28.7 / 48.9; 16, 5120 27.9 / 38.0 / 67.2 and 27.7 / 39.1 / 67.8; 24, 5120 30.3 / 39.7 / 76.4 and 32.2 / 43.2 / 83.7; 48, 3200 27.5 / 34.8 /
// 55.6 and 24.4 / 33.4 / 62.5; past 64 tiles 128, 768 30.7 and 32.0.  A single tile has one part, so there is no second launch to be
// saved: d = 3200 13.8 and 15.8, d = 5120 15.7 and 19.8.
inline bool lora_grads_by_quads(int Tt, int d, int F) {
  return Tt >= 2 && Tt <= 64 && (Tt + 10ll) * (d / 64 + F / 64) <= 12500;
}

}  // namespace lx
