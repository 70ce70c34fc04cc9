// 16-bit sparse FFN kernels for gfx950 (Sec. VI-B: neuron-centric tiled matrix
// products that take the list of active neuron blocks and load / compute only
// those).  fp32 accumulation on the 16x16x32 MFMA for 16-bit operands.  The kernels are
// templates over the element type DT (bfloat16 or IEEE half, same layouts and data movement).
//
// Both products of a pass are "NT" contractions whose operands are read along
// their contiguous dimension in 128-byte segments (one 64-element K-chunk
// of one row), which is what the weight layouts of Sec. VI-B are for:
//   sdd  out block (i, j) = A_i [64 x K] . W[j-block rows, :]^T, K = d
//        a workgroup owns TM token tiles that share a list row and up to TN consecutive
//        entries of that row.
//   dsd  out tile (i, 64*TN columns) = sum over listed j of Act_ij [64 x 64] .
//        W[rows n0.., j-block columns]^T: the K loop walks the active list, one
//        64-wide K-step per active block; inactive blocks are never touched.
// The products themselves, and how their operands travel, are in ffn_tile.h.  Every output element
// sees the same products in the same order whatever the tile, so results do not depend on it.
//
// The LoRA branch on the up-projection (Sec. II-C / II-D) is one more step of either product; the
// calls that add it are at the end of this file, its small products in lora_bf16.hip.
#include "ffn_plan.h"
#include "ffn_tile.h"

namespace lx {

// The tiles of ffn_plan.h.  TM TN WM WN NST PH
using Tile44 = Tile<4, 4, 4, 2, 2, 2>;
using Tile24 = Tile<2, 4, 2, 4, 3, 2>;
using Tile22 = Tile<2, 2, 2, 2, 2, 2>;
using Tile22Deep = Tile<2, 2, 2, 4, 4, 1>;
using Tile14 = Tile<1, 4, 1, 4, 2, 2>;
using Tile14Lean = Tile<1, 4, 1, 4, 1, 4, 4, 32>;  // four workgroups on a CU: see sdd_lean, dsd_lean
using Tile18Lean = Tile<1, 8, 1, 8, 1, 4, 4, 32>;  // two workgroups on a CU: see sdd_even
using Tile14Deep = Tile<1, 4, 2, 4, 4, 2>;
using Tile12 = Tile<1, 2, 1, 4, 3, 2>;
using Tile11 = Tile<1, 1, 2, 2, 4, 1, 2, 32>;
using Tile11Many = Tile<1, 1, 2, 2, 3, 1, 3>;
template <class Tl>
constexpr int kRingElems = Tl::NST * Tl::kElems;

// Work items of the sdd kernel are (token tile, group of `per` consecutive list entries); `rows` counts token
// tiles, and gt consecutive tiles share one row of the list (gt = 1: a list row per tile).  The launch grid is
// the host-known upper bound on their number and every wavefront finds its item from row_ptr with 64-wide
// scans, so the active workgroups are the FIRST ones of the grid and spread evenly over shader engines and
// CUs (a 2-D grid with early exits piles them onto a few CUs).
// The items are numbered by the first halves of all lists, tile after tile, and then the second halves; without `halves` (see
// sdd_halves) by the whole lists, which are then the first halves.
// Workgroup w runs on XCD w % 8; it takes item of the range (w % 8) * L .. + L - 1 with L = ceil(total / 8), so
// each XCD owns a quarter of the token tiles and, the lists being sorted, about half of the neuron axis.  Its L2
// then fetches the rows of a quarter of the tokens and the listed ones of half of the weights, fewer bytes than
// an eighth of the tokens and all listed weights (by the masks of 128 tiles, d = 4096, 8 % of the blocks: 470 MB over
// the XCDs against 593 if all its workgroups kept step, d = 2048, 11 %: 156 and 184).  Returns false past the end.
__device__ __forceinline__ bool find_work(const int* __restrict__ row_ptr, int rows, int gt, int w,
                                          int per, int nnz_cap, bool halves, int& row, int& chunk) {
  const int lane = threadIdx.x % kWave;
  // groups of entries of a token tile.  Entries of its list row count that lie within the capacity of the list buffers,
  // so that the number of items never exceeds the bound the grid was sized from
  auto groups = [&](int r) {
    if (r >= rows) return 0;
    const int lr = r / gt;
    return (min(row_ptr[lr + 1], nnz_cap) - min(row_ptr[lr], nnz_cap) + per - 1) / per;
  };
  // those of its first half
  auto first_half = [&](int c) { return halves ? (c + 1) / 2 : c; };
  // inclusive sums over the lanes
  auto scan = [&](int v) {
#pragma unroll
    for (int dlt = 1; dlt < kWave; dlt <<= 1) {
      const int up = __shfl_up(v, dlt);
      if (lane >= dlt) v += up;
    }
    return v;
  };
  // Item w of the launch's: which one of all; -1 past the end.  Inside an XCD's range consecutive workgroups are a quarter
  // of the range apart: the workgroups that run at the same time come from different token tiles and, the lists
  // being sorted, from the same region of the neuron axis, whose weight blocks are then fetched into its L2 once; four
  // of them at a time, as tiles that walk along the same blocks in step wait for the same lines (an eighth / a quarter / half of
  // the range apart / one after the other, us: 128 tiles, d = 2048, lists that have a hot set in common 57.0 / 51.0 / 49.9 / 50.3,
  // skewed ones 51.8 / 52.6 / 51.7 / 54.6; 128, 4096 173 / 163 / 164 / 161; 16, 5120, 80 % 321 / 263 / 308; 15 sizes 1.03 and 1.01 times as
  // fast by a quarter and by half).
  auto item_of = [&](int total) {
    const int L = (total + 7) / 8, q = (L + 3) / 4, slot = w / 8, pos = (slot % 4) * q + slot / 4;
    const int work = (w % 8) * L + pos;
    return slot >= 4 * q || pos >= L || work >= total ? -1 : work;
  };
  // The row among this wavefront's 64 whose items, `mine` up to the inclusive sum `incl`, hold item `work`.
  auto place = [&](int work, int incl, int mine, int h, bool second) {
    const int first = __ffsll((long long)__ballot(incl > work)) - 1;
    chunk = work - __shfl(incl - mine, first) + (second ? __shfl(h, first) : 0);
    return first;
  };
  // One scan of both halves, 16 bits each; beyond 64 rows two of them per lane (81 tiles, d = 704: first
  // product 11.9 us by the loops below, 10.9 so).
  if (rows <= 2 * kWave && (long long)nnz_cap * gt < 1 << 16) {
    const bool two = rows > kWave;
    const int c0 = groups(two ? 2 * lane : lane), c1 = two ? groups(2 * lane + 1) : 0, h0 = first_half(c0), h1 = first_half(c1);
    const int c = c0 + c1, h = h0 + h1, both = scan(h | (c - h) << 16), all = __shfl(both, kWave - 1), firsts = all & 0xFFFF;
    int work = item_of(firsts + (int)((unsigned)all >> 16));
    if (work < 0) return false;
    const bool second = work >= firsts;
    if (second) work -= firsts;
    const int incl = second ? (int)((unsigned)both >> 16) : both & 0xFFFF, mine = second ? c - h : h;
    const int l = __ffsll((long long)__ballot(incl > work)) - 1, first = __shfl(h0, l);
    work -= __shfl(incl - mine, l);
    row = two ? 2 * l : l;
    const int held = second ? __shfl(c0, l) - first : first;        // by the lane's first row
    if (work >= held) {
      ++row;
      chunk = work - held + (second ? __shfl(h1, l) : 0);
    } else {
      chunk = work + (second ? first : 0);
    }
    return true;
  }
  int total = 0, firsts = 0;           // of all lists; of their first halves
  for (int base = 0; base < rows; base += kWave) {
    int c = groups(base + lane);
    firsts += __popcll(__ballot(c & 1));
#pragma unroll
    for (int dlt = 32; dlt > 0; dlt >>= 1) c += __shfl_xor(c, dlt);
    total += c;
  }
  firsts = halves ? (total + firsts) / 2 : total;       // (a first half is the longer one)
  int work = item_of(total);
  if (work < 0) return false;
  const bool second = work >= firsts;
  if (second) work -= firsts;
  for (int base = 0; base < rows; base += kWave) {
    const int c = groups(base + lane), h = first_half(c), mine = second ? c - h : h, incl = scan(mine);
    const int seg = __shfl(incl, kWave - 1);
    if (work < seg) {
      row = base + place(work, incl, mine, h, second);
      return true;
    }
    work -= seg;
  }
  return false;
}

// Items of the sdd kernel as pieces of lists of about equal length (sdd_even, whose arithmetic these scans serve): with `per`,
// their most entries, a tile's list of n entries falls into k = ceil(n / per) pieces of n / k entries, rounded up or down.
// Numbered by halves of the lists as in find_work; an XCD takes its eighth in order.  A list per token tile, up to kEvenTiles
// of them and 2^16 entries.  Returns false past the end.
__device__ __forceinline__ bool find_piece(const int* __restrict__ row_ptr, int Tt, int w, int nnz_cap, int& tile, int& first,
                                           int& count, int& per) {
  if (w >= sdd_even_grid(Tt, min(row_ptr[Tt], nnz_cap))) return false;      // before the scans
  const int lane = threadIdx.x % kWave;
  auto entries = [&](int i) { return i < Tt ? min(row_ptr[i + 1], nnz_cap) - min(row_ptr[i], nnz_cap) : 0; };
  const bool two = Tt > kWave;
  EvenLane own = {two ? entries(2 * lane) : entries(lane), two ? entries(2 * lane + 1) : 0};
  constexpr int kPers = kEvenMost - kEvenLeast + 1;
  int sum[(kPers + 1) / 2];     // pieces of all tiles by at most kEvenLeast + i entries, 16 bits each
#pragma unroll
  for (int i = 0; i < kPers; ++i) {
    const int k = own.pieces(kEvenLeast + i);
    sum[i / 2] = i % 2 ? sum[i / 2] | k << 16 : k;
  }
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1)
#pragma unroll
    for (int i = 0; i < (kPers + 1) / 2; ++i) sum[i] += __shfl_xor(sum[i], d);
  per = even_per([&](int p) { return (int)((unsigned)sum[(p - kEvenLeast) / 2] >> ((p - kEvenLeast) % 2 ? 16 : 0) & 0xFFFFu); },
                 [&] {
                   int k = own.pieces(kEvenShort);
                   for (int d = 1; d < kWave; d <<= 1) k += __shfl_xor(k, d);
                   return k;
                 });
  own.cut(per);
  int both = own.firsts() | (own.k0 + own.k1 - own.firsts()) << 16;
  const int mine = both;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int up = __shfl_up(both, d);
    if (lane >= d) both += up;
  }
  const int all = __shfl(both, kWave - 1), firsts = all & 0xFFFF, total = firsts + (int)((unsigned)all >> 16);
  int work = even_place(w, total);
  if (work < 0) return false;
  const bool second = work >= firsts;
  if (second) work -= firsts;
  const int incl = second ? (int)((unsigned)both >> 16) : both & 0xFFFF;
  const int l = __ffsll((long long)__ballot(incl > work)) - 1;
  work -= __shfl(incl - (second ? (int)((unsigned)mine >> 16) : mine & 0xFFFF), l);
  const EvenLane at = {__shfl(own.n0, l), __shfl(own.n1, l), __shfl(own.k0, l), __shfl(own.k1, l)};
  const EvenPiece p = at.piece(second, work);
  tile = __builtin_amdgcn_readfirstlane((two ? 2 * l : l) + p.odd);
  first = __builtin_amdgcn_readfirstlane(p.first);
  count = __builtin_amdgcn_readfirstlane(p.count);
  return true;
}

template <class Tl>
__device__ __forceinline__ void zero_acc(typename Tl::Acc (&acc)[Tl::NI][Tl::TI]) {
#pragma unroll
  for (int x = 0; x < Tl::NI; ++x)
#pragma unroll
    for (int y = 0; y < Tl::TI; ++y)
#pragma unroll
      for (int v = 0; v < Tl::MF * Tl::MF / kWave; ++v) acc[x][y][v] = 0.f;
}

// Epilogue.  The accumulators hold four consecutive columns of a lane's token; stored as they are, the 8-byte
// pieces of 32 rows per instruction took up to two fifths of a launch (4096 tokens, d = 2048, one list of 14
// blocks, second product: 24 us, 14 without the stores).  They go through LDS instead, as [64 x 64] blocks
// (tile t, group of 64 columns e at index t * TN + e) whose 128-byte rows have their 16-byte slots XOR-swizzled
// with the row, and leave in 16-byte pieces, eight lanes to a full row of a block.
__device__ __forceinline__ uint32_t out_slot(int block, int row, int slot) {
  return (uint32_t)(block * 8192 + row * 128 + ((slot ^ (row & 7)) << 4));
}
// Four consecutive columns of a token row -> LDS at `at`, rounded; bias: theirs (or null), then ReLU.
template <int DT>
__device__ __forceinline__ void cols_to_lds(f32x4 v, uint32_t at, const uint16_t* __restrict__ bias, bool relu) {
  if (bias) {
    const uint2 bb = *reinterpret_cast<const uint2*>(bias);
    v[0] += to_f32<DT>(bb.x & 0xFFFFu); v[1] += to_f32<DT>(bb.x >> 16);
    v[2] += to_f32<DT>(bb.y & 0xFFFFu); v[3] += to_f32<DT>(bb.y >> 16);
  }
  if (relu) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
  }
  lds_write8(at, make_uint2(pack2<DT>(v[0], v[1]), pack2<DT>(v[2], v[3])));
}
// One accumulator (token rows th .., columns nh .. of the block) -> LDS; bias: its columns' (or null).
template <int DT>
__device__ __forceinline__ void acc_to_lds(const f32x16& acc, uint32_t lds, int block, int th, int nh,
                                           const uint16_t* __restrict__ bias, bool relu) {
  const int lane = threadIdx.x % kWave, tl = th + lane % 32, h2 = lane / 32;
#pragma unroll
  for (int g = 0; g < 4; ++g)
    cols_to_lds<DT>(f32x4{acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]},
                    lds + out_slot(block, tl, nh / 8 + g) + 8 * h2, bias ? bias + 8 * g + 4 * h2 : nullptr, relu);
}
template <int DT>
__device__ __forceinline__ void acc_to_lds(const f32x4& acc, uint32_t lds, int block, int th, int nh,
                                           const uint16_t* __restrict__ bias, bool relu) {
  const int lane = threadIdx.x % kWave, tl = th + lane % 16, q = lane / 16;
  cols_to_lds<DT>(acc, lds + out_slot(block, tl, nh / 8 + q / 2) + 8 * (q % 2), bias ? bias + 4 * q : nullptr, relu);
}
// The elements of v whose gate is positive, 0 for the others (two packed 16-bit elements each).
template <int DT>
__device__ __forceinline__ uint32_t gate2(uint32_t v, uint32_t g) {
  return (to_f32<DT>(g & 0xFFFFu) > 0.f ? v & 0xFFFFu : 0u) | (to_f32<DT>(g >> 16) > 0.f ? v & 0xFFFF0000u : 0u);
}
// The blocks in LDS -> memory: block_at(t, e) is the first element of block (t, e), its rows ld elements apart,
// or negative: not stored.  gate: indexed like out (or null).  THROUGH: the lines are written through the L2 at
// once instead of when the kernel ends, which is when all workgroups of a round store: second product, 4096 tokens,
// d = 2048, one list of 14 blocks 21.0 -> 19.2 us, 8192 tokens with a list per tile 51 -> 48; no use for the first
// product, whose outputs the second reads again.
template <class Tl, int DT, bool THROUGH, class BlockAt>
__device__ __forceinline__ void lds_to_out(uint32_t lds, uint16_t* __restrict__ out, long long ld,
                                           const uint16_t* __restrict__ gate, BlockAt block_at) {
  constexpr int kPieces = Tl::TM * Tl::TN * 512, kT = Tl::kTileThreads, kPer = kPieces / kT;
  constexpr int kGroup = kPer < 8 ? kPer : 8;      // gate loads in flight
#pragma unroll
  for (int u0 = 0; u0 < kPer; u0 += kGroup) {
    uint4 g[kGroup];
    long long o[kGroup];
#pragma unroll
    for (int u = 0; u < kGroup; ++u) {
      const int x = (u0 + u) * kT + (int)threadIdx.x, block = x / 512, row = x % 512 / 8, slot = x % 8;
      const long long first = block_at(block / Tl::TN, block % Tl::TN);
      o[u] = first < 0 ? -1 : first + row * ld + slot * 8;
      if (gate && o[u] >= 0) g[u] = *reinterpret_cast<const uint4*>(gate + o[u]);
    }
#pragma unroll
    for (int u = 0; u < kGroup; ++u) {
      const int x = (u0 + u) * kT + (int)threadIdx.x;
      uint4 v = lds_read16(lds + out_slot(x / 512, x % 512 / 8, x % 8));
      if (o[u] < 0) continue;
      if (gate) v = make_uint4(gate2<DT>(v.x, g[u].x), gate2<DT>(v.y, g[u].y), gate2<DT>(v.z, g[u].z), gate2<DT>(v.w, g[u].w));
      if (THROUGH)  // (s_nop: the store still reads its registers for two wait states, unknown to the compiler)
        asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(out + o[u]), "v"(__builtin_bit_cast(u32x4, v)) : "memory");
      else
        *reinterpret_cast<uint4*>(out + o[u]) = v;
    }
  }
}

// Offsets of the two products' transfer instructions: instruction u of wavefront w brings the stage
// rows 8g .. 8g+7 with g = w + kWaves*u (token rows first); lane l brings the 16-byte slot l % 8 of row
// l / 8, i.e. the segment of that row's 128 bytes that tile_swz puts there.
template <class Tl>
__device__ __forceinline__ uint32_t lane_voff(long long ld, int g) {
  const int lane = threadIdx.x % kWave, lr = lane / 8;
  return (uint32_t)(lr * ld * 2 + (((lane % 8) ^ tile_swz<Tl>(8 * g + lr)) << 4));
}

struct SddArgs {
  const uint16_t *A, *W, *bias;
  const int *row_ptr, *col_idx;
  int Tt, gt, K, nnz_cap;      // gt token tiles share a list row
  int rows, blocks;            // list rows, and blocks that the list could hold
  int own, grid;               // of SddPlan
  unsigned allowed;
  bool mix, halves;            // sdd_may_mix, sdd_halves
  uint16_t* out;
  const uint16_t* gate;        // null: ReLU
  const uint16_t *A2, *W2;     // LORA
};

// Sources of the sdd kernel's transfers; step K/64, if there is one, is the low-rank step.  It is the last
// one, so its sources replace the others; a choice at each transfer instruction instead was a branch between
// the matrix instructions and cost a 64 x 64 tile 90 ns per step (704 tokens, 4928 -> 19712: 26.6 -> 19.9 us).
// EVEN: an item's transfers and products are those of the entries that it has; else of as many as the tile holds.
template <class Tl, bool LORA, bool EVEN>
struct SddSrc {
  const uint16_t* base[Tl::kIss];
  const uint16_t* base2[LORA ? Tl::kIss : 1];
  uint32_t voff[2], voff2[2];
  long long off;
  int ksteps, entries, lines;     // EVEN, of the item: entries; entries whose transfers are issued
  __device__ __forceinline__ int live() const { return EVEN ? Tl::kIssA + lines * 8 / Tl::kWaves : Tl::kIss; }
  __device__ __forceinline__ bool busy(int wn) const { return !EVEN || wn * Tl::TN < entries * Tl::WN; }
  __device__ __forceinline__ void begin(int s) {
    off = (long long)s * kBK;
    if (LORA && s == ksteps) {
      off = 0;
      voff[0] = voff2[0];
      voff[1] = voff2[1];
#pragma unroll
      for (int u = 0; u < Tl::kIss; ++u) base[u] = base2[LORA ? u : 0];
    }
  }
  __device__ __forceinline__ void dma(int u, uint32_t lds) const {
    dma16_s(base[u] + off, voff[Tl::kWaves == 4 ? u & 1 : 0], lds + u * (Tl::kWaves * 1024));
  }
};

// out block (tile, entry) = relu(A_tile W_entry^T + bias) or gated by `gate`; compact activation blocks
// [entry][tile within the row's group of gt tiles].
// LORA: one more 64-deep step after the K loop with the operands A2 [T,64] (rows of the token
// tile) and W2 [F,64] (rows of the listed blocks): acc += A2_i W2_j^T, the low-rank branch
// z = W x + B (A x) of Sec. II-C with A2 = X A^T computed beforehand and W2 = B, both padded to
// rank 64.
// placed: the item's number along the tokens and along the list where the caller has chosen it (one list row), -1: this
// workgroup's of a launch of such tiles.  EVEN: the items are those of find_piece.
template <class Tl, int DT, bool LORA, bool EVEN = false>
__device__ __forceinline__ void sdd_tile(const SddArgs& a, uint16_t* ring, GridItem placed = {-1, -1}) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (wave >= Tl::kWaves) return;      // (barriers wait for the wavefronts that are left)
  int m, first, nb, rs, lines;
  if constexpr (EVEN) {
    if (!find_piece(a.row_ptr, a.Tt, blockIdx.x, a.nnz_cap, m, first, nb, lines)) return;
    rs = a.row_ptr[m];
  } else {
    int chunk, n_i;
    if (a.gt == a.Tt) {
      rs = min(a.row_ptr[0], a.nnz_cap);
      n_i = min(a.row_ptr[1], a.nnz_cap) - rs;
      if (placed.m < 0) {
        const int GM = (a.Tt + Tl::TM - 1) / Tl::TM, GN = (n_i + Tl::TN - 1) / Tl::TN;
        const int total = GM * GN, L = (total + 7) / 8, slot = blockIdx.x / 8, idx = (blockIdx.x % 8) * L + slot;
        if (slot >= L || idx >= total) return;
        placed = grid_item(idx, GM, GN, Tl::TM == 4 ? 4 : 8);
      }
      m = placed.m;
      chunk = placed.n;
    } else {
      if (!find_work(a.row_ptr, a.Tt / Tl::TM, a.gt / Tl::TM, blockIdx.x, Tl::TN, a.nnz_cap, a.halves, m, chunk)) return;
      m = __builtin_amdgcn_readfirstlane(m);
      chunk = __builtin_amdgcn_readfirstlane(chunk);
      const int lr = m * Tl::TM / a.gt;
      rs = a.row_ptr[lr];
      n_i = min(a.row_ptr[lr + 1], a.nnz_cap) - rs;   // entries beyond the capacity of the list buffers are ignored
    }
    first = chunk * Tl::TN;
    nb = lines = min(Tl::TN, n_i - first);
  }
  const int i0 = m * Tl::TM, p0 = rs + first;
  if (nb <= 0) return;

  SddSrc<Tl, LORA, EVEN> src;
  src.ksteps = a.K / kBK;
  src.entries = nb;
  src.lines = lines;
  src.voff[0] = lane_voff<Tl>(a.K, wave);
  src.voff[1] = lane_voff<Tl>(a.K, wave + 4);
  if (LORA) {
    src.voff2[0] = lane_voff<Tl>(64, wave);
    src.voff2[1] = lane_voff<Tl>(64, wave + 4);
  }
#pragma unroll
  for (int u = 0; u < Tl::kIss; ++u) {
    const int g = wave + Tl::kWaves * u;
    if (u < Tl::kIssA) {     // (token tiles past the end: the last one again, not stored)
      const long long row = (long long)min(i0 + g / 8, a.Tt - 1) * 64 + 8 * (g % 8);
      src.base[u] = a.A + row * a.K;
      if (LORA) src.base2[LORA ? u : 0] = a.A2 + row * 64;
    } else {                 // blocks past the end of the list are filled from the first block (not stored)
      const int e = (g - 8 * Tl::TM) / 8;
      const long long row = (long long)a.col_idx[p0 + (e < nb ? e : 0)] * 64 + 8 * (g % 8);
      src.base[u] = a.W + row * a.K;
      if (LORA) src.base2[LORA ? u : 0] = a.W2 + row * 64;
    }
  }
  const int wm = wave / Tl::WN, wn = wave % Tl::WN;
  typename Tl::Acc acc[Tl::NI][Tl::TI];
  zero_acc<Tl>(acc);
  run_tile<Tl, DT>(src.ksteps + (LORA ? 1 : 0), lds_addr(ring), wm, wn, src, acc);
  lds_barrier();       // nobody reads the ring any more
#pragma unroll
  for (int ni = 0; ni < Tl::NI; ++ni) {
    const int c = wn * Tl::NI + ni, e = c / Tl::kPer, nh = Tl::MF * (c % Tl::kPer);
    const uint16_t* bias = a.bias && e < nb ? a.bias + a.col_idx[p0 + e] * 64 + nh : nullptr;
#pragma unroll
    for (int ti = 0; ti < Tl::TI; ++ti)
      acc_to_lds<DT>(acc[ni][ti], lds_addr(ring), (wm * Tl::TI + ti) / Tl::kPer * Tl::TN + e,
                     Tl::MF * ((wm * Tl::TI + ti) % Tl::kPer), nh, bias, !a.gate);
  }
  lds_barrier();
  lds_to_out<Tl, DT, false>(lds_addr(ring), a.out, 64, a.gate, [&](int t, int e) {
    const int i = i0 + t;
    return i < a.Tt && e < nb ? (((long long)rs + first + e) * a.gt + i % a.gt) * 4096 : -1ll;
  });
}

template <class Tl, int DT, bool LORA>
__global__ __launch_bounds__(Tl::kTileThreads, Tl::kMinWaves) void ffn_sdd(SddArgs a) {
  __shared__ __attribute__((aligned(1024))) uint16_t ring[kRingElems<Tl>];
  sdd_tile<Tl, DT, LORA>(a, ring);
}
template <int DT, bool LORA>
__global__ __launch_bounds__(Tile18Lean::kTileThreads, Tile18Lean::kMinWaves) void ffn_sdd_even(SddArgs a) {
  __shared__ __attribute__((aligned(1024))) uint16_t ring[kRingElems<Tile18Lean>];
  sdd_tile<Tile18Lean, DT, LORA, true>(a, ring);
}
// The tile that suits the list as it is, of the set with RESIDENT workgroups per CU: see SddSet.  First product with
// the list's length / four times that / every block as capacity: 4096 tokens, d = 2048, 14 blocks 24.2 / 24.1 / 24.2 us
// (by the capacity's tile 23.3 / 46.3 / 45.9), 2048 tokens, d = 2560, 20 blocks 25.8 / 25.4 / 25.4 (25.7 / 54.8 /
// 35.6), 1024 tokens, d = 4096, 26 blocks 26.6 / 28.2 / 28.0 (26.3 / 46.3 / 76.8); four token tiles per list row, 1024
// tokens, d = 4096, every block as capacity 31 us (79).  With the low-rank step, rank 64: 4096 tokens, d = 2048, 14
// blocks, capacities 14 / 56 / 128 25 / 25 / 25 us (23 / 48 / 48), 1024 tokens, d = 4096, 26 blocks, capacities 26 / 104 /
// 256 28 / 30 / 30 (27 / 47 / 80), four token tiles per row as above 33 (82).
template <int DT, bool LORA, int RESIDENT>
__global__ __launch_bounds__(RESIDENT == 1 ? 512 : 256, 2) void ffn_sdd_any(SddArgs a) {
  __shared__ __attribute__((aligned(1024))) uint16_t ring[RESIDENT == 1 ? kRingElems<Tile14Deep> : kRingElems<Tile14>];
  const int n = min(a.row_ptr[a.rows], a.nnz_cap) - min(a.row_ptr[0], a.nnz_cap);
  int id = a.own;
  GridItem it = {-1, -1};
  if (sdd_keeps_own(a.nnz_cap, n)) {
    if (RESIDENT == 1 && a.mix) {
      const SddMix mix = sdd_mix(a.Tt, n);
      if (sdd_mixes(mix) && !sdd_mix_item(mix, a.Tt, n, blockIdx.x, id, it)) return;
    }
  } else {
    const int limit = sdd_limit<RESIDENT>(a.own, a.grid, a.Tt, a.gt, n);
    if ((int)blockIdx.x >= limit) return;
    id = sdd_pick<RESIDENT>(a.own, a.allowed, limit, a.Tt, a.gt, a.K, n);
  }
  if constexpr (RESIDENT == 1) {
    switch (id) {
      case kT44: sdd_tile<Tile44, DT, LORA>(a, ring, it); break;
      case kT24: sdd_tile<Tile24, DT, LORA>(a, ring, it); break;
      case kT22Deep: sdd_tile<Tile22Deep, DT, LORA>(a, ring, it); break;
      case kT14Deep: sdd_tile<Tile14Deep, DT, LORA>(a, ring); break;
      case kT12: sdd_tile<Tile12, DT, LORA>(a, ring); break;
      case kT11: sdd_tile<Tile11, DT, LORA>(a, ring); break;
    }
  } else {
    switch (id) {
      case kT22: sdd_tile<Tile22, DT, LORA>(a, ring); break;
      case kT14: sdd_tile<Tile14, DT, LORA>(a, ring); break;
      case kT12: sdd_tile<Tile12, DT, LORA>(a, ring); break;
      case kT11: sdd_tile<Tile11, DT, LORA>(a, ring); break;
    }
  }
}

// The token tile whose list has rank `want` by length (longest first, ties by index), out of up to kBalTiles; every
// workgroup computes the same ranking, so the assignment is a permutation.  Beyond: tile `want`.
__device__ __forceinline__ int tile_of_rank(const int* __restrict__ row_ptr, int Tt, int gt,
                                            int nnz_cap, int want, int* lens) {
  if (Tt > kBalTiles || Tt < 3) return want;
  const int tid = threadIdx.x;
  if (tid < Tt) {
    const int r = tid / gt;
    lens[tid] = min(row_ptr[r + 1], nnz_cap) - row_ptr[r];
  }
  __syncthreads();
  if (tid < Tt) {
    const int n = lens[tid];
    int rank = 0;
    for (int u = 0; u < Tt; ++u) {
      const int m = lens[u];
      rank += (m > n || (m == n && u < tid)) ? 1 : 0;
    }
    if (rank == want) lens[kBalTiles] = tid;
  }
  __syncthreads();
  const int tile = __builtin_amdgcn_readfirstlane(lens[kBalTiles]);
  __syncthreads();   // lens is memory the caller reuses
  return tile;
}


struct DsdArgs {
  const uint16_t *act, *W, *bias;
  long long ldw;
  const int *row_ptr, *col_idx;
  int Tt, gt, ncols, nnz_cap;
  int band;                    // h of grid_item (one list row)
  int full, rest, pieces;      // one list row: units that run whole, then units whose list is cut
  int GM, GN, order;           // otherwise: token groups, column chunks, DsdOrder
  uint16_t* out;
  float* part;
  const uint16_t *A2, *W2;     // LORA
};

template <class Tl, bool LORA>
struct DsdSrc {
  const uint16_t* base[Tl::kIss];
  const uint16_t* base2[LORA ? Tl::kIss : 1];
  uint32_t voffA[2], voffW[2];
  long long off_a, off_w, step_a;
  const int* list;             // col_idx of the range
  int lsteps, next;            // list entries of 64 steps, one per lane
  __device__ __forceinline__ int live() const { return Tl::kIss; }
  __device__ __forceinline__ bool busy(int) const { return true; }
  // Loads the entries of steps s .. s + 63.  In assembly, with its own wait: a load that the compiler
  // tracks would make it wait for vmcnt(0), and so for the whole ring, at every step's use of `next`
  // (twice the time with three stages).  The drain that is left costs about 1 us per 64 steps.
  __device__ __forceinline__ void fetch(int s) {
    const int e = s + (int)(threadIdx.x % kWave);
    const uint32_t off = (uint32_t)(e < lsteps ? e : lsteps - 1) * 4u;
    asm volatile("global_load_dword %0, %1, %2\n\ts_waitcnt vmcnt(0)" : "=v"(next) : "v"(off), "s"(list) : "memory");
  }
  __device__ __forceinline__ void begin(int s) {
    if (LORA && s == lsteps) {  // (the last step, as in SddSrc)
      off_a = off_w = 0;
      voffW[0] = voffA[0];     // rows of 64 elements too
      voffW[1] = voffA[1];
#pragma unroll
      for (int u = 0; u < Tl::kIss; ++u) base[u] = base2[LORA ? u : 0];
      return;
    }
    if (s > 0 && s % kWave == 0) fetch(s);
    off_a = s * step_a;
    off_w = (long long)__builtin_amdgcn_readlane(next, s % kWave) * 64;
  }
  __device__ __forceinline__ void dma(int u, uint32_t lds) const {
    const uint32_t to = lds + u * (Tl::kWaves * 1024);
    const int q = Tl::kWaves == 4 ? u & 1 : 0;
    if (u < Tl::kIssA)
      dma16_s(base[u] + off_a, voffA[q], to);
    else
      dma16_s(base[u] + off_w, voffW[q], to);
  }
};

// out[tile rows, n0 .. n0 + 64*TN - 1] = sum_s act[p_s] [64 x 64] . W[n0.., j_s*64 ..]^T (+ bias)
// LORA: one more step with the operands A2 [T,64] (the token tile's 64 x 64 block) and
// W2 [ncols_out, 64]: out += A2_i W2[n0..]^T, the low-rank part (dZ B) A of the input gradient.
// One list row for all tiles: 1-D grid over units (tile group, column chunk); the first `full` run
// whole, the list of each of the following `rest` is cut into `pieces` whose accumulators go to
// `part` as they are, fp32, for ffn_dsd_reduce to add in order.  Otherwise: 1-D grid of (column chunk, tile group),
// see dsd_unit.
// placed: as in sdd_tile.
template <class Tl, int DT, bool LORA>
__device__ __forceinline__ void dsd_tile(const DsdArgs& a, uint16_t* ring, GridItem placed = {-1, -1}) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  int i0, n0, s_lo = 0, n_i, rs, slot = -1;
  if (a.gt == a.Tt) {
    const int GM = (a.Tt + Tl::TM - 1) / Tl::TM, GN = (a.ncols + 64 * Tl::TN - 1) / (64 * Tl::TN);
    int piece = -1;
    if (placed.m < 0) {
      const int Lf = (a.full + 7) / 8, s = blockIdx.x / 8, x = blockIdx.x % 8;
      int unit;
      if (s < Lf) {
        unit = x * Lf + s;
        if (unit >= a.full) return;
      } else {
        const int cut = a.rest * a.pieces, Lr = (cut + 7) / 8, y = x * Lr + s - Lf;
        if (s - Lf >= Lr || y >= cut) return;
        piece = y / a.rest;                 // an XCD works on few pieces: their weights and activations
        unit = a.full + y % a.rest;
        slot = (y % a.rest) * a.pieces + piece;
      }
      placed = grid_item(unit, GM, GN, a.band);
    }
    i0 = placed.m * Tl::TM;
    n0 = placed.n * (64 * Tl::TN);
    rs = min(a.row_ptr[0], a.nnz_cap);
    n_i = min(a.row_ptr[1], a.nnz_cap) - rs;
    if (piece >= 0) {
      s_lo = (int)((long long)n_i * piece / a.pieces);
      n_i = (int)((long long)n_i * (piece + 1) / a.pieces) - s_lo;
    }
  } else {
    int chunk, rank;
    if (!dsd_unit(a.order, a.GM, a.GN, blockIdx.x, chunk, rank)) return;
    chunk = __builtin_amdgcn_readfirstlane(chunk);
    rank = __builtin_amdgcn_readfirstlane(rank);
    if (a.order != kUnranked)
      rank = tile_of_rank(a.row_ptr, a.GM, a.gt / Tl::TM, a.nnz_cap, rank, reinterpret_cast<int*>(ring));
    i0 = Tl::TM * rank;
    n0 = chunk * (64 * Tl::TN);
    rs = a.row_ptr[i0 / a.gt];
    n_i = min(a.row_ptr[i0 / a.gt + 1], a.nnz_cap) - rs;
  }
  if (n_i < 0) n_i = 0;     // nothing within the capacity

  DsdSrc<Tl, LORA> src;
  src.list = a.col_idx + rs + s_lo;
  src.lsteps = n_i;
  src.next = 0;
  if (n_i > 0) src.fetch(0);
  src.step_a = (long long)a.gt * 4096;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    src.voffA[q] = lane_voff<Tl>(64, wave + 4 * q);
    src.voffW[q] = lane_voff<Tl>(a.ldw, wave + 4 * q);
  }
#pragma unroll
  for (int u = 0; u < Tl::kIss; ++u) {
    const int g = wave + Tl::kWaves * u;
    if (u < Tl::kIssA) {     // (token tiles past the end: the last one again, not stored)
      const int i = min(i0 + g / 8, a.Tt - 1);
      src.base[u] = a.act + (((long long)rs + s_lo) * a.gt + i % a.gt) * 4096 + 8 * (g % 8) * 64;
      if (LORA) src.base2[LORA ? u : 0] = a.A2 + ((long long)i * 64 + 8 * (g % 8)) * 64;
    } else {                 // columns past the edge: the last 64 again, not stored
      const long long n = min(n0 + (g / 8 - Tl::TM) * 64, a.ncols - 64) + 8 * (g % 8);
      src.base[u] = a.W + n * a.ldw;
      if (LORA) src.base2[LORA ? u : 0] = a.W2 + n * 64;
    }
  }
  const int wm = wave / Tl::WN, wn = wave % Tl::WN;
  typename Tl::Acc acc[Tl::NI][Tl::TI];
  zero_acc<Tl>(acc);
  run_tile<Tl, DT>(n_i + (LORA ? 1 : 0), lds_addr(ring), wm, wn, src, acc);
  // (the lists of tiles of 32-row accumulators are never cut, which launch_dsd sees to)
  if constexpr (Tl::MF == 16)
    if (slot >= 0) {   // the piece's partial sums: [wave][accumulator][lane][4 registers]
      f32x4* dst = reinterpret_cast<f32x4*>(a.part) + ((size_t)slot * Tl::kWaves + wave) * (Tl::NI * Tl::TI) * kWave + threadIdx.x % kWave;
#pragma unroll
      for (int x = 0; x < Tl::NI; ++x)
#pragma unroll
        for (int y = 0; y < Tl::TI; ++y) dst[(x * Tl::TI + y) * kWave] = acc[x][y];
      return;
    }
  lds_barrier();       // nobody reads the ring any more
#pragma unroll
  for (int ni = 0; ni < Tl::NI; ++ni) {
    const int c = wn * Tl::NI + ni, n = n0 + Tl::MF * c;
#pragma unroll
    for (int ti = 0; ti < Tl::TI; ++ti)
      acc_to_lds<DT>(acc[ni][ti], lds_addr(ring), (wm * Tl::TI + ti) / Tl::kPer * Tl::TN + c / Tl::kPer,
                     Tl::MF * ((wm * Tl::TI + ti) % Tl::kPer), Tl::MF * (c % Tl::kPer), a.bias && n < a.ncols ? a.bias + n : nullptr, false);
  }
  lds_barrier();
  lds_to_out<Tl, DT, true>(lds_addr(ring), a.out, a.ncols, nullptr, [&](int t, int e) {
    return i0 + t < a.Tt && n0 + 64 * e < a.ncols ? (long long)(i0 + t) * 64 * a.ncols + n0 + 64 * e : -1ll;
  });
}
template <class Tl, int DT, bool LORA>
__global__ __launch_bounds__(Tl::kTileThreads, Tl::kMinWaves) void ffn_dsd(DsdArgs a) {
  __shared__ __attribute__((aligned(1024))) uint16_t ring[Tl::NST * Tl::kElems];
  dsd_tile<Tl, DT, LORA>(a, ring);
}
// 4 x 4 tiles and the rest of a round by narrower ones (SddMix).
template <int DT, bool LORA>
__global__ __launch_bounds__(512, 2) void ffn_dsd_mix(DsdArgs a) {
  constexpr int kRing = Tile24::NST * Tile24::kElems;          // the longest of the three
  static_assert(Tile44::NST * Tile44::kElems <= kRing && Tile22Deep::NST * Tile22Deep::kElems <= kRing, "shared memory");
  __shared__ __attribute__((aligned(1024))) uint16_t ring[kRing];
  int id;
  GridItem it;
  if (!sdd_mix_item(sdd_mix(a.Tt, a.ncols / 64), a.Tt, a.ncols / 64, blockIdx.x, id, it)) return;
  if (id == kT44)
    dsd_tile<Tile44, DT, LORA>(a, ring, it);
  else if (id == kT24)
    dsd_tile<Tile24, DT, LORA>(a, ring, it);
  else
    dsd_tile<Tile22Deep, DT, LORA>(a, ring, it);
}

// Adds the pieces of each cut unit (piece 0 first, fixed order: reproducible) and stores like the kernel's own
// epilogue: workgroup (b, y) is unit full + b and the y-th 64 x 64 block of its tile; wavefront w adds the
// four accumulators that hold quadrant (w % 2, w / 2) of the block.
template <class Tl, int DT>
__global__ __launch_bounds__(256) void ffn_dsd_reduce(DsdArgs a) {
  static_assert(Tl::MF == 16, "partial sums are stored per 16 x 16 accumulator");
  __shared__ __attribute__((aligned(1024))) uint16_t block[64 * 64];
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  const int t = blockIdx.y / Tl::TN, e = blockIdx.y % Tl::TN, nh = w % 2, th = w / 2;
  const int GM = (a.Tt + Tl::TM - 1) / Tl::TM, GN = (a.ncols + 64 * Tl::TN - 1) / (64 * Tl::TN);
  const GridItem it = grid_item(a.full + blockIdx.x, GM, GN, a.band);
  const int i = it.m * Tl::TM + t, n = (it.n * Tl::TN + e) * 64;
  if (i >= a.Tt || n >= a.ncols) return;
  const f32x4* src[2][2];
  f32x4 acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const int ng = 4 * e + 2 * nh + x, tg = 4 * t + 2 * th + y;        // 16-row groups of the tile
      const int wave = tg / Tl::TI * Tl::WN + ng / Tl::NI, acc_i = ng % Tl::NI * Tl::TI + tg % Tl::TI;
      src[x][y] = reinterpret_cast<const f32x4*>(a.part) +
                  (((size_t)blockIdx.x * a.pieces * Tl::kWaves + wave) * (Tl::NI * Tl::TI) + acc_i) * kWave + lane;
      acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  for (int p = 0; p < a.pieces; ++p)
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y) acc[x][y] += src[x][y][(size_t)p * (Tl::kWaves * Tl::NI * Tl::TI * kWave)];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
      acc_to_lds<DT>(acc[x][y], lds_addr(block), 0, 32 * th + 16 * y, 32 * nh + 16 * x,
                     a.bias ? a.bias + n + 32 * nh + 16 * x : nullptr, false);
  lds_barrier();
  lds_to_out<Tile<1, 1, 2, 2, 2, 2>, DT, true>(lds_addr(block), a.out, a.ncols, nullptr,
                                         [&](int, int) { return (long long)i * 64 * a.ncols + n; });
}

// ---------------------------------------------------------------------------
// Few tiles: a workgroup per quarter (32 x 32) of a 64 x 64 tile.  The quarters of a tile sit eight workgroups
// apart, on one XCD and on different CUs.  Results are those of the other tiles, to the last bit.
// ---------------------------------------------------------------------------
struct QuarterOf {
  int tile, th, nh;        // number of the tile's workgroup; token half, column half
  __device__ __forceinline__ QuarterOf() {
    const int w = blockIdx.x, q = w / 8 % 4;
    tile = w / 32 * 8 + w % 8;
    th = q % 2;
    nh = q / 2;
  }
};
// This lane's two 16-byte pieces of the quarter: element offsets of piece u from the quarter's first element.
__device__ __forceinline__ long long quarter_piece(int u, long long ld) {
  const int x = u * kWave + (int)threadIdx.x;
  return x / 4 * ld + x % 4 * 8;
}
// By the first wavefront, which is the only one left.
template <int DT, bool THROUGH>
__device__ __forceinline__ void store_quarter(const f32x16& acc, uint32_t lds, const uint16_t* __restrict__ bias, bool relu,
                                              bool gated, const uint4 (&gate)[2], uint16_t* __restrict__ out, long long ld) {
  lds_barrier();
  acc_to_lds<DT>(acc, lds, 0, 0, 0, bias, relu);
  lds_barrier();
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int x = u * kWave + (int)threadIdx.x;
    uint4 v = lds_read16(lds + out_slot(0, x / 4, x % 4));
    if (gated) v = make_uint4(gate2<DT>(v.x, gate[u].x), gate2<DT>(v.y, gate[u].y), gate2<DT>(v.z, gate[u].z), gate2<DT>(v.w, gate[u].w));
    uint16_t* p = out + quarter_piece(u, ld);
    if (THROUGH)
      asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(__builtin_bit_cast(u32x4, v)) : "memory");
    else
      *reinterpret_cast<uint4*>(p) = v;
  }
}
// A wave-uniform pointer, for an operand that has to be scalar.  (readfirstlane returns a signed int.)
__device__ __forceinline__ const uint16_t* scalar(const uint16_t* p) {
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return reinterpret_cast<const uint16_t*>((unsigned long long)hi << 32 | lo);
}
template <bool LORA>
struct QuarterSddSrc {
  const uint16_t *rows, *rows2;          // the operand's first element; of the low-rank step
  QuarterRows t, t2;
  uint32_t at;                           // of the operand in a step
  int ksteps;
  __device__ __forceinline__ void issue(int s, uint32_t lds) const {
    if (LORA && s == ksteps)
      t2.issue(scalar(rows2), lds + at);
    else
      t.issue(LORA ? scalar(rows + (long long)s * kBK) : rows + (long long)s * kBK, lds + at);
  }
};

template <int DT, bool LORA, int NST>
__global__ __launch_bounds__(Quarter::kTileThreads, NST == 8 ? 1 : 2) void ffn_sdd_quarter(SddArgs a) {
  __shared__ __attribute__((aligned(1024))) uint16_t ring[NST * 2 * Quarter::kElems];
  const QuarterOf q;
  int m, e, rs;
  if (a.gt == a.Tt) {
    rs = min(a.row_ptr[0], a.nnz_cap);
    const int n_i = min(a.row_ptr[1], a.nnz_cap) - rs;
    const int total = a.Tt * n_i, L = (total + 7) / 8, slot = q.tile / 8, idx = (q.tile % 8) * L + slot;
    if (slot >= L || idx >= total) return;
    const GridItem it = grid_item(idx, a.Tt, n_i, 8);
    m = it.m;
    e = it.n;
  } else {
    if (!find_work(a.row_ptr, a.Tt, a.gt, q.tile, 1, a.nnz_cap, a.halves, m, e)) return;
    m = __builtin_amdgcn_readfirstlane(m);
    e = __builtin_amdgcn_readfirstlane(e);
    rs = a.row_ptr[m / a.gt];
  }
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), col = a.col_idx[rs + e];
  const long long row_a = m * 64ll + 32 * q.th, row_w = col * 64ll + 32 * q.nh;
  uint16_t* out = a.out + (((long long)rs + e) * a.gt + m % a.gt) * 4096 + 32 * q.th * 64 + 32 * q.nh;
  uint4 gate[2] = {};
  QuarterSddSrc<LORA> src;
  src.ksteps = a.K / kBK;
  if (wave == 0) {
    if (a.gate) {
#pragma unroll
      for (int u = 0; u < 2; ++u) gate[u] = *reinterpret_cast<const uint4*>(a.gate + (out - a.out) + quarter_piece(u, 64));
    }
  } else {
    const bool weights = wave == 2;
    src.rows = weights ? a.W + row_w * a.K : a.A + row_a * a.K;
    src.at = weights ? 32 * kBK * 2 : 0;
    src.t.init(a.K, weights);
    if (LORA) {
      src.rows2 = weights ? a.W2 + row_w * 64 : a.A2 + row_a * 64;
      src.t2.init(64, weights);
    }
  }
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  run_quarter<DT, NST>(src.ksteps + (LORA ? 1 : 0), lds_addr(ring), src, acc);
  if (wave > 0) return;
  store_quarter<DT, false>(acc, lds_addr(ring), a.bias ? a.bias + row_w : nullptr, !a.gate, a.gate != nullptr, gate, out, 64);
}

template <bool LORA>
struct QuarterDsdSrc {
  const uint16_t *rows, *rows2;
  QuarterRows t, t2;
  uint32_t at;
  long long step;                        // of the token rows from list entry to list entry
  const int* list;                       // null: the token rows
  int lsteps, next;                      // as in DsdSrc
  __device__ __forceinline__ void fetch(int s) {
    const int e = s + (int)(threadIdx.x % kWave);
    const uint32_t off = (uint32_t)(e < lsteps ? e : lsteps - 1) * 4u;
    asm volatile("global_load_dword %0, %1, %2\n\ts_waitcnt vmcnt(0)" : "=v"(next) : "v"(off), "s"(list) : "memory");
  }
  __device__ __forceinline__ void issue(int s, uint32_t lds) {
    if (LORA && s == lsteps) {
      t2.issue(rows2, lds + at);
    } else if (!list) {
      t.issue(rows + s * step, lds + at);
    } else {
      if (s > 0 && s % kWave == 0) fetch(s);
      t.issue(rows + (long long)__builtin_amdgcn_readlane(next, s % kWave) * 64, lds + at);
    }
  }
};

template <int DT, bool LORA, int NST>
__global__ __launch_bounds__(Quarter::kTileThreads, NST == 8 ? 1 : 2) void ffn_dsd_quarter(DsdArgs a) {
  __shared__ __attribute__((aligned(1024))) uint16_t ring[NST * 2 * Quarter::kElems];
  const QuarterOf q;
  int chunk, i;
  if (!dsd_unit(kUnranked, a.GM, a.GN, q.tile, chunk, i)) return;
  chunk = __builtin_amdgcn_readfirstlane(chunk);
  i = __builtin_amdgcn_readfirstlane(i);
  const int rs = min(a.row_ptr[i / a.gt], a.nnz_cap), n_i = min(a.row_ptr[i / a.gt + 1], a.nnz_cap) - rs, n0 = chunk * 64 + 32 * q.nh;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  QuarterDsdSrc<LORA> src;
  src.lsteps = n_i;
  src.next = 0;
  src.list = nullptr;
  src.step = 0;
  if (wave == 1) {
    src.rows = a.act + ((long long)rs * a.gt + i % a.gt) * 4096 + 32 * q.th * 64;
    src.step = (long long)a.gt * 4096;
    src.at = 0;
    src.t.init(64, false);
    if (LORA) src.rows2 = a.A2 + (i * 64ll + 32 * q.th) * 64, src.t2 = src.t;
  } else if (wave == 2) {
    src.list = a.col_idx + rs;
    if (n_i > 0) src.fetch(0);
    src.rows = a.W + n0 * a.ldw;
    src.at = 32 * kBK * 2;
    src.t.init(a.ldw, true);
    if (LORA) src.rows2 = a.W2 + n0 * 64ll, src.t2.init(64, true);
  }
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  run_quarter<DT, NST>(n_i + (LORA ? 1 : 0), lds_addr(ring), src, acc);
  if (wave > 0) return;
  const uint4 none[2] = {};
  store_quarter<DT, true>(acc, lds_addr(ring), a.bias ? a.bias + n0 : nullptr, false, false, none,
                          a.out + (i * 64ll + 32 * q.th) * a.ncols + n0, a.ncols);
}

// pass 0 (forward):  A = X,  W1 = W_up [F,d],     W2 = W_down [d,F], act_out = H_act, out = Y
// pass 1 (backward): A = dY, W1 = W_down_t [F,d], W2 = W_up_t [d,F], act_out = dZ_act,
//                    act_gate = H_act, out = dX

// Token tiles per workgroup: 0 = chosen here; 1, 2 or 4 = at most that many, asked for by the caller.
// One value per host thread: a thread that sets the knob changes its own later calls only.
static thread_local int g_ffn_tiles_per_wg = 0;
hipError_t set_ffn_tiles_per_wg(int n) {
  if (n != 0 && n != 1 && n != 2 && n != 4) return hipErrorInvalidValue;
  g_ffn_tiles_per_wg = n;
  return hipSuccess;
}

// Bytes of partial sums with which the second product, given one list row of at most nnz_cap entries
// for all Tt token tiles, may cut lists (0: never), whatever the caller's tiles per workgroup.
size_t ffn_dsd_split_bytes(int Tt, int d, int nnz_cap) {
  size_t need = 0;
  for (int want : {0, 1, 2, 4}) {
    const size_t b = choose_dsd(Tt, Tt, d, nnz_cap, ~(size_t)0, want).part_bytes();
    need = b > need ? b : need;
  }
  return need;
}

// Calls CALL(Tile) for the tile `id`.
#define LX_TILES(id, CALL)                     \
  switch (id) {                                \
    case kT44: CALL(Tile44); break;            \
    case kT24: CALL(Tile24); break;            \
    case kT22: CALL(Tile22); break;            \
    case kT22Deep: CALL(Tile22Deep); break;    \
    case kT14: CALL(Tile14); break;            \
    case kT14Deep: CALL(Tile14Deep); break;    \
    case kT12: CALL(Tile12); break;            \
    case kT11: CALL(Tile11); break;            \
    default: CALL(Tile11Many); break;          \
  }

template <int DT, bool LORA>
static void launch_sdd(SddArgs a, hipStream_t st) {
  const SddRoute r = sdd_route(a.Tt, a.gt, a.K, a.nnz_cap, a.blocks, g_ffn_tiles_per_wg);
  const dim3 grid(r.grid);
  a.halves = r.halves;
  a.own = r.plan.id;
  a.grid = r.grid;
  a.allowed = r.plan.allowed;
  a.mix = r.mix;
#define LX_CALL(TL) hipLaunchKernelGGL((ffn_sdd<TL, DT, LORA>), grid, dim3(TL::kTileThreads), 0, st, a)
  if (r.by == kByQuarters && r.items <= kQuarterTilesAlone)
    hipLaunchKernelGGL((ffn_sdd_quarter<DT, LORA, 8>), grid, dim3(Quarter::kTileThreads), 0, st, a);
  else if (r.by == kByQuarters)
    hipLaunchKernelGGL((ffn_sdd_quarter<DT, LORA, 4>), grid, dim3(Quarter::kTileThreads), 0, st, a);
  else if (r.by == kBySet && kTileInfo[r.plan.id].resident == 1)
    hipLaunchKernelGGL((ffn_sdd_any<DT, LORA, 1>), grid, dim3(512), 0, st, a);
  else if (r.by == kBySet)
    hipLaunchKernelGGL((ffn_sdd_any<DT, LORA, 2>), grid, dim3(256), 0, st, a);
  else if (r.by == kByPieces)
    hipLaunchKernelGGL((ffn_sdd_even<DT, LORA>), grid, dim3(Tile18Lean::kTileThreads), 0, st, a);
  else if (r.by == kByLean)
    LX_CALL(Tile14Lean);
  else if (r.by == kByTile)
    LX_TILES(r.plan.id, LX_CALL)
#undef LX_CALL
}
template <int DT, bool LORA>
static void launch_dsd(DsdArgs a, size_t part_bytes, hipStream_t st) {
  const DsdRoute r = dsd_route(a.Tt, a.gt, a.ncols, a.ldw, a.nnz_cap, LORA || !a.part ? 0 : part_bytes, g_ffn_tiles_per_wg);
  const DsdPlan& p = r.plan;
  const dim3 grid(r.grid);
  a.GM = r.GM;
  a.GN = r.GN;
  a.order = r.order;
  if (r.by == kByQuarters) {
    if (r.items <= kQuarterTilesAlone)
      hipLaunchKernelGGL((ffn_dsd_quarter<DT, LORA, 8>), grid, dim3(Quarter::kTileThreads), 0, st, a);
    else
      hipLaunchKernelGGL((ffn_dsd_quarter<DT, LORA, 4>), grid, dim3(Quarter::kTileThreads), 0, st, a);
    return;
  }
  if (r.by == kByMix) {
    hipLaunchKernelGGL((ffn_dsd_mix<DT, LORA>), grid, dim3(512), 0, st, a);
    return;
  }
  a.band = kTileInfo[p.id].tm == 4 ? 4 : 8;
  a.full = p.full;
  a.rest = p.rest;
  a.pieces = p.pieces;
#define LX_CALL(TL) hipLaunchKernelGGL((ffn_dsd<TL, DT, LORA>), grid, dim3(TL::kTileThreads), 0, st, a)
  if (r.by == kByLean)
    LX_CALL(Tile14Lean);
  else
    LX_TILES(p.id, LX_CALL)
#undef LX_CALL
#define LX_CALL(TL) \
  hipLaunchKernelGGL((ffn_dsd_reduce<TL, DT>), dim3(p.rest, TL::TM * TL::TN), dim3(256), 0, st, a)
  static_assert(kLastCut == kT22, "the tiles whose lists may be cut are those that are reduced here");
  if (p.rest > 0) {
    if (p.id == kT44)
      LX_CALL(Tile44);
    else if (p.id == kT24)
      LX_CALL(Tile24);
    else
      LX_CALL(Tile22);
  }
#undef LX_CALL
}

template <int DT>
static hipError_t launch_ffn_bf16_t(int pass, int Tt, int gt, int Fb, int d, int F, const uint16_t* A,
                                    const uint16_t* W1, const uint16_t* b1, const uint16_t* W2,
                                    const uint16_t* b2, const int* row_ptr, const int* col_idx, int nnz_cap,
                                    uint16_t* act_out, const uint16_t* act_gate, uint16_t* out,
                                    float* part, size_t part_bytes, hipStream_t st) {
  (void)Fb;
  if (((long long)nnz_cap * gt + 3) / 4 + Tt > (1ll << 30)) return hipErrorInvalidValue;
  {
    ProfScope ps(pass == 0 ? kKFfnUp : kKFfnDh, st);
    launch_sdd<DT, false>({A, W1, pass == 0 ? b1 : nullptr, row_ptr, col_idx, Tt, gt, d, nnz_cap, Tt / gt, Tt / gt * (F / 64), 0, 0, 0u, false, false, act_out,
                           pass == 0 ? nullptr : act_gate, nullptr, nullptr}, st);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  ProfScope ps(pass == 0 ? kKFfnDown : kKFfnDx, st);
  launch_dsd<DT, false>({act_out, W2, b2, (long long)F, row_ptr, col_idx, Tt, gt, d, nnz_cap, 0, 0, 0, 1, 0, 0, 0, out, part,
                         nullptr, nullptr}, part_bytes, st);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// LoRA branch on the up-projection (Sec. II-C: z = W x + B A x; Sec. II-D: its gradients).
// A_pad [64, d] and B_pad [F, 64] hold A [r, d] and B [F, r] zero-padded to rank 64.
// ---------------------------------------------------------------------------

// forward: U = X A_pad^T [T,64];  H_act = ReLU(X W_up^T + U B_pad^T) on the listed blocks;
// Y = H W_down^T.
template <int DT>
static hipError_t launch_ffn_lora_fwd_bf16_t(int Tt, int gt, int d, int F, const uint16_t* X,
                                    const uint16_t* W_up, const uint16_t* A_pad,
                                    const uint16_t* B_pad, const uint16_t* W_down,
                                    const int* row_ptr, const int* col_idx, int nnz_cap,
                                    uint16_t* U, uint16_t* H_act, uint16_t* Y,
                                    hipStream_t st) {
  if (((long long)nnz_cap * gt + 3) / 4 + Tt > (1ll << 30)) return hipErrorInvalidValue;
  {
    ProfScope ps(kKLora, st);
    const hipError_t eu = launch_lora_u(DT, Tt, d, X, A_pad, U, st);
    if (eu != hipSuccess) return eu;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  {
    ProfScope ps(kKFfnUp, st);
    launch_sdd<DT, true>({X, W_up, nullptr, row_ptr, col_idx, Tt, gt, d, nnz_cap, Tt / gt, Tt / gt * (F / 64), 0, 0, 0u, false, false, H_act, nullptr, U, B_pad}, st);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  ProfScope ps(kKFfnDown, st);
  launch_dsd<DT, false>({H_act, W_down, nullptr, (long long)F, row_ptr, col_idx, Tt, gt, d, nnz_cap, 0, 0, 0, 1, 0, 0, 0, Y,
                         nullptr, nullptr, nullptr}, 0, st);
  return hipGetLastError();
}

// backward: dZ = (dY W_down) (.) [H > 0] on the listed blocks;  G = dZ B_pad [T,64];
// dX = dZ W_up + G A_pad;  dB = dZ^T U;  dA = G^T X.
// Scratch: A_t [d,64], G [T,64], da_part [lora_da_split][64][d] and db_part [lora_db_split][F][64] (the latter
// unused for a split of 1).
template <int DT>
static hipError_t launch_ffn_lora_bwd_bf16_t(int Tt, int gt, int d, int F, const uint16_t* X,
                                    const uint16_t* dY, const uint16_t* H_act, const uint16_t* U,
                                    const uint16_t* W_down_t, const uint16_t* W_up_t,
                                    const uint16_t* A_pad, const uint16_t* B_pad,
                                    const int* row_ptr, const int* col_idx, int nnz_cap,
                                    uint16_t* dZ, uint16_t* A_t, uint16_t* G,
                                    float* da_part, float* db_part, uint16_t* dX,
                                    float* dA, float* dB, hipStream_t st) {
  if (((long long)nnz_cap * gt + 3) / 4 + Tt > (1ll << 30)) return hipErrorInvalidValue;
  {
    ProfScope ps(kKFfnDh, st);
    launch_sdd<DT, false>({dY, W_down_t, nullptr, row_ptr, col_idx, Tt, gt, d, nnz_cap, Tt / gt, Tt / gt * (F / 64), 0, 0, 0u, false, false, dZ, H_act, nullptr, nullptr},
                          st);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  {
    ProfScope ps(kKLora, st);
    const hipError_t eg = launch_lora_g(DT, Tt, gt, d, dZ, B_pad, row_ptr, col_idx, nnz_cap, G, A_pad, A_t, st);
    if (eg != hipSuccess) return eg;
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  {
    ProfScope ps(kKFfnDx, st);
    launch_dsd<DT, true>({dZ, W_up_t, nullptr, (long long)F, row_ptr, col_idx, Tt, gt, d, nnz_cap, 0, 0, 0, 1, 0, 0, 0, dX,
                          nullptr, G, A_t}, 0, st);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  ProfScope ps(kKLora, st);
  return launch_lora_grads(DT, Tt, gt, d, F, dZ, U, G, X, row_ptr, col_idx, nnz_cap, da_part, db_part, dA,
                           dB, st);
}

// Entry points of this file: dt selects the element type (kBf16 or kF16).
hipError_t launch_ffn_bf16(int dt, int pass, int Tt, int gt, int Fb, int d, int F, const uint16_t* A,
                           const uint16_t* W1, const uint16_t* b1, const uint16_t* W2,
                           const uint16_t* b2, const int* row_ptr, const int* col_idx, int nnz_cap,
                           uint16_t* act_out, const uint16_t* act_gate, uint16_t* out,
                           float* part, size_t part_bytes, hipStream_t st) {
  return LX_BY_DT(launch_ffn_bf16_t, pass, Tt, gt, Fb, d, F, A, W1, b1, W2, b2, row_ptr, col_idx,
                  nnz_cap, act_out, act_gate, out, part, part_bytes, st);
}
hipError_t launch_ffn_lora_fwd_bf16(int dt, int Tt, int gt, int d, int F, const uint16_t* X,
                                    const uint16_t* W_up, const uint16_t* A_pad,
                                    const uint16_t* B_pad, const uint16_t* W_down,
                                    const int* row_ptr, const int* col_idx, int nnz_cap,
                                    uint16_t* U, uint16_t* H_act, uint16_t* Y,
                                    hipStream_t st) {
  return LX_BY_DT(launch_ffn_lora_fwd_bf16_t, Tt, gt, d, F, X, W_up, A_pad, B_pad, W_down, row_ptr,
                  col_idx, nnz_cap, U, H_act, Y, st);
}
hipError_t launch_ffn_lora_bwd_bf16(int dt, int Tt, int gt, int d, int F, const uint16_t* X,
                                    const uint16_t* dY, const uint16_t* H_act, const uint16_t* U,
                                    const uint16_t* W_down_t, const uint16_t* W_up_t,
                                    const uint16_t* A_pad, const uint16_t* B_pad,
                                    const int* row_ptr, const int* col_idx, int nnz_cap,
                                    uint16_t* dZ, uint16_t* A_t, uint16_t* G,
                                    float* da_part, float* db_part, uint16_t* dX,
                                    float* dA, float* dB, hipStream_t st) {
  return LX_BY_DT(launch_ffn_lora_bwd_bf16_t, Tt, gt, d, F, X, dY, H_act, U, W_down_t, W_up_t,
                  A_pad, B_pad, row_ptr, col_idx, nnz_cap, dZ, A_t, G, da_part, db_part, dX,
                  dA, dB, st);
}

}  // namespace lx
