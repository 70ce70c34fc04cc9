// Block-sparse attention for gfx950 (Sec. VI-A).  The two block-sparse products
// of the paper -- SDD (scores on listed blocks) and DSD (probabilities times
// V) -- are fused with the softmax in flash style, so the score blocks live
// only in registers; the unit of work is the listed block, which is what keeps
// heads with different patterns balanced (Sec. VI-A, online combination).
//
// Layout of one workgroup (256 threads = 4 wavefronts): it works on a 64-row
// query block (forward, dQ) or a 64-row key block (dK/dV) at a time -- its OWN
// rows -- and streams the [64 x D] tiles of the blocks listed for that row of
// the mask through LDS.  Wavefront w owns 16 of the own rows and works on ALL
// 64 rows of every streamed tile, on the 16x16x32 MFMA with fp32 accumulators:
// no two wavefronts share own rows, so a row of the mask ends without any
// exchange -- each wavefront normalises and stores its own 16 rows -- and the
// accumulators are small enough (D/4 registers per product) for dK and dV to
// be summed in one pass at both head sizes.
//
// At the block densities of the paper a row of the mask lists only a few
// blocks, so a workgroup that handled one row would spend most of its life in
// the chain of dependent loads that starts it (row pointer -> list -> tiles).
// A workgroup therefore owns up to eight rows and walks
// their lists as ONE sequence of ring entries, written once into an LDS table:
// per row an entry that brings the row's own tiles, then its listed blocks.
// The transfers of the entries ahead -- of the same row or of the next -- are
// in flight while the current one is computed, and nothing in the walk reads
// global memory directly.  Which rows: those of a group of up to four
// consecutive heads of a batch entry are ranked by the length of their lists and
// dealt to the group's workgroups in a snake over the ranks, which evens out the
// number of blocks per workgroup for any mask and between heads with long and
// short lists (where all workgroups of a launch are resident at once, it lasts as
// long as its longest workgroup); or, where a launch's rows do not divide evenly
// that way, one row of each of several cohorts of (batch entry, head) pairs, again
// by the rank of its list (by turns: attn_turns).
//
// Data movement: tiles go from global memory straight into LDS
// (global_load_lds, 16 bytes per lane) through a ring of two or three stages.
// Transfers AND result stores are issued as assembly and waited for by
// counting instructions (vmcnt retires them in order), so that no
// compiler-inserted wait drains the stages in flight.  Tiles are row-major,
// unpadded, with the 16-byte slots of a row XOR-swizzled by the row index
// (bank spreading).
//
// Two tricks keep everything in one LDS layout and out of cross-lane shuffles:
//  * the first product is computed transposed (S^T = K Q^T), so every lane
//    holds scores of ONE query and the accumulator registers are fed straight
//    back as the B operand of the second product; the MFMA's k index may be
//    permuted freely as long as both operands agree;
//  * the operands that are needed k-major (V^T, K^T, Q^T, dO^T) are read from
//    the same row-major tile with the transposing LDS read (ds_read_b64_tr_b16:
//    within 16 lanes, lane j receives column c0+j of the four rows addressed by
//    lanes 0-3, 4-7, 8-11, 12-15).
#include <type_traits>

#include "attn_plan.h"
#include "lx_dev.h"
#include "lx_launch.h"

namespace lx {

constexpr int kAT = 256;                 // threads per workgroup
constexpr int kAW = kAT / kWave;         // wavefronts per workgroup
// ring stages / resident workgroups per CU (= wavefronts per SIMD) the kernels are compiled
// for, head size 64: forward 2 / 4, dQ 2 / 4, dK/dV 3 / 3
// (measured against 3 / 3, 3 / 3 and 2 / 3, and 2 / 2 or 4 / 2); head size 128: 2 / 2
// everywhere (a stage is 32 KiB)
constexpr int kFwdNs64 = 2, kFwdOcc64 = 4, kDqNs64 = 2, kDqOcc64 = 4, kDkvNs64 = 3, kDkvOcc64 = 3;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kSlack = 8.f;            // log2 units; see the forward kernel

// What the 16-byte slots of a row are XORed with.  A 16-byte read takes four clocks if no two lanes of 0 .. 3, 12 .. 15 and
// 20 .. 27, or of the others of a half wavefront, meet in a bank (64 of them), and a transposing read two if none of the 32
// lanes of a half do; both hold for the two access patterns below.  (Measured in a loop of such reads, eight wavefronts:
// with row ^ row / 8 at D = 64 and row at D = 128, conflict-free for eight lanes in a row, the 16-byte reads took 8 clocks
// at D = 64 and the transposing ones 4.2 at D = 128.)  Rows 16 apart have the same.
template <int D>
__device__ __forceinline__ constexpr int tswz(int row) {
  return D == 64 ? row & 7 : (row & 3) << 1 | ((row >> 2 ^ row >> 3) & 1) << 3 | (row >> 2 & 1);
}

// The DMA instructions this wave issues for one [64 x D] tile: one moves 1 KiB = 64*16/(2D) rows, up to eight.  All of them
// have the tile's address as their wave-uniform base and a 32-bit offset per lane, which reaches over token strides below
// kWideStride, and one assembly block steps their LDS address: a wavefront does nothing else while it issues them, once
// per block.  (A base and an LDS address per instruction and 64-bit products for the tile's address were 85 scalar
// instructions for the two tiles of a block instead of 31.  Forward / dQ / dK and dV, us: 32 heads of 4096 tokens, D = 128, half of
// the blocks 102.9 / 132.9 / 164.2 -> 100.2 / 131.1 / 161.7; 16 of 4096, D = 64, all blocks 54.7 / 67.6 / 95.5 -> 53.6
// / 66.0 / 93.5; over ten sizes 1.8 / 1.2 / 1.4 % less.)  WIDE, for longer strides: a 64-bit address per lane.
constexpr long long kWideStride = 1ll << 25;      // elements; 63 rows of 2 * 2^25 bytes and a row's 240 fit 32 bits
template <int D, bool WIDE>
struct TileDma {
  static constexpr int kSlots = D / 8;            // 16-byte slots per row
  static constexpr int kRowsPer = 64 / kSlots;    // rows per DMA instruction
  static constexpr int kPerWave = 64 / kRowsPer / kAW;
  using Off = std::conditional_t<WIDE, long long, uint32_t>;
  Off off[kPerWave];                              // bytes from the tile's address: row, swizzled slot
  uint32_t wave_lds;
  __device__ __forceinline__ void init(long long ld) {
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    wave_lds = wave * 1024;
#pragma unroll
    for (int u = 0; u < kPerWave; ++u) {
      const int row = kRowsPer * (wave + kAW * u) + lane / kSlots, slot = (lane % kSlots) ^ tswz<D>(row);
      off[u] = (Off)(row * ld * 2) + slot * 16;
    }
  }
  // tile_addr: LDS byte address of the destination tile; g0: wave-uniform.  (No memory clobber: see dma16_s.)
  __device__ __forceinline__ void issue(uint32_t tile_addr, const char* g0) const {
    const uint32_t to = tile_addr + wave_lds;
    if constexpr (WIDE) {
#pragma unroll
      for (int u = 0; u < kPerWave; ++u) dma16(g0 + off[u], to + u * (kAW * 1024));
    } else {
#define LX_FIRST "s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %1"
#define LX_NEXT(V) "\n\ts_add_u32 m0, m0, 4096\n\ts_nop 0\n\tglobal_load_lds_dwordx4 " V ", %1"
      static_assert(kAW * 1024 == 4096 && (kPerWave == 2 || kPerWave == 4), "the assembly's steps");
      if constexpr (kPerWave == 2)
        asm volatile(LX_FIRST LX_NEXT("%3") ::"s"(to), "s"(g0), "v"(off[0]), "v"(off[1]) : "m0", "scc");
      else
        asm volatile(LX_FIRST LX_NEXT("%3") LX_NEXT("%4") LX_NEXT("%5") ::"s"(to), "s"(g0), "v"(off[0]), "v"(off[1]),
                     "v"(off[2]), "v"(off[3])
                     : "m0", "scc");
#undef LX_FIRST
#undef LX_NEXT
    }
  }
};

// LDS byte offsets inside a [64 x D] tile.  Element (row, col) sits at
// row*2D + (((col/8) ^ tswz(row)) << 4) + (col%8)*2.  tswz is linear over XOR and the row, slot
// and in-slot parts occupy disjoint bits, so the offset of (r0 + dr, c0 + dc) is the offset of
// (r0, c0) XOR a compile-time constant whenever r0/dr and c0/dc have disjoint bits.  Of that constant
// the row part only adds (bits that r0 leaves clear), so it goes into the LDS instruction's immediate
// offset; what is left are D / 32 or D / 16 different XORs of the slot bits per access pattern, each kept as one
// per-lane offset to which the stage's address is added once per tile (an XOR per LDS read was a
// sixth of the forward kernel's vector instructions).
template <int D>
__device__ __forceinline__ constexpr uint32_t tile_off(int row, int col) {
  return (uint32_t)(row * 2 * D + ((((col >> 3) ^ tswz<D>(row)) << 4)) + (col & 7) * 2);
}

// ---------------------------------------------------------------------------
// rows of a workgroup and the walk over their blocks
// ---------------------------------------------------------------------------
// The rows (query blocks, or key blocks for dK/dV) that a workgroup owns: of one batch entry's group of heads, as number g of
// the group's G workgroups (see init for how they are chosen; with more than 64 blocks per head: slot j holds block
// j*G + g for even j and (j+1)*G - 1 - g for odd j, counted from the last block if `mirror`, so
// that with the group index as the slowest grid dimension the longest rows of a causal mask are
// dispatched first), or by turns (init_turns).  The row pointers of all slots are fetched once and kept in a small LDS table.
// TURNS: the rows' batch entries differ (attn_turns); kernels of calls that do not run so are compiled without.
template <bool TURNS>
struct RowSet {
  const int* tab;   // LDS: blk[kRMax] (-1 = slot not used), rs[kRMax], n[kRMax], head[kRMax], batch entry[kRMax]
  int reg;          // the same table, entry i in lane i of every wavefront (one LDS read for all accessors)
  int b0, Hh;       // the batch entry of all rows, without TURNS; heads
  // How many of 64 lists are longer than this lane's, of n entries (-1: none, shorter than any), or as long and of a lower
  // lane: by a radix walk over the bits of the length with one ballot per bit.  `gt` collects the lanes known to be
  // longer, `eq` those equal in the bits seen so far.
  static __device__ __forceinline__ int rank_of(int n) {
    const unsigned key = (unsigned)(n + 1);
    unsigned long long gt = 0, eq = ~0ull;
#pragma unroll
    for (int bit = 6; bit >= 0; --bit) {     // a list has at most 64 entries here
      const unsigned long long set = __ballot((key >> bit) & 1u);
      if ((key >> bit) & 1u) {
        eq &= set;
      } else {
        gt |= eq & set;
        eq &= ~set;
      }
    }
    return __popcll(gt) + __popcll(eq & ((1ull << threadIdx.x % kWave) - 1ull));
  }
  // By turns (see attn_turns): slot k is a row of the k-th cohort that this workgroup's place takes part in.  Like init.
  __device__ __forceinline__ void init_turns(int* tab_lds, const int* __restrict__ row_ptr, int cap, const AttnArgs& a, int nblk, int w) {
    tab = tab_lds;
    const int lane = threadIdx.x % kWave, turns = a.by_turns.turns, V = a.by_turns.pairs, G = V * nblk, Z = a.by_turns.places,
              cohorts = a.by_turns.cohorts;
    const int x = w % 8, s = w / 8, place = s / G, r = s - place * G;
    const int mine = lane / nblk, k0 = threadIdx.x / kWave;
    constexpr int kMine = kRMax / kAW;          // slots k0, k0 + kAW, .. are this wavefront's; the loads of all before any is ranked
    bool valid[kMine], head_on[kMine];
    int hh[kMine], b[kMine], rs[kMine], end[kMine];
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
      const int k = k0 + kAW * i;
      // (every XCD begins elsewhere, so that what they read at a time lies in all parts of the tensors)
      const int number = k * Z + place, from = number + cohorts * x / 8, cohort = from < cohorts ? from : from - cohorts;
      const int pair = x + 8 * (cohort * V + mine);
      valid[i] = k < turns && number < cohorts && lane < G && pair < a.B * a.Hh;
      hh[i] = valid[i] ? pair / a.B : 0;
      b[i] = valid[i] ? pair - hh[i] * a.B : 0;
      rs[i] = end[i] = 0;
      head_on[i] = true;
      if (valid[i]) {
        const long long at = (long long)((a.mask_batch == 1 ? 0 : b[i]) * a.Hh + hh[i]) * nblk + lane - mine * nblk;
        if (a.head_active) head_on[i] = a.head_active[hh[i]] != 0;
        rs[i] = row_ptr[at];
        end[i] = row_ptr[at + 1];
      }
    }
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
      const int k = k0 + kAW * i;
      // entries beyond the capacity of the index buffer are ignored
      const int n = !valid[i] ? -1 : head_on[i] ? max(min(end[i], cap) - rs[i], 0) : 0;
      const int rank = rank_of(n), want = turn_rank(r, k, G, turns);
      if (valid[i] && rank == want) {
        tab_lds[k] = lane - mine * nblk;
        tab_lds[kRMax + k] = rs[i];
        tab_lds[2 * kRMax + k] = n;
        tab_lds[3 * kRMax + k] = hh[i];
        tab_lds[4 * kRMax + k] = b[i];
      }
      if (want >= __popcll(__ballot(valid[i])) && lane < 5) tab_lds[lane * kRMax + k] = lane == 0 ? -1 : 0;
    }
    __syncthreads();
    // behind the table's copy the slots' numbers of their (batch entry, head) pair
    const int k = lane % kRMax, own = tab_lds[min(lane, 5 * kRMax - 1)];
    reg = lane < 5 * kRMax ? own : tab_lds[4 * kRMax + k] * a.Hh + tab_lds[3 * kRMax + k];
  }
  // The rows are those of `heads` consecutive heads, h0 .. (nb1 blocks each, their list rows one
  // after the other from head_row0), ranked and dealt together: heads whose lists differ in
  // length then share their workgroups instead of each keeping G of its own.
  // tab_lds: 4 * kRMax ints of LDS (init_turns: 5); contains a barrier: call from uniform control flow
  __device__ __forceinline__ void init(int* tab_lds, const int* __restrict__ row_ptr,
                                       int cap, int head_row0, int nb1, int heads, int h0,
                                       const uint8_t* __restrict__ head_active, int g, int G, int R,
                                       bool mirror, int batch, int n_heads) {
    tab = tab_lds;
    const int tid = threadIdx.x;
    b0 = batch;
    const int nblk = nb1 * heads;
    if (nblk <= kWave) {
      // Groups balanced by the actual lengths of the lists: the rows of the head are ranked by
      // length (longest first, ties by index) and dealt to the G workgroups in a snake over the
      // ranks, rank k going to slot k / G of workgroup k % G or G - 1 - k % G.  Every workgroup
      // of the head computes the same ranking, one row per lane of its first wavefront.
      if (tid < kWave) {
        const bool valid = tid < nblk;
        const int hh = valid ? tid / nb1 : 0;       // head of this lane's row, relative to h0
        int rs = 0, n = -1;
        if (valid) {
          const bool head_on = !head_active || head_active[h0 + hh] != 0;
          rs = row_ptr[head_row0 + tid];
          // entries beyond the capacity of the index buffer are ignored
          n = head_on ? max(min(row_ptr[head_row0 + tid + 1], cap) - rs, 0) : 0;
        }
        const int rank = rank_of(n);     // (lanes past the last row are behind every row)
        const int j = rank / G, pos = rank - j * G;
        if (valid && ((j & 1) ? G - 1 - pos : pos) == g) {
          tab_lds[j] = tid - hh * nb1;
          tab_lds[kRMax + j] = rs;
          tab_lds[2 * kRMax + j] = n;
          tab_lds[3 * kRMax + j] = h0 + hh;
        }
      } else if (tid < kWave + kRMax) {
        // slots whose rank does not exist (the head has fewer rows than G * kRMax)
        const int j = tid - kWave;
        const int rank = j * G + ((j & 1) ? G - 1 - g : g);
        if (j >= R || rank >= nblk) {
          tab_lds[j] = -1;
          tab_lds[kRMax + j] = 0;
          tab_lds[2 * kRMax + j] = 0;
          tab_lds[3 * kRMax + j] = h0;
        }
      }
    } else if (tid < kRMax) {
      // more rows than lanes: fixed snake over the block index (balanced under a causal mask)
      const int j = tid;                       // (heads == 1 here: the launcher groups heads only
      int bj = (j & 1) ? (j + 1) * G - 1 - g : j * G + g;   //  when their rows fit one wavefront)
      const bool used = j < R && bj < nblk;
      if (mirror) bj = nblk - 1 - bj;
      const bool head_on = !head_active || head_active[h0] != 0;
      int rs = 0, n = 0;
      if (used) {
        rs = row_ptr[head_row0 + bj];
        n = head_on ? max(min(row_ptr[head_row0 + bj + 1], cap) - rs, 0) : 0;
      }
      tab_lds[j] = used ? bj : -1;
      tab_lds[kRMax + j] = rs;
      tab_lds[2 * kRMax + j] = n;
      tab_lds[3 * kRMax + j] = h0;
    }
    __syncthreads();
    Hh = n_heads;
    reg = tab_lds[threadIdx.x % (4 * kRMax)];
  }
  // k is wave-uniform; the results are scalars taken from the register copy of the table
  __device__ __forceinline__ int blk(int k) const { return __builtin_amdgcn_readlane(reg, k); }
  __device__ __forceinline__ int rs(int k) const { return __builtin_amdgcn_readlane(reg, kRMax + k); }
  __device__ __forceinline__ int n(int k) const { return __builtin_amdgcn_readlane(reg, 2 * kRMax + k); }
  __device__ __forceinline__ int head(int k) const { return __builtin_amdgcn_readlane(reg, 3 * kRMax + k); }
  __device__ __forceinline__ int batch(int k) const { return TURNS ? __builtin_amdgcn_readlane(reg, 4 * kRMax + k) : b0; }
  __device__ __forceinline__ int pair(int k) const { return TURNS ? __builtin_amdgcn_readlane(reg, 5 * kRMax + k) : b0 * Hh + head(k); }
};

// One 64-bit byte offset per row slot (its head's in a tensor), in the lanes of a register pair; with an entry's block added.
struct SlotOffset {
  uint32_t lo, hi;
  template <bool TURNS, class OfHead>
  __device__ __forceinline__ void init(const RowSet<TURNS>& rows, OfHead of_head) {
    const long long v = of_head(TURNS ? rows.tab[4 * kRMax + threadIdx.x % kRMax] : rows.b0, rows.tab[3 * kRMax + threadIdx.x % kRMax]);
    lo = (uint32_t)v;
    hi = (uint32_t)((unsigned long long)v >> 32);
  }
  // + blk blocks of `step` bytes; Step: uint32_t where a step fits it (two instructions for the product instead of four)
  template <class Step>
  __device__ __forceinline__ long long at(int slot, uint32_t blk, Step step) const {
    const uint32_t l = (uint32_t)__builtin_amdgcn_readlane((int)lo, slot), h = (uint32_t)__builtin_amdgcn_readlane((int)hi, slot);
    return (long long)(((unsigned long long)h << 32 | l) + (unsigned long long)blk * step);
  }
};

// ---------------------------------------------------------------------------
// products of a wavefront: its 16 own rows against the 64 rows of a streamed tile
// ---------------------------------------------------------------------------
// Per-lane offsets of the two access patterns into a streamed [64 x D] tile, for every XOR of the slot
// bits that the patterns' rows and columns make.
template <int D>
struct LaneOff16 {
  uint32_t rows[D / 32];   // element (lane%16, 8*(lane/16)) of k slice kk; row tile t: + 16t rows
  uint32_t tr[D / 16];     // element (4*(lane/16) + (lane%16)/4, 4*(lane%4)) of column tile ct; + 32kk + 16i rows
  __device__ __forceinline__ void init() {
    const int lane = threadIdx.x % kWave, g = lane / 16, j = lane % 16;
#pragma unroll
    for (int kk = 0; kk < D / 32; ++kk) rows[kk] = tile_off<D>(j, 8 * g) ^ (kk << 6);
#pragma unroll
    for (int ct = 0; ct < D / 16; ++ct) tr[ct] = tile_off<D>(4 * g + j / 4, 4 * (j % 4)) ^ (ct << 5);
  }
};
// v + s, opaque to the compiler: constants added to the result stay in the LDS instructions' immediates
__device__ __forceinline__ uint32_t add_lds(uint32_t v, uint32_t s) {
  uint32_t r;
  asm("v_add_u32 %0, %1, %2" : "=v"(r) : "s"(s), "v"(v));
  return r;
}

// acc[t] = R[rows 16t + lane%16][:] . F^T for the four row tiles t of a row-major tile R in LDS
// (byte address `tile`); F: per-lane fragments of the own rows (column index = lane%16).
// Result register v of acc[t]: element (row 16t + 4*(lane/16) + v, own row lane%16).
template <int D, int DT>
__device__ __forceinline__ void mma_rows16(uint32_t tile, const LaneOff16<D>& lo,
                                           const uint4 (&frag)[D / 32], f32x4 (&acc)[4]) {
  const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
  uint32_t a0[D / 32];
#pragma unroll
  for (int kk = 0; kk < D / 32; ++kk) a0[kk] = add_lds(lo.rows[kk], tile);
  uint4 a[D / 32][4];
#pragma unroll
  for (int kk = 0; kk < D / 32; ++kk)
#pragma unroll
    for (int t = 0; t < 4; ++t) a[kk][t] = lds_read16(a0[kk] + 16 * t * 2 * D);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int kk = 0; kk < D / 32; ++kk)
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = mfma16<DT>(a[kk][t], frag[kk], kk == 0 ? zero4 : acc[t]);
}

// Operands of out[ct] += T^T . P over all 64 rows of the row-major tile T (two k slices of 32
// rows), read with the transposing read.  k slot 8*(lane/16) + e of slice kk is row
// 32kk + 4*(lane/16) + e (e < 4) or 32kk + 16 + 4*(lane/16) + e - 4: the order in which the
// accumulator tiles 2kk and 2kk+1 of the first product hold their rows.
template <int D>
struct TrOps16 {
  uint4 a[2][D / 16];
};
template <int D>
__device__ __forceinline__ void load_tr16(uint32_t tile, const LaneOff16<D>& lo, TrOps16<D>& t) {
  uint32_t a0[D / 16];
#pragma unroll
  for (int ct = 0; ct < D / 16; ++ct) a0[ct] = add_lds(lo.tr[ct], tile);
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
#pragma unroll
    for (int ct = 0; ct < D / 16; ++ct) {
      const uint2 l = lds_read8_tr(a0[ct] + (32 * kk) * 2 * D);
      const uint2 h = lds_read8_tr(a0[ct] + (32 * kk + 16) * 2 * D);
      t.a[kk][ct] = make_uint4(l.x, l.y, h.x, h.y);
    }
}
// p[t][v]: accumulator-layout values of the [64 x 16] factor (rounded to the element type here)
template <int D, int DT>
__device__ __forceinline__ void mma_tr16(const TrOps16<D>& t, const f32x4 (&p)[4], f32x4 (&out)[D / 16]) {
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    uint4 b;
    b.x = pack2<DT>(p[2 * kk][0], p[2 * kk][1]);
    b.y = pack2<DT>(p[2 * kk][2], p[2 * kk][3]);
    b.z = pack2<DT>(p[2 * kk + 1][0], p[2 * kk + 1][1]);
    b.w = pack2<DT>(p[2 * kk + 1][2], p[2 * kk + 1][3]);
#pragma unroll
    for (int ct = 0; ct < D / 16; ++ct) out[ct] = mfma16<DT>(t.a[kk][ct], b, out[ct]);
  }
}

// The products of the two backward kernels issue a slot at a time: a matrix instruction, then the vector and LDS work of
// other products that needs nothing of it, with the compiler's scheduler held off between slots.  kMmaSlots: of a first product
// (D / 32 slices, four row tiles), and of a second one (two slices, D / 16 column tiles).
// The LDS operand reads bound these kernels, and the matrix and vector instructions that they hold up: with all blocks both
// sides take 61 % of the time at D = 128 (71 % at 64) without the reads, 87 % (74 %) without the matrix instructions,
// 93 % (88 %) without the exponentials.  Reads therefore go out a product ahead, into the registers that the operands
// before them leave, as far as the kernel's wavefronts per SIMD leave registers; not further: a register in scratch memory
// costs a drained ring (10 in dK/dV at D = 128: 1.2 times the time).  Both backward launches, us, product after product / in
// slots: 4 x 32 heads of 2048 tokens, D = 128, all blocks 1007 / 987, causal 566 / 554, causal 25 % 207 / 205; 16 of 4096,
// D = 128, causal 25 % 90.3 / 86.8; the same at D = 64 61.3 / 58.9; 2 x 40 of 2048, D = 64, causal 25 % 82.0 / 81.3.  (The
// forward kernel by slots: no difference.)
template <int D>
constexpr int kMmaSlots = D / 8;
__device__ __forceinline__ void end_slot() { __builtin_amdgcn_sched_barrier(0); }
// a first product's operand of slot i, from a row-major tile
template <int D>
__device__ __forceinline__ uint4 read_rows16(uint32_t tile, const LaneOff16<D>& lo, int i) {
  return lds_read16(add_lds(lo.rows[i / 4], tile) + 16 * (i % 4) * 2 * D);
}
// a second product's, from a row-major tile
template <int D>
__device__ __forceinline__ uint4 read_tr16(uint32_t tile, const LaneOff16<D>& lo, int i) {
  const int kk = i / (D / 16), ct = i % (D / 16);
  const uint32_t a0 = add_lds(lo.tr[ct], tile);
  const uint2 l = lds_read8_tr(a0 + (32 * kk) * 2 * D), h = lds_read8_tr(a0 + (32 * kk + 16) * 2 * D);
  return make_uint4(l.x, l.y, h.x, h.y);
}
// slice kk of a second product's [64 x 16] factor, rounded to the element type
template <int DT>
__device__ __forceinline__ uint4 pack_slice(const f32x4 (&p)[4], int kk) {
  return make_uint4(pack2<DT>(p[2 * kk][0], p[2 * kk][1]), pack2<DT>(p[2 * kk][2], p[2 * kk][3]),
                    pack2<DT>(p[2 * kk + 1][0], p[2 * kk + 1][1]), pack2<DT>(p[2 * kk + 1][2], p[2 * kk + 1][3]));
}
// acc = R F^T as in mma_rows16; meanwhile the operands of a first product with the tile `next` are read
template <int D, int DT>
__device__ __forceinline__ void mma_rows16_ahead(uint32_t tile, uint32_t next, const LaneOff16<D>& lo, const uint4 (&frag)[D / 32],
                                                 f32x4 (&acc)[4], uint4 (&ahead)[kMmaSlots<D>]) {
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  uint4 a[kMmaSlots<D>];
#pragma unroll
  for (int i = 0; i < kMmaSlots<D>; ++i) a[i] = read_rows16<D>(tile, lo, i);
  end_slot();
#pragma unroll
  for (int i = 0; i < kMmaSlots<D>; ++i) {
    acc[i % 4] = mfma16<DT>(a[i], frag[i / 4], i < 4 ? zero : acc[i % 4]);
    ahead[i] = read_rows16<D>(next, lo, i);
    end_slot();
  }
}

// Scores in the layout of mma_rows16 with the streamed rows (16t + 4*(lane/16) + v) being KEYS
// and the lane (own row `ql` of the block) the QUERY: keys after the query get -inf; `above`: the
// whole block lies on the excluded side of the diagonal.  mask_diag16_t: the roles exchanged
// (streamed rows are queries, the lane's own row is the key).
__device__ __forceinline__ void mask_diag16(f32x4 (&s)[4], int ql, bool above) {
  const int g = (threadIdx.x % kWave) / 16;
  const int x = above ? -1 : ql - 4 * g;     // key 16t + v > x: excluded
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (16 * t + v > x) s[t][v] = -INFINITY;
}
__device__ __forceinline__ void mask_diag16_t(f32x4 (&s)[4], int kl, bool above) {
  const int g = (threadIdx.x % kWave) / 16;
  const int x = above ? 64 : kl - 4 * g;     // query 16t + v < x: excluded
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (16 * t + v < x) s[t][v] = -INFINITY;
}

// accumulator layout [c-tile][v] (c = 16ct + 4*(lane/16) + v, row = lane%16) -> global
template <int D, int DT>
__device__ __forceinline__ void store_acc16(const f32x4 (&acc)[D / 16], float mul,
                                            uint16_t* __restrict__ dst_row) {
  const int g = (threadIdx.x % kWave) / 16;
#pragma unroll
  for (int ct = 0; ct < D / 16; ++ct) {
    uint2 o;
    o.x = pack2<DT>(acc[ct][0] * mul, acc[ct][1] * mul);
    o.y = pack2<DT>(acc[ct][2] * mul, acc[ct][3] * mul);
    *reinterpret_cast<uint2*>(dst_row + 16 * ct + 4 * g) = o;
  }
}
template <int N>
__device__ __forceinline__ void zero4(f32x4 (&a)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) a[i] = f32x4{0.f, 0.f, 0.f, 0.f};
}
// sum / maximum over the four lanes that share lane%16.  The rows of 16 lanes are exchanged in the vector
// unit: a swap of two copies of x leaves x of the even row (lower half) in both rows (halves) of one and
// x of the odd row (upper half) in the other.  In assembly: clang's builtin returns the first result
// twice; the s_nop is the distance a swap needs from the instruction that wrote its operands.
template <class T>
__device__ __forceinline__ void swap16(T& a, T& b) {
  asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void swap32(float& a, float& b) {
  asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ float sum_g(float x) {
  float y = x;
  swap16(x, y);
  x += y;
  y = x;
  swap32(x, y);
  return x + y;
}
__device__ __forceinline__ float max_g(float x) {
  float y = x;
  swap16(x, y);
  x = fmaxf(x, y);
  y = x;
  swap32(x, y);
  return fmaxf(x, y);
}
// (fmaxf makes the compiler quiet each argument first)
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// ---------------------------------------------------------------------------
// The work of a workgroup as ONE sequence of ring entries, built once into an LDS table: for
// every row slot with a non-empty list an OWN entry (the row's own tiles travel through the
// ring like any block, so a row starts without a load of its own), in the dQ kernel an AUX entry
// (a third own tile), then its listed blocks, the last one flagged.  Entry: bits 0..23 block
// index, 24..26 row slot.
// ---------------------------------------------------------------------------
constexpr int kTabCap = 512;                       // entries per fill of the table
constexpr int kTabInts = kTabCap + 4;              // its size: a walk reads up to a ring past the last entry
constexpr int kEOwn = 1 << 30, kELast = 1 << 29, kEAux = 1 << 28;

__device__ __forceinline__ int entry_blk(int e) { return e & 0xFFFFFF; }
__device__ __forceinline__ int entry_slot(int e) { return (e >> 24) & 7; }

// Entries first .. first+cnt-1 of the sequence -> tab[0 .. cnt).  Uniform control flow; ends
// with a barrier.  offs[i]: first entry of slot i (offs[kRMax] = length of the sequence); pre:
// entries of a row before its first block (1: OWN; 2: OWN, AUX).
template <class Rows>
__device__ __forceinline__ void fill_table(int* tab, const Rows& rows, const int* __restrict__ col_idx,
                                           const int (&offs)[kRMax + 1], int first, int cnt, int pre) {
  for (int e = first + (int)threadIdx.x; e < first + cnt; e += kAT) {
    int j = 0, o = 0;
#pragma unroll
    for (int i = 1; i < kRMax; ++i)
      if (e >= offs[i]) {
        j = i;
        o = offs[i];
      }
    const int it = e - o - pre;                    // < 0: the row's OWN (first) or AUX entry
    const int n = rows.tab[2 * kRMax + j];
    const int blk = it < 0 ? rows.tab[j] : col_idx[rows.tab[kRMax + j] + it];
    tab[e - first] = blk | (j << 24) | (it == -pre ? kEOwn : 0) | (it < 0 && it > -pre ? kEAux : 0) |
                     (it == n - 1 ? kELast : 0);
  }
  __syncthreads();
}

// s_waitcnt vmcnt(n') with the largest supported n' <= n (n wave-uniform): waiting for more than
// asked is always safe.
__device__ __forceinline__ void wait_vmcnt_dyn(int n) {
  switch (n) {
#define LX_W(N) case N: wait_vmcnt<N>(); break;
    LX_W(0) LX_W(1) LX_W(2) LX_W(3) LX_W(4) LX_W(5) LX_W(6) LX_W(7) LX_W(8) LX_W(9) LX_W(10)
    LX_W(11) LX_W(12) LX_W(13) LX_W(14) LX_W(15) LX_W(16) LX_W(17) LX_W(18) LX_W(19) LX_W(20)
    LX_W(21) LX_W(22) LX_W(23) LX_W(24) LX_W(25) LX_W(26) LX_W(27) LX_W(28) LX_W(29) LX_W(30)
    LX_W(31)
#undef LX_W
    default: wait_vmcnt<32>(); break;
  }
}

// Stores issued as assembly: the walk below counts every vector-memory instruction a wavefront
// issues (vmcnt retires loads and stores in order), so their number must not be the compiler's choice.
// (a store of more than 8 bytes still reads its registers for two wait states, which the compiler keeps for
// its own stores only)
__device__ __forceinline__ void store16(uint16_t* p, uint4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off\n\ts_nop 1" ::"v"(p), "v"(__builtin_bit_cast(u32x4, v)) : "memory");
}
__device__ __forceinline__ void store4(float* p, float v) {
  asm volatile("global_store_dword %0, %1, off" ::"v"(p), "v"(v) : "memory");
}
// accumulator layout -> global, D/32 store instructions: the lanes of a row hold four consecutive columns
// each; a swap of the odd rows of 16 lanes between two column tiles leaves eight in a lane, so an
// instruction writes 64 bytes of each of its 16 rows.  With 32-byte pieces (8 bytes per lane) the stores
// held up the walk's next transfers: forward / dQ / dK and dV over 48 sizes took 4.5 / 3.6 / 7.5 % longer.
template <int D, int DT>
__device__ __forceinline__ void store_acc16_asm(const f32x4 (&acc)[D / 16], float mul,
                                                uint16_t* __restrict__ dst_row) {
  const int g = (threadIdx.x % kWave) / 16;
  uint16_t* dst = dst_row + 16 * (g % 2) + 8 * (g / 2);
#pragma unroll
  for (int ct = 0; ct < D / 16; ct += 2) {
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      w[2 * e] = pack2<DT>(acc[ct + e][0] * mul, acc[ct + e][1] * mul);
      w[2 * e + 1] = pack2<DT>(acc[ct + e][2] * mul, acc[ct + e][3] * mul);
    }
    swap16(w[0], w[2]);
    swap16(w[1], w[3]);
    store16(dst + 16 * ct, make_uint4(w[0], w[1], w[2], w[3]));
  }
}

// Walk over the sequence with a ring of NS stages: the transfers of entry t + NS - 1 are issued
// while entry t is computed.  issue_own / issue_aux / issue_blk(stage, e) start the transfers of an
// entry and issue exactly XOWN / XAUX / XBLK vector-memory instructions per wavefront (XAUX < 0: the
// rows have no AUX entry); row_begin(stage, e) takes the own rows' operands out of the stage of an
// OWN entry; aux(stage, e) consumes an AUX entry and issues exactly YAUX store instructions;
// comp(stage, e) consumes a block; row_end(e) stores the row's results with exactly YST store
// instructions per wavefront.  No other vector-memory instruction may be issued inside the walk: a
// wavefront waits for the transfers of entry t by counting what it has issued since (in order: the
// transfers of the entries after t and the stores issued meanwhile).
struct NoAux {
  __device__ __forceinline__ void operator()(int, int) const {}
};
template <int NS, int XOWN, int XAUX, int XBLK, int YAUX, int YST, class IssueOwn, class IssueAux, class IssueBlk,
          class RowBegin, class Aux, class Comp, class RowEnd, class Rows>
__device__ __forceinline__ void walk_table(int* tab, const Rows& rows, const int* __restrict__ col_idx,
                                           IssueOwn issue_own, IssueAux issue_aux, IssueBlk issue_blk,
                                           RowBegin row_begin, Aux aux, Comp comp, RowEnd row_end) {
  static_assert(NS >= 2 && NS <= 4, "ring depth");
  static_assert(YAUX < 256 && YST < 256, "store counts are kept a byte each");
  constexpr int kPre = XAUX >= 0 ? 2 : 1;
  int offs[kRMax + 1];
  offs[0] = 0;
#pragma unroll
  for (int i = 0; i < kRMax; ++i) {
    const int ni = rows.n(i);
    offs[i + 1] = offs[i] + (ni > 0 ? ni + kPre : 0);
  }
  const int total = offs[kRMax];
  auto entry = [&](int i) { return __builtin_amdgcn_readfirstlane(tab[i]); };
  auto issue_entry = [&](int stage, int e) {
    if (e & kEOwn)
      issue_own(stage, e);
    else if (XAUX >= 0 && (e & kEAux))
      issue_aux(stage, e);
    else
      issue_blk(stage, e);
  };
  auto issued_by = [&](int e) { return (e & kEOwn) ? XOWN : (XAUX >= 0 && (e & kEAux)) ? XAUX : XBLK; };
  for (int first = 0; first < total; first += kTabCap) {
    const int cnt = min(kTabCap, total - first);
    if (first > 0) lds_barrier();        // the previous table and the stages are no longer read
    fill_table(tab, rows, col_idx, offs, first, cnt, kPre);
#pragma unroll
    for (int i = 0; i < NS - 1; ++i)
      if (i < cnt) issue_entry(i, entry(i));
    unsigned hist = 0;                   // byte i: store instructions issued while entry t-1-i was consumed
    int stage = 0, istage = NS - 1;      // stage of entry t; that of t - 1, which entry t + NS - 1 goes to
    int q[NS];                           // entries t .. t + NS - 1, read from the table a step before they are needed
#pragma unroll
    for (int u = 0; u < NS; ++u) q[u] = entry(u);
    for (int t = 0; t < cnt; ++t) {
      const int e = q[0];
      const int ahead = tab[t + NS];     // (past the end: not used)
      if constexpr (NS == 2) {           // what was issued since: the stores of the previous entry
        const unsigned st = hist & 0xFF;
        if (st == 0)
          wait_vmcnt<0>();
        else if (YAUX > 0 && YAUX != YST && st == YAUX)
          wait_vmcnt<YAUX>();
        else
          wait_vmcnt<YST>();
      } else {
        int n = 0;
#pragma unroll
        for (int u = 0; u < NS - 1; ++u) n += (hist >> (8 * u)) & 0xFF;
#pragma unroll
        for (int u = 1; u <= NS - 2; ++u)
          if (t + u < cnt) n += issued_by(q[u]);
        wait_vmcnt_dyn(n);
      }
      lds_barrier();
      if (t + NS - 1 < cnt) issue_entry(istage, q[NS - 1]);
      int stores = 0;
      if (e & kEOwn) {
        row_begin(stage, e);
      } else if (XAUX >= 0 && (e & kEAux)) {
        aux(stage, e);
        stores = YAUX;
      } else {
        comp(stage, e);
        if (e & kELast) {
          row_end(e);
          stores = YST;
        }
      }
      hist = (hist << 8) | (unsigned)stores;
      istage = stage;
      stage = NS == 2 ? stage ^ 1 : stage + 1 == NS ? 0 : stage + 1;
#pragma unroll
      for (int u = 0; u < NS - 1; ++u) q[u] = q[u + 1];
      q[NS - 1] = __builtin_amdgcn_readfirstlane(ahead);
    }
  }
}

// Which workgroup of which (batch entry, head group) pair this is.  Workgroup w runs on XCD w % 8.  Whole
// rounds of eight pairs are dealt to the XCDs in turn, all `gz` workgroups of a pair to one XCD: they
// stream the same tiles, so these are fetched into one L2 only, whatever the batch and head counts
// (dealt by the plain linear index, only multiples of eight pairs had that: 5 x 31 heads of 1536 tokens,
// 68 % of the blocks, forward 91 us, see the launcher).  The workgroups of the last P % 8 pairs are spread over all XCDs in
// runs.  The batch entry is the fast index of a pair: the masks of the batch entries are the same or
// alike, those of the heads are not, so every XCD gets about the same mix of heads.
// The longest workgroups of a pair have the smallest numbers z.  Where all workgroups of a launch are resident at
// once and own few rows (a.spread: otherwise the deal of the rows makes them equal), it matters which of them share
// a CU: an XCD's go to its 32 CUs in turn, so they are ordered by z, the first 32 the other way round: a CU's first
// workgroup is short where its second one is long, and the longest are alone where there are not two per CU.
// Against z after z of one pair and then the next (forward / dQ / dK and dV, us): 4 x 12 heads of 512 tokens, D = 128,
// all blocks 18.2 / 23.1 / 28.0 -> 15.7 / 20.2 / 23.5; 16 heads of 4096, D = 64, 25 % of the blocks 29.5 / 37.3 / 47.5
// -> 24.8 / 30.6 / 43.7; 32 heads of 2048, D = 128, dK and dV at 25 % 43.3 -> 36.1, with all blocks 90.4 -> 94.6 (the
// largest loss of 204 launches; with four or more rows per workgroup the order costs up to 8 % there, and gains little).
struct PairWork {
  int b, group, z;
};
__device__ __forceinline__ bool pair_work(const AttnArgs& a, int w, PairWork& p) {
  const int P = a.B * (a.Hh / a.vheads), gz = a.gz;
  const int x = w % 8, whole = P / 8 * gz;
  int s = w / 8, pair;
  if (a.spread && s < kCUs / 8 && whole >= kCUs / 8) s = kCUs / 8 - 1 - s;
  if (s < whole) {
    const int W = P / 8;
    pair = (a.spread ? s % W : s / gz) * 8 + x;
    p.z = a.spread ? s / W : s % gz;
  } else {
    const int rest = P % 8 * gz, L = (rest + 7) / 8, r = x * L + (s - whole);
    if (s - whole >= L || r >= rest) return false;
    pair = P / 8 * 8 + r / gz;
    p.z = r % gz;
  }
  p.b = pair % a.B;
  p.group = pair / a.B;
  return true;
}

// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------
template <int D, int DT, int NS, int OCC, bool WIDE, bool TURNS>
__global__ __launch_bounds__(kAT, OCC) void attn_fwd_bf16(const AttnArgs a) {
  __shared__ __attribute__((aligned(2 * 64 * D))) uint16_t st[NS][2 * 64 * D];   // stage: K tile, V tile
  __shared__ int rowtab[TURNS ? 5 * kRMax : 4 * kRMax];
  __shared__ int btab[kTabInts];
  constexpr uint32_t kStage = 4 * 64 * D, kTile = 2 * 64 * D;   // bytes
  const int nqb = a.S / 64;
  PairWork pw;
  if (!TURNS && !pair_work(a, blockIdx.x, pw)) return;
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int g = lane / 16, ql = 16 * wave + lane % 16;    // this lane's query inside the block
  auto base_of = [&](int b, int hh) { return (long long)b * a.sb + (long long)hh * a.sh; };
  auto stat_of = [&](int b, int hh) { return ((long long)b * a.Hh + hh) * a.S; };
  const uint32_t st_addr = lds_addr(&st[0][0]);
  const uint32_t own_off = tile_off<D>(ql, 8 * g);       // this lane's fragments inside an own tile

  RowSet<TURNS> rows;
  if constexpr (TURNS)
    rows.init_turns(rowtab, a.row_ptr, a.nnz_cap, a, nqb, blockIdx.x);
  else
    rows.init(rowtab, a.row_ptr, a.nnz_cap, ((a.mask_batch == 1 ? 0 : pw.b) * a.Hh + pw.group * a.vheads) * nqb, nqb,
              a.vheads, pw.group * a.vheads, a.head_active, pw.z, a.gz, a.rows_per_wg, true, pw.b, a.Hh);
  // rows without a listed block (or of an inactive head): O = 0, LSE = -inf, nothing to read
  for (int j = 0; j < kRMax; ++j)
    if (rows.blk(j) >= 0 && rows.n(j) == 0) {
      f32x4 z[D / 16];
      zero4(z);
      const int hh = rows.head(j), b = rows.batch(j);
      store_acc16<D, DT>(z, 0.f, a.Out + base_of(b, hh) + (long long)(rows.blk(j) * 64 + ql) * a.ss);
      if (g == 0) a.LSE[stat_of(b, hh) + rows.blk(j) * 64 + ql] = -INFINITY;
    }

  TileDma<D, WIDE> dma;
  dma.init(a.ss);
  using Step = std::conditional_t<WIDE, unsigned long long, uint32_t>;
  SlotOffset heads;
  heads.init(rows, [&](int b, int hh) { return 2 * base_of(b, hh); });
  // the element offset of this lane's own row in block blk of a slot, and of its head's statistics.  (Without TURNS from the head's number: from the
  // table's registers the machine code is another one and layer-sized launches of head size 64 were no faster, 0.99 - 1.02.)
  auto row_of = [&](int slot, int blk) -> long long {
    if constexpr (TURNS)
      return heads.at(slot, blk, (Step)(128 * a.ss)) / 2 + ql * a.ss;
    else
      return base_of(rows.b0, rows.head(slot)) + (long long)(blk * 64 + ql) * a.ss;
  };
  auto stats_of = [&](int slot) -> long long {
    if constexpr (TURNS)
      return (long long)rows.pair(slot) * a.S;
    else
      return stat_of(rows.b0, rows.head(slot));
  };
  // tensor p's tile of an entry
  auto tile_of = [&](const uint16_t* p, int e) {
    return reinterpret_cast<const char*>(p) + heads.at(entry_slot(e), entry_blk(e), (Step)(128 * a.ss));
  };
  LaneOff16<D> lo;
  lo.init();
  const float sc = a.scale * kLog2e;
  int qb = 0;
  long long qoff = 0, soff = 0;
  uint4 qf[D / 32];
  f32x4 o_acc[D / 16];
  float m = -INFINITY, m_use = 0.f, lsum = 0.f;   // reference point of the query (0 for -inf); this lane's share of its sum

  auto issue_own = [&](int stage, int e) {
    dma.issue(st_addr + stage * kStage, tile_of(a.Q, e));
  };
  auto issue_blk = [&](int stage, int e) {
    const uint32_t dst = st_addr + stage * kStage;
    dma.issue(dst, tile_of(a.K, e));
    dma.issue(dst + kTile, tile_of(a.V, e));
  };
  auto row_begin = [&](int stage, int e) {
    qb = entry_blk(e);
    const int slot = entry_slot(e);
    qoff = row_of(slot, qb);
    soff = stats_of(slot) + qb * 64 + ql;
    const uint32_t q0 = (st_addr + stage * kStage) | own_off;
#pragma unroll
    for (int kk = 0; kk < D / 32; ++kk) qf[kk] = lds_read16(q0 ^ tile_off<D>(0, 32 * kk));
    zero4(o_acc);
    m = -INFINITY;
    m_use = 0.f;
    lsum = 0.f;
  };
  auto comp = [&](int stage, int e) {
    const int col = entry_blk(e);
    const uint32_t stg = st_addr + stage * kStage;
    f32x4 s[4];
    mma_rows16<D, DT>(stg, lo, qf, s);          // S^T[key][q]
    TrOps16<D> vt;                              // independent of the scores: latency hides behind the softmax
    load_tr16<D>(stg + kTile, lo, vt);
    __builtin_amdgcn_sched_barrier(0);
    if (a.causal && col >= qb) mask_diag16(s, ql, col > qb);
    float mloc = max3(s[0][0], s[0][1], s[0][2]);
    mloc = max3(mloc, s[0][3], s[1][0]);
#pragma unroll
    for (int t = 1; t < 4; ++t) {
      mloc = max3(mloc, s[t][1], s[t][2]);
      mloc = max3(mloc, s[t][3], s[t < 3 ? t + 1 : t][0]);
    }
    // The reference point m of the running sums only has to bound the scores from above up to a
    // factor that fp32 holds comfortably: it follows the running maximum only when that has moved
    // by more than kSlack (then exp2(score - m) <= 2^kSlack).  Most blocks move it for no query of
    // the wavefront, which every lane sees from its own scores: no exchange, no rescaling.
    if (__any(mloc * sc > m + kSlack)) {
      const float cand = max_g(mloc) * sc;
      const float m_new = cand > m + kSlack ? cand : m;
      // a query none of whose keys so far is allowed keeps m = -inf; subtracting 0 instead keeps
      // the exponentials below at exp2(-inf) = 0 rather than exp2(-inf + inf)
      m_use = m_new == -INFINITY ? 0.f : m_new;
      const float alpha = __builtin_amdgcn_exp2f(m - m_use);
      lsum *= alpha;
      if (__any(alpha != 1.f && m != -INFINITY)) {
#pragma unroll
        for (int ct = 0; ct < D / 16; ++ct) o_acc[ct] *= alpha;
      }
      m = m_new;
    }
    float psum = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float p = __builtin_amdgcn_exp2f(fmaf(s[t][v], sc, -m_use));
        s[t][v] = p;
        psum += p;
      }
    lsum += psum;                   // the four lanes of a query add their shares at the row's end
    mma_tr16<D, DT>(vt, s, o_acc);              // O^T += V^T P^T
  };
  auto row_end = [&](int) {
    const float l = sum_g(lsum);
    const bool any = l > 0.f;
    const float inv = any ? 1.f / l : 0.f;
    store_acc16_asm<D, DT>(o_acc, inv, a.Out + qoff);
    // (the four lanes of a query store the same value)
    store4(a.LSE + soff, any ? (m + __builtin_amdgcn_logf(l)) * kLn2 : -INFINITY);
  };
  walk_table<NS, TileDma<D, WIDE>::kPerWave, -1, 2 * TileDma<D, WIDE>::kPerWave, 0, D / 32 + 1>(
      btab, rows, a.col_idx, issue_own, NoAux(), issue_blk, row_begin, NoAux(), comp, row_end);
}

// ---------------------------------------------------------------------------
// backward, query side
// ---------------------------------------------------------------------------
// sum + the products of eight elements of two operands
template <int DT>
__device__ __forceinline__ float dot8(uint4 a, uint4 b, float sum) {
  const uint32_t x[4] = {a.x, a.y, a.z, a.w}, y[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
  for (int q = 0; q < 4; ++q)
    sum += to_f32<DT>(x[q] & 0xFFFFu) * to_f32<DT>(y[q] & 0xFFFFu) + to_f32<DT>(x[q] >> 16) * to_f32<DT>(y[q] >> 16);
  return sum;
}
template <int D, int NS, bool TURNS>
struct DqLds {                       // (aligned to a tile where it is declared)
  uint16_t st[NS][2 * 64 * D];       // stage: K, V (or Q, dO; or O) tile
  float slse[NS][4][16];             // stage, wavefront: LSE of its 16 own rows
  int rowtab[TURNS ? 5 * kRMax : 4 * kRMax];
  int btab[kTabInts];
};
template <int D, int DT, int NS, bool WIDE, bool TURNS>
__device__ __forceinline__ void attn_bwd_dq(const AttnArgs& a, int w, DqLds<D, NS, TURNS>& sh) {
  auto& st = sh.st;
  auto& slse = sh.slse;
  constexpr uint32_t kStage = 4 * 64 * D, kTile = 2 * 64 * D;
  const int nqb = a.S / 64;
  PairWork pw;
  if (!TURNS && !pair_work(a, w, pw)) return;
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int g = lane / 16, ql = 16 * wave + lane % 16;
  auto base_of = [&](int b, int hh) { return (long long)b * a.sb + (long long)hh * a.sh; };
  auto stat_of = [&](int b, int hh) { return ((long long)b * a.Hh + hh) * a.S; };
  const uint32_t st_addr = lds_addr(&st[0][0]), slse_addr = lds_addr(&slse[0][0][0]);
  const uint32_t own_off = tile_off<D>(ql, 8 * g);

  RowSet<TURNS> rows;
  if constexpr (TURNS)
    rows.init_turns(sh.rowtab, a.row_ptr, a.nnz_cap, a, nqb, w);
  else
    rows.init(sh.rowtab, a.row_ptr, a.nnz_cap, ((a.mask_batch == 1 ? 0 : pw.b) * a.Hh + pw.group * a.vheads) * nqb, nqb,
              a.vheads, pw.group * a.vheads, a.head_active, pw.z, a.gz, a.rows_per_wg, true, pw.b, a.Hh);
  // rows without a listed block (or of an inactive head): dQ = 0, Delta = 0, nothing to read
  for (int j = 0; j < kRMax; ++j)
    if (rows.blk(j) >= 0 && rows.n(j) == 0) {
      f32x4 z[D / 16];
      zero4(z);
      const int hh = rows.head(j), b = rows.batch(j);
      store_acc16<D, DT>(z, 0.f, a.dQ + base_of(b, hh) + (long long)(rows.blk(j) * 64 + ql) * a.ss);
      if (g == 0) {
        a.Delta[stat_of(b, hh) + rows.blk(j) * 64 + ql] = 0.f;
        a.NegLse2[stat_of(b, hh) + rows.blk(j) * 64 + ql] = -INFINITY;      // no probability, if a column list names the row
      }
    }

  TileDma<D, WIDE> dma;
  dma.init(a.ss);
  using Step = std::conditional_t<WIDE, unsigned long long, uint32_t>;
  SlotOffset heads;
  heads.init(rows, [&](int b, int hh) { return 2 * base_of(b, hh); });
  // the element offset of this lane's own row in block blk of a slot, and of its head's statistics
  auto row_of = [&](int slot, int blk) -> long long {
    if constexpr (TURNS)
      return heads.at(slot, blk, (Step)(128 * a.ss)) / 2 + ql * a.ss;
    else
      return base_of(rows.b0, rows.head(slot)) + (long long)(blk * 64 + ql) * a.ss;
  };
  auto stats_of = [&](int slot) -> long long {
    if constexpr (TURNS)
      return (long long)rows.pair(slot) * a.S;
    else
      return stat_of(rows.b0, rows.head(slot));
  };
  // tensor p's tile of an entry
  auto tile_of = [&](const uint16_t* p, int e) {
    return reinterpret_cast<const char*>(p) + heads.at(entry_slot(e), entry_blk(e), (Step)(128 * a.ss));
  };
  LaneOff16<D> lo;
  lo.init();
  const float sc = a.scale * kLog2e;
  int qb = 0;
  long long qoff = 0;
  long long soff = 0;
  uint4 qf[D / 32], dof[D / 32];
  float delta = 0.f, lse2 = 0.f;
  f32x4 dq_acc[D / 16];

  auto issue_own = [&](int stage, int e) {
    const uint32_t dst = st_addr + stage * kStage;
    dma.issue(dst, tile_of(a.Q, e));
    dma.issue(dst + kTile, tile_of(a.dO, e));
  };
  // the row's O tile, needed once for Delta = rowsum(dO . O), and the LSE of its 64 queries
  // (lanes 0-15 of wavefront w bring those of its own rows 16w .. 16w+15)
  auto issue_aux = [&](int stage, int e) {
    const long long stats = stats_of(entry_slot(e));
    const int blk = entry_blk(e);
    dma.issue(st_addr + stage * kStage, tile_of(a.O, e));
    if (lane < 16) dma4(a.LSEin + stats + blk * 64 + ql, slse_addr + stage * 256 + wave * 64);
  };
  auto issue_blk = [&](int stage, int e) {
    const uint32_t dst = st_addr + stage * kStage;
    dma.issue(dst, tile_of(a.K, e));
    dma.issue(dst + kTile, tile_of(a.V, e));
  };
  auto row_begin = [&](int stage, int e) {
    qb = entry_blk(e);
    const int slot = entry_slot(e);
    qoff = row_of(slot, qb);
    soff = stats_of(slot) + qb * 64 + ql;
    const uint32_t q0 = (st_addr + stage * kStage) | own_off;
#pragma unroll
    for (int kk = 0; kk < D / 32; ++kk) {
      qf[kk] = lds_read16(q0 ^ tile_off<D>(0, 32 * kk));
      dof[kk] = lds_read16((q0 + kTile) ^ tile_off<D>(0, 32 * kk));
    }
    zero4(dq_acc);
  };
  // Delta and -LSE in log2 units of the row, kept for its blocks and written for the key-side kernel
  auto aux = [&](int stage, int) {
    const uint32_t o0 = (st_addr + stage * kStage) | own_off;
    float sum = 0.f;
#pragma unroll
    for (int kk = 0; kk < D / 32; ++kk) {
      sum = dot8<DT>(dof[kk], lds_read16(o0 ^ tile_off<D>(0, 32 * kk)), sum);
    }
    delta = sum_g(sum);
    // a row whose listed blocks hold no allowed key has LSE = -inf: +inf here makes every
    // probability exp2(score - inf) = 0, also for excluded scores (-inf), which -(-inf) would not
    const float lse_in = slse[stage][wave][lane % 16];
    lse2 = lse_in == -INFINITY ? INFINITY : lse_in * kLog2e;
    // (the four lanes of a query store the same values)
    store4(a.Delta + soff, delta);
    store4(a.NegLse2 + soff, -lse2);
  };
  auto comp = [&](int stage, int e) {
    const int col = entry_blk(e);
    const uint32_t stg = st_addr + stage * kStage;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    constexpr int N = kMmaSlots<D>, E = 16 / N, NC = D / 16;     // slots; score elements of a slot; column tiles
    f32x4 s[4], dp[4];
    uint4 vt[N], kt[N];
    // S^T[key][q]; with room for them (at D = 64 four wavefronts share a SIMD) meanwhile V's operands
    if constexpr (D == 64) {
      mma_rows16<D, DT>(stg, lo, qf, s);
#pragma unroll
      for (int i = 0; i < N; ++i) vt[i] = read_rows16<D>(stg + kTile, lo, i);
    } else {
      mma_rows16_ahead<D, DT>(stg, stg + kTile, lo, qf, s, vt);
    }
    if (a.causal && col >= qb) mask_diag16(s, ql, col > qb);   // excluded keys: P = exp2(-inf) = 0
    // dP^T[key][q]; meanwhile P, and with room for them K's operands
#pragma unroll
    for (int i = 0; i < N; ++i) {
      dp[i % 4] = mfma16<DT>(vt[i], dof[i / 4], i < 4 ? zero : dp[i % 4]);
      if (D == 128) kt[i] = read_tr16<D>(stg, lo, i);
#pragma unroll
      for (int x = E * i; x < E * (i + 1); ++x) s[x / 4][x % 4] = __builtin_amdgcn_exp2f(fmaf(s[x / 4][x % 4], sc, -lse2));
      end_slot();
    }
    auto ds = [&](int x) { s[x / 4][x % 4] *= dp[x / 4][x % 4] - delta; };      // dS^T
#pragma unroll
    for (int x = 0; x < 8; ++x) ds(x);
    uint4 f = pack_slice<DT>(s, 0);
    if (D == 64) {
#pragma unroll
      for (int i = 0; i < N; ++i) kt[i] = read_tr16<D>(stg, lo, i);
    }
    end_slot();
    // dQ^T += K^T dS^T
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      dq_acc[i] = mfma16<DT>(kt[i], f, dq_acc[i]);
#pragma unroll
      for (int x = 8 + 8 / NC * i; x < 8 + 8 / NC * (i + 1); ++x) ds(x);
      end_slot();
    }
    f = pack_slice<DT>(s, 1);
#pragma unroll
    for (int i = 0; i < NC; ++i) dq_acc[i] = mfma16<DT>(kt[NC + i], f, dq_acc[i]);
  };
  auto row_end = [&](int) { store_acc16_asm<D, DT>(dq_acc, a.scale, a.dQ + qoff); };
  walk_table<NS, 2 * TileDma<D, WIDE>::kPerWave, TileDma<D, WIDE>::kPerWave + 1, 2 * TileDma<D, WIDE>::kPerWave, 2, D / 32>(
      sh.btab, rows, a.col_idx, issue_own, issue_aux, issue_blk, row_begin, aux, comp, row_end);
}
template <int D, int DT, int NS, int OCC, bool WIDE, bool TURNS>
__global__ __launch_bounds__(kAT, OCC) void attn_bwd_dq_bf16(const AttnArgs a) {
  __shared__ __attribute__((aligned(2 * 64 * D))) DqLds<D, NS, TURNS> sh;
  attn_bwd_dq<D, DT, NS, WIDE, TURNS>(a, blockIdx.x, sh);
}

// ---------------------------------------------------------------------------
// backward, key side: a wavefront owns 16 keys; the streamed tiles are Q and dO of the listed
// query blocks, with the queries' -LSE*log2(e) and Delta beside them.  ALONE: O is streamed too and they are made here,
// as the query side makes them, so that the two sides need not follow each other
// ---------------------------------------------------------------------------
template <int D, int NS, bool ALONE, bool TURNS>
struct DkvLds {                      // (aligned to a tile where it is declared)
  uint16_t st[NS][(ALONE ? 3 : 2) * 64 * D];      // stage: Q, dO (or K, V), O tile
  float sstat[NS][4][32];            // stage, query tile: -LSE*log2e [16], Delta [16]
  int rowtab[TURNS ? 5 * kRMax : 4 * kRMax];
  int btab[kTabInts];
};
template <int D, int DT, int NS, bool WIDE, bool ALONE, bool TURNS>
__device__ __forceinline__ void attn_bwd_dkv(const AttnArgs& a, int w, DkvLds<D, NS, ALONE, TURNS>& sh) {
  auto& st = sh.st;
  auto& sstat = sh.sstat;
  constexpr uint32_t kTile = 2 * 64 * D, kStage = (ALONE ? 3 : 2) * kTile;
  const int nkb = a.S / 64;
  PairWork pw;
  if (!TURNS && !pair_work(a, w, pw)) return;
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int g = lane / 16, kl = 16 * wave + lane % 16;    // this lane's key inside the block
  auto base_of = [&](int b, int hh) { return (long long)b * a.sb + (long long)hh * a.sh; };
  auto stat_of = [&](int b, int hh) { return ((long long)b * a.Hh + hh) * a.S; };
  const uint32_t st_addr = lds_addr(&st[0][0]), sstat_addr = lds_addr(&sstat[0][0][0]);
  const uint32_t own_off = tile_off<D>(kl, 8 * g);

  RowSet<TURNS> rows;
  if constexpr (TURNS)
    rows.init_turns(sh.rowtab, a.crow_ptr, a.cnnz_cap, a, nkb, w);
  else
    rows.init(sh.rowtab, a.crow_ptr, a.cnnz_cap, ((a.mask_batch == 1 ? 0 : pw.b) * a.Hh + pw.group * a.vheads) * nkb, nkb,
              a.vheads, pw.group * a.vheads, a.head_active, pw.z, a.gz, a.rows_per_wg, false, pw.b, a.Hh);
  // key blocks used by no query block: zero gradients, nothing to read
  for (int j = 0; j < kRMax; ++j)
    if (rows.blk(j) >= 0 && rows.n(j) == 0) {
      f32x4 z[D / 16];
      zero4(z);
      const long long koff = base_of(rows.batch(j), rows.head(j)) + (long long)(rows.blk(j) * 64 + kl) * a.ss;
      store_acc16<D, DT>(z, 0.f, a.dV + koff);
      store_acc16<D, DT>(z, 0.f, a.dK + koff);
    }

  TileDma<D, WIDE> dma;
  dma.init(a.ss);
  using Step = std::conditional_t<WIDE, unsigned long long, uint32_t>;
  SlotOffset heads;
  heads.init(rows, [&](int b, int hh) { return 2 * base_of(b, hh); });
  // the element offset of this lane's own row in block blk of a slot
  auto row_of = [&](int slot, int blk) -> long long {
    if constexpr (TURNS)
      return heads.at(slot, blk, (Step)(128 * a.ss)) / 2 + kl * a.ss;
    else
      return base_of(rows.b0, rows.head(slot)) + (long long)(blk * 64 + kl) * a.ss;
  };
  // tensor p's tile of an entry
  auto tile_of = [&](const uint16_t* p, int e) {
    return reinterpret_cast<const char*>(p) + heads.at(entry_slot(e), entry_blk(e), (Step)(128 * a.ss));
  };
  LaneOff16<D> lo;
  lo.init();
  const float sc = a.scale * kLog2e;
  // lanes 0-15 of wave w bring -LSE*log2(e), lanes 16-31 Delta of queries 16w .. 16w+15 of a block; ALONE: lanes 0-15 LSE
  const char* stat_src = reinterpret_cast<const char*>((ALONE ? a.LSEin : lane < 16 ? a.NegLse2 : a.Delta) + 16 * wave + lane % 16);
  SlotOffset stats;
  stats.init(rows, [&](int b, int hh) { return 4 * stat_of(b, hh); });
  int kb = 0;
  long long koff = 0;
  uint4 kf[D / 32], vf[D / 32];
  f32x4 dk_acc[D / 16], dv_acc[D / 16];

  auto issue_own = [&](int stage, int e) {
    const uint32_t dst = st_addr + stage * kStage;
    dma.issue(dst, tile_of(a.K, e));
    dma.issue(dst + kTile, tile_of(a.V, e));
  };
  auto issue_blk = [&](int stage, int e) {
    const uint32_t dst = st_addr + stage * kStage;
    dma.issue(dst, tile_of(a.Q, e));
    dma.issue(dst + kTile, tile_of(a.dO, e));
    if (ALONE) dma.issue(dst + 2 * kTile, tile_of(a.O, e));
    if (lane < (ALONE ? 16 : 32)) dma4(stat_src + stats.at(entry_slot(e), entry_blk(e), 256u), sstat_addr + stage * 512 + wave * 128);
  };
  auto row_begin = [&](int stage, int e) {
    kb = entry_blk(e);
    koff = row_of(entry_slot(e), kb);
    const uint32_t k0 = (st_addr + stage * kStage) | own_off;
#pragma unroll
    for (int kk = 0; kk < D / 32; ++kk) {
      kf[kk] = lds_read16(k0 ^ tile_off<D>(0, 32 * kk));
      vf[kk] = lds_read16((k0 + kTile) ^ tile_off<D>(0, 32 * kk));
    }
    zero4(dk_acc);
    zero4(dv_acc);
  };
  auto comp = [&](int stage, int e) {
    const int col = entry_blk(e);
    const uint32_t stg = st_addr + stage * kStage;
    if (ALONE) {      // the same sums in the same order as the query side's
      const uint32_t o0 = stg + kTile + own_off;
      float sum = 0.f;
#pragma unroll
      for (int kk = 0; kk < D / 32; ++kk) {
        const uint4 df = lds_read16(o0 ^ tile_off<D>(0, 32 * kk)), of = lds_read16((o0 + kTile) ^ tile_off<D>(0, 32 * kk));
        sum = dot8<DT>(df, of, sum);
      }
      const float delta = sum_g(sum), lse = sstat[stage][wave][lane % 16];
      if (g == 0) {
        sstat[stage][wave][lane] = lse == -INFINITY ? -INFINITY : -(lse * kLog2e);
        sstat[stage][wave][16 + lane] = delta;
      }
      lds_barrier();
    }
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    constexpr int N = kMmaSlots<D>, E = 16 / N, NC = D / 16;     // slots; score elements of a slot; column tiles
    f32x4 s[4], dp[4], stat[2];        // stat: -LSE or Delta of the row tile's queries, a tile ahead
    uint4 ops[N], tr[N];
    mma_rows16_ahead<D, DT>(stg, stg + kTile, lo, kf, s, ops);      // S[q][key]
    // diagonal block: here the rows of the score tile are queries and the lane is the key
    if (a.causal && col <= kb) mask_diag16_t(s, kl, col < kb);
    auto read_stat = [&](int t, int which) { stat[t % 2] = *reinterpret_cast<const f32x4*>(&sstat[stage][t][16 * which + 4 * g]); };
    read_stat(0, 0);
    end_slot();
    // dP[q][key]; meanwhile P
#pragma unroll
    for (int i = 0; i < N; ++i) {
      dp[i % 4] = mfma16<DT>(ops[i], vf[i / 4], i < 4 ? zero : dp[i % 4]);
      if (E * i % 4 == 0 && i + 4 / E < N) read_stat(E * i / 4 + 1, 0);
#pragma unroll
      for (int x = E * i; x < E * (i + 1); ++x)
        s[x / 4][x % 4] = __builtin_amdgcn_exp2f(fmaf(s[x / 4][x % 4], sc, stat[x / 4 % 2][x % 4]));
      end_slot();
    }
    uint4 p16[2], ds16[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) p16[kk] = pack_slice<DT>(s, kk);
    read_stat(0, 1);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (t < 3) read_stat(t + 1, 1);
#pragma unroll
      for (int v = 0; v < 4; ++v) dp[t][v] = s[t][v] * (dp[t][v] - stat[t % 2][v]);
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) ds16[kk] = pack_slice<DT>(dp, kk);
#pragma unroll
    for (int i = 0; i < N; ++i) tr[i] = read_tr16<D>(stg + kTile, lo, i);
    end_slot();
    // dV^T += dO^T P; meanwhile Q's operands
#pragma unroll
    for (int i = 0; i < N; ++i) {
      dv_acc[i % NC] = mfma16<DT>(tr[i], p16[i / NC], dv_acc[i % NC]);
      ops[i] = read_tr16<D>(stg, lo, i);
      end_slot();
    }
    // dK^T += Q^T dS
#pragma unroll
    for (int i = 0; i < N; ++i) dk_acc[i % NC] = mfma16<DT>(ops[i], ds16[i / NC], dk_acc[i % NC]);
  };
  auto row_end = [&](int) {
    store_acc16_asm<D, DT>(dv_acc, 1.f, a.dV + koff);
    store_acc16_asm<D, DT>(dk_acc, a.scale, a.dK + koff);
  };
  walk_table<NS, 2 * TileDma<D, WIDE>::kPerWave, -1, (ALONE ? 3 : 2) * TileDma<D, WIDE>::kPerWave + 1, 0, 2 * (D / 32)>(
      sh.btab, rows, a.ccol_idx, issue_own, NoAux(), issue_blk, row_begin, NoAux(), comp, row_end);
}
template <int D, int DT, int NS, int OCC, bool WIDE, bool TURNS>
__global__ __launch_bounds__(kAT, OCC) void attn_bwd_dkv_bf16(const AttnArgs a) {
  __shared__ __attribute__((aligned(2 * 64 * D))) DkvLds<D, NS, false, TURNS> sh;
  attn_bwd_dkv<D, DT, NS, WIDE, false, TURNS>(a, blockIdx.x, sh);
}

// Both sides in one launch (bwd_in_one): the first `half` workgroups take the key side, which is the longer one.
template <int D, int DT, int NS, int OCC>
__global__ __launch_bounds__(kAT, OCC) void attn_bwd_both_bf16(const AttnArgs a, int half) {
  __shared__ __attribute__((aligned(2 * 64 * D))) DkvLds<D, NS, true, false> sh;
  static_assert(sizeof(DqLds<D, NS, false>) <= sizeof(sh), "shared memory");
  if ((int)blockIdx.x < half)
    attn_bwd_dkv<D, DT, NS, false, true, false>(a, blockIdx.x, sh);
  else
    attn_bwd_dq<D, DT, NS, false, false>(a, blockIdx.x - half, reinterpret_cast<DqLds<D, NS, false>&>(sh));
}


static thread_local int g_rows_per_wg = 0;   // one value per host thread
hipError_t set_attn_rows_per_wg(int r) {
  if (r < 0 || r > kRMax) return hipErrorInvalidValue;
  g_rows_per_wg = r;
  return hipSuccess;
}

// Completes the arguments for workgroups of which `slots` fit the chip; returns the grid (see pair_work and
// RowSet::init_turns: a.by_turns.turns > 0).
static int attn_grid(AttnArgs& a, int B, int slots, bool may_turn) {
  const AttnShape s = attn_shape(B, a.Hh, a.S / 64, slots, may_turn, g_rows_per_wg);
  a.B = B;
  a.vheads = s.vheads;
  a.rows_per_wg = s.rows_per_wg;
  a.gz = s.gz;
  a.spread = s.spread;
  a.by_turns = s.by_turns;
  return s.grid;
}

template <int D, int DT, bool WIDE>
static hipError_t launch_fwd_t(AttnArgs a, int B, hipStream_t st) {
  ProfScope ps(kKAttnFwd, st);
  constexpr int kNs = D == 64 ? kFwdNs64 : 2, kOcc = D == 64 ? kFwdOcc64 : 2;
  const int grid = attn_grid(a, B, kCUs * kOcc, true);
  if (a.by_turns.turns > 0)
    hipLaunchKernelGGL((attn_fwd_bf16<D, DT, kNs, kOcc, WIDE, true>), dim3(grid), dim3(kAT), 0, st, a);
  else
    hipLaunchKernelGGL((attn_fwd_bf16<D, DT, kNs, kOcc, WIDE, false>), dim3(grid), dim3(kAT), 0, st, a);
  return hipGetLastError();
}
template <int D, int DT>
static hipError_t launch_fwd(const AttnArgs& a, int B, hipStream_t st) {
  return a.ss < kWideStride ? launch_fwd_t<D, DT, false>(a, B, st) : launch_fwd_t<D, DT, true>(a, B, st);
}

// Whether the two sides of a backward pass run in one launch: results are the same to the last bit.
constexpr int kBothOcc(int D) { return D == 64 ? 3 : 1; }
static bool bwd_in_one(const AttnArgs& a, int D, int B) {
  const int nblk = a.S / 64;
  const long long rows = (long long)a.mask_batch * a.Hh * nblk, stats = (long long)B * a.Hh * a.S * 4;
  const double mean = (double)(a.nnz_cap > a.cnnz_cap ? a.nnz_cap : a.cnnz_cap) / rows;
  if (!bwd_one_launch_pays(D, (long long)B * a.Hh * nblk, nblk, a.causal != 0, mean)) return false;
  return bwd_sides_apart({{{B, a.Hh, a.S}, {2 * a.sb, 2 * a.sh, 2 * a.ss}, 2 * D},
                          {a.Q, a.K, a.V, a.O, a.dO},
                          {a.dQ, a.dK, a.dV},
                          {a.LSEin, stats},
                          {{a.row_ptr, 4 * (rows + 1)}, {a.col_idx, 4ll * a.nnz_cap}},
                          {{a.Delta, stats}, {a.NegLse2, stats}}});
}
template <int D, int DT, bool WIDE>
static hipError_t launch_bwd_t(AttnArgs a, int B, hipStream_t st) {
  if constexpr (!WIDE)      // (long strides: see bwd_one_launch_pays)
    if (bwd_in_one(a, D, B)) {
      ProfScope ps(kKAttnDkv, st);
      constexpr int kOcc = kBothOcc(D);
      const int half = attn_grid(a, B, kCUs * kOcc / 2, false);
      hipLaunchKernelGGL((attn_bwd_both_bf16<D, DT, 2, kOcc>), dim3(2 * half), dim3(kAT), 0, st, a, half);
      return hipGetLastError();
    }
  {
    ProfScope ps(kKAttnDq, st);
    constexpr int kNs = D == 64 ? kDqNs64 : 2, kOcc = D == 64 ? kDqOcc64 : 2;
    const int grid = attn_grid(a, B, kCUs * kOcc, true);
    if (a.by_turns.turns > 0)
      hipLaunchKernelGGL((attn_bwd_dq_bf16<D, DT, kNs, kOcc, WIDE, true>), dim3(grid), dim3(kAT), 0, st, a);
    else
      hipLaunchKernelGGL((attn_bwd_dq_bf16<D, DT, kNs, kOcc, WIDE, false>), dim3(grid), dim3(kAT), 0, st, a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  {
    ProfScope ps(kKAttnDkv, st);
    constexpr int kNs = D == 64 ? kDkvNs64 : 2, kOcc = D == 64 ? kDkvOcc64 : 2;
    const int grid = attn_grid(a, B, kCUs * kOcc, true);
    if (a.by_turns.turns > 0)
      hipLaunchKernelGGL((attn_bwd_dkv_bf16<D, DT, kNs, kOcc, WIDE, true>), dim3(grid), dim3(kAT), 0, st, a);
    else
      hipLaunchKernelGGL((attn_bwd_dkv_bf16<D, DT, kNs, kOcc, WIDE, false>), dim3(grid), dim3(kAT), 0, st, a);
  }
  return hipGetLastError();
}
template <int D, int DT>
static hipError_t launch_bwd(const AttnArgs& a, int B, hipStream_t st) {
  return a.ss < kWideStride ? launch_bwd_t<D, DT, false>(a, B, st) : launch_bwd_t<D, DT, true>(a, B, st);
}

// dt: element type (kBf16 or kF16)
hipError_t launch_attn_fwd_bf16(int dt, int D, int B, const AttnArgs& a, hipStream_t st) {
  if (dt == kF16) return D == 64 ? launch_fwd<64, kF16>(a, B, st) : launch_fwd<128, kF16>(a, B, st);
  return D == 64 ? launch_fwd<64, kBf16>(a, B, st) : launch_fwd<128, kBf16>(a, B, st);
}
hipError_t launch_attn_bwd_bf16(int dt, int D, int B, const AttnArgs& a, hipStream_t st) {
  if (dt == kF16) return D == 64 ? launch_bwd<64, kF16>(a, B, st) : launch_bwd<128, kF16>(a, B, st);
  return D == 64 ? launch_bwd<64, kBf16>(a, B, st) : launch_bwd<128, kBf16>(a, B, st);
}

}  // namespace lx
