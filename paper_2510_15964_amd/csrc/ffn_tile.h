// The tile product of the 16-bit FFN kernels (gfx950): a workgroup multiplies 64*TM token rows with
// 64*TN weight rows, 64 of the contraction index per step, through the transfer ring of ffn_ring.h's
// layout (128-byte LDS rows, 16-byte slots XOR-swizzled with the row index).
//
// One barrier per step, and operands of the next phase on their way from LDS to registers while the
// matrix instructions of the current one run (a plain "barrier, read, multiply" step leaves the matrix
// cores idle for as long as all wavefronts of the CU read their operands at once: 256 x 256 x 64 steps
// took 1800 ns that way).  A step is cut into PH phases; before the last phase of step s a wavefront has
// all its operands of the step in registers, so past the barrier that also tells it that step s + 1 has
// landed it may refill the stage of step s.
//
// The matrix instruction is the 16x16x32 one.  The 32x32x16 one reads half the operand bytes per product, but its
// accumulators cross the register file once per 16 of the contraction index instead of 32, and power bounds the wide
// tiles: on registers, with normally distributed operands, it reaches 1680 TFLOP/s and the 16x16x32 one 1930 (2300 and
// 2340 with zeros).  Bits are the same.  4 x 4 tiles, first / second product, us: 4096 tokens, d = 5120, all 320 blocks 698 / 918
// -> 638 / 857, 3840 tokens, 96 blocks 220 / 249 -> 206 / 233, 8192 tokens, d = 4096, 64 blocks 213 / 202 -> 194 / 186; over the 52
// launches of profiles/ffn_tile_sweep.txt, small ones most of them, 4 x 4 tiles 3 % less time, 2 x 4, 2 x 2 and 1 x 4 ones 2, the others 1,
// which is also what two runs of the tile that did not change are apart.  Tile11, the 1 x 1 tile of a ring of four stages, keeps the larger
// one: it is a chain of few instructions, and with them half as many it takes 1.3 % less.  (Three of its kind to a CU, Tile11Many, take as
// long with either: 30 launches 0.975 - 1.05, 1.00 in the mean.)
#pragma once
#include <type_traits>

#include "ffn_ring.h"

namespace lx {

// TM x TN groups of 64 token / weight rows, WM x WN wavefronts over them, NST ring stages, PH phases per
// step, MINW wavefronts per SIMD the registers have to leave room for, MF rows of the matrix instruction's tile (16; 32 for
// Tile11, and for a ring of one stage, which has no registers for slices 32 deep).
template <int MF>
struct AccOf {
  using T = f32x4;
};
template <>
struct AccOf<32> {
  using T = f32x16;
};
template <int TM_, int TN_, int WM_, int WN_, int NST_, int PH_, int MINW_ = 2, int MF_ = 16>
struct Tile {
  static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, NST = NST_, PH = PH_, kMinWaves = MINW_, MF = MF_;
  static constexpr int kWaves = WM * WN, kTileThreads = kWaves * kWave;
  static constexpr int kElems = 64 * (TM + TN) * kBK;        // one stage
  static constexpr int kIss = 8 * (TM + TN) / kWaves;        // transfer instructions per wavefront and stage
  static constexpr int kIssA = 8 * TM / kWaves;              // the first of them bring token rows
  static constexpr int kPer = 64 / MF;                       // accumulators along 64 rows
  static constexpr int NI = kPer * TN / WN, TI = kPer * TM / WM;      // MF x MF accumulators of a wavefront
  static constexpr int kSlices = MF / 16 * 2, KS = kSlices / PH;      // slices of a step, 512 / MF deep; of a phase
  using Acc = typename AccOf<MF>::T;
  static_assert(8 * TM % kWaves == 0 && 8 * TN % kWaves == 0 && (kWaves == 4 || kWaves == 8), "wavefronts");
  static_assert(NI >= 1 && TI >= 1 && (NST == 1 ? PH == kSlices : PH == 1 || PH == 2), "wave tile");
};
template <int DT>
__device__ __forceinline__ f32x16 mfma(uint4 a, uint4 b, f32x16 c) { return mfma32<DT>(a, b, c); }
template <int DT>
__device__ __forceinline__ f32x4 mfma(uint4 a, uint4 b, f32x4 c) { return mfma16<DT>(a, b, c); }

template <class Tl>
struct Frag {
  uint4 a[Tl::KS][Tl::NI], b[Tl::KS][Tl::TI];   // weight rows, token rows
};

// What the 16-byte slots of a stage's row are XORed with, so that the lanes of an operand read that are served together
// (0 .. 3, 12 .. 15 and 20 .. 27 of a half wavefront, and the others) meet in no bank: 16 rows of two slots, or 32 of one.
template <class Tl>
__device__ __forceinline__ int tile_swz(int row) {
  return (Tl::MF == 16 ? row : row ^ row >> 3) & 7;
}
// LDS byte offsets of this lane's operand rows inside a stage, per slice.
template <class Tl>
struct LaneOff {
  uint32_t a[Tl::kSlices], b[Tl::kSlices];
  __device__ __forceinline__ LaneOff(int wm, int wn) {
    const int lane = threadIdx.x % kWave, r = lane % Tl::MF;
    const int ra = Tl::MF * Tl::NI * wn + r, rb = Tl::MF * Tl::TI * wm + r;
#pragma unroll
    for (int k = 0; k < Tl::kSlices; ++k) {
      const int seg = k * (kWave / Tl::MF) + lane / Tl::MF;
      a[k] = (uint32_t)((64 * Tl::TM + ra) * 128 + ((seg ^ tile_swz<Tl>(ra)) << 4));
      b[k] = (uint32_t)(rb * 128 + ((seg ^ tile_swz<Tl>(rb)) << 4));
    }
  }
};

// Operand number x of phase ph of the stage at LDS address `stage`.  (Every other group of 32 rows has bit 2 of
// tile_swz flipped, which is a slice two further on.)
template <class Tl>
__device__ __forceinline__ void read_operand(Frag<Tl>& f, const LaneOff<Tl>& lo, uint32_t stage, int ph, int x) {
  constexpr int per = Tl::NI + Tl::TI;
  const int e = x / per, y = x % per, k = ph * Tl::KS + e, i = y < Tl::NI ? y : y - Tl::NI;
  const int at = Tl::MF == 32 ? k ^ 2 * (i & 1) : k;
  if (y < Tl::NI)
    f.a[e][i] = lds_read16(stage + lo.a[at] + i * (Tl::MF * 128));
  else
    f.b[e][i] = lds_read16(stage + lo.b[at] + i * (Tl::MF * 128));
}

// One phase: the products of `cur`, meanwhile the operands of phase ph of the stage at `stage` go to
// `nxt` and, with DMA, the transfers of a later step are issued (src.dma(u, LDS address)).
template <class Tl, int DT, bool DMA, class Src>
__device__ __forceinline__ void tile_phase(const Frag<Tl>& cur, Frag<Tl>& nxt, const LaneOff<Tl>& lo,
                                           uint32_t stage, int ph, Src& src, uint32_t dma_lds,
                                           typename Tl::Acc (&acc)[Tl::NI][Tl::TI]) {
  constexpr int NM = Tl::KS * Tl::NI * Tl::TI, NR = Tl::KS * (Tl::NI + Tl::TI), ND = Tl::kIss;
  // operand reads over the first three quarters of the matrix instructions, transfers over all of them
  constexpr int RM = NM * 3 / 4 > 0 ? NM * 3 / 4 : 1;
  int m = 0, xr = 0, xd = 0;
#pragma unroll
  for (int e = 0; e < Tl::KS; ++e)
#pragma unroll
    for (int ni = 0; ni < Tl::NI; ++ni)
#pragma unroll
      for (int ti = 0; ti < Tl::TI; ++ti) {
        const int r_to = m + 1 >= RM ? NR : ((m + 1) * NR + RM - 1) / RM;
#pragma unroll
        for (int z = 0; z < NR; ++z)
          if (z >= xr && z < r_to) read_operand<Tl>(nxt, lo, stage, ph, z);
        xr = r_to;
        if constexpr (DMA) {
          const int d_to = ((m + 1) * ND + NM - 1) / NM;
#pragma unroll
          for (int z = 0; z < ND; ++z)
            if (z >= xd && z < d_to) src.dma(z, dma_lds);
          xd = d_to;
        }
        acc[ni][ti] = mfma<DT>(cur.a[e][ni], cur.b[e][ti], acc[ni][ti]);
        __builtin_amdgcn_sched_barrier(0);
        ++m;
      }
}

// run_tile with a ring of one stage: a workgroup waits for the transfers of its next step, and the others that such a stage
// leaves room for on the CU compute meanwhile.  A wavefront issues the first src.live() transfer instructions of a step, and
// multiplies if src.busy(wn): an item may have fewer weight groups than the tile.
template <class Tl, int DT, class Src>
__device__ __forceinline__ void run_tile_one_stage(int nsteps, uint32_t ring, int wm, int wn, Src& src,
                                                   typename Tl::Acc (&acc)[Tl::NI][Tl::TI]) {
  if (nsteps <= 0) return;
  const LaneOff<Tl> lo(wm, wn);
  const uint32_t to = ring + (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave) * 1024;
  Frag<Tl> f[2];
  auto read = [&](int ph) {
#pragma unroll
    for (int x = 0; x < Tl::NI + Tl::TI; ++x) read_operand<Tl>(f[ph % 2], lo, ring, ph, x);
  };
  const int live = src.live();
  auto issue = [&](int s) {
    src.begin(s);
#pragma unroll
    for (int u = 0; u < Tl::kIss; ++u)
      if (u < live) src.dma(u, to);
  };
  issue(0);
  if (!src.busy(wn)) {       // the two barriers of a step and its transfers
    for (int s = 0; s < nsteps; ++s) {
      wait_vmcnt<0>();
      lds_barrier();
      lds_barrier();
      if (s + 1 < nsteps) issue(s + 1);
    }
    return;
  }
  for (int s = 0; s < nsteps; ++s) {
    wait_vmcnt<0>();
    lds_barrier();
    read(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ph = 0; ph < Tl::PH; ++ph) {
      if (ph + 1 < Tl::PH) {
        read(ph + 1);
      } else {
        lds_barrier();     // every wavefront has the step's operands in registers
        if (s + 1 < nsteps) issue(s + 1);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ni = 0; ni < Tl::NI; ++ni)
#pragma unroll
        for (int ti = 0; ti < Tl::TI; ++ti) acc[ni][ti] = mfma<DT>(f[ph % 2].a[0][ni], f[ph % 2].b[0][ti], acc[ni][ti]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// acc[ni][ti] += sum over nsteps steps.  src.begin(s) prepares the sources of step s, src.dma(u, lds)
// issues its transfer instruction u to the stage at that LDS address.
template <class Tl, int DT, class Src>
__device__ __forceinline__ void run_tile_ring(int nsteps, uint32_t ring, int wm, int wn, Src& src,
                                         typename Tl::Acc (&acc)[Tl::NI][Tl::TI]) {
  constexpr int NST = Tl::NST, NISS = Tl::kIss;
  static_assert(NST >= 2 && NISS * (NST - 1) < 64, "ring depth");
  if (nsteps <= 0) return;
  const LaneOff<Tl> lo(wm, wn);
  constexpr uint32_t kStage = Tl::kElems * 2;
  const uint32_t wave_lds = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x / kWave) * 1024;
#pragma unroll
  for (int p = 0; p < NST; ++p)
    if (p < nsteps) {
      src.begin(p);
#pragma unroll
      for (int u = 0; u < NISS; ++u) src.dma(u, ring + p * kStage + wave_lds);
    }
  // step 0 has landed when at most the transfers of the others are outstanding
  if (nsteps >= NST)
    wait_vmcnt<NISS * (NST - 1)>();
  else
    wait_tail<NISS, NST - 2>(nsteps - 1);
  lds_barrier();
  Frag<Tl> f0, f1;
#pragma unroll
  for (int x = 0; x < Tl::KS * (Tl::NI + Tl::TI); ++x) read_operand<Tl>(f0, lo, ring, 0, x);
  __builtin_amdgcn_sched_barrier(0);
  int stage = 0;       // of step s
  // everything of step s but its last phase; then the last one, behind the barrier
  auto step = [&](int s, auto dma, Frag<Tl>& fa, Frag<Tl>& fb) {
    constexpr bool D = decltype(dma)::value;
    const uint32_t here = ring + stage * kStage;
    stage = stage + 1 == NST ? 0 : stage + 1;
    const uint32_t next = ring + stage * kStage;
    if constexpr (Tl::PH == 2) tile_phase<Tl, DT, false>(fa, fb, lo, here, 1, src, 0u, acc);
    // step s + 1 has landed: at most the transfers of steps s + 2 .. s + NST - 1 are outstanding
    if constexpr (D) {
      wait_vmcnt<NISS * (NST - 2)>();
    } else {
      const int younger = nsteps - 2 - s;
      if (younger >= NST - 2)
        wait_vmcnt<NISS * (NST - 2)>();
      else
        wait_tail<NISS, NST - 3>(younger > 0 ? younger : 0);
    }
    lds_barrier();
    if constexpr (D) src.begin(s + NST);
    if constexpr (Tl::PH == 2)
      tile_phase<Tl, DT, D>(fb, fa, lo, next, 0, src, here + wave_lds, acc);
    else
      tile_phase<Tl, DT, D>(fa, fb, lo, next, 0, src, here + wave_lds, acc);
  };
  int s = 0;
  if constexpr (Tl::PH == 2) {
    for (; s + NST < nsteps; ++s) step(s, std::true_type{}, f0, f1);
    for (; s < nsteps; ++s) step(s, std::false_type{}, f0, f1);
  } else {      // the two operand sets swap roles every step
    for (; s + 1 + NST < nsteps; s += 2) {
      step(s, std::true_type{}, f0, f1);
      step(s + 1, std::true_type{}, f1, f0);
    }
    if (s + NST < nsteps) {
      step(s, std::true_type{}, f0, f1);
      ++s;
      for (; s < nsteps; s += 2) {
        step(s, std::false_type{}, f1, f0);
        if (s + 1 < nsteps) step(s + 1, std::false_type{}, f0, f1);
      }
    } else {
      for (; s < nsteps; s += 2) {
        step(s, std::false_type{}, f0, f1);
        if (s + 1 < nsteps) step(s + 1, std::false_type{}, f1, f0);
      }
    }
  }
}

template <class Tl, int DT, class Src>
__device__ __forceinline__ void run_tile(int nsteps, uint32_t ring, int wm, int wn, Src& src,
                                         typename Tl::Acc (&acc)[Tl::NI][Tl::TI]) {
  if constexpr (Tl::NST == 1)
    run_tile_one_stage<Tl, DT>(nsteps, ring, wm, wn, src, acc);
  else
    run_tile_ring<Tl, DT>(nsteps, ring, wm, wn, src, acc);
}

// The quarter tile: 32 token rows times 32 weight rows by ONE wavefront that multiplies and two that transfer, the one the
// token rows, the other the weight rows.  For launches of few tiles: a 64 x 64 tile of four wavefronts takes 390 clocks per
// step, of which the CU's memory path is busy for 256 with its 16 KB; four quarters on four CUs have 128 each, as
// many as the chain of a step's matrix instructions takes, if nothing else has to be issued between them (one wavefront
// that does it all is 3 - 8 % faster than the 64 x 64 tile).  By that tile and by quarters, us, first / second product: 192
// tokens, d = 768, 15 blocks 6.6 / 6.1 -> 5.4 / 5.2; 64, 1792, 44 9.5 / 11.2 -> 7.5 / 9.2; 64, 2560, 16 12.1 / 5.8 -> 9.3 / 5.1; 64,
// 4288, 14 15.3 / 5.6 -> 12.3 / 4.9; 64 tokens, d = 2496,
// 92 blocks 11.5 / 19.8 -> 11.1 / 15.4; 192 tokens, d = 832, a list per tile, 128 tiles 7.8 / 5.2 -> 6.0 / 4.4.
struct Quarter {
  static constexpr int kWaves = 3, kTileThreads = kWaves * kWave;
  static constexpr int kElems = 64 * kBK;               // of a step: 32 token rows, 32 weight rows, laid out like the others
  static constexpr int kIss = 4;                        // transfer instructions of a wavefront per step
};
// The transfers of one operand's 32 rows: this lane's offsets from their first element, rows ld elements apart (32 of
// them within 4 GiB: quarters_pay); `second`: the weight rows, which come after the token rows in a stage.
struct QuarterRows {
  uint32_t voff[4];
  __device__ __forceinline__ void init(long long ld, bool second) {
    const int lane = threadIdx.x % kWave, lr = lane / 8;
#pragma unroll
    for (int u = 0; u < 4; ++u) voff[u] = (uint32_t)((8 * u + lr) * ld * 2 + (((lane % 8) ^ lr ^ (second ? 4 + u : u)) << 4));
  }
  __device__ __forceinline__ void issue(const uint16_t* first, uint32_t lds) const {
    dma16_s_at<0>(first, voff[0], lds);
    dma16_s_at<1024>(first, voff[1], lds);
    dma16_s_at<2048>(first, voff[2], lds);
    dma16_s_at<3072>(first, voff[3], lds);
  }
};
// acc += sum over nsteps steps, in the order of run_tile, in the first wavefront.  NST stages of two steps each.
// src.issue(step, LDS address) starts the calling wavefront's transfers of a step (steps past the end: the last one again).
template <int DT, int NST, class Src>
__device__ __forceinline__ void run_quarter(int nsteps, uint32_t ring, Src& src, f32x16& acc) {
  constexpr uint32_t kStep = Quarter::kElems * 2, kStage = 2 * kStep;
  const int pairs = (nsteps + 1) / 2, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (wave > 0) {
    auto issue = [&](int d) {
      const uint32_t to = ring + (uint32_t)(d % NST) * kStage;
      src.issue(2 * d, to);
      src.issue(2 * d + 1 < nsteps ? 2 * d + 1 : 2 * d, to + kStep);
    };
    for (int d = 0; d < NST - 1 && d < pairs; ++d) issue(d);
    for (int d = 0; d < pairs; ++d) {
      // pair d has landed; behind the barrier pair d - 1 is in the registers of the first wavefront
      const int younger = pairs - 1 - d;
      wait_tail<2 * Quarter::kIss, NST - 2>(younger < NST - 2 ? younger : NST - 2);
      lds_barrier();
      if (d + NST - 1 < pairs) issue(d + NST - 1);
    }
    return;
  }
  const int lane = threadIdx.x % kWave, r = lane % 32, h2 = lane / 32, sw = (r & 7) ^ (r >> 3);
  uint32_t a_off[4], b_off[4];       // weight rows, token rows
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    b_off[k] = ring + (uint32_t)(r * 128 + (((2 * k + h2) ^ sw) << 4));
    a_off[k] = ring + (uint32_t)((32 + r) * 128 + (((2 * k + h2) ^ sw ^ 4) << 4));
  }
  struct Operands {
    uint4 a[8], b[8];
  } f[2];
  auto read = [&](Operands& o, int d) {
    const uint32_t st = (uint32_t)(d % NST) * kStage;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      o.a[k] = lds_read16(a_off[k % 4] + st + k / 4 * kStep);
      o.b[k] = lds_read16(b_off[k % 4] + st + k / 4 * kStep);
    }
  };
  auto multiply = [&](const Operands& o) {
#pragma unroll
    for (int k = 0; k < 8; ++k) acc = mfma32<DT>(o.a[k], o.b[k], acc);
  };
  if (pairs > 0) {
    lds_barrier();
    read(f[0], 0);
  }
  int d = 1;
  for (; d + 1 < pairs; d += 2) {
    lds_barrier();                   // (waits for the reads of pair d - 1)
    read(f[1], d);
    __builtin_amdgcn_sched_barrier(0);
    multiply(f[0]);
    lds_barrier();
    read(f[0], d + 1);
    __builtin_amdgcn_sched_barrier(0);
    multiply(f[1]);
  }
  if (d < pairs) {
    lds_barrier();
    read(f[1], d);
    __builtin_amdgcn_sched_barrier(0);
    multiply(f[0]);
    f[0] = f[1];
  }
  const int last = pairs > 0 ? nsteps - 2 * (pairs - 1) : 0;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (last > 0) acc = mfma32<DT>(f[0].a[k], f[0].b[k], acc);
  if (last > 1) {
#pragma unroll
    for (int k = 4; k < 8; ++k) acc = mfma32<DT>(f[0].a[k], f[0].b[k], acc);
  }
}

}  // namespace lx
