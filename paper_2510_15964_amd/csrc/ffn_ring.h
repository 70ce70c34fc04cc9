// The global -> LDS transfer ring of the predictor and LoRA kernels (gfx950); the FFN kernels' own
// pipeline (ffn_tile.h) has the same LDS layout.
//
// Data movement: global memory -> LDS directly (global_load_lds, 16 bytes per lane, no registers
// in between), a ring of stages; the loads of the next K-steps are in flight while the MFMAs of
// the current one run.  LDS rows are 128 bytes (one 64-element K-chunk of one row), unpadded (a
// DMA instruction writes 1 KiB = 8 rows contiguously); the 16-byte slots of a row are
// XOR-swizzled with the row index so that the MFMA operand reads of 16 consecutive rows hit
// distinct banks.
#pragma once
#include "lx_dev.h"
#include "lx_launch.h"

namespace lx {

constexpr int kFW = 8;             // wavefronts per workgroup
constexpr int kThreads = kFW * kWave;
constexpr int kBK = 64;            // K-chunk per step: 64 bf16 = 128 bytes per row
constexpr int kRowsB = 64;         // shared operand (token rows)

__device__ __forceinline__ int swz(int row) { return (row ^ (row >> 3)) & 7; }

// One stage = NISS DMA instructions per wave.
// Instruction u of wave w fills stage rows 8g .. 8g+7 with g = w + kFW*u (g < 8: the 64 shared
// rows, then the weight blocks); lane l brings the 16-byte slot l%8 of row 8g + l/8.  src[u]
// already points at this lane's (row, swizzled segment); offB / offA are the element offsets of
// the current K-step for the shared rows (the first NSH instructions of a wave) and the weight
// rows.
template <int NISS, int NSH>
__device__ __forceinline__ void issue_stage(uint16_t* stage, const uint16_t* const (&src)[NISS], long long offB,
                                            long long offA) {
  const uint32_t base = lds_addr(stage) + (threadIdx.x / kWave) * 1024;
#pragma unroll
  for (int u = 0; u < NISS; ++u) dma16(src[u] + (u < NSH ? offB : offA), base + u * (kFW * 1024));
}

// Pipeline over nsteps K-steps through a ring of NST stages: while step s is multiplied, the
// DMA of steps s+1 .. s+NST-1 is in flight (what bounds these kernels is how many bytes a CU
// keeps in flight towards memory, so the ring is as deep as LDS allows).  offs(s, offB, offA)
// yields the element offsets of step s.  A wave first waits until its own DMA of step s has
// landed (its loads retire in order, so the loads of the younger steps may stay outstanding),
// the barrier then guarantees that the whole stage is there and that nobody still reads the
// stage about to be refilled.
// Wait until at most NISS * y DMA instructions are outstanding, for a run-time y <= M (the last
// steps of a ring, when fewer stages than its depth are in flight).
template <int NISS, int M>
__device__ __forceinline__ void wait_tail(int y) {
  if constexpr (M <= 0) {
    wait_vmcnt<0>();
  } else {
    if (y == M)
      wait_vmcnt<NISS * M>();
    else
      wait_tail<NISS, M - 1>(y);
  }
}

// step(stage pointer) is the multiplication of one landed stage; a stage holds SE elements.
template <int NST, int NISS, int SE, int NSH = 1, class Offs, class Step>
__device__ __forceinline__ void run_ring_of(int nsteps, const uint16_t* const (&src)[NISS], Offs offs, uint16_t* ring,
                                            Step step) {
  static_assert(NST >= 2 && NISS * (NST - 2) < 64, "ring depth");
  auto issue = [&](int s, int stage) {
    long long ob, oa;
    offs(s, ob, oa);
    issue_stage<NISS, NSH>(ring + stage * SE, src, ob, oa);
  };
#pragma unroll
  for (int p = 0; p < NST - 1; ++p)
    if (p < nsteps) issue(p, p);
  int stage = 0;
  for (int s = 0; s < nsteps; ++s) {
    const int younger = nsteps - 1 - s;   // steps after s whose DMA has been issued: min(., NST-2)
    if (younger >= NST - 2)
      wait_vmcnt<NISS * (NST - 2)>();
    else
      wait_tail<NISS, NST - 3>(younger);
    lds_barrier();
    if (s + NST - 1 < nsteps) issue(s + NST - 1, stage == 0 ? NST - 1 : stage - 1);
    step(ring + stage * SE);
    stage = stage + 1 == NST ? 0 : stage + 1;
  }
}

// Host side: calls fn<kF16> or fn<kBf16> according to the run-time element type `dt`.
#define LX_BY_DT(fn, ...) (dt == kF16 ? fn<kF16>(__VA_ARGS__) : fn<kBf16>(__VA_ARGS__))

}  // namespace lx
