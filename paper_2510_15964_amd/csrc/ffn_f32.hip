// fp32 sparse FFN kernels (Sec. VI-B neuron-centric tiled products), used for the fp32 correctness
// configuration.  fp32 operands and accumulation throughout, on the 16x16x4 fp32 MFMA, whose rate is
// that of the vector unit, but an operand element is read once per 16 products instead of once per
// one to two.
//
// Two kernel shapes serve all four products:
//   sdd: out block (i, j) = A_i [TB x K] . B_j [TB x K]^T for every listed
//        (token tile i, neuron block j); epilogue ReLU (+bias) or gating by the
//        stored activation sign.          (up-projection, dH)
//   dsd: out tile  = sum over listed j of Act_ij [TB x TB] . B[:, j-block]^T
//        (down-projection, dX), the contraction runs over active blocks only.
//
// The output tile of a workgroup is as small as a list block (32 or 64 tokens x 32 or 64 columns), which fills the
// chip at the sizes this configuration runs at.  What bounds a product is the chain of a wavefront's matrix
// instructions: 8 clocks per term of the sum whatever the instruction (16x16x1 with four blocks: 32 clocks a term),
// and few SIMDs have more than one or two chains.  So a wavefront owns 16 columns of 16 tokens (32 with 64 x 64 blocks),
// the wavefronts of a workgroup share a ring of stages in LDS, 32 terms of all rows each, and the operands of the next
// stage are read while the matrix instructions of the current one run, one barrier per stage.  Where the order of the
// sum is free, two sets of wavefronts take half of it each.  Four stages: deeper rings cost resident workgroups and
// won nothing (six: 13 -> 15.5 us for the second product below).
// The instruction adds its four terms one after the other, each with one rounding: a chain of them is the same sum, to
// the last bit, as one fused multiply-add per term in ascending order (tested).
// Up / gate / second product, us, against wavefronts of 32 x 32 (16x16x1 and 32x32x2) with stages of their own:
//   512 tokens, 768 -> 3072, 30 % of 32 x 32 blocks    22 / 17.3 / 16 -> 12.4 / 12.2 / 12.8
//   160 tokens, 1024 -> 4096, 7 %                      25 / 8.4 / 5.0 -> 9.8 / 8.7 / 4.9
//   96 tokens, 544 -> 2176, 15 %                       15 / 6.7 / 5.0 -> 6.6 / 6.3 / 4.9
// and forward / backward calls: 1024 tokens, 1024 -> 4096, 60 % 152 / 129 -> 98 / 108; 64 x 64 blocks of the same 135 /
// 133 -> 105 / 114; 4096 tokens, 2048 -> 8192, 30 % of 64 x 64 blocks 995 / 907 -> 762 / 730 (112 TFLOP/s; the vendor
// library's GEMM reaches 150).  Against sums in 64 bits the errors are those of before (2.7e-7 and 1.3e-7 of the norm).
#include <type_traits>

#include "ffn_ring.h"

namespace lx {

constexpr int kF32Batch = 32;      // contraction elements of a stage: a 128-byte row piece, eight MFMAs of depth four

// Stages of RA token rows and RW weight rows, NST of them; KS parts of the contraction index, each with wavefronts and a
// ring of its own.
template <int RA_, int RW_, int NST_, int KS_>
struct TileF32 {
  static constexpr int RA = RA_, RW = RW_, NST = NST_, KS = KS_;
  static constexpr int TA = RA / 32;                       // groups of 16 tokens of a wavefront
  static constexpr int kWaves = 2 * (RW / 16);             // of a part
  static constexpr int kTileThreads = KS * kWaves * kWave;
  static constexpr int kStage = (RA + RW) * 128, kRing = NST * kStage;           // bytes
  static constexpr int kIssA = RA / 8 / kWaves, kIss = (RA + RW) / 8 / kWaves;   // transfer instructions per wavefront
  static_assert(RA / 8 % kWaves == 0 && RW / 8 % kWaves == 0, "transfers");
};
template <int TB>
using UpF32 = TileF32<TB, TB, 4, 1>;
template <int TB>
using GateF32 = TileF32<TB, TB, 4, 2>;
template <int TB>
using DsdF32 = TileF32<TB, 32, 4, 2>;

// Instruction u of wavefront w brings the stage rows 8g .. 8g+7 with g = w + kWaves*u (token rows first), lane l the
// 16-byte slot l % 8 of row 8g + l/8: a wave-uniform base per instruction and a 32-bit offset per lane, which reaches
// over row strides below kWideF32.  WIDE, for longer ones: a 64-bit offset per lane.
constexpr int kWideF32 = 1 << 27;      // elements; 7 rows of 2^29 bytes and a row's 128 fit 32 bits
template <class Tl, bool WIDE>
struct SourcesF32 {
  using Off = std::conditional_t<WIDE, long long, uint32_t>;
  const float* base[Tl::kIss];
  Off voff[Tl::kIss];
  uint32_t wave_lds;
  __device__ __forceinline__ SourcesF32(const float* A, long long lda, const float* W, long long ldw) {
    const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) % Tl::kWaves;
    wave_lds = wave * 1024;
#pragma unroll
    for (int u = 0; u < Tl::kIss; ++u) {
      const bool is_a = u < Tl::kIssA;
      const long long ld = is_a ? lda : ldw;
      const int first = 8 * (wave + Tl::kWaves * u) - (is_a ? 0 : Tl::RA);
      base[u] = (is_a ? A : W) + first * ld;
      voff[u] = (Off)((lane / 8) * ld * 4) + (((lane % 8) ^ swz(first + lane / 8)) << 4);
    }
  }
  // oa, ow: elements from the operands' first rows; stage: LDS address
  __device__ __forceinline__ void issue(uint32_t stage, long long oa, long long ow) const {
#pragma unroll
    for (int u = 0; u < Tl::kIss; ++u) {
      const float* b = base[u] + (u < Tl::kIssA ? oa : ow);
      const uint32_t to = stage + wave_lds + u * (Tl::kWaves * 1024);
      if constexpr (WIDE)
        dma16(reinterpret_cast<const char*>(b) + voff[u], to);
      else
        dma16_s(b, voff[u], to);
    }
  }
};

__device__ __forceinline__ float lds_readf(uint32_t addr) {
  return *reinterpret_cast<const LX_AS3 float*>((uintptr_t)addr);
}
// (volatile: the compiler would read the four elements one by one)
__device__ __forceinline__ f32x4 lds_readf4(uint32_t addr) {
  return *reinterpret_cast<const volatile LX_AS3 f32x4*>((uintptr_t)addr);
}
// This lane's operands of a step of eight MFMAs: row lane%16 of the wavefront's groups of 16.  ASCENDING: MFMA m takes
// the elements 4m .. 4m+3, one per 16 lanes, so that its sum goes on in ascending order; read one by one, two lanes to
// a bank.  Otherwise MFMA 4h + e takes the elements 16h + 4g + e (g = lane/16): 16 bytes per read.  `lo` are the
// addresses in the first stage; `stage`, bytes from there, is a constant that goes into the instructions.  The 16-byte
// slots of a row are XOR-swizzled with the row; rows 16 further on have bit 1 of the slot flipped.
template <class Tl, bool ASCENDING>
struct OperandsF32;
template <class Tl>
struct OperandsF32<Tl, true> {
  struct Lane {
    uint32_t a[8], w[8];
    __device__ __forceinline__ Lane(uint32_t ring, int wa, int ww) {
      const int lane = threadIdx.x % kWave, g = lane / 16, ra = 16 * Tl::TA * wa + lane % 16, rw = 16 * ww + lane % 16;
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        a[m] = ring + (uint32_t)(ra * 128 + ((m ^ swz(ra)) << 4) + 4 * g);
        w[m] = ring + (uint32_t)((Tl::RA + rw) * 128 + ((m ^ swz(rw)) << 4) + 4 * g);
      }
    }
  };
  float va[Tl::TA][8], vw[8];
  __device__ __forceinline__ void read(const Lane& lo, int stage, int m) {     // what MFMA m needs
    vw[m] = lds_readf(lo.w[m] + stage);
#pragma unroll
    for (int t = 0; t < Tl::TA; ++t) va[t][m] = lds_readf(lo.a[m ^ (2 * t)] + (stage + t * 2048));
  }
  __device__ __forceinline__ float a(int t, int m) const { return va[t][m]; }
  __device__ __forceinline__ float w(int m) const { return vw[m]; }
};
template <class Tl>
struct OperandsF32<Tl, false> {
  struct Lane {
    uint32_t a[Tl::TA][2], w[2];
    __device__ __forceinline__ Lane(uint32_t ring, int wa, int ww) {
      const int lane = threadIdx.x % kWave, g = lane / 16, rw = 16 * ww + lane % 16;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int t = 0; t < Tl::TA; ++t) {
          const int ra = 16 * (Tl::TA * wa + t) + lane % 16;
          a[t][h] = ring + (uint32_t)(ra * 128 + (((4 * h + g) ^ swz(ra)) << 4));
        }
        w[h] = ring + (uint32_t)((Tl::RA + rw) * 128 + (((4 * h + g) ^ swz(rw)) << 4));
      }
    }
  };
  f32x4 va[Tl::TA][2], vw[2];
  __device__ __forceinline__ void read(const Lane& lo, int stage, int m) {     // spread over the MFMAs
    if (m % 4 == 0) vw[m / 4] = lds_readf4(lo.w[m / 4] + stage);
#pragma unroll
    for (int t = 0; t < Tl::TA; ++t)
      if (m % 4 == 1 + t) va[t][m / 4] = lds_readf4(lo.a[t][m / 4] + stage);
  }
  __device__ __forceinline__ float a(int t, int m) const { return va[t][m / 4][m % 4]; }
  __device__ __forceinline__ float w(int m) const { return vw[m / 4][m % 4]; }
};

// acc[t] = sum over n steps, element v of lane l: token 16t + l%16, column 4*(l/16) + v of the wavefront's groups.
// off(s, a, w): element offsets of step s from the sources; ring: LDS address of the part's stages; the parts of a
// workgroup go through `most` >= n steps.  ASCENDING: one term after the other, in ascending order; otherwise the sums of
// the even and of the odd steps, added at the end.
// The steps are unrolled over the stages, so that a step has no vector instruction but the LDS reads and the MFMAs:
// every other one holds up the chain (16 additions for the addresses took a step from 290 clocks to 500).
template <class Tl, bool ASCENDING, class Src, class Off>
__device__ __forceinline__ void run_f32(int n, int most, uint32_t ring, const Src& src, int wa, int ww, Off off,
                                        f32x4 (&acc)[Tl::TA]) {
  constexpr int NST = Tl::NST, SUMS = ASCENDING ? 1 : 2;
  using Ops = OperandsF32<Tl, ASCENDING>;
  static_assert(NST % 2 == 0, "two sets of operands");
  f32x4 sum[SUMS][Tl::TA];
#pragma unroll
  for (int x = 0; x < SUMS; ++x)
#pragma unroll
    for (int t = 0; t < Tl::TA; ++t) sum[x][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto issue = [&](int s, int stage) {
    long long oa, ow;
    off(s, oa, ow);
    src.issue(ring + stage * Tl::kStage, oa, ow);
  };
#pragma unroll
  for (int p = 0; p < NST; ++p)
    if (p < n) issue(p, p);
  wait_tail<Tl::kIss, NST - 1>(n <= 0 ? 0 : n < NST ? n - 1 : NST - 1);
  lds_barrier();
  const typename Ops::Lane lo(ring, wa, ww);
  Ops f[2];
#pragma unroll
  for (int m = 0; m < 8; ++m) f[0].read(lo, 0, m);
  for (int s0 = 0; s0 < most; s0 += NST)
#pragma unroll
    for (int q = 0; q < NST; ++q) {
      const int s = s0 + q;
      if (s >= most) break;
      // step s + 1 has landed; past the barrier every wavefront has the operands of step s in registers
      const int younger = n - 2 - s;
      if (younger >= NST - 2)
        wait_vmcnt<Tl::kIss * (NST - 2)>();
      else
        wait_tail<Tl::kIss, NST - 3>(younger > 0 ? younger : 0);
      lds_barrier();
      if (s >= n) continue;      // (the other part has steps left)
      if (s + NST < n) issue(s + NST, q);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        f[(q + 1) % 2].read(lo, (q + 1) % NST * Tl::kStage, m);      // (past the last step: an old stage, not used)
#pragma unroll
        for (int t = 0; t < Tl::TA; ++t)
          sum[q % SUMS][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[q % 2].w(m), f[q % 2].a(t, m), sum[q % SUMS][t], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
  for (int t = 0; t < Tl::TA; ++t) acc[t] = ASCENDING ? sum[0][t] : sum[0][t] + sum[SUMS - 1][t];
}
// Adds the second part's sums to the first one's, over the rings; true in the wavefronts that hold the result.
template <class Tl>
__device__ __forceinline__ bool fold_parts_f32(float* ring, f32x4 (&acc)[Tl::TA]) {
  static_assert(Tl::KS == 2, "two parts");
  const int wave = threadIdx.x / kWave % Tl::kWaves, part = threadIdx.x / kWave / Tl::kWaves;
  f32x4* area = reinterpret_cast<f32x4*>(ring) + wave * Tl::TA * kWave + threadIdx.x % kWave;
  lds_barrier();       // nobody reads the rings any more
  if (part == 1) {
#pragma unroll
    for (int t = 0; t < Tl::TA; ++t) area[t * kWave] = acc[t];
  }
  lds_barrier();
  if (part == 1) return false;
#pragma unroll
  for (int t = 0; t < Tl::TA; ++t) acc[t] += area[t * kWave];
  return true;
}

// Last of the `rows` list rows whose entries start at or before lp: 64 probes a round, one per lane.
__device__ __forceinline__ int row_of_entry(const int* __restrict__ row_ptr, int rows, int lp) {
  const int lane = threadIdx.x % kWave;
  int lo = 0, len = rows;
  while (len > 1) {
    const int each = (len + kWave - 1) / kWave, x = lane * each;
    const unsigned long long at = __ballot(x < len && row_ptr[lo + (x < len ? x : 0)] <= lp);
    const int k = __popcll(at) - 1;
    lo += k * each;
    len = min(each, len - k * each);
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

// Workgroup = (list entry, token tile of its group of gt), numbered in list order; the grid is the capacity's, and
// an eighth of the items that there are goes to each XCD, whose L2 then holds the rows of an eighth of the tokens.
// GATE false: out = max(A W^T + bias, 0), one fused multiply-add per term in ascending order: what the ReLU decides on
// does not depend on how the kernel is cut.  GATE: out = gate > 0 ? A W^T : 0.
template <int TB, bool GATE>
using SddF32 = std::conditional_t<GATE, GateF32<TB>, UpF32<TB>>;
template <int TB, bool GATE, bool WIDE>
__global__ __launch_bounds__((SddF32<TB, GATE>::kTileThreads), 2) void ffn_sdd_f32(
    const float* __restrict__ A, const float* __restrict__ W, const float* __restrict__ bias,
    const int* __restrict__ row_ptr, const int* __restrict__ col_idx, int rows, int gt, int K, int nnz_cap, int gx,
    float* __restrict__ out_act, const float* __restrict__ gate_act) {
  using Tl = SddF32<TB, GATE>;
  __shared__ __attribute__((aligned(1024))) float ring[Tl::KS * Tl::kRing / 4];
  const int w = blockIdx.y * gx + blockIdx.x;     // gx: the grid's first dimension
  // entries beyond the capacity of the list buffers are ignored
  const int first = min(row_ptr[0], nnz_cap), total = (min(row_ptr[rows], nnz_cap) - first) * gt, L = (total + 7) / 8;
  const int item = (w % 8) * L + w / 8;
  if (w / 8 >= L || item >= total) return;
  const int lp = first + item / gt, j = col_idx[lp];
  const int i = row_of_entry(row_ptr, rows, lp) * gt + item % gt;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int wa = wave % 2, ww = wave % Tl::kWaves / 2, part = wave / Tl::kWaves;
  // this lane's four columns of token t + 16x; activation blocks are stored as [entry][tile within the row's group]
  const int t = 16 * Tl::TA * wa + lane % 16, n = 16 * ww + 4 * (lane / 16);
  const long long o = ((long long)lp * gt + i % gt) * (TB * TB) + t * TB + n;
  f32x4 gate[Tl::TA];
  if (GATE && part == 0) {
#pragma unroll
    for (int x = 0; x < Tl::TA; ++x) gate[x] = *reinterpret_cast<const f32x4*>(gate_act + o + x * 16 * TB);
  }
  const int steps = K / kF32Batch, most = (steps + Tl::KS - 1) / Tl::KS, s_lo = part * most;
  const SourcesF32<Tl, WIDE> src(A + (long long)i * TB * K + s_lo * kF32Batch, K, W + (long long)j * TB * K + s_lo * kF32Batch, K);
  f32x4 acc[Tl::TA];
  run_f32<Tl, !GATE>(min(most, steps - s_lo), most, lds_addr(ring) + part * Tl::kRing, src, wa, ww,
                            [](int s, long long& oa, long long& ow) { oa = ow = (long long)s * kF32Batch; }, acc);
  if constexpr (Tl::KS > 1)
    if (!fold_parts_f32<Tl>(ring, acc)) return;
#pragma unroll
  for (int x = 0; x < Tl::TA; ++x) {
    f32x4 v = acc[x];
    if (!GATE && bias) v += *reinterpret_cast<const f32x4*>(bias + j * TB + n);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (GATE ? gate[x][e] : v[e]) > 0.f ? v[e] : 0.f;
    *reinterpret_cast<f32x4*>(out_act + o + x * 16 * TB) = v;
  }
}

// out[i-tile, n0..n0+31] = sum_s act[p_s] [TB x TB] . W[n0.., j_s*TB ..]^T  (+ bias).  The second part takes the second
// half of the entries.
template <int TB, bool WIDE>
__global__ __launch_bounds__(DsdF32<TB>::kTileThreads, 2) void ffn_dsd_f32(
    const float* __restrict__ act, const float* __restrict__ W, long long ldw,
    const float* __restrict__ bias, const int* __restrict__ row_ptr,
    const int* __restrict__ col_idx, int gt, int ncols_out, int nnz_cap,
    float* __restrict__ out) {
  using Tl = DsdF32<TB>;
  __shared__ __attribute__((aligned(1024))) float ring[Tl::KS * Tl::kRing / 4];
  const int i = blockIdx.y, n0 = blockIdx.x * 32;
  const int rs = row_ptr[i / gt], n_i = max(min(row_ptr[i / gt + 1], nnz_cap) - rs, 0);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int wa = wave % 2, ww = wave % Tl::kWaves / 2, part = wave / Tl::kWaves;
  const int most = (n_i + 1) / 2, e_lo = rs + part * most, cnt = min(most, rs + n_i - e_lo);    // this part's entries
  const SourcesF32<Tl, WIDE> src(act + ((long long)e_lo * gt + i % gt) * (TB * TB), TB, W + (long long)n0 * ldw, ldw);
  // the columns of 64 entries, one per lane; in assembly with its own wait (a load that the compiler tracks would
  // make it wait for the whole ring at every step)
  int cols = 0;
  const int* list = col_idx + e_lo;
  auto fetch = [&](int e) {
    const uint32_t at = (uint32_t)min(e + lane, cnt - 1) * 4u;
    asm volatile("global_load_dword %0, %1, %2\n\ts_waitcnt vmcnt(0)" : "=v"(cols) : "v"(at), "s"(list) : "memory");
  };
  constexpr int kPer = TB / kF32Batch;      // steps per entry
  f32x4 acc[Tl::TA];
  run_f32<Tl, false>(cnt * kPer, most * kPer, lds_addr(ring) + part * Tl::kRing, src, wa, ww,
                 [&](int s, long long& oa, long long& ow) {
                   const int e = s / kPer, h = s % kPer * kF32Batch;
                   if (e % kWave == 0 && h == 0) fetch(e);
                   oa = (long long)e * gt * (TB * TB) + h;
                   ow = (long long)__builtin_amdgcn_readlane(cols, e % kWave) * TB + h;
                 },
                 acc);
  if (!fold_parts_f32<Tl>(ring, acc)) return;
  const int n = n0 + 16 * ww + 4 * (lane / 16);
#pragma unroll
  for (int x = 0; x < Tl::TA; ++x) {
    const int t = i * TB + 16 * (Tl::TA * wa + x) + lane % 16;
    f32x4 v = acc[x];
    if (bias) v += *reinterpret_cast<const f32x4*>(bias + n);
    *reinterpret_cast<f32x4*>(out + (long long)t * ncols_out + n) = v;
  }
}

template <int TB, bool WIDE>
static void launch_sdd_f32(int Tt, int gt, int d, const float* A, const float* W, const float* bias, const int* row_ptr,
                           const int* col_idx, int nnz_cap, float* act_out, const float* act_gate, hipStream_t st) {
  const int items = (nnz_cap * gt + 7) / 8 * 8, gx = items < (1 << 20) ? items : 1 << 20;
  if (items == 0) return;
  const dim3 grid(gx, (items + gx - 1) / gx);
  if (act_gate)
    hipLaunchKernelGGL((ffn_sdd_f32<TB, true, WIDE>), grid, dim3(GateF32<TB>::kTileThreads), 0, st, A, W, bias, row_ptr, col_idx, Tt / gt, gt, d,
                       nnz_cap, gx, act_out, act_gate);
  else
    hipLaunchKernelGGL((ffn_sdd_f32<TB, false, WIDE>), grid, dim3(UpF32<TB>::kTileThreads), 0, st, A, W, bias, row_ptr, col_idx, Tt / gt, gt, d,
                       nnz_cap, gx, act_out, act_gate);
}

template <int TB>
static hipError_t launch_f32(int pass, int Tt, int gt, int d, int F, const float* A, const float* W1, const float* b1,
                             const float* W2, const float* b2, const int* row_ptr, const int* col_idx, int nnz_cap,
                             float* act_out, const float* act_gate, float* out, hipStream_t st) {
  // W1: [F, d] rows = neurons (contraction over d).  W2: [d, F] (contraction over active f).
  {
    ProfScope ps(pass == 0 ? kKFfnUp : kKFfnDh, st);
    auto* launch = d < kWideF32 ? launch_sdd_f32<TB, false> : launch_sdd_f32<TB, true>;
    launch(Tt, gt, d, A, W1, pass == 0 ? b1 : nullptr, row_ptr, col_idx, nnz_cap, act_out, pass == 0 ? nullptr : act_gate, st);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  ProfScope ps(pass == 0 ? kKFfnDown : kKFfnDx, st);
  auto* kernel = F < kWideF32 ? ffn_dsd_f32<TB, false> : ffn_dsd_f32<TB, true>;
  hipLaunchKernelGGL(kernel, dim3(d / 32, Tt), dim3(DsdF32<TB>::kTileThreads), 0, st, (const float*)act_out, W2, (long long)F, b2,
                     row_ptr, col_idx, gt, d, nnz_cap, out);
  return hipGetLastError();
}

// pass 0 (forward):  A = X,  W1 = W_up [F,d],     W2 = W_down [d,F], act_out = H_act, out = Y
// pass 1 (backward): A = dY, W1 = W_down_t [F,d], W2 = W_up_t [d,F], act_out = dZ_act,
//                    act_gate = H_act, out = dX
hipError_t launch_ffn_f32(int pass, int tile, int Tt, int gt, int Fb, int d, int F, const float* A,
                          const float* W1, const float* b1, const float* W2, const float* b2,
                          const int* row_ptr, const int* col_idx, int nnz_cap, float* act_out,
                          const float* act_gate, float* out, hipStream_t st) {
  (void)Fb;
  if (tile == 32)
    return launch_f32<32>(pass, Tt, gt, d, F, A, W1, b1, W2, b2, row_ptr, col_idx, nnz_cap,
                              act_out, act_gate, out, st);
  return launch_f32<64>(pass, Tt, gt, d, F, A, W1, b1, W2, b2, row_ptr, col_idx, nnz_cap,
                            act_out, act_gate, out, st);
}

// ---------------------------------------------------------------------------
// Transpose for the one-time weight repack: dst[c][r] = src[r][c].
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void transpose_kernel(const T* __restrict__ src, int R, int C,
                                                        T* __restrict__ dst) {
  __shared__ T tile[64][65];
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  const int tx = threadIdx.x % 64, ty = threadIdx.x / 64;
  for (int rr = ty; rr < 64; rr += 4)
    if (r0 + rr < R && c0 + tx < C) tile[rr][tx] = src[(long long)(r0 + rr) * C + c0 + tx];
  __syncthreads();
  for (int cc = ty; cc < 64; cc += 4)
    if (c0 + cc < C && r0 + tx < R) dst[(long long)(c0 + cc) * R + r0 + tx] = tile[tx][cc];
}

hipError_t launch_transpose(int elem_bytes, const void* src, int R, int C, void* dst,
                            hipStream_t st) {
  dim3 grid((C + 63) / 64, (R + 63) / 64);
  ProfScope ps(kKTranspose, st);
  if (elem_bytes == 4)
    hipLaunchKernelGGL(transpose_kernel<float>, grid, dim3(256), 0, st, (const float*)src, R, C,
                       (float*)dst);
  else
    hipLaunchKernelGGL(transpose_kernel<uint16_t>, grid, dim3(256), 0, st, (const uint16_t*)src, R,
                       C, (uint16_t*)dst);
  return hipGetLastError();
}

}  // namespace lx
