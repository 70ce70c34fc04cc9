// fp32 sparse FFN kernels (Sec. VI-B neuron-centric tiled products), used for the fp32 correctness
// configuration.  fp32 operands and accumulation throughout, on the 32x32x2 fp32 MFMA: its rate is
// that of the vector unit, but an operand element is read once per 32 products instead of once per
// one to two, and that is what the products are made of here.
//
// Two kernel shapes serve all four products:
//   sdd: out block (i, j) = A_i [TT x K] . B_j [BN x K]^T for every listed
//        (token tile i, neuron block j); epilogue ReLU (+bias) or gating by the
//        stored activation sign.          (up-projection, dH)
//   dsd: out tile  = sum over listed j of Act_ij [TT x BN] . B[:, j-block]^T
//        (down-projection, dX), the contraction runs over active blocks only.
//
// The output tile of a workgroup is as small as a list block (32 or 64 tokens x 32 or 64 columns),
// which fills the chip at the sizes this configuration runs at; its wavefronts share it by 32 x 32
// quadrants and, beyond those, by ranges of the contraction index, whose partial sums are added
// through LDS in a fixed order.  No two wavefronts of a range share an operand pair, so every
// wavefront streams its own operands through its own two stages of LDS and the loop has no barrier.
// The detour over LDS is for the loads: a lane's row is fixed by the MFMA's layout, and a load of 16
// bytes from each of 32 rows occupies the CU's memory pipeline for 64 clocks where eight rows of 128
// bytes take 16.
// Measured at 512 tokens, 768 -> 3072 -> 768, 30 % of 32 x 32 blocks (460 blocks): 16-20 us per
// product, of which 6 us are the MFMAs (0.73 GFLOP, at most two blocks per CU) and about 7 the launch
// and the three dependent loads in front of the first operand; operands straight into registers 20-22,
// 2 x 2 register tiles on the vector unit 58-62.  The up-projection, whose signs decide the ReLU gate,
// adds its terms one by one in ascending order (23 us): a sum in another order would flip the gate of
// activations within rounding of zero.  With 64 x 64 blocks one workgroup fits a CU (128 KB of LDS: eight
// wavefronts of two stages, four of four in the up-projection): the same layer 20-24 us per product, 4096 tokens, 2048 -> 8192 (30 %, 2469 blocks) 450-550 us; on the
// vector unit 88-92 and 1008-1077.
#include "ffn_ring.h"

namespace lx {

constexpr int kF32Batch = 32;      // contraction elements per step: a 128-byte row piece, sixteen MFMAs of depth two
constexpr int kF32Stage = 64 * kF32Batch * 4;   // bytes of a stage: 32 token rows, 32 weight rows
constexpr int kF32Stages = 2;

// How the wavefronts of a workgroup with NQ quadrants share the work: KS ranges of the contraction
// index per quadrant.
template <int NQ>
struct F32Split {
  static constexpr int kRanges = NQ == 4 ? 2 : 4;
  static constexpr int kWaves = NQ * kRanges;
  static constexpr int kThreads = kWaves * kWave;
};

__device__ __forceinline__ f32x16 mfma32_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// acc += W[32 rows] . A[32 rows]^T over n batches of 32 contraction elements; at(s, a, w) yields the
// first element of batch s in row 0 of either operand, lda / ldw are the row strides.  `lds`: byte
// address of this wavefront's stages.
template <class At>
__device__ __forceinline__ void mma_batches_f32(uint32_t lds, int n, long long lda, long long ldw, At at,
                                                f32x16& acc) {
  const int lane = threadIdx.x % kWave, r = lane % 32, h2 = lane / 32;
  // instruction g of a stage brings rows 8g .. 8g+7 (g < 4: tokens), lane l slot l % 8 of row 8g + l/8
  long long off[8];
#pragma unroll
  for (int g = 0; g < 8; ++g) {
    const int row = 8 * g + lane / 8, seg = (lane % 8) ^ swz(row);
    off[g] = (row % 32) * (g < 4 ? lda : ldw) + seg * 4;
  }
  auto issue = [&](int s) {
    const float *a, *w;
    at(s, a, w);
    const uint32_t dst = lds + (s % kF32Stages) * kF32Stage;
#pragma unroll
    for (int g = 0; g < 8; ++g) dma16((g < 4 ? a : w) + off[g], dst + g * 1024);
  };
#pragma unroll
  for (int p = 0; p < kF32Stages; ++p)
    if (p < n) issue(p);
  for (int s = 0; s < n; ++s) {
    if (s + 1 < n) wait_vmcnt<8>(); else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    const uint32_t st = lds + (s % kF32Stages) * kF32Stage;
    f32x4 x[4], y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int slot = 2 * u + h2;
      x[u] = __builtin_bit_cast(f32x4, lds_read16(st + r * 128 + ((slot ^ swz(r)) << 4)));
      y[u] = __builtin_bit_cast(f32x4, lds_read16(st + (32 + r) * 128 + ((slot ^ swz(32 + r)) << 4)));
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the stage has been read
    if (s + kF32Stages < n) issue(s + kF32Stages);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = mfma32_f32(y[u][e], x[u][e], acc);
  }
}

// The same product with ONE fused multiply-add per term in ascending order of the contraction index,
// on the 16x16x1 MFMA (four 16 x 16 blocks, the 2 x 2 of the 32 x 32 tile; as fast per product): what
// the ReLU decides on does not depend on how the kernel is cut.  Lane l holds row l % 16 of block l / 16
// of either operand; accumulator register 4b + i is C[4 * (l / 16) + i][l % 16] of block b.
constexpr int kSeqStages = 4;
template <class At>
__device__ __forceinline__ void mma_batches_seq_f32(uint32_t lds, int n, long long lda, long long ldw, At at,
                                                    f32x16& acc) {
  const int lane = threadIdx.x % kWave, r = lane % 16, b = lane / 16;
  long long off[8];
#pragma unroll
  for (int g = 0; g < 8; ++g) {
    const int row = 8 * g + lane / 8, seg = (lane % 8) ^ swz(row);
    off[g] = (row % 32) * (g < 4 ? lda : ldw) + seg * 4;
  }
  auto issue = [&](int s) {
    const float *a, *w;
    at(s, a, w);
    const uint32_t dst = lds + (s % kSeqStages) * kF32Stage;
#pragma unroll
    for (int g = 0; g < 8; ++g) dma16((g < 4 ? a : w) + off[g], dst + g * 1024);
  };
  const int ra = 16 * (b / 2) + r, rw = 32 + 16 * (b % 2) + r;     // token row, weight row of the stage
#pragma unroll
  for (int p = 0; p < kSeqStages; ++p)
    if (p < n) issue(p);
  for (int s = 0; s < n; ++s) {
    const int younger = n - 1 - s;
    if (younger >= 3) wait_vmcnt<24>(); else wait_tail<8, 2>(younger);
    asm volatile("" ::: "memory");
    const uint32_t st = lds + (s % kSeqStages) * kF32Stage;
    f32x4 x[8], y[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      x[u] = __builtin_bit_cast(f32x4, lds_read16(st + ra * 128 + ((u ^ swz(ra)) << 4)));
      y[u] = __builtin_bit_cast(f32x4, lds_read16(st + rw * 128 + ((u ^ swz(rw)) << 4)));
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the stage has been read
    if (s + kSeqStages < n) issue(s + kSeqStages);
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x1f32(y[u][e], x[u][e], acc, 0, 0, 0);
  }
}

// out = max(A W^T + bias, 0), one fused multiply-add per term in ascending order.
// Workgroup (token tile, list entry): the tile index is the fast one, so that the workgroups without
// an entry come last in dispatch order.  A wavefront per 32 x 32 quadrant of the block.
template <int TB>
__global__ __launch_bounds__(TB * TB / 1024 * kWave) void ffn_up_f32(
    const float* __restrict__ A, const float* __restrict__ W, const float* __restrict__ bias,
    const int* __restrict__ row_ptr, const int* __restrict__ col_idx, int gt, int K, int nnz_cap,
    float* __restrict__ out_act) {
  constexpr int Q1 = TB / 32, NQ = Q1 * Q1;
  __shared__ __attribute__((aligned(1024))) float stages[NQ * kSeqStages * kF32Stage / 4];
  const int i = blockIdx.x;
  // gt consecutive token tiles share row i / gt of the list; the activation blocks of a list
  // row are stored as [entry][tile within the row's group]
  const int rs = row_ptr[i / gt], n_i = row_ptr[i / gt + 1] - rs;
  if ((int)blockIdx.y >= n_i) return;
  const int lp = rs + blockIdx.y;
  if (lp >= nnz_cap) return;       // entries beyond the capacity of the list buffers are ignored
  const int j = col_idx[lp];
  const long long p = (long long)lp * gt + i % gt;
  const int quad = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int t0 = 32 * (quad % Q1), n0 = 32 * (quad / Q1);      // this wavefront's quadrant
  const float* a0 = A + ((long long)i * TB + t0) * K;
  const float* w0 = W + ((long long)j * TB + n0) * K;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  mma_batches_seq_f32(lds_addr(stages) + quad * (kSeqStages * kF32Stage), K / kF32Batch, K, K,
                      [=](int s, const float*& a, const float*& w) {
                        a = a0 + s * kF32Batch;
                        w = w0 + s * kF32Batch;
                      },
                      acc);
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int t = t0 + 16 * (b / 2) + lane % 16, n = n0 + 16 * (b % 2) + 4 * (lane / 16);
    const long long o = p * (TB * TB) + t * TB + n;
    f32x4 v = {acc[4 * b], acc[4 * b + 1], acc[4 * b + 2], acc[4 * b + 3]};
    if (bias) v += *reinterpret_cast<const f32x4*>(bias + j * TB + n);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
    *reinterpret_cast<f32x4*>(out_act + o) = v;
  }
}

// Leaves the accumulators in LDS ([wave][16][lane] floats, over the stages) for folded_f32, which
// adds group g of four accumulator elements over the KS ranges of a quadrant (wavefront = quadrant +
// NQ * range), range 0 first.
__device__ __forceinline__ void spill_f32(float* area, const f32x16& acc) {
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 16; ++v) area[(wave * 16 + v) * kWave + lane] = acc[v];
  __syncthreads();
}
template <int NQ, int KS>
__device__ __forceinline__ f32x4 folded_f32(const float* area, int quadrant, int g) {
  const int lane = threadIdx.x % kWave;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < KS; ++k)
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] += area[((quadrant + NQ * k) * 16 + 4 * g + e) * kWave + lane];
  return s;
}

// out = gate > 0 ? A W^T : 0; same grid as above, the contraction in ranges.
template <int TB>
__global__ __launch_bounds__(F32Split<TB * TB / 1024>::kThreads) void ffn_gate_f32(
    const float* __restrict__ A, const float* __restrict__ W,
    const int* __restrict__ row_ptr, const int* __restrict__ col_idx, int gt, int K, int nnz_cap,
    float* __restrict__ out_act, const float* __restrict__ gate_act) {
  constexpr int Q1 = TB / 32, NQ = Q1 * Q1, KS = F32Split<NQ>::kRanges;
  __shared__ __attribute__((aligned(1024))) float stages[F32Split<NQ>::kWaves * kF32Stages * kF32Stage / 4];
  const int i = blockIdx.x;
  // gt consecutive token tiles share row i / gt of the list; the activation blocks of a list
  // row are stored as [entry][tile within the row's group]
  const int rs = row_ptr[i / gt], n_i = row_ptr[i / gt + 1] - rs;
  if ((int)blockIdx.y >= n_i) return;
  const int lp = rs + blockIdx.y;
  if (lp >= nnz_cap) return;       // entries beyond the capacity of the list buffers are ignored
  const int j = col_idx[lp];
  const long long p = (long long)lp * gt + i % gt;
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int quad = wave % NQ, range = wave / NQ;
  const int t0 = 32 * (quad % Q1), n0 = 32 * (quad / Q1);      // this wavefront's quadrant
  const int batches = K / kF32Batch;
  const int b_lo = batches * range / KS, b_hi = batches * (range + 1) / KS;
  const float* a0 = A + ((long long)i * TB + t0) * K + b_lo * kF32Batch;
  const float* w0 = W + ((long long)j * TB + n0) * K + b_lo * kF32Batch;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  mma_batches_f32(lds_addr(stages) + wave * (kF32Stages * kF32Stage), b_hi - b_lo, K, K,
                  [=](int s, const float*& a, const float*& w) {
                    a = a0 + s * kF32Batch;
                    w = w0 + s * kF32Batch;
                  },
                  acc);
  spill_f32(stages, acc);
  // accumulator group g: columns n0 + 8g + 4*(lane/32) .. +3 of token t0 + lane%32
#pragma unroll
  for (int g = range; g < 4; g += KS) {
    f32x4 v = folded_f32<NQ, KS>(stages, quad, g);
    const int t = t0 + lane % 32, n = n0 + 8 * g + 4 * (lane / 32);
    const long long o = p * (TB * TB) + t * TB + n;
    const f32x4 gg = *reinterpret_cast<const f32x4*>(gate_act + o);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = gg[e] > 0.f ? v[e] : 0.f;
    *reinterpret_cast<f32x4*>(out_act + o) = v;
  }
}

// out[i-tile, n0..n0+31] = sum_s act[p_s] [TB x TB] . W[n0.., j_s*TB ..]^T  (+ bias).  The list
// entries are dealt to the KS ranges in turn.
template <int TB>
__global__ __launch_bounds__(F32Split<TB / 32>::kThreads) void ffn_dsd_f32(
    const float* __restrict__ act, const float* __restrict__ W, long long ldw,
    const float* __restrict__ bias, const int* __restrict__ row_ptr,
    const int* __restrict__ col_idx, int gt, int ncols_out, int nnz_cap,
    float* __restrict__ out) {
  constexpr int NQ = TB / 32, KS = F32Split<NQ>::kRanges;
  __shared__ __attribute__((aligned(1024))) float stages[F32Split<NQ>::kWaves * kF32Stages * kF32Stage / 4];
  const int i = blockIdx.y, n0 = blockIdx.x * 32;
  const int rs = row_ptr[i / gt], n_i = min(row_ptr[i / gt + 1], nnz_cap) - rs;
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int quad = wave % NQ, range = wave / NQ;
  const int t0 = 32 * quad;
  const float* a0 = act + t0 * TB;
  const float* w0 = W + (long long)n0 * ldw;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  // entries range, range + KS, ...; their columns are fetched 64 at a time, one per lane
  for (int base = range; base < n_i; base += KS * kWave) {
    const int mine = base + KS * lane;
    const int col = mine < n_i ? col_idx[rs + mine] : 0;
    const int cnt = min(kWave, (n_i - base + KS - 1) / KS);
    constexpr int kPer = TB / kF32Batch;      // batches per entry
    mma_batches_f32(lds_addr(stages) + wave * (kF32Stages * kF32Stage), cnt * kPer, TB, ldw,
                    [&](int s, const float*& a, const float*& w) {
                      const int e = s / kPer, h = (s % kPer) * kF32Batch;
                      const long long p = (long long)(rs + base + KS * e) * gt + i % gt;
                      const int j = __builtin_amdgcn_readlane(col, e);
                      a = a0 + p * (TB * TB) + h;
                      w = w0 + (long long)j * TB + h;
                    },
                    acc);
  }
  spill_f32(stages, acc);
#pragma unroll
  for (int g = range; g < 4; g += KS) {
    f32x4 v = folded_f32<NQ, KS>(stages, quad, g);
    const int t = i * TB + t0 + lane % 32, n = n0 + 8 * g + 4 * (lane / 32);
    if (bias) v += *reinterpret_cast<const f32x4*>(bias + n);
    *reinterpret_cast<f32x4*>(out + (long long)t * ncols_out + n) = v;
  }
}

template <int TB>
static hipError_t launch_f32(int pass, int Tt, int gt, int Fb, int d, int F, const float* A, const float* W1,
                             const float* b1, const float* W2, const float* b2, const int* row_ptr,
                             const int* col_idx, int nnz_cap, float* act_out,
                             const float* act_gate, float* out, hipStream_t st) {
  // W1: [F, d] rows = neurons (contraction over d).  W2: [d, F] (contraction over active f).
  {
    ProfScope ps(pass == 0 ? kKFfnUp : kKFfnDh, st);
    if (pass == 0)
      hipLaunchKernelGGL(ffn_up_f32<TB>, dim3(Tt, Fb), dim3(TB * TB / 1024 * kWave), 0, st, A, W1, b1, row_ptr,
                         col_idx, gt, d, nnz_cap, act_out);
    else
      hipLaunchKernelGGL(ffn_gate_f32<TB>, dim3(Tt, Fb), dim3(F32Split<TB * TB / 1024>::kThreads), 0, st, A, W1,
                         row_ptr, col_idx, gt, d, nnz_cap, act_out, act_gate);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  ProfScope ps(pass == 0 ? kKFfnDown : kKFfnDx, st);
  hipLaunchKernelGGL(ffn_dsd_f32<TB>, dim3(d / 32, Tt), dim3(F32Split<TB / 32>::kThreads), 0, st,
                     (const float*)act_out, W2, (long long)F, b2, row_ptr, col_idx, gt, d, nnz_cap, out);
  return hipGetLastError();
}

// pass 0 (forward):  A = X,  W1 = W_up [F,d],     W2 = W_down [d,F], act_out = H_act, out = Y
// pass 1 (backward): A = dY, W1 = W_down_t [F,d], W2 = W_up_t [d,F], act_out = dZ_act,
//                    act_gate = H_act, out = dX
hipError_t launch_ffn_f32(int pass, int tile, int Tt, int gt, int Fb, int d, int F, const float* A,
                          const float* W1, const float* b1, const float* W2, const float* b2,
                          const int* row_ptr, const int* col_idx, int nnz_cap, float* act_out,
                          const float* act_gate, float* out, hipStream_t st) {
  if (tile == 32)
    return launch_f32<32>(pass, Tt, gt, Fb, d, F, A, W1, b1, W2, b2, row_ptr, col_idx, nnz_cap,
                              act_out, act_gate, out, st);
  return launch_f32<64>(pass, Tt, gt, Fb, d, F, A, W1, b1, W2, b2, row_ptr, col_idx, nnz_cap,
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
