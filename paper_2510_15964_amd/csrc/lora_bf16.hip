// The small products of the LoRA branch on the up-projection (Sec. II-C: z = W x + B A x;
// Sec. II-D: its gradients) for gfx950: U = X A^T, G = dZ B and dB = dZ^T U over the listed blocks,
// dA = G^T X, and the transpose of A.  A_pad [64, d] and B_pad [F, 64] hold
// A [r, d] and B [F, r] zero-padded to rank 64.  The branch's steps inside the up-projection and
// the input-gradient product live in the FFN kernels themselves.
#include "ffn_plan.h"
#include "ffn_ring.h"

namespace lx {

// The small products of the branch work on pairs of [64 x 64] bf16 tiles: a stage of the ring
// holds tile P in rows 0..63 and tile Q in rows 64..127 (16 KiB, two DMA instructions per wave:
// rows 8*wave + lane/8 of each).  Four stages = 64 KiB: two workgroups per CU.
constexpr int kPairElems = 128 * kBK;
constexpr int kPairStages = 4;

// Byte offset of element (row, col) inside a staged [64 x 64] tile.
__device__ __forceinline__ uint32_t tile64_off(int row, int col) {
  return (uint32_t)(row * 128 + (((col >> 3) ^ swz(row)) << 4) + (col & 7) * 2);
}

// This lane's source pointers of the two instructions: P and Q point at the first element of the
// tiles of step 0, ldp / ldq are their row strides in elements.
__device__ __forceinline__ void pair_src(const uint16_t* P, long long ldp, const uint16_t* Q,
                                         long long ldq, const uint16_t* (&src)[2]) {
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int row = 8 * wave + lane / 8, seg = (lane % 8) ^ swz(row);
  src[0] = P + row * ldp + seg * 8;
  src[1] = Q + row * ldq + seg * 8;
}

// The eight wavefronts of such a product: wavefront w owns the 32 x 32 quadrant (w % 2, (w / 2) % 2)
// of the 64 x 64 result and half w / 4 of the contraction index.  fold_khalves adds the second
// halves to the first ones through 16 KiB of LDS, in a fixed order; it returns true in the
// wavefronts 0 .. 3, which then hold the sums.
__device__ __forceinline__ bool fold_khalves(float* area, f32x16& acc) {
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  lds_barrier();   // nobody reads the ring any more
  if (wave >= 4) {
#pragma unroll
    for (int v = 0; v < 16; ++v) area[((wave - 4) * 16 + v) * kWave + lane] = acc[v];
  }
  lds_barrier();
  if (wave >= 4) return false;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] += area[(wave * 16 + v) * kWave + lane];
  return true;
}

// dst[c][r] = src[r][c] of a 64 x 64 tile, by 128 or more threads; t: 64 x 72 elements of LDS.
__device__ __forceinline__ void transpose64(const uint16_t* __restrict__ src, long long lds, uint16_t* __restrict__ dst,
                                            long long ldd, uint16_t* t) {
  for (int piece = threadIdx.x; piece < 512; piece += blockDim.x) {
    const int r = piece / 8, c8 = (piece % 8) * 8;
    const uint4 v = *reinterpret_cast<const uint4*>(src + r * lds + c8);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      t[(c8 + 2 * e) * 72 + r] = (uint16_t)(w[e] & 0xFFFFu);
      t[(c8 + 2 * e + 1) * 72 + r] = (uint16_t)(w[e] >> 16);
    }
  }
  __syncthreads();
  for (int piece = threadIdx.x; piece < 512; piece += blockDim.x) {
    const int r = piece / 8, c8 = (piece % 8) * 8;
    *reinterpret_cast<uint4*>(dst + r * ldd + c8) = *reinterpret_cast<const uint4*>(t + r * 72 + c8);
  }
}

// out[t][q] = sum over steps of sum_k P_s[t][k] Q_s[q][k], a 64 x 64 tile per token tile i.
// MODE 0, U = X A_pad^T (Sec. II-C: the inner factor A x of the branch): P = X, Q = A_pad, row
//   stride ld of both; the steps are the ld / 64 chunks of K.
// MODE 1, G = dZ B_pad (Sec. II-D: the gradient that reaches A x): P = the compact blocks dZ_ij of
//   the tile's list, Q_s[q][k] = B_pad[64 j_s + k][q]; the steps are the list entries.  The last ld / 64
//   workgroups of the launch transpose A_pad [64,ld] into A_t [ld,64] meanwhile, which the
//   input-gradient product reads.
// Two kernels: up to kNtQuadTiles token tiles a workgroup per 32 x 32 quadrant with the steps cut into ranges,
// beyond that a workgroup per tile.  At d = 2048, U (bf16; one range per quadrant from 256 tiles on, two from
// 128): 64 tiles 10.5 us by quadrants and 13.6 by tiles, 72 tiles 15.4 and 13.7, 128 tiles 14.7 and 14.3, 256
// tiles 34.7 and 16.3, 512 tiles 64.6 and 33.3 (134 MB of X: 4 TB/s, the copy rate).  Tiles lose where they leave
// half of the CUs idle over a long K: 128 tiles, d = 5120 35.6 us, 25.1 with K cut in two and a launch that adds.
constexpr int kNtQuadTiles = 64;

// Few tiles: what bounds the product is latency.  A quadrant per workgroup gives every CU one at 64 tiles; a
// wavefront owns one half (32 of the 64 k) of the steps of one range (lora_u_split / lora_g_split of them) and
// streams its own operands through its own stages, 4 KB each, without a barrier; halves and ranges are added at
// the end through LDS, in that order.  The quadrants of a tile sit eight workgroups apart, on one XCD, so that a
// tile's rows are fetched into one L2 only (neighbours, on four XCDs: 64 tiles, d = 2048 U 13.7 us, now 10.5).
constexpr int kNtStage = 4096;                 // bytes: 32 rows of 64 bytes of P, 32 of Q
constexpr int kNtStages(int waves) { return waves <= 4 ? 8 : 32 / waves; }
constexpr int kNtLds = 32 * kNtStage;          // stages of all wavefronts (one workgroup per CU, see above)
// Workgroups of the quadrants of Tt tiles, in whole groups of eight tiles.
__host__ __device__ constexpr int nt_quads(int Tt) { return 32 * ((Tt + 7) / 8); }
template <int DT, int MODE>
__global__ __launch_bounds__(1024) void lora_nt_kernel(
    const uint16_t* __restrict__ P, const uint16_t* __restrict__ Q, int ld,
    const int* __restrict__ row_ptr, const int* __restrict__ col_idx, int Tt, int gt, int nnz_cap,
    uint16_t* __restrict__ out, const uint16_t* __restrict__ A_pad, uint16_t* __restrict__ A_t) {
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kNtLds];
  const int w = blockIdx.x, quads = nt_quads(Tt);
  if (MODE == 1 && w >= quads) {
    transpose64(A_pad + (w - quads) * 64ll, ld, A_t + (w - quads) * 4096ll, 64, reinterpret_cast<uint16_t*>(lds));
    return;
  }
  const int i = w / 32 * 8 + w % 8, quad = w / 8 % 4;
  if (i >= Tt) return;
  const int th = quad % 2, qh = quad / 2;
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int waves = blockDim.x / kWave, split = waves / 2, range = wave / 2, kh = wave % 2;
  const int nst = kNtStages(waves);
  int rs = 0, nsteps = ld / kBK;
  if (MODE == 1) {
    rs = row_ptr[i / gt];
    nsteps = max(min(row_ptr[i / gt + 1], nnz_cap) - rs, 0);   // entries beyond the capacity are ignored
  }
  const int per = (nsteps + split - 1) / split;
  const int s_lo = range * per, n = min(nsteps, s_lo + per) - s_lo;
  // Transfer: 16 rows of 64 bytes per instruction, two for P and two for Q.  Slot c of row r (16 bytes) sits at
  // 64 r + 16 (c ^ (r / 2) % 4): eight consecutive rows of a slot then lie in different banks.
  const int tr = lane / 4, tc = (lane % 4) ^ ((tr / 2) % 4);
  const uint32_t p_off = (uint32_t)(tr * (MODE == 0 ? ld : 64) * 2 + tc * 16);
  const uint32_t q_off = (uint32_t)(tr * (MODE == 0 ? ld : 64) * 2 + tc * 16);
  const uint32_t ring = lds_addr(lds) + wave * (nst * kNtStage);
  auto issue = [&](int s) {
    const uint32_t to = ring + (s % nst) * kNtStage;
    const uint16_t *p, *q;
    long long ldp, ldq;
    if (MODE == 0) {
      p = P + ((long long)i * 64 + 32 * th) * ld + (s_lo + s) * 64 + 32 * kh;
      q = Q + 32ll * qh * ld + (s_lo + s) * 64 + 32 * kh;
      ldp = ldq = ld;
    } else {
      const int e = rs + s_lo + s;
      p = P + ((long long)e * gt + i % gt) * 4096 + 32 * th * 64 + 32 * kh;
      q = Q + ((long long)col_idx[e] * 64 + 32 * kh) * 64 + 32 * qh;      // rows are k
      ldp = ldq = 64;
    }
    dma16_s(p, p_off, to);
    dma16_s(p + 16 * ldp, p_off, to + 1024);
    dma16_s(q, q_off, to + 2048);
    dma16_s(q + 16 * ldq, q_off, to + 3072);
  };
  const int r = lane % 32, h2 = lane / 32;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  for (int s = 0; s < nst - 1; ++s)
    if (s < n) issue(s);
  for (int s = 0; s < n; ++s) {
    if (s + nst - 1 < n) issue(s + nst - 1);
    switch (min(n - 1 - s, nst - 1)) {         // younger steps in flight
      case 0: wait_vmcnt<0>(); break;
      case 1: wait_vmcnt<4>(); break;
      case 2: wait_vmcnt<8>(); break;
      case 3: wait_vmcnt<12>(); break;
      case 4: wait_vmcnt<16>(); break;
      case 5: wait_vmcnt<20>(); break;
      case 6: wait_vmcnt<24>(); break;
      default: wait_vmcnt<28>(); break;
    }
    asm volatile("" ::: "memory");
    const uint32_t st = ring + (s % nst) * kNtStage;
    uint4 a[2], b[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      if (MODE == 0) {
        const uint32_t o = r * 64 + (((2 * e + h2) ^ ((r / 2) % 4)) << 4);
        b[e] = lds_read16(st + o);
        a[e] = lds_read16(st + 2048 + o);
      } else {
        // Q by rows of k: the transposing read gives this lane's rank index the k 4*h2 .. +3 and 8 + 4*h2 .. +3
        // of the 16; P is read in the same order
        const uint32_t sw = (r / 2) % 4, p0 = r * 64 + 8 * h2;
        const uint2 pl = lds_read8(st + p0 + (((2 * e) ^ sw) << 4)), ph = lds_read8(st + p0 + (((2 * e + 1) ^ sw) << 4));
        b[e] = make_uint4(pl.x, pl.y, ph.x, ph.y);
        const int j = lane % 16, c = 2 * ((lane / 16) % 2) + (j % 4) / 2;    // slot of column 16*((lane/16)%2) + 4*(j%4)
        const int k0 = 16 * e + 4 * h2 + j / 4, k1 = k0 + 8;
        const uint2 ql = lds_read8_tr(st + 2048 + k0 * 64 + ((c ^ ((k0 / 2) % 4)) << 4) + (j % 2) * 8);
        const uint2 qu = lds_read8_tr(st + 2048 + k1 * 64 + ((c ^ ((k1 / 2) % 4)) << 4) + (j % 2) * 8);
        a[e] = make_uint4(ql.x, ql.y, qu.x, qu.y);
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the stage has been read: the next issue refills it
#pragma unroll
    for (int e = 0; e < 2; ++e) acc = mfma32<DT>(a[e], b[e], acc);
  }
  float* area = reinterpret_cast<float*>(lds);
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 16; ++v) area[(wave * 16 + v) * kWave + lane] = acc[v];
  __syncthreads();
  // element v of lane l: rank index 32*qh + 8*(v/4) + 4*(l/32) + v%4, token 32*th + l%32; a group of four per thread
  for (int x = threadIdx.x; x < 256; x += blockDim.x) {
    const int g = x / kWave, l = x % kWave;
    float v[4] = {};
    for (int p = 0; p < split; ++p)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float half = area[((2 * p) * 16 + 4 * g + e) * kWave + l] + area[((2 * p + 1) * 16 + 4 * g + e) * kWave + l];
        v[e] = split == 1 ? half : v[e] + half;
      }
    uint2 ov;
    ov.x = pack2<DT>(v[0], v[1]);
    ov.y = pack2<DT>(v[2], v[3]);
    *reinterpret_cast<uint2*>(out + ((long long)i * 64 + 32 * th + l % 32) * 64 + 32 * qh + 8 * g + 4 * (l / 32)) = ov;
  }
}

// More tiles: a workgroup per tile, which reads the tile's rows once in whole 128-byte lines and shares them between
// its wavefronts (a quadrant and a half of k each) through the ring; two workgroups per CU.
template <int DT, int MODE>
__global__ __launch_bounds__(kThreads) void lora_nt_tile_kernel(
    const uint16_t* __restrict__ P, const uint16_t* __restrict__ Q, int ld,
    const int* __restrict__ row_ptr, const int* __restrict__ col_idx, int Tt, int gt, int nnz_cap,
    uint16_t* __restrict__ out, const uint16_t* __restrict__ A_pad, uint16_t* __restrict__ A_t) {
  __shared__ __attribute__((aligned(1024))) uint16_t ring[kPairStages * kPairElems];
  const int i = blockIdx.x;
  if (MODE == 1 && i >= Tt) {
    transpose64(A_pad + (i - Tt) * 64ll, ld, A_t + (i - Tt) * 4096ll, 64, ring);
    return;
  }
  int rs = 0, nsteps = ld / kBK;
  if (MODE == 1) {
    rs = row_ptr[i / gt];
    nsteps = max(min(row_ptr[i / gt + 1], nnz_cap) - rs, 0);   // entries beyond the capacity are ignored
  }
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int th = wave % 2, qh = (wave / 2) % 2, kh = wave / 4;
  const int r = lane % 32, h2 = lane / 32;
  const uint16_t* src[2];
  if (MODE == 0)
    pair_src(P + (long long)i * 64 * ld, ld, Q, ld, src);
  else
    pair_src(P, 64, Q, 64, src);
  // byte offsets inside a stage, per 16-deep slice of this wavefront's half of k
  uint32_t po[2][2], qo[2][2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int k = 32 * kh + 16 * e;
    if (MODE == 0) {
      po[e][0] = tile64_off(32 * th + r, k + 8 * h2);
      qo[e][0] = 64 * 128 + tile64_off(32 * qh + r, k + 8 * h2);
    } else {
      const int j = lane % 16, col = 32 * qh + 16 * ((lane / 16) % 2) + 4 * (j % 4);
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        po[e][x] = tile64_off(32 * th + r, k + 8 * x + 4 * h2);
        qo[e][x] = 64 * 128 + tile64_off(k + 8 * x + 4 * h2 + j / 4, col);
      }
    }
  }
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  run_ring_of<kPairStages, 2, kPairElems>(
      nsteps, src,
      [=](int s, long long& ob, long long& oa) {
        if (MODE == 0) {
          ob = oa = (long long)s * kBK;
        } else {
          ob = ((long long)(rs + s) * gt + i % gt) * 4096;
          oa = (long long)col_idx[rs + s] * 4096;
        }
      },
      ring,
      [&](const uint16_t* stage) {
        const uint32_t st = lds_addr(stage);
        uint4 a[2], b[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          if (MODE == 0) {
            a[e] = lds_read16(st + qo[e][0]);
            b[e] = lds_read16(st + po[e][0]);
          } else {
            const uint2 pl = lds_read8(st + po[e][0]), ph = lds_read8(st + po[e][1]);
            const uint2 ql = lds_read8_tr(st + qo[e][0]), qu = lds_read8_tr(st + qo[e][1]);
            b[e] = make_uint4(pl.x, pl.y, ph.x, ph.y);
            a[e] = make_uint4(ql.x, ql.y, qu.x, qu.y);
          }
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) acc = mfma32<DT>(a[e], b[e], acc);
      });
  if (!fold_khalves(reinterpret_cast<float*>(ring), acc)) return;
  // register v: rank index 32*qh + 8*(v/4) + 4*h2 + v%4, token 32*th + lane%32
  uint16_t* o = out + ((long long)i * 64 + 32 * th + r) * 64 + 32 * qh + 4 * h2;
#pragma unroll
  for (int g = 0; g < 4; ++g)
    *reinterpret_cast<uint2*>(o + 8 * g) =
        make_uint2(pack2<DT>(acc[4 * g], acc[4 * g + 1]), pack2<DT>(acc[4 * g + 2], acc[4 * g + 3]));
}

// Per-lane LDS offsets of the operands of a product out[a][b] = sum_t P[t][a] Q[t][b] whose
// contraction index is the ROW of both staged tiles: both are read with the transposing read.
// For the 16-row slice i of this wavefront's half of t, a lane gets rows
// {4*h2 .. +3} and {8 + 4*h2 .. +3} of the slice (h2 = lane / 32) of column lane % 32 of its
// quadrant, for P and Q alike, so the two operands of the MFMA agree on the order of t.
struct TnLane {
  uint32_t p[2][2], q[2][2];   // [slice][rows +0 / +8]
  __device__ __forceinline__ void init(int ah, int bh, int kh) {
    const int lane = threadIdx.x % kWave, h2 = lane / 32, j = lane % 16;
    const int col = 16 * ((lane / 16) % 2) + 4 * (j % 4);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int row = 32 * kh + 16 * i + 8 * e + 4 * h2 + j / 4;
        p[i][e] = tile64_off(row, 32 * ah + col);
        q[i][e] = 64 * 128 + tile64_off(row, 32 * bh + col);
      }
  }
};
template <int DT>
__device__ __forceinline__ void tn_step(uint32_t stage, const TnLane& lo, f32x16& acc) {
  uint4 a[2], b[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const uint2 al = lds_read8_tr(stage + lo.p[i][0]), ah = lds_read8_tr(stage + lo.p[i][1]);
    const uint2 bl = lds_read8_tr(stage + lo.q[i][0]), bh = lds_read8_tr(stage + lo.q[i][1]);
    a[i] = make_uint4(al.x, al.y, ah.x, ah.y);
    b[i] = make_uint4(bl.x, bl.y, bh.x, bh.y);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) acc = mfma32<DT>(a[i], b[i], acc);
}

// The token tiles i_lo .. i_hi - 1, at most kThreads of them, whose list holds neuron block j: calls put(place in their
// order, tile, compact activation block) in one thread each, returns their number to all.  wcount: kFW ints of LDS.
template <class Put>
__device__ __forceinline__ int listed_tiles(const int* __restrict__ row_ptr, const int* __restrict__ col_idx, int gt, int nnz_cap,
                                            int j, int i_lo, int i_hi, int* wcount, Put put) {
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave, i = i_lo + (int)threadIdx.x;
  long long blk = -1;
  if (i < i_hi) {
    const int rs = row_ptr[i / gt];
    int lo_ = 0, hi_ = min(row_ptr[i / gt + 1], nnz_cap) - rs;   // entries beyond the capacity are ignored
    while (lo_ < hi_) {
      const int mid = (lo_ + hi_) / 2, c = col_idx[rs + mid];
      if (c == j) {
        blk = ((long long)rs + mid) * gt + i % gt;
        break;
      }
      if (c < j) lo_ = mid + 1; else hi_ = mid;
    }
  }
  const unsigned long long hit = __ballot(blk >= 0);
  if (lane == 0) wcount[wave] = __popcll(hit);
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kFW; ++w) {
    const int c = wcount[w];
    if (w < wave) before += c;
    total += c;
  }
  if (blk >= 0) put(before + __popcll(hit & ((1ull << lane) - 1ull)), i, blk);
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(total);
}

// Gradients of the two LoRA matrices (Sec. II-D), fp32, as sums of 64 x 64 products
// out[a][b] = sum over steps of sum_t P[t][a] Q[t][b] on the MFMA:
// MODE 0, dB = dZ^T U over the listed blocks: x = neuron block j; the steps are the
//   token tiles i of range y whose list row holds j (found by bisection of the
//   sorted row, one tile per thread, and kept in list order): P = dZ_ij, Q = U_i;
//   out = rows 64j .. of dB [F,64].
// MODE 1, dA = G^T X: x = 64-column chunk c of X; the steps are all tiles of the range:
//   P = G_i, Q = X_i[:, 64c ..]; out = columns 64c .. of dA [64,d].
// The sums over the tile ranges y go to part[y] (part_stride elements apart; with one
// range, part is the result itself) and are added by lora_grad_reduce_kernel.
struct TnArgs {
  const uint16_t *P, *Q;
  long long ldq;
  float* part;
  long long part_stride;
  int ld_out, nx, ny;          // products x = 0 .. nx - 1 times ranges y = 0 .. ny - 1
};
struct TnLds {
  uint16_t ring[kPairStages * kPairElems];
  long long p[kThreads], q[kThreads];
  int wcount[kFW];
};
template <int DT, int MODE>
__device__ __forceinline__ void lora_tn(const TnArgs& args, int x, int y, const int* __restrict__ row_ptr,
                                        const int* __restrict__ col_idx, int Tt, int gt, int nnz_cap, TnLds& sh) {
  const uint16_t* __restrict__ P = args.P;
  const uint16_t* __restrict__ Q = args.Q;
  const long long ldq = args.ldq;
  uint16_t* ring = sh.ring;
  long long *s_p = sh.p, *s_q = sh.q;
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int per = (Tt + args.ny - 1) / args.ny;
  const int i_lo = y * per, i_hi = min(Tt, i_lo + per);
  const int ah = wave % 2, bh = (wave / 2) % 2;
  const uint16_t* src[2];
  pair_src(P, 64, Q + (MODE == 1 ? x * 64 : 0), ldq, src);
  TnLane lo;
  lo.init(ah, bh, wave / 4);
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  auto step = [&](const uint16_t* stage) { tn_step<DT>(lds_addr(stage), lo, acc); };
  if (MODE == 1) {
    run_ring_of<kPairStages, 2, kPairElems>(
        i_hi - i_lo, src,
        [=](int s, long long& ob, long long& oa) {
          ob = (long long)(i_lo + s) * 4096;
          oa = (long long)(i_lo + s) * 64 * ldq;
        },
        ring, step);
  } else {
    // (the host splits so that a range holds at most kThreads tiles)
    const int total = listed_tiles(row_ptr, col_idx, gt, nnz_cap, x, i_lo, i_hi, sh.wcount, [&](int k, int i, long long blk) {
      s_p[k] = blk * 4096;
      s_q[k] = (long long)i * 64 * ldq;
    });
    run_ring_of<kPairStages, 2, kPairElems>(
        total, src,
        [&](int s, long long& ob, long long& oa) {
          ob = s_p[s];
          oa = s_q[s];
        },
        ring, step);
  }
  if (!fold_khalves(reinterpret_cast<float*>(ring), acc)) return;
  // register v: a = 32*ah + 8*(v/4) + 4*(lane/32) + v%4, b = 32*bh + lane%32
  const long long row0 = MODE == 0 ? (long long)x * 64 : 0;
  const int col0 = MODE == 0 ? 0 : x * 64;
  float* o = args.part + y * args.part_stride + (row0 + 32 * ah + 4 * (lane / 32)) * args.ld_out + col0 +
             32 * bh + lane % 32;
#pragma unroll
  for (int v = 0; v < 16; ++v) o[(long long)(8 * (v / 4) + v % 4) * args.ld_out] = acc[v];
}
// Both gradients in one launch, independent of each other: workgroups 0 .. of the one, then those of the other.
// The longer ones go first, or the launch ends on them alone.  With lists per group of tiles those are dA's, which
// sum all tiles of their range where a neuron block is listed by a part of them (d = 2048, F = 8192, 11 % of the
// blocks, 512 tiles: both gradients 57.3 us in launches of their own, 70.7 with dB first; backward LoRA products
// with dB / dA first: 512 tiles 97.5 / 75.9 us, 256 tiles 59.4 / 49.8, 64 tiles 31.6 / 28.8).  With one list for
// all tiles dB's listed blocks are as long as dA's, and few: 512 tiles, 28 blocks 123.7 / 139.1, 80 tiles, d = 5120,
// 32 blocks 49.4 / 54.1.
template <int DT>
__global__ __launch_bounds__(kThreads) void lora_tn_kernel(TnArgs db, TnArgs da, const int* __restrict__ row_ptr,
                                                           const int* __restrict__ col_idx, int Tt, int gt, int nnz_cap) {
  __shared__ __attribute__((aligned(1024))) TnLds sh;
  const int nb = db.nx * db.ny, na = da.nx * da.ny;
  const bool db_first = gt == Tt;
  const int w = blockIdx.x, w_b = db_first ? w : w - na, w_a = db_first ? w - nb : w;
  if (db_first ? w < nb : w >= na)
    lora_tn<DT, 0>(db, w_b % db.nx, w_b / db.nx, row_ptr, col_idx, Tt, gt, nnz_cap, sh);
  else
    lora_tn<DT, 1>(da, w_a % da.nx, w_a / da.nx, row_ptr, col_idx, Tt, gt, nnz_cap, sh);
}
// Few token tiles: a workgroup per 32 x 32 quadrant of a product, whose eight wavefronts take a range of its token tiles
// each, in steps of 32 token rows through stages of their own (4 KB, no barrier), and add up through LDS in a fixed
// order: there are no parts in memory and no launch that adds them.  The quadrants of a product sit eight
// workgroups apart, on one XCD.  What bounds it is latency while all workgroups are resident at once, two per CU, and
// the products that they add beyond that (see lora_grads_by_quads).  Errors of dA and dB against 64 bits over eleven sizes are
// 0.91 - 1 and 0.87 - 1 times those by parts.
constexpr int kTnQuadStages = 2, kTnQuadStage = 4096;
struct TnQuadLds {
  uint8_t ring[kFW * kTnQuadStages * kTnQuadStage];     // (the sums at the end: 32 KB)
  int tile[kThreads], wcount[kFW];
  long long blk[kThreads];
};
constexpr int tn_quads(int nx) { return 32 * ((nx + 7) / 8); }
template <int DT, int MODE>
__device__ __forceinline__ void lora_tn_quad(const TnArgs& args, int w, const int* __restrict__ row_ptr,
                                             const int* __restrict__ col_idx, int Tt, int gt, int nnz_cap, TnQuadLds& sh) {
  const int x = w / 32 * 8 + w % 8, quad = w / 8 % 4;
  if (x >= args.nx) return;
  const int ah = quad % 2, bh = quad / 2;
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  int tiles = Tt;
  if (MODE == 0)
    tiles = listed_tiles(row_ptr, col_idx, gt, nnz_cap, x, 0, Tt, sh.wcount, [&](int k, int i, long long blk) {
      sh.tile[k] = i;
      sh.blk[k] = blk;
    });
  const int per = (tiles + kFW - 1) / kFW, t_lo = min(wave * per, tiles), n = 2 * (min(tiles, t_lo + per) - t_lo);
  // 16 rows of 64 bytes per transfer, two for P and two for Q; slot c (16 bytes) of row r sits at 64 r + 16 (c ^ (r / 2) % 4)
  const int tr = lane / 4, tc = (lane % 4) ^ ((tr / 2) % 4);
  const uint32_t p_off = (uint32_t)(tr * 128 + tc * 16), q_off = (uint32_t)(tr * args.ldq * 2 + tc * 16);
  const uint32_t ring = lds_addr(sh.ring) + wave * (kTnQuadStages * kTnQuadStage);
  auto issue = [&](int s) {
    const uint32_t to = ring + (s % kTnQuadStages) * kTnQuadStage;
    const int k = t_lo + s / 2, half = 32 * (s % 2);
    long long blk = k, i = k;
    if (MODE == 0) {
      i = __builtin_amdgcn_readfirstlane(sh.tile[k]);
      blk = (long long)__builtin_amdgcn_readfirstlane((int)(sh.blk[k] >> 32)) << 32 |
            (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.blk[k]);
    }
    const uint16_t* p = args.P + blk * 4096 + half * 64 + 32 * ah;
    const uint16_t* q = args.Q + (i * 64 + half) * args.ldq + (MODE == 1 ? x * 64 : 0) + 32 * bh;
    dma16_s(p, p_off, to);
    dma16_s(p + 16 * 64, p_off, to + 1024);
    dma16_s(q, q_off, to + 2048);
    dma16_s(q + 16 * args.ldq, q_off, to + 3072);
  };
  // operands: column 16*((lane/16)%2) + lane%16 of the rows 16e + 4*(lane/32) .. + 3 and those eight further on
  const int h2 = lane / 32, j = lane % 16, c = 2 * ((lane / 16) % 2) + (j % 4) / 2;
  uint32_t off[2][2];
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int k = 16 * e + 8 * u + 4 * h2 + j / 4;
      off[e][u] = ring + k * 64 + ((c ^ ((k / 2) % 4)) << 4) + (j % 2) * 8;
    }
  // the halves of a tile are summed apart, as by parts: shorter sums, smaller errors, and products that need not wait
  f32x16 acc, odd;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = odd[v] = 0.f;
  for (int s = 0; s < kTnQuadStages; ++s)
    if (s < n) issue(s);
  auto step = [&](int s, f32x16& sum) {
    wait_tail<4, kTnQuadStages - 1>(min(n - 1 - s, kTnQuadStages - 1));    // younger steps in flight
    asm volatile("" ::: "memory");
    const uint32_t st = (s % kTnQuadStages) * kTnQuadStage;
    uint4 a[2], b[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const uint2 al = lds_read8_tr(off[e][0] + st), au = lds_read8_tr(off[e][1] + st);
      const uint2 bl = lds_read8_tr(off[e][0] + st + 2048), bu = lds_read8_tr(off[e][1] + st + 2048);
      a[e] = make_uint4(al.x, al.y, au.x, au.y);
      b[e] = make_uint4(bl.x, bl.y, bu.x, bu.y);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the stage has been read
    if (s + kTnQuadStages < n) issue(s + kTnQuadStages);
#pragma unroll
    for (int e = 0; e < 2; ++e) sum = mfma32<DT>(a[e], b[e], sum);
  };
  for (int s = 0; s < n; s += 2) {
    step(s, acc);
    step(s + 1, odd);
  }
  float* area = reinterpret_cast<float*>(sh.ring);
  __syncthreads();
#pragma unroll
  for (int v = 0; v < 16; ++v) area[(wave * 16 + v) * kWave + lane] = acc[v] + odd[v];
  __syncthreads();
  // element v of lane l: row 32*ah + 8*(v/4) + 4*(l/32) + v%4, column 32*bh + l%32
  float* o = args.part + ((MODE == 0 ? x * 64ll : 0) + 32 * ah) * args.ld_out + (MODE == 1 ? x * 64 : 0) + 32 * bh;
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int v = wave + kFW * u;
    float sum[kFW];
#pragma unroll
    for (int q = 0; q < kFW; ++q) sum[q] = area[(q * 16 + v) * kWave + lane];
#pragma unroll
    for (int n2 = 1; n2 < kFW; n2 *= 2)     // by pairs: smaller errors than one after the other
#pragma unroll
      for (int q = 0; q < kFW; q += 2 * n2) sum[q] += sum[q + n2];
    o[(8 * (v / 4) + 4 * (lane / 32) + v % 4) * (long long)args.ld_out + lane % 32] = sum[0];
  }
}
template <int DT>
__global__ __launch_bounds__(kThreads, 4) void lora_tn_quad_kernel(TnArgs db, TnArgs da, const int* __restrict__ row_ptr,
                                                                   const int* __restrict__ col_idx, int Tt, int gt, int nnz_cap) {
  __shared__ __attribute__((aligned(1024))) TnQuadLds sh;
  const int nb = tn_quads(db.nx), na = tn_quads(da.nx);
  const bool db_first = gt == Tt;
  const int w = blockIdx.x, w_b = db_first ? w : w - na, w_a = db_first ? w - nb : w;
  if (db_first ? w < nb : w >= na)
    lora_tn_quad<DT, 0>(db, w_b, row_ptr, col_idx, Tt, gt, nnz_cap, sh);
  else
    lora_tn_quad<DT, 1>(da, w_a, row_ptr, col_idx, Tt, gt, nnz_cap, sh);
}

// dB and dA = sums of their parts, in order, four elements per thread; a result with one part
// was written in place and has n4 = 0 here.
__global__ void lora_grad_reduce_kernel(const float* __restrict__ part_b, int parts_b, long long n4_b,
                                        float* __restrict__ dB, const float* __restrict__ part_a,
                                        int parts_a, long long n4_a, float* __restrict__ dA) {
  long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const float* part = part_b;
  int parts = parts_b;
  long long n4 = n4_b;
  float* out = dB;
  if (idx >= n4_b) {
    idx -= n4_b;
    part = part_a; parts = parts_a; n4 = n4_a; out = dA;
    if (idx >= n4_a) return;
  }
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int p = 0; p < parts; ++p) {
    const float4 v = *reinterpret_cast<const float4*>(part + ((long long)p * n4 + idx) * 4);
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  *reinterpret_cast<float4*>(out + idx * 4) = s;
}

// U = X A_pad^T [T,64].
template <int DT>
static hipError_t launch_lora_u_t(int Tt, int d, const uint16_t* X, const uint16_t* A_pad, uint16_t* U,
                                  hipStream_t st) {
  const int* none = nullptr;
  const uint16_t* none16 = nullptr;
  if (Tt <= kNtQuadTiles)
    hipLaunchKernelGGL((lora_nt_kernel<DT, 0>), dim3(nt_quads(Tt)), dim3(2 * kWave * lora_u_split(Tt, d)), 0, st, X, A_pad,
                       d, none, none, Tt, 1, 0, U, none16, (uint16_t*)nullptr);
  else
    hipLaunchKernelGGL((lora_nt_tile_kernel<DT, 0>), dim3(Tt), dim3(kThreads), 0, st, X, A_pad, d, none, none, Tt, 1, 0, U,
                       none16, (uint16_t*)nullptr);
  return hipGetLastError();
}
hipError_t launch_lora_u(int dt, int Tt, int d, const uint16_t* X, const uint16_t* A_pad, uint16_t* U,
                         hipStream_t st) {
  return LX_BY_DT(launch_lora_u_t, Tt, d, X, A_pad, U, st);
}

// G = dZ B_pad [T,64] from the compact blocks dZ, and A_t = A_pad^T [d,64].
template <int DT>
static hipError_t launch_lora_g_t(int Tt, int gt, int d, const uint16_t* dZ, const uint16_t* B_pad,
                                  const int* row_ptr, const int* col_idx, int nnz_cap, uint16_t* G,
                                  const uint16_t* A_pad, uint16_t* A_t, hipStream_t st) {
  if (Tt <= kNtQuadTiles)
    hipLaunchKernelGGL((lora_nt_kernel<DT, 1>), dim3(nt_quads(Tt) + d / 64), dim3(2 * kWave * lora_g_split(Tt)), 0, st, dZ,
                       B_pad, d, row_ptr, col_idx, Tt, gt, nnz_cap, G, A_pad, A_t);
  else
    hipLaunchKernelGGL((lora_nt_tile_kernel<DT, 1>), dim3(Tt + d / 64), dim3(kThreads), 0, st, dZ, B_pad, d, row_ptr,
                       col_idx, Tt, gt, nnz_cap, G, A_pad, A_t);
  return hipGetLastError();
}
hipError_t launch_lora_g(int dt, int Tt, int gt, int d, const uint16_t* dZ, const uint16_t* B_pad,
                         const int* row_ptr, const int* col_idx, int nnz_cap, uint16_t* G, const uint16_t* A_pad,
                         uint16_t* A_t, hipStream_t st) {
  return LX_BY_DT(launch_lora_g_t, Tt, gt, d, dZ, B_pad, row_ptr, col_idx, nnz_cap, G, A_pad, A_t, st);
}

// dB = dZ^T U over the listed blocks and dA = G^T X.  Scratch: da_part [lora_da_split][64][d] and
// db_part [lora_db_split][F][64] (each unused for a split of 1, both by quadrants).
template <int DT>
static hipError_t launch_lora_grads_t(int Tt, int gt, int d, int F, const uint16_t* dZ,
                                      const uint16_t* U, const uint16_t* G, const uint16_t* X,
                                      const int* row_ptr, const int* col_idx, int nnz_cap,
                                      float* da_part, float* db_part, float* dA, float* dB,
                                      hipStream_t st) {
  if (lora_grads_by_quads(Tt, d, F)) {
    const TnArgs db = {dZ, U, 64, dB, 0, 64, F / 64, 1}, da = {G, X, d, dA, 0, d, d / 64, 1};
    hipLaunchKernelGGL(lora_tn_quad_kernel<DT>, dim3(tn_quads(db.nx) + tn_quads(da.nx)), dim3(kThreads), 0, st, db, da,
                       row_ptr, col_idx, Tt, gt, nnz_cap);
    return hipGetLastError();
  }
  const int sb = lora_db_split(Tt, F), sa = lora_da_split(Tt, d);
  const long long nb = (long long)F * 64, na = (long long)64 * d;
  const TnArgs db = {dZ, U, 64, sb > 1 ? db_part : dB, nb, 64, F / 64, sb};
  const TnArgs da = {G, X, d, sa > 1 ? da_part : dA, na, d, d / 64, sa};
  hipLaunchKernelGGL(lora_tn_kernel<DT>, dim3(db.nx * db.ny + da.nx * da.ny), dim3(kThreads), 0, st, db, da, row_ptr,
                     col_idx, Tt, gt, nnz_cap);
  const long long n4b = sb > 1 ? nb / 4 : 0, n4a = sa > 1 ? na / 4 : 0;
  if (n4b + n4a > 0)
    hipLaunchKernelGGL(lora_grad_reduce_kernel, dim3((unsigned)((n4b + n4a + 255) / 256)), dim3(256), 0,
                       st, (const float*)db_part, sb, n4b, dB, (const float*)da_part, sa, n4a, dA);
  return hipGetLastError();
}
hipError_t launch_lora_grads(int dt, int Tt, int gt, int d, int F, const uint16_t* dZ,
                             const uint16_t* U, const uint16_t* G, const uint16_t* X,
                             const int* row_ptr, const int* col_idx, int nnz_cap, float* da_part,
                             float* db_part, float* dA, float* dB, hipStream_t st) {
  return LX_BY_DT(launch_lora_grads_t, Tt, gt, d, F, dZ, U, G, X, row_ptr, col_idx, nnz_cap, da_part,
                  db_part, dA, dB, st);
}

}  // namespace lx
