// Which attention backward calls run their two sides in one launch.  Plain C++, without the device's headers.
#pragma once

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

}  // namespace lx
