// How a mask compaction job is divided among workgroups and which of the kernel's ways takes it: rules over sizes and
// strides.  Plain C++.
#pragma once
#include <stdint.h>

namespace lx {

constexpr int kChunkRows = 4096;    // rows scanned per pass (kByRow)
constexpr int kStageBytes = 32768;  // mask bytes staged in LDS per pass (kTurned, kByRow)

// One compaction job: `batch` masks of rows x cols bytes -> one list (see lx_mask_compact).
struct CompactJob {
  const uint8_t* mask;
  int batch, rows, cols;
  long long bstride, rstride, cstride;
  int* row_ptr;
  int* col_idx;
  int cap;
};

// How the bytes of a job lie: the rows of all masks one after the other, or every mask contiguous in
// the other orientation (the column list of contiguous masks), or anything else.
enum MaskLayout { kRowMajor, kColMajor, kStrided };
inline MaskLayout mask_layout(const CompactJob& j) {
  const bool whole = j.batch == 1 || j.bstride == (long long)j.rows * j.cols;
  if (whole && j.cstride == 1 && j.rstride == j.cols) return kRowMajor;
  if (whole && j.rstride == 1 && j.cstride == j.rows) return kColMajor;
  return kStrided;
}
// Workgroups (blockIdx.x = job, blockIdx.y = part of the job's rows): a launch builds one list,
// the row list and the column list of the same masks, or the lists of several independent masks
// side by side.  A large mask is divided by rows; a workgroup that does not start at row 0 first
// counts the active entries of all rows before its own (a plain count over bytes it would otherwise
// wait for another workgroup to scan), so the parts need no communication.  Where several masks that
// fit the stage lie one after the other, the parts are whole masks: what precedes a part is then one
// range of bytes, and the part another, in either orientation (16 bytes per load for both).  A part
// is about 1 KB: both lists of 32 heads of 32 x 32, staged and scanned row by row, took 13 us in eight parts of
// bytes loaded one by one for the column list, 7 in 32 parts (one list 4.5 by the present kernel).  Strided bytes are slow to count, so
// those parts are larger.
// kFlat numbers the bytes of a part in 32 bits: rows one after the other go row by row only where one alone has 2^30 bytes and
// more.  (2^18 rows of 4096 bytes, 1 GiB, flat 25.5 ms, row by row 34.8.)
enum CompactBy { kFlat, kTurned, kByRow };
struct CompactParts {
  int parts, rows;      // rows per part
  int chunk;            // rows per pass (kTurned, kByRow)
  int by, layout;       // CompactBy, MaskLayout
};
constexpr long long kPartBytes = 1ll << 29;      // of a part of many; a row more at most
inline CompactParts compact_parts(const CompactJob& j) {
  const long long total = (long long)j.batch * j.rows, bytes = total * j.cols;
  const MaskLayout lay = mask_layout(j);
  const bool masks = lay != kStrided && j.batch > 1 && j.rows <= kChunkRows && (long long)j.rows * j.cols <= kStageBytes;
  const int unit = masks ? j.rows : 1;
  const bool fast = masks || lay == kRowMajor;
  const long long units = total / unit;
  long long p = (bytes + (fast ? 1023 : 4095)) / (fast ? 1024 : 4096);
  p = p > (fast ? 64 : 16) ? (fast ? 64 : 16) : p;
  if (lay == kRowMajor && bytes > 64 * kPartBytes) p = (bytes + kPartBytes - 1) / kPartBytes;
  p = p > units ? units : p < 1 ? 1 : p;
  const long long per = (units + p - 1) / p;
  CompactParts c = {(int)((units + per - 1) / per), (int)per * unit, 1, kByRow, lay};
  if (lay == kRowMajor && j.cols < 1 << 30) {
    c.by = kFlat;
  } else if (lay == kColMajor && j.rows <= kChunkRows && (long long)j.rows * j.cols <= kStageBytes && c.rows % j.rows == 0) {
    c.by = kTurned;
    c.chunk = kStageBytes / (j.rows * j.cols) * j.rows;
  } else if (j.cols <= kStageBytes) {
    const int fit = kStageBytes / j.cols;
    c.chunk = fit < 1 ? 1 : fit < kChunkRows ? fit : kChunkRows;
  }
  return c;
}

}  // namespace lx
