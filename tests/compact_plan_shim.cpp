// How a compaction job is divided (csrc/compact_plan.h), as a C function.
#include "../paper_2510_15964_amd/csrc/compact_plan.h"

using namespace lx;

extern "C" void parts(int batch, int rows, int cols, long long bs, long long rs, long long cs, int* out) {
  const CompactParts p = compact_parts({nullptr, batch, rows, cols, bs, rs, cs, nullptr, nullptr, 1});
  out[0] = p.parts, out[1] = p.rows, out[2] = p.chunk, out[3] = p.by;
}
