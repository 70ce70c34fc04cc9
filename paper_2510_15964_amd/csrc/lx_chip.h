// The chip, for host and device code and for plain C++ (gfx950 only).
#pragma once
#if defined(__HIPCC__)
#define LX_HD __host__ __device__ inline
#else
#define LX_HD inline
#endif
namespace lx {
constexpr int kCUs = 256;   // compute units
}
