// The chip, for host and device code and for plain C++ (gfx950 only).
#pragma once
namespace lx {
constexpr int kCUs = 256;   // compute units
}
