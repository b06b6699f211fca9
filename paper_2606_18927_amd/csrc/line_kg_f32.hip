// Line-lane right-hand side, mixed precision, Kennedy-Gruber / Lax-Friedrichs pair.
#include "line_device.hpp"

namespace dg {

hipError_t launch_line_kg_f32(int N, bool rk, const LineLaunch& l, hipStream_t s) {
  return line_dispatch<float, false>(N, rk, LineArgs{l.U, l.ffv, l.out, l.U_out, l.status, *l.m, *l.p, *l.b, *l.st}, s);
}

}  // namespace dg
