// Line-lane right-hand side, mixed precision, entropy-conserving / Roe pair.
#include "line_device.hpp"

namespace dg {

hipError_t launch_line_ec_f32(int N, bool rk, const LineLaunch& l, hipStream_t s) {
  return line_dispatch<float, true>(N, rk, LineArgs{l.U, l.ffv, l.out, l.U_out, l.status, *l.m, *l.p, *l.b, *l.st}, s);
}

}  // namespace dg
