// Right-hand side on curvilinear elements, FP64, Kennedy-Gruber / Lax-Friedrichs pair.
#include "curv_line.hpp"

namespace dg {

hipError_t launch_curv_kg_f64(int N, bool rk, const LineLaunch& l, hipStream_t s) {
  return curv_line_dispatch<double, false>(N, rk, LineArgs{l.U, l.ffv, l.out, l.U_out, l.status, *l.m, *l.p, *l.b, *l.st}, s);
}

}  // namespace dg
