// Choice between the sum-factorised stage kernels and the others.
#include "dg_device.h"

bool dg::launch_line(const dg_ctx *c, const double *w, double *out, const double *dt, int mode, const Mix &mx,
                     const RateOp &ro, hipStream_t s, int *err) {
  if (ro.op == RATE_NONE && march3d_takes(c)) {
    *err = launch_march3d(c, w, out, dt, mode, mx, s);
    return true;
  }
  if (ro.op == RATE_NONE && split3d_takes(c)) {
    *err = launch_split3d(c, w, out, dt, mode, mx, s);
    return true;
  }
  if (split2d_takes(c)) {
    *err = launch_split2d(c, w, out, dt, mode, mx, ro, s);
    return true;
  }
  return false;
}
