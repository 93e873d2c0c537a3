// The double-double operations of the integrated Green's function (ddmath.hpp) evaluated on the
// device, with the hardware reciprocals that the host build replaces, for unit tests of the kernels'
// math.  Not used by libpic.so.
#include "ddmath.hpp"

namespace {

__global__ __launch_bounds__(256) void k_dd(int fn, int count, const double* __restrict__ in,
                                            double* __restrict__ out) {
  const int t = (int)(blockIdx.x * 256 + threadIdx.x);
  if (t >= count) return;
  const pic::ddv a{in[4 * t], in[4 * t + 1]}, b{in[4 * t + 2], in[4 * t + 3]};
  const pic::ddv r = fn == 0   ? pic::dd_log(a)
                     : fn == 1 ? pic::dd_atan2(a, b)
                     : fn == 2 ? pic::dd_sqrt(a)
                               : pic::dd_div(a, b);
  out[2 * t] = r.hi;
  out[2 * t + 1] = r.lo;
}

}  // namespace

// fn 0: log a, 1: atan(a / b), 2: sqrt a, 3: a / b of device pairs in[4k..4k+3] = (a.hi, a.lo, b.hi,
// b.lo) into the device pairs out[2k], out[2k+1]
extern "C" int pic_devcheck_dd(int fn, int count, const double* in, double* out, void* stream) {
  if (fn < 0 || fn > 3 || count < 1 || count > (1 << 24) || !in || !out) return -1;
  hipLaunchKernelGGL(k_dd, dim3((count + 255) / 256), dim3(256), 0, (hipStream_t)stream, fn, count,
                     in, out);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}
