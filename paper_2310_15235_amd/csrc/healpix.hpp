// HEALPix pixel of a direction: the FP64 form whose decisions the oracle
// shares, and an FP32 form that gives the same pixel or says that it may not.
#pragma once

#include <cmath>
#include <cstdint>

namespace trevr {

constexpr double kPi = 3.14159265358979323846;

// Square root for the conservative FP32 culling tests: the hardware
// instruction (within about an ulp), far inside their margins; the correctly
// rounded sqrtf expands to a dozen instructions.
__device__ inline float cull_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// HEALPix ring-scheme pixel containing direction v (Gorski et al. 2005).
__device__ inline int healpix_pixel(int N, double x, double y, double zz) {
  const double r = sqrt(x * x + y * y + zz * zz);
  const double z = zz / r;
  const double za = fabs(z);
  double phi = atan2(y, x);
  if (phi < 0.0) phi += 2.0 * kPi;
  const double tt = phi / (0.5 * kPi);
  const int ncap = 2 * N * (N - 1);
  if (za <= 2.0 / 3.0) {
    const double t1 = N * (0.5 + tt);
    const double t2 = N * z * 0.75;
    const long jp = (long)floor(t1 - t2);
    const long jm = (long)floor(t1 + t2);
    const long ir = N + 1 + jp - jm;
    const long kshift = 1 - (ir & 1);
    long ip = (jp + jm - N + kshift + 1) / 2;
    ip = ((ip % (4 * N)) + 4 * N) % (4 * N);
    return (int)(ncap + (ir - 1) * 4 * N + ip);
  }
  const double tp = tt - floor(tt);
  const double tmp = N * sqrt(3.0 * (1.0 - za));
  const long jp = (long)floor(tp * tmp);
  const long jm = (long)floor((1.0 - tp) * tmp);
  const long ir = jp + jm + 1;
  long ip = (long)floor(tt * ir);
  ip = ((ip % (4 * ir)) + 4 * ir) % (4 * ir);
  if (z > 0) return (int)(2 * ir * (ir - 1) + ip);
  return (int)(12 * N * N - 2 * ir * (ir + 1) + ip);
}

// Pixel of direction (x, y, z) as healpix_pixel gives it, in FP32 where that
// decides it surely, -1 where it may not: the floors' arguments must be 1e-5 N
// away from integers and |z| 1e-5 from the belt's edge, several times the
// error of the FP32 values (quarter turns to 2e-7 by a polynomial fitted to
// (2/pi) atan(a)/a, a <= 1; |z| and the cap's root to 1e-6).  The FP64 form's
// arc tangent, root and divisions were a third of what the walk issued (2^18
// elements 1.25 -> 0.85 ms); about one direction in 10^4 needs it now.
__device__ inline int fast_pixel(int N, float x, float y, float z) {
  const float rho2 = x * x + y * y, r2 = rho2 + z * z;
  if (!(r2 > 1e-30f && r2 < 1e30f)) return -1;
  const float ir = __builtin_amdgcn_rsqf(r2);
  const float zn = z * ir, za = fabsf(zn);
  const float ax = fabsf(x), ay = fabsf(y);
  const float a = fminf(ax, ay) * __builtin_amdgcn_rcpf(fmaxf(fmaxf(ax, ay), 1e-30f));
  const float q = a * a;
  float p = -0.0029722690f;
  p = __builtin_fmaf(p, q, 0.0153848557f);
  p = __builtin_fmaf(p, q, -0.0377946161f);
  p = __builtin_fmaf(p, q, 0.0630644932f);
  p = __builtin_fmaf(p, q, -0.0892325044f);
  p = __builtin_fmaf(p, q, 0.1271281391f);
  p = __builtin_fmaf(p, q, -0.2121978551f);
  p = __builtin_fmaf(p, q, 0.6366196871f);
  float tt = p * a;                       // quarter turns, [0, 1/2]
  if (ay > ax) tt = 1.0f - tt;
  if (x < 0.0f) tt = 2.0f - tt;
  if (y < 0.0f) tt = 4.0f - tt;
  const float Nf = (float)N, marg = 1e-5f * Nf;
  const bool belt = za <= 2.0f / 3.0f;
  // the two floors: edges crossed in the belt, or from the pole in a cap
  const float tp = tt - floorf(tt);
  const float root = Nf * cull_sqrt(3.0f * rho2 * ir * ir * __builtin_amdgcn_rcpf(1.0f + za));
  const float u = belt ? Nf * (0.5f + tt) - Nf * zn * 0.75f : tp * root;
  const float v = belt ? Nf * (0.5f + tt) + Nf * zn * 0.75f : (1.0f - tp) * root;
  const float fu = floorf(u), fv = floorf(v);
  const int jp = (int)fu, jm = (int)fv;
  const int ir2 = belt ? N + 1 + jp - jm : jp + jm + 1;   // ring
  const float w = tt * (float)ir2;                        // place in a cap's ring
  const float fw = floorf(w);
  auto sure = [&](float s, float f) { return s - f > marg && s - f < 1.0f - marg; };
  if (!(sure(u, fu) && sure(v, fv) && fabsf(za - 2.0f / 3.0f) > 1e-5f && (belt || sure(w, fw))))
    return -1;
  if (belt) {
    int ip = (jp + jm - N + 1 - (ir2 & 1) + 1) / 2;
    if (ip >= 4 * N) ip -= 4 * N;
    if (ip < 0) ip += 4 * N;
    return 2 * N * (N - 1) + (ir2 - 1) * 4 * N + ip;
  }
  int ip = (int)fw;
  if (ip >= 4 * ir2) ip -= 4 * ir2;
  return z > 0.0f ? 2 * ir2 * (ir2 - 1) + ip : 12 * N * N - 2 * ir2 * (ir2 + 1) + ip;
}

}  // namespace trevr
