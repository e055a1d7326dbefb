// The FP32 pixel of csrc/healpix.hpp against its FP64 form, on the CPU: the
// hardware's reciprocals and roots (1 ulp) are the exact ones here, moved by up
// to an ulp at random.  Prints directions, undecided ones and wrong pixels per
// N_side.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <random>

#define __device__
static std::mt19937_64 gen(1);
static float ulp(float v) { return v * (1.0f + 1.2e-7f * (float)((int)(gen() % 3) - 1)); }
static float __builtin_amdgcn_rsqf(float x) { return ulp(1.0f / std::sqrt(x)); }
static float __builtin_amdgcn_rcpf(float x) { return ulp(1.0f / x); }
static float __builtin_amdgcn_sqrtf(float x) { return ulp(std::sqrt(x)); }
using std::floor;
using std::fabs;
#include "healpix.hpp"

int main() {
  std::normal_distribution<double> d;
  std::uniform_real_distribution<double> U(-1.0, 1.0);
  for (int N = 1; N <= 16; N *= 2) {
    long unsure = 0, wrong = 0, plain = 0, plain_unsure = 0;
    auto check = [&](double x, double y, double z) {
      const int f = trevr::fast_pixel(N, (float)x, (float)y, (float)z);
      if (f < 0) return true;
      if (f != trevr::healpix_pixel(N, x, y, z)) ++wrong;
      return false;
    };
    for (long i = 0; i < 400000; ++i) {
      double x = d(gen), y = d(gen), z = d(gen);
      ++plain;
      plain_unsure += check(x, y, z);
      switch (i % 8) {   // near the axes, the poles, the diagonals and the belt's edge
        case 0: x *= 1e-6; break;
        case 1: y *= 1e-7; break;
        case 2: x *= 1e-5; y *= 1e-5; break;
        case 3: z *= 1e-7; break;
        case 4: y = x * (1.0 + 1e-7 * U(gen)); break;
        case 5: { const double s = std::exp(20.0 * U(gen)); x *= s; y *= s; z *= s; break; }
        case 6: z = std::copysign(std::sqrt((x * x + y * y) * 0.8) * (1.0 + 1e-5 * U(gen)), z); break;
        default: x = std::round(x); y = std::round(y); z = std::round(z); break;
      }
      if (x != 0.0 || y != 0.0 || z != 0.0) unsure += check(x, y, z);
    }
    std::printf("%d %ld %ld %ld %ld\n", N, plain, plain_unsure, unsure, wrong);
  }
  return 0;
}
