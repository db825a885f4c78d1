// ppe_plan_util.hpp -- host-side FFT factorisation and twiddle tables.
#pragma once

#include <algorithm>
#include <cmath>
#include <vector>

#include "ppe_device.hpp"

namespace ppe {
namespace {

constexpr int kMaxN = 2048;  // longest FFT / y extent supported

// ---------------------------------------------------------------------------
// FFT plans
// ---------------------------------------------------------------------------
struct HostFft {
  int n = 0, e = 1, tc = 1, nst = 0;
  int radix[kMaxStages] = {0};
  int ns[kMaxStages] = {0};
  int tstep[kMaxStages] = {0};
  float inv_ns[kMaxStages] = {0};
  double* tw = nullptr;  // device, 2n doubles
};

inline int gcd_i(int a, int b) { return b ? gcd_i(b, a % b) : a; }

// Radices for n = 2^a 3^b: all 3s first, then 8s (pure powers of two) or 4s,
// then a final 2 or 4.  E = lcm of the radices.  Returns false if n has
// another prime factor.
inline bool fft_factor(int n, HostFft& f) {
  if (n < 1 || n > kMaxN) return false;
  int m = n, a = 0, b = 0;
  while (m % 2 == 0) { m /= 2; ++a; }
  while (m % 3 == 0) { m /= 3; ++b; }
  if (m != 1) return false;
  // (a fixed array: planning allocates no memory)
  int r[kMaxStages + 16];
  int nr = 0;
  for (int q = 0; q < b; ++q) r[nr++] = 3;
  if (b == 0) {
    while (a >= 3) { r[nr++] = 8; a -= 3; }
    if (a == 2) r[nr++] = 4;
    else if (a == 1) r[nr++] = 2;
  } else {
    while (a >= 2) { r[nr++] = 4; a -= 2; }
    if (a == 1) r[nr++] = 2;
  }
  if (nr > kMaxStages) return false;
  int e = 1;
  for (int q = 0; q < nr; ++q) e = e / gcd_i(e, r[q]) * r[q];
  f.n = n;
  f.e = e;
  f.tc = n / e;
  f.nst = nr;
  int ns = 1;
  for (int s = 0; s < f.nst; ++s) {
    f.radix[s] = r[s];
    f.ns[s] = ns;
    f.tstep[s] = n / (ns * r[s]);
    f.inv_ns[s] = 1.0f / (float)ns;
    ns *= r[s];
  }
  return true;
}

// exp(-2 pi i t / n) for t = 0..n-1, computed in extended precision.
inline std::vector<double> twiddles(int n) {
  std::vector<double> w(2 * (size_t)n);
  const long double two_pi = 6.283185307179586476925286766559005768L;
  for (int t = 0; t < n; ++t) {
    // 64-bit-mantissa evaluation, rounded once to double
    const long double a = two_pi * (long double)t / (long double)n;
    w[2 * t] = (double)cosl(a);
    w[2 * t + 1] = (double)(-sinl(a));
  }
  // exact values where the circle hits the axes
  for (int t = 0; t < n; ++t) {
    long long q4 = 4LL * t;
    if (q4 % n == 0) {
      const long long qq = (q4 / n) % 4;
      const double c[4] = {1, 0, -1, 0}, s[4] = {0, -1, 0, 1};
      w[2 * t] = c[qq];
      w[2 * t + 1] = s[qq];
    }
  }
  return w;
}

// ---------------------------------------------------------------------------
// Planes per block of a marching kernel whose instance has `ntile` tiles a
// plane, and planes per record of its partial sums.
//
// kc, the planes a block marches, follows the instances of a launch: a block
// pays about 0.7 of a plane for the planes at its ends, and a grid of a few
// blocks per CU should load the CUs evenly, with at least two on each for their
// loads to overlap (64x64x64 x 8 k_correct 48 -> 40 us, k_resid 16.3 -> 14.1,
// 128x512x96 k_correct 121 -> 111 against 2048 blocks an instance).
//
// kr, the planes of a record, follows the grid alone -- it is the kc of a single
// instance -- and kc is a multiple of it: an instance's sums are split in the
// same way, and so round in the same way, whatever shares its launch.
// ---------------------------------------------------------------------------
struct MarchChunks {
  int kr, kc;
};
inline MarchChunks march_chunks(int ntile, int nz, int nb, int max_planes) {
  const auto best_kc = [&](int instances, int kr) {
    int kc = 0;
    double best = 0.0;
    for (int nkc = (nz + max_planes - 1) / max_planes; nkc <= std::max(1, nz / 2); ++nkc) {
      const int even = (nz + nkc - 1) / nkc, k = (even + kr - 1) / kr * kr;
      const double per_cu = (double)ntile * instances * ((nz + k - 1) / k) / 256.0;
      const double score = per_cu / std::ceil(per_cu) * std::min(1.0, per_cu / 2.0) * even / (k + 0.7);
      if (k <= std::max(max_planes, kr) && score > best * 1.001) {
        best = score;
        kc = k;
      }
    }
    return kc > 0 ? kc : std::max(kr, std::min(nz, max_planes));
  };
  const int kr = best_kc(1, 1);
  return {kr, nb > 1 ? best_kc(nb, kr) : kr};
}

}  // namespace
}  // namespace ppe
