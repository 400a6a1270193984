"""The device formulas of the face flux and the refined roots they use, compiled
for the host: properties that hold for every estimate the hardware may return, so the reciprocal and the
reciprocal root are stand-ins off by as much as an estimate can be (FP64: a
relative 2^-22, refined by the code under test; FP32: one unit in the last
place, used as it is)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2501_15923_amd", "csrc")

RUNTIME = r"""
#pragma once
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>
using std::fabs;
using std::fmax;
using std::fmin;
using std::sqrt;
#define __device__
#define __forceinline__ inline
extern int est_sign;  // which way the estimates are off
inline float next(float x) { return std::nextafterf(x, est_sign > 0 ? INFINITY : 0.f); }
inline double off(double x) { return x * (1.0 + est_sign * 0x1p-22); }
inline double rcp64(double x) { return off(1.0 / x); }
inline double rsq64(double x) { return off(1.0 / std::sqrt(x)); }
inline float rcp32(float x) { return next(1.f / x); }
inline float sqrt32(float x) { return next(std::sqrt(x)); }
inline float rsq32(float x) { return next(1.f / std::sqrt(x)); }
#define __builtin_amdgcn_rcp rcp64
#define __builtin_amdgcn_rsq rsq64
#define __builtin_amdgcn_rcpf rcp32
#define __builtin_amdgcn_sqrtf sqrt32
#define __builtin_amdgcn_rsqf rsq32
"""

MAIN = r"""
#include "icr_device.hpp"
int est_sign = 1;
using namespace icr;
double uni(double a, double b) { return a + (b - a) * (rand() / (double)RAND_MAX); }
// a cell moving at v along component n, faster than its fast speed
template <typename R>
void cell(R (&w)[NV], int n, double v) {
  w[0] = (R)uni(0.5, 2.0);
  for (int q = 1; q < 4; ++q) w[q] = (R)uni(-0.5, 0.5);
  w[n] = (R)(v * uni(1.0, 1.3));
  w[4] = (R)uni(0.1, 0.5);
  for (int q = 5; q < 8; ++q) w[q] = (R)uni(-0.4, 0.4);
}
template <typename R, int N>
int upwind_faces(double v) {
  int wrong = 0;
  for (int q = 0; q < 4000; ++q) {
    R a[NV], b[NV], c[NV], f[NV], g[NV];
    cell<R>(a, N, v);
    cell<R>(b, N, v);
    cell<R>(c, N, v);
    const R gam = R(1.5), igm1 = R(2);
    if (v > 0) {
      face_flux<R, N, FLUX_HLL, true>(a, b, gam, igm1, f);
      face_flux<R, N, FLUX_HLL, true>(a, c, gam, igm1, g);
    } else {
      face_flux<R, N, FLUX_HLL, true>(b, a, gam, igm1, f);
      face_flux<R, N, FLUX_HLL, true>(c, a, gam, igm1, g);
    }
    bool same = f[0] == a[0] * a[N];
    for (int k = 0; k < NV; ++k) same = same && f[k] == g[k];
    wrong += !same;
  }
  return wrong;
}
template <typename R>
int upwind() {
  int n = 0;
  for (int s = -1; s <= 1; s += 2) {
    est_sign = s;
    for (double v : {4.0, -4.0})
      n += upwind_faces<R, 1>(v) + upwind_faces<R, 2>(v) + upwind_faces<R, 3>(v);
  }
  return n;
}
// largest distance in ulps of the refined values from the rounded exact ones
long ulps(double a, long double b) {
  const double r = (double)b;
  long x, y;
  memcpy(&x, &a, 8);
  memcpy(&y, &r, 8);
  return labs(x - y);
}
void refined(long (&most)[3]) {
  for (int s = -1; s <= 1; s += 2) {
    est_sign = s;
    for (int q = 0; q < 200000; ++q) {
      const double x = q % 2 ? uni(1.0, 4.0) : pow(10.0, uni(-280.0, 280.0));
      const long double l = x;
      const long u[3] = {ulps(rcp_fast(x), 1 / l), ulps(sqrt_fast(x), sqrtl(l)),
                         ulps(rsqrt_fast(x), 1 / sqrtl(l))};
      for (int k = 0; k < 3; ++k) most[k] = u[k] > most[k] ? u[k] : most[k];
    }
  }
}
int main() {
  long most[3] = {0, 0, 0};
  refined(most);
  printf("%d %d %ld %ld %ld\n", upwind<double>(), upwind<float>(), most[0], most[1], most[2]);
}
"""


@pytest.fixture(scope="module")
def counts(tmp_path_factory):
    d = tmp_path_factory.mktemp("device_forms")
    os.makedirs(d / "hip")
    (d / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (d / "main.cpp").write_text(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-Wno-unknown-pragmas",
                           f"-I{d}", f"-I{CSRC}", "-o", str(d / "main"), str(d / "main.cpp")])
    return [int(x) for x in subprocess.check_output([str(d / "main")], text=True).split()]


def test_supersonic_hll_face_takes_the_upwind_flux_alone(counts):
    """Mass flux bitwise rho v_n of the upwind state, and no bit of the flux
    depends on the other state, in FP64 and FP32."""
    assert counts[:2] == [0, 0]


def test_refined_reciprocal_and_roots_are_within_one_ulp(counts):
    """1/x, sqrt(x) and 1/sqrt(x) in FP64 from estimates at the end of their
    error range.  One rounding at the end and the one in x y of the residual
    (halved) are 0.75 ulp at most, so one from the rounded exact value."""
    assert max(counts[2:]) <= 1
