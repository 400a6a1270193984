// icr_device.hpp -- device-side pieces of the heliospheric MHD update for
// CDNA4 (gfx950): state conversions (Eq. 6, mu0 = 1), fast speeds, the
// physical flux of Eqs. (1)-(4), slope limiters, the TVDLF/HLL face flux and
// the cell-centred source terms (spherical geometry, gravity, centrifugal
// and Coriolis force of the co-rotating frame, Sect. 2).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace icr {

constexpr int NV = 8;  // rho, m_r, m_t, m_p, e, B_r, B_t, B_p

enum : int { FLUX_TVDLF = 0, FLUX_HLL = 1, FLUX_HLLD = 2 };
enum : int { LIM_MINMOD = 0, LIM_MC = 1, LIM_WENO5 = 2 };  // WENO5: 3 ghost layers

constexpr int BAD_NONE = 0x7fffffff;

// Device-resident clock and step control.  Written by the kernel that ends a
// step (or reduces a new state's CFL partials) and by the begin-of-call kernel;
// read by every kernel of a step so that no host round trip is needed.
struct DevClock {
  double t;        // current time (code units)
  double dt;       // dt of the next step (clipped to t_end)
  double dt_cfl;   // CFL dt of the next step before clipping
  double t_end;    // <= 0: no end time
  double last_dt;  // dt of the last completed step
  double resid;    // last ||rho^{n+1} - rho^n|| / ||rho^n||
  long long step;  // completed steps
  long long taken; // steps completed in the current icr_step call
  int active;      // 1: the next step advances the state
  int clip;        // 1: the next step ends exactly at t_end
  int bad;         // first invalid cell index or BAD_NONE
  int advanced;    // 1: a step completed since the probe logger last ran
  unsigned int counter;  // arrival counter of the last-block reduction
  int pad0;
  long long n_log;       // probe records written
  long long last_sample; // floor(t / cadence) of the last probe record
};

// Metric factors of one precision (see k_metric for definitions).
template <typename R>
struct Metric {
  const R *rm2, *rp2, *ivr, *hr, *gr, *irc, *grav, *idr, *rc;  // per r cell
  const R *sm, *sp, *ict, *cot, *snc, *csc, *phf, *ilph;  // per theta cell
  R ilth;                                                 // 1 / dtheta
};

// Element idx of a device array: a 32-bit byte offset from a wave-uniform
// base (the grid setup keeps every array below 4 GiB).  Loads of several
// arrays at the same index then share one offset register instead of each
// holding a 64-bit address.
template <typename T>
__device__ __forceinline__ T ldg(const T* base, unsigned idx) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) +
                                     idx * (unsigned)sizeof(T));
}
template <typename T>
__device__ __forceinline__ void stg(T* base, unsigned idx, T x) {
  *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + idx * (unsigned)sizeof(T)) = x;
}

// Reflecting colatitude edges: a row index beyond [0, nt) reads the mirror
// row (-1 - j below, 2 nt - 1 - j above, clamped to the grid) with the theta
// components of velocity and field negated (flip = true).
__device__ __forceinline__ int mirror_row(int j, int nt, bool& flip) {
  flip = j < 0 || j >= nt;
  const int m = j < 0 ? -1 - j : (j >= nt ? 2 * nt - 1 - j : j);
  return m < 0 ? 0 : (m >= nt ? nt - 1 : m);
}

template <typename R>
__device__ __forceinline__ void flip_theta(R (&w)[NV]) {
  w[2] = -w[2];
  w[6] = -w[6];
}

template <typename R>
__device__ __forceinline__ R rmax(R a, R b) { return a > b ? a : b; }
template <typename R>
__device__ __forceinline__ R rmin(R a, R b) { return a < b ? a : b; }

// Reciprocal and square root for the face-once kernel.  FP64: the hardware
// estimate y (relative error e below 2^-22) refined once: reciprocal
// y (1 + e + e^2), third order; square root by one step of Goldschmidt's
// coupled iteration for g ~ sqrt(x), h ~ 1/(2 sqrt(x)) and the residual
// correction g + h (x - g^2), whose two errors of order e^2 multiply.  Both
// end with one rounding of a value right to about 2^-66, like the two
// second-order steps (and, for the root, one correction) that took 4 and 10
// operations instead of 3 and 7.  FP32: the single hardware op.
__device__ __forceinline__ double rcp_fast(double x) {
  const double y = __builtin_amdgcn_rcp(x);
  double e = __builtin_fma(-x, y, 1.0);
  e = __builtin_fma(e, e, e);
  return __builtin_fma(y, e, y);
}
__device__ __forceinline__ float rcp_fast(float x) { return __builtin_amdgcn_rcpf(x); }

__device__ __forceinline__ double sqrt_fast(double x) {  // x > 0
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double r = __builtin_fma(-g, h, 0.5);
  g = __builtin_fma(g, r, g);
  h = __builtin_fma(h, r, h);
  const double d = __builtin_fma(-g, g, x);
  return __builtin_fma(d, h, g);
}
__device__ __forceinline__ float sqrt_fast(float x) { return __builtin_amdgcn_sqrtf(x); }

// Smallest positive argument passed to sqrt_fast for a square root that may
// be exactly zero (keeps the estimate finite; far below any resolved value).
template <typename R>
__device__ __forceinline__ R sqrt_floor();
template <>
__device__ __forceinline__ double sqrt_floor<double>() { return 1e-280; }
template <>
__device__ __forceinline__ float sqrt_floor<float>() { return 1e-30f; }

__device__ __forceinline__ double fma_(double a, double b, double c) {
  return __builtin_fma(a, b, c);
}
__device__ __forceinline__ float fma_(float a, float b, float c) {
  return __builtin_fmaf(a, b, c);
}

template <typename R, bool FAST = false>
__device__ __forceinline__ void cons2prim(const R (&u)[NV], R (&w)[NV], R gm1) {
  const R rho = u[0];
  const R ir = FAST ? rcp_fast(rho) : R(1) / rho;
  w[0] = rho;
  w[1] = u[1] * ir;
  w[2] = u[2] * ir;
  w[3] = u[3] * ir;
  const R kin = R(0.5) * (u[1] * w[1] + u[2] * w[2] + u[3] * w[3]);
  const R mag = R(0.5) * (u[5] * u[5] + u[6] * u[6] + u[7] * u[7]);
  w[4] = gm1 * (u[4] - kin - mag);
  w[5] = u[5];
  w[6] = u[6];
  w[7] = u[7];
}

template <typename R>
__device__ __forceinline__ void prim2cons(const R (&w)[NV], R (&u)[NV], R igm1) {
  const R rho = w[0];
  u[0] = rho;
  u[1] = rho * w[1];
  u[2] = rho * w[2];
  u[3] = rho * w[3];
  const R kin = R(0.5) * (u[1] * w[1] + u[2] * w[2] + u[3] * w[3]);
  const R mag = R(0.5) * (w[5] * w[5] + w[6] * w[6] + w[7] * w[7]);
  u[4] = w[4] * igm1 + kin + mag;
  u[5] = w[5];
  u[6] = w[6];
  u[7] = w[7];
}

// Fast magnetosonic speed along local component N (1..3):
// c_f^2 = [a^2 + b^2 + sqrt((a^2 + b^2)^2 - 4 a^2 B_n^2 / rho)] / 2.
// FAST form, with S = gamma p + B^2 = rho (a^2 + b^2) and b2 = B^2 given:
// c_f^2 = [S + sqrt(S^2 - 4 gamma p B_n^2)] / (2 rho), one division by rho
// instead of one in every term.
template <typename R, int N>
__device__ __forceinline__ R cfast_b2(const R (&w)[NV], R gam, R b2) {
  const R gp = gam * w[4];
  const R S = gp + b2;
  const R bn = w[4 + N];
  // floors keep exact zeros (possible only for invalid states) at ~0
  const R D = rmax(fma_(R(-4) * gp, bn * bn, S * S), sqrt_floor<R>());
  return sqrt_fast(rmax(R(0.5) * (S + sqrt_fast(D)) * rcp_fast(w[0]), sqrt_floor<R>()));
}
template <typename R>
__device__ __forceinline__ R field2(const R (&w)[NV]) {
  return fma_(w[7], w[7], fma_(w[6], w[6], w[5] * w[5]));
}

template <typename R, int N, bool FAST = false>
__device__ __forceinline__ R cfast(const R (&w)[NV], R gam) {
  if constexpr (FAST) return cfast_b2<R, N>(w, gam, field2<R>(w));
  const R ir = R(1) / w[0];
  const R a2 = gam * w[4] * ir;
  const R b2 = (w[5] * w[5] + w[6] * w[6] + w[7] * w[7]) * ir;
  const R bn = w[4 + N];
  const R s = a2 + b2;
  const R disc = rmax(s * s - R(4) * a2 * bn * bn * ir, R(0));
  return sqrt(R(0.5) * (s + sqrt(disc)));
}

// Physical flux through a face normal to local component N.
template <typename R, int N>
__device__ __forceinline__ void phys_flux(const R (&w)[NV], const R (&u)[NV], R (&f)[NV]) {
  const R vn = w[N], bn = w[4 + N];
  const R ptot = w[4] + R(0.5) * (w[5] * w[5] + w[6] * w[6] + w[7] * w[7]);
  const R vb = w[1] * w[5] + w[2] * w[6] + w[3] * w[7];
  f[0] = w[0] * vn;
#pragma unroll
  for (int d = 1; d <= 3; ++d) f[d] = u[d] * vn - bn * w[4 + d];
  f[N] += ptot;
  f[4] = (u[4] + ptot) * vn - bn * vb;
#pragma unroll
  for (int d = 1; d <= 3; ++d) f[4 + d] = vn * w[4 + d] - bn * w[d];
}

// minmod(a, b): 0 if a b <= 0, else the argument of smaller magnitude.
// MC(a, b): 0 if a b <= 0, else sign(a) min(2|a|, 2|b|, |a + b|/2).
template <typename R, int LIM>
__device__ __forceinline__ R limiter(R a, R b) {
  if (a * b <= R(0)) return R(0);
  if (LIM == LIM_MINMOD) return fabs(a) < fabs(b) ? a : b;
  R m = rmin(R(2) * fabs(a), R(2) * fabs(b));
  m = rmin(m, R(0.5) * fabs(a + b));
  return a > R(0) ? m : -m;
}

// Half the limited slope of a cell with one-sided differences x and y, where
// lo, hi = min(y, 0), max(y, 0) (shared by the two cells of a face, y being
// the difference across it).  minmod(x, y) is the median of x, y and 0, i.e.
// x clamped to [lo, hi]; MC / 2 = sign min(|x|, |y|, |x + y|/4) is (x + y)/4
// clamped to the interval between 0 and that minmod.  Branch-free, and the
// same values as the definitions above.  FP32 has a median instruction for
// each clamp; FP64, which has none, takes the smaller magnitude with the
// minmod's sign, two instructions where the second clamp took four (FP64 MC
// stage 2281 -> 2153 instructions a cell; in FP32 that form costs 5 % more).
template <typename R, int LIM>
__device__ __forceinline__ R half_slope(R x, R y, R lo, R hi) {
  const R m = fmax(lo, fmin(x, hi));
  if (LIM == LIM_MINMOD) return R(0.5) * m;
  const R c = R(0.25) * (x + y);
  if constexpr (sizeof(R) == 8) return __builtin_copysign(fmin(fabs(m), fabs(c)), m);
  return fmax(fmin(m, R(0)), fmin(c, fmax(m, R(0))));
}

// Face states from four consecutive cells (m-2, m-1, m, m+1) around face
// m-1/2: W_L = W_{m-1} + s_{m-1}/2, W_R = W_m - s_m/2, limited undivided
// slopes on primitives.
template <typename R, int LIM, bool FAST>
__device__ __forceinline__ void face_states(R a, R b, R c, R d, R& wl, R& wr) {
  const R db = b - a, dc = c - b, dd = d - c;
  if constexpr (FAST) {
    const R lo = fmin(dc, R(0)), hi = fmax(dc, R(0));
    if (LIM == LIM_MINMOD) {  // (one fused multiply-add with the half)
      wl = fma_(R(0.5), fmax(lo, fmin(db, hi)), b);
      wr = fma_(R(-0.5), fmax(lo, fmin(dd, hi)), c);
    } else {
      wl = b + half_slope<R, LIM>(db, dc, lo, hi);
      wr = c - half_slope<R, LIM>(dd, dc, lo, hi);
    }
  } else {
    wl = b + R(0.5) * limiter<R, LIM>(db, dc);
    wr = c - R(0.5) * limiter<R, LIM>(dc, dd);
  }
}
// A cell's states at its lower and upper face from its value w and the
// differences x (to the cell below) and y (to the cell above): the values
// face_states gives its two faces.
template <typename R, int LIM>
__device__ __forceinline__ void cell_states(R w, R x, R y, R& dn, R& up) {
  const R lo = fmin(y, R(0)), hi = fmax(y, R(0));
  if (LIM == LIM_MINMOD) {
    const R m = fmax(lo, fmin(x, hi));
    dn = fma_(R(-0.5), m, w);
    up = fma_(R(0.5), m, w);
  } else {
    const R h = half_slope<R, LIM>(x, y, lo, hi);
    dn = w - h;
    up = w + h;
  }
}
template <typename R, int LIM, bool FAST = false>
__device__ __forceinline__ void reconstruct(const R (&a)[NV], const R (&b)[NV],
                                            const R (&c)[NV], const R (&d)[NV],
                                            R (&wl)[NV], R (&wr)[NV]) {
#pragma unroll
  for (int v = 0; v < NV; ++v)
    face_states<R, LIM, FAST>(a[v], b[v], c[v], d[v], wl[v], wr[v]);
}

// WENO5 (Jiang & Shu 1996) value at the face between cells c and d from the
// five cells a..e: the three third-order candidates of the stencils ending
// at, centred on and starting at c, weighted by d_k / (eps + beta_k)^2 with
// linear weights (1, 6, 3)/10 and smoothness indicators beta_k; eps is 1e-6
// of the stencil's mean square (plus 1e-40), so the weights are free of units.
template <typename R, bool FAST = false>
__device__ __forceinline__ R weno5(R a, R b, R c, R d, R e) {
  constexpr R sixth = R(1) / R(6);
  const R q0 = (R(2) * a - R(7) * b + R(11) * c) * sixth;
  const R q1 = (-b + R(5) * c + R(2) * d) * sixth;
  const R q2 = (R(2) * c + R(5) * d - e) * sixth;
  const R s0 = a - R(2) * b + c, t0 = a - R(4) * b + R(3) * c;
  const R s1 = b - R(2) * c + d, t1 = b - d;
  const R s2 = c - R(2) * d + e, t2 = R(3) * c - R(4) * d + e;
  const R b0 = R(13) / R(12) * s0 * s0 + R(0.25) * t0 * t0;
  const R b1 = R(13) / R(12) * s1 * s1 + R(0.25) * t1 * t1;
  const R b2 = R(13) / R(12) * s2 * s2 + R(0.25) * t2 * t2;
  // absolute floor: (floor)^2 must stay a normal number (FP32: 1e-15)
  const R eps = R(1e-6) * (a * a + b * b + c * c + d * d + e * e) * R(0.2) +
                (sizeof(R) == 8 ? R(1e-40) : R(1e-15));
  const R g0 = (eps + b0) * (eps + b0), g1 = (eps + b1) * (eps + b1), g2 = (eps + b2) * (eps + b2);
  if constexpr (sizeof(R) == 8) {
    // weights d_k / g_k scaled by g0 g1 g2: one division (products stay in
    // range in FP64: g >= 1e-80)
    const R a0 = R(0.1) * g1 * g2, a1 = R(0.6) * g0 * g2, a2 = R(0.3) * g0 * g1;
    if constexpr (FAST) return (a0 * q0 + a1 * q1 + a2 * q2) * rcp_fast(a0 + a1 + a2);
    return (a0 * q0 + a1 * q1 + a2 * q2) / (a0 + a1 + a2);
  } else {
    const R a0 = R(0.1) / g0, a1 = R(0.6) / g1, a2 = R(0.3) / g2;
    return (a0 * q0 + a1 * q1 + a2 * q2) / (a0 + a1 + a2);
  }
}

// WENO5 face states of face m-1/2 from the six cells m-3 .. m+2 (p0..p5);
// a face state with rho or p <= 0 falls back to its cell value.
template <typename R, bool FAST = false>
__device__ __forceinline__ void reconstruct_weno5(const R (&p0)[NV], const R (&p1)[NV],
                                                  const R (&p2)[NV], const R (&p3)[NV],
                                                  const R (&p4)[NV], const R (&p5)[NV],
                                                  R (&wl)[NV], R (&wr)[NV]) {
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    wl[v] = weno5<R, FAST>(p0[v], p1[v], p2[v], p3[v], p4[v]);
    wr[v] = weno5<R, FAST>(p5[v], p4[v], p3[v], p2[v], p1[v]);
  }
  if (!(wl[0] > R(0) && wl[4] > R(0)))
#pragma unroll
    for (int v = 0; v < NV; ++v) wl[v] = p2[v];
  if (!(wr[0] > R(0) && wr[4] > R(0)))
#pragma unroll
    for (int v = 0; v < NV; ++v) wr[v] = p3[v];
}

// Numerical flux from the two face states: TVDLF
// F = (F_L + F_R)/2 - alpha (U_R - U_L)/2, alpha = max(|v_n| + c_f), or HLL
// with S_L = min(v_nL - c_fL, v_nR - c_fR), S_R = max(v_nL + c_fL, ...).
// HLLD flux (Miyoshi & Kusano 2005) through a face with normal component N:
// the outer fast waves, the two rotational waves and the contact bound four
// intermediate states sharing the contact speed S_M and total pressure;
// density is continuous across the rotational waves.  Both face states use
// the mean normal field; the normal field's own flux is the HLL value with
// the same outer speeds.
template <typename R, int N>
__device__ __forceinline__ void hlld_flux(const R (&wl0)[NV], const R (&wr0)[NV], R gam, R igm1,
                                          R (&fs)[NV]) {
  constexpr int T1 = N == 1 ? 2 : 1, T2 = N == 3 ? 2 : 3;
  auto rcp = [](R x) { return R(1) / x; };
  const R bn = R(0.5) * (wl0[4 + N] + wr0[4 + N]);
  const R dbn = wr0[4 + N] - wl0[4 + N];
  R w[2][NV], u[2][NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    w[0][v] = wl0[v];
    w[1][v] = wr0[v];
  }
  w[0][4 + N] = bn;
  w[1][4 + N] = bn;
  prim2cons<R>(w[0], u[0], igm1);
  prim2cons<R>(w[1], u[1], igm1);
  const R cmax = rmax(cfast<R, N>(w[0], gam), cfast<R, N>(w[1], gam));
  const R sl = rmin(w[0][N], w[1][N]) - cmax, sr = rmax(w[0][N], w[1][N]) + cmax;
  const R fbn = (sl < R(0) && sr > R(0)) ? sl * sr * dbn * rcp(sr - sl) : R(0);
  // every region's flux needs the physical flux of one side only
  if (sl >= R(0) || sr <= R(0)) {
    const bool left = sl >= R(0);
    R wa[NV], ua[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      wa[v] = left ? w[0][v] : w[1][v];
      ua[v] = left ? u[0][v] : u[1][v];
    }
    phys_flux<R, N>(wa, ua, fs);
    fs[4 + N] = fbn;
    return;
  }
  R pt[2], d[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    pt[a] = w[a][4] + R(0.5) * (w[a][5] * w[a][5] + w[a][6] * w[a][6] + w[a][7] * w[a][7]);
    d[a] = ((a ? sr : sl) - w[a][N]) * w[a][0];  // mass flux relative to the outer wave
  }
  const R idd = rcp(d[1] - d[0]);
  const R sm = (d[1] * w[1][N] - d[0] * w[0][N] - pt[1] + pt[0]) * idd;
  const R pts = (d[1] * pt[0] - d[0] * pt[1] + d[0] * d[1] * (w[1][N] - w[0][N])) * idd;
  // outer star states of both sides (the double-star state needs both)
  R us[2][NV], sq[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const R s = a ? sr : sl;
    const R ism = rcp(s - sm);
    const R rho = d[a] * ism;
    const R den = d[a] * (s - sm) - bn * bn;
    R vt1 = w[a][T1], vt2 = w[a][T2], bt1 = w[a][4 + T1], bt2 = w[a][4 + T2];
    if (fabs(den) > R(1e-12) * (fabs(d[a] * (s - sm)) + bn * bn)) {
      const R iden = rcp(den);
      const R fv = bn * (sm - w[a][N]) * iden;
      const R fb = (d[a] * (s - w[a][N]) - bn * bn) * iden;
      vt1 -= bt1 * fv;
      vt2 -= bt2 * fv;
      bt1 *= fb;
      bt2 *= fb;
    }
    const R vb = w[a][1] * w[a][5] + w[a][2] * w[a][6] + w[a][3] * w[a][7];
    const R vbs = sm * bn + vt1 * bt1 + vt2 * bt2;
    us[a][0] = rho;
    us[a][N] = rho * sm;
    us[a][T1] = rho * vt1;
    us[a][T2] = rho * vt2;
    us[a][4] = ((s - w[a][N]) * u[a][4] - pt[a] * w[a][N] + pts * sm + bn * (vb - vbs)) * ism;
    us[a][4 + N] = bn;
    us[a][4 + T1] = bt1;
    us[a][4 + T2] = bt2;
    sq[a] = sqrt(rho);
  }
  // the side of the contact the face lies on: F*_a = F_a + S_a (U*_a - U_a)
  const bool left = sm >= R(0);
  R q[NV], fa[NV];
  {
    R wa[NV], ua[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      wa[v] = left ? w[0][v] : w[1][v];
      ua[v] = left ? u[0][v] : u[1][v];
      q[v] = left ? us[0][v] : us[1][v];
    }
    phys_flux<R, N>(wa, ua, fa);
    const R sa = left ? sl : sr;
#pragma unroll
    for (int v = 0; v < NV; ++v) fa[v] += sa * (q[v] - ua[v]);
  }
  const R ssl = sm - fabs(bn) * rcp(sq[0]), ssr = sm + fabs(bn) * rcp(sq[1]);
  if (ssl >= R(0) || ssr <= R(0)) {
#pragma unroll
    for (int v = 0; v < NV; ++v) fs[v] = fa[v];
    fs[4 + N] = fbn;
    return;
  }
  // double-star state between the rotational waves
  const R sg = bn >= R(0) ? R(1) : R(-1);
  const R isq = rcp(sq[0] + sq[1]);
  const R vl1 = us[0][T1] / us[0][0], vl2 = us[0][T2] / us[0][0];
  const R vr1 = us[1][T1] / us[1][0], vr2 = us[1][T2] / us[1][0];
  const R v1 = (sq[0] * vl1 + sq[1] * vr1 + (us[1][4 + T1] - us[0][4 + T1]) * sg) * isq;
  const R v2 = (sq[0] * vl2 + sq[1] * vr2 + (us[1][4 + T2] - us[0][4 + T2]) * sg) * isq;
  const R b1 = (sq[0] * us[1][4 + T1] + sq[1] * us[0][4 + T1] + sq[0] * sq[1] * (vr1 - vl1) * sg) *
               isq;
  const R b2 = (sq[0] * us[1][4 + T2] + sq[1] * us[0][4 + T2] + sq[0] * sq[1] * (vr2 - vl2) * sg) *
               isq;
  const R vbs = (q[N] * q[4 + N] + q[T1] * q[4 + T1] + q[T2] * q[4 + T2]) / q[0];
  const R vbss = sm * bn + v1 * b1 + v2 * b2;
  R uss[NV];
  uss[0] = q[0];
  uss[N] = q[0] * sm;
  uss[T1] = q[0] * v1;
  uss[T2] = q[0] * v2;
  uss[4] = q[4] + (left ? -sq[0] : sq[1]) * (vbs - vbss) * sg;
  uss[4 + N] = bn;
  uss[4 + T1] = b1;
  uss[4 + T2] = b2;
  const R ssa = left ? ssl : ssr;
#pragma unroll
  for (int v = 0; v < NV; ++v) fs[v] = fa[v] + ssa * (uss[v] - q[v]);
  fs[4 + N] = fbn;
}

// 1 / sqrt(x), x > 0: the hardware estimate y refined by y (1 + e/2 + 3 e^2/8),
// e = 1 - x y^2.
__device__ __forceinline__ double rsqrt_fast(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = __builtin_fma(-x * y, y, 1.0);
  return __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
}
__device__ __forceinline__ float rsqrt_fast(float x) { return __builtin_amdgcn_rsqf(x); }

// The same flux for the face-once kernels.  Each region's flux is the physical
// flux of its state (the jump conditions hold across every wave by
// construction), with the contact speed and the shared total pressure in the
// star regions: so the state at the face is selected first and one flux
// formed, energies included; only the transverse star states are needed from
// both sides.  Where a side's transverse jump is degenerate it keeps v_t and
// B_t, and its induction flux the side's own v_n.  Faces outside the fan (the
// radial ones in supersonic wind) and those outside the rotational waves leave
// early: without these two branches the step below was 2.5 % slower than with
// the general form, although it counts fewer operations.  The stage kernels
// are bound by VALU issue: 2281 instructions a cell (FP64, MC) instead of
// 3014, a step at 331 x 47 x 91 with the tracer 364 us instead of 391.
template <typename R, int N>
__device__ __forceinline__ void hlld_flux_fast(const R (&wl)[NV], const R (&wr)[NV], R gam, R igm1,
                                               R (&fs)[NV]) {
  constexpr int T1 = N == 1 ? 2 : 1, T2 = N == 3 ? 2 : 3;
  constexpr R half = R(0.5);
  const R bn = half * (wl[4 + N] + wr[4 + N]), bn2 = bn * bn, abn = fabs(bn);
  const R dbn = wr[4 + N] - wl[4 + N];
  const R (*w[2])[NV] = {&wl, &wr};
  R b2[2], pt[2], c[2];
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const R* q = *w[a];
    b2[a] = fma_(q[4 + T2], q[4 + T2], fma_(q[4 + T1], q[4 + T1], bn2));
    pt[a] = fma_(half, b2[a], q[4]);
    const R gp = gam * q[4], S = gp + b2[a];
    const R D = rmax(fma_(R(-4) * gp, bn2, S * S), sqrt_floor<R>());
    c[a] = half * (S + sqrt_fast(D)) * rcp_fast(q[0]);
  }
  // the larger fast speed needs one outer root only
  const R cmax = sqrt_fast(rmax(rmax(c[0], c[1]), sqrt_floor<R>()));
  const R vl = wl[N], vr = wr[N];
  const R sl = rmin(vl, vr) - cmax, sr = rmax(vl, vr) + cmax;
  const R dl = (sl - vl) * wl[0], dr = (sr - vr) * wr[0];  // mass flux relative to the outer wave
  const R sm = fma_(dr, vr, fma_(-dl, vl, pt[0] - pt[1])) * rcp_fast(dr - dl);
  const bool outer = sl >= R(0) || sr <= R(0);
  // the side of the contact the face lies on
  const bool left = sl >= R(0) || (sr > R(0) && sm >= R(0));
  R u[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) u[v] = left ? wl[v] : wr[v];
  R P = left ? pt[0] : pt[1];
  const R b2u = left ? b2[0] : b2[1];
  const R k2 = fma_(u[0], fma_(u[3], u[3], fma_(u[2], u[2], u[1] * u[1])), b2u);
  R E = fma_(half, k2, u[4] * igm1);
  R vb = fma_(u[T2], u[4 + T2], fma_(u[T1], u[4 + T1], u[N] * bn));
  R V = u[N], m = u[0] * V, v1 = u[T1], v2 = u[T2], b1 = u[4 + T1], b3 = u[4 + T2];
  R f1 = fma_(V, b1, -bn * v1), f2 = fma_(V, b3, -bn * v2);
  fs[4 + N] = R(0);
  if (!outer) {
    fs[4 + N] = sl * sr * dbn * rcp_fast(sr - sl);
    const R pts = fma_(dl, sm - vl, pt[0]);
    // transverse star states of both sides
    R rho[2], y[2], vt[2][2], bt[2][2];
    bool keep[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      const R* q = *w[a];
      const R s = a ? sr : sl, d = a ? dr : dl, ds = d * (s - sm);
      rho[a] = d * rcp_fast(s - sm);
      y[a] = rsqrt_fast(rho[a]);
      const R den = ds - bn2;
      keep[a] = !(fabs(den) > R(1e-12) * (fabs(ds) + bn2));
      const R id = rcp_fast(den);
      const R fv = keep[a] ? R(0) : bn * (sm - q[N]) * id;
      const R fb = keep[a] ? R(1) : (d * (s - q[N]) - bn2) * id;
      vt[a][0] = fma_(-q[4 + T1], fv, q[T1]);
      vt[a][1] = fma_(-q[4 + T2], fv, q[T2]);
      bt[a][0] = q[4 + T1] * fb;
      bt[a][1] = q[4 + T2] * fb;
    }
    const R su = left ? sl : sr;
    v1 = left ? vt[0][0] : vt[1][0];
    v2 = left ? vt[0][1] : vt[1][1];
    b1 = left ? bt[0][0] : bt[1][0];
    b3 = left ? bt[0][1] : bt[1][1];
    const R vbs = fma_(v2, b3, fma_(v1, b1, sm * bn));
    E = fma_(su - V, E, fma_(-P, V, fma_(pts, sm, bn * (vb - vbs)))) * rcp_fast(su - sm);
    const R vi = (left ? keep[0] : keep[1]) ? V : sm;
    f1 = fma_(vi, b1, -bn * v1);
    f2 = fma_(vi, b3, -bn * v2);
    V = sm;
    P = pts;
    m = (left ? rho[0] : rho[1]) * sm;
    vb = vbs;
    // double-star state between the rotational waves
    const R ssl = fma_(-abn, y[0], sm), ssr = fma_(abn, y[1], sm);
    if (ssl < R(0) && ssr > R(0)) {
      const R ql = rho[0] * y[0], qr = rho[1] * y[1];
      const R sg = bn >= R(0) ? R(1) : R(-1);
      const R isq = rcp_fast(ql + qr), qq = ql * qr * sg;
      const R x1 = (fma_(ql, vt[0][0], qr * vt[1][0]) + (bt[1][0] - bt[0][0]) * sg) * isq;
      const R x2 = (fma_(ql, vt[0][1], qr * vt[1][1]) + (bt[1][1] - bt[0][1]) * sg) * isq;
      const R z1 = fma_(ql, bt[1][0], fma_(qr, bt[0][0], qq * (vt[1][0] - vt[0][0]))) * isq;
      const R z2 = fma_(ql, bt[1][1], fma_(qr, bt[0][1], qq * (vt[1][1] - vt[0][1]))) * isq;
      vb = fma_(x2, z2, fma_(x1, z1, sm * bn));
      const R ss = left ? ssl : ssr;
      E = fma_((left ? -ql : qr) * sg, vbs - vb, E);
      f1 = fma_(ss, z1 - b1, f1);
      f2 = fma_(ss, z2 - b3, f2);
      v1 = x1;
      v2 = x2;
      b1 = z1;
      b3 = z2;
    }
  }
  fs[0] = m;
  fs[N] = fma_(m, V, P - bn2);
  fs[T1] = fma_(m, v1, -bn * b1);
  fs[T2] = fma_(m, v2, -bn * b3);
  fs[4] = fma_(E + P, V, -bn * vb);
  fs[4 + T1] = f1;
  fs[4 + T2] = f2;
}

// TVDLF and HLL in one form for the face-once kernels: with the bounding
// speeds s_L = -alpha, s_R = alpha (TVDLF) or s_L = min(S_L, 0), s_R =
// max(S_R, 0) (HLL, whose one-sided cases are then included) and the weights
// h_R = -s_L / (s_R - s_L), h_L = 1 - h_R,
//   F = h_L (F_L - s_L U_L) + h_R (F_R - s_R U_R).
// A flux component is u v_n plus magnetic and pressure terms, so each side's
// F - s U needs u (v_n - s) only: neither the physical fluxes nor the
// momenta are formed.  About 215 FP64 operations a face with minmod states,
// where separate fluxes, states and their differences took about 285; with
// the stage kernels bound by VALU issue the step at 600 x 60 x 120 went from
// 0.66 to 0.59 ms (FP64, minmod + TVDLF) and 0.35 to 0.31 ms (FP32, MC +
// HLL), the error against a 64-bit reference staying where it was.
template <typename R, int N, int FLUX>
__device__ __forceinline__ void two_wave_flux(const R (&wl)[NV], const R (&wr)[NV], R gam, R igm1,
                                              R (&fs)[NV]) {
  constexpr R half = R(0.5);
  const R b2l = field2<R>(wl), b2r = field2<R>(wr);
  const R cl = cfast_b2<R, N>(wl, gam, b2l), cr = cfast_b2<R, N>(wr, gam, b2r);
  R sl, sr, hl, hr;
  if constexpr (FLUX == FLUX_TVDLF) {
    sr = rmax(fabs(wl[N]) + cl, fabs(wr[N]) + cr);
    sl = -sr;
    hl = hr = half;
  } else {
    sl = rmin(rmin(wl[N] - cl, wr[N] - cr), R(0));
    sr = rmax(rmax(wl[N] + cl, wr[N] + cr), R(0));
    // one-sided cases exactly: a product of s_R and the reciprocal of s_R is
    // 1 to an ulp only, and the upwind flux would carry that error
    hr = sr > R(0) ? -sl * rcp_fast(sr - sl) : R(1);
    hl = R(1) - hr;
  }
  const R al = hl * (wl[N] - sl), ar = hr * (wr[N] - sr);
  const R bl = hl * wl[4 + N], br = hr * wr[4 + N];
  // densities of kinetic + magnetic energy (twice) and of the total
  const R kl = wl[0] * fma_(wl[3], wl[3], fma_(wl[2], wl[2], wl[1] * wl[1])) + b2l;
  const R kr = wr[0] * fma_(wr[3], wr[3], fma_(wr[2], wr[2], wr[1] * wr[1])) + b2r;
  const R el = fma_(half, kl, wl[4] * igm1), er = fma_(half, kr, wr[4] * igm1);
  const R pl = hl * fma_(half, b2l, wl[4]), pr = hr * fma_(half, b2r, wr[4]);
  const R vbl = fma_(wl[3], wl[7], fma_(wl[2], wl[6], wl[1] * wl[5]));
  const R vbr = fma_(wr[3], wr[7], fma_(wr[2], wr[6], wr[1] * wr[5]));
  const R ml = wl[0] * al, mr = wr[0] * ar;
  fs[0] = ml + mr;
#pragma unroll
  for (int d = 1; d <= 3; ++d)
    fs[d] = fma_(ml, wl[d], fma_(mr, wr[d], -fma_(bl, wl[4 + d], br * wr[4 + d])));
  fs[N] += pl + pr;
  fs[4] = fma_(el, al, fma_(pl, wl[N], -bl * vbl)) + fma_(er, ar, fma_(pr, wr[N], -br * vbr));
#pragma unroll
  for (int d = 1; d <= 3; ++d)
    fs[4 + d] = d == N ? -fma_(bl, sl, br * sr)
                       : fma_(al, wl[4 + d], fma_(ar, wr[4 + d], -fma_(bl, wl[d], br * wr[d])));
}

template <typename R, int N, int FLUX, bool FAST = false>
__device__ __forceinline__ void face_flux(const R (&wl)[NV], const R (&wr)[NV],
                                          R gam, R igm1, R (&fs)[NV]) {
  if constexpr (FLUX == FLUX_HLLD) {
    if constexpr (FAST)
      hlld_flux_fast<R, N>(wl, wr, gam, igm1, fs);
    else
      hlld_flux<R, N>(wl, wr, gam, igm1, fs);
    return;
  } else if constexpr (FAST) {
    two_wave_flux<R, N, FLUX>(wl, wr, gam, igm1, fs);
    return;
  }
  R ul[NV], ur[NV], fl[NV], fr[NV];
  prim2cons<R>(wl, ul, igm1);
  prim2cons<R>(wr, ur, igm1);
  phys_flux<R, N>(wl, ul, fl);
  phys_flux<R, N>(wr, ur, fr);
  const R cl = cfast<R, N>(wl, gam), cr = cfast<R, N>(wr, gam);
  if (FLUX == FLUX_TVDLF) {
    const R alpha = rmax(fabs(wl[N]) + cl, fabs(wr[N]) + cr);
#pragma unroll
    for (int v = 0; v < NV; ++v)
      fs[v] = R(0.5) * (fl[v] + fr[v]) - R(0.5) * alpha * (ur[v] - ul[v]);
  } else {
    const R sl = rmin(wl[N] - cl, wr[N] - cr);
    const R sr = rmax(wl[N] + cl, wr[N] + cr);
    if (sl >= R(0)) {
#pragma unroll
      for (int v = 0; v < NV; ++v) fs[v] = fl[v];
    } else if (sr <= R(0)) {
#pragma unroll
      for (int v = 0; v < NV; ++v) fs[v] = fr[v];
    } else {
      const R id = R(1) / (sr - sl);
#pragma unroll
      for (int v = 0; v < NV; ++v)
        fs[v] = (sr * fl[v] - sl * fr[v] + sl * sr * (ur[v] - ul[v])) * id;
    }
  }
}

// Cell-centred sources: spherical geometric terms with area-difference
// pressure factors G_r = dA_r/V, H_r*cot(theta_c) = dA_theta/V; gravity
// g = -GM/r^2 e_r (momentum rho g, energy rho v.g); co-rotating frame with
// Omega along the polar axis: F = rho (Omega x r) x Omega + 2 rho v x Omega
// and energy source v.F.
//
// The metric factors of the cell come through an accessor: CellMetric reads
// the global arrays at (i, j); the face-once stage kernel passes one that
// reads its tile's copy in LDS (the same values).
enum MetricR { MR_RM2, MR_RP2, MR_IVR, MR_HR, MR_GR, MR_IRC, MR_GRAV, MR_IDR, MR_RC, MR_N };
enum MetricT { MT_SM, MT_SP, MT_ICT, MT_COT, MT_SNC, MT_CSC, MT_PHF, MT_ILPH, MT_N };

template <typename R>
__device__ __forceinline__ const R* metric_r(const Metric<R>& m, int a) {
  switch (a) {
    case MR_RM2: return m.rm2;
    case MR_RP2: return m.rp2;
    case MR_IVR: return m.ivr;
    case MR_HR: return m.hr;
    case MR_GR: return m.gr;
    case MR_IRC: return m.irc;
    case MR_GRAV: return m.grav;
    case MR_IDR: return m.idr;
    default: return m.rc;
  }
}
template <typename R>
__device__ __forceinline__ const R* metric_t(const Metric<R>& m, int a) {
  switch (a) {
    case MT_SM: return m.sm;
    case MT_SP: return m.sp;
    case MT_ICT: return m.ict;
    case MT_COT: return m.cot;
    case MT_SNC: return m.snc;
    case MT_CSC: return m.csc;
    case MT_PHF: return m.phf;
    default: return m.ilph;
  }
}

template <typename R>
struct CellMetric {
  const Metric<R>& m;
  int i, j;
  __device__ __forceinline__ R r(int a) const { return ldg(metric_r(m, a), (unsigned)i); }
  __device__ __forceinline__ R t(int a) const { return ldg(metric_t(m, a), (unsigned)j); }
  __device__ __forceinline__ R ilth() const { return m.ilth; }
};

template <typename R, typename CM>
__device__ __forceinline__ void add_sources_cm(const R (&w)[NV], const CM& cm, R omega,
                                               int gravity, int corot, R (&L)[NV]) {
  const R rho = w[0], vr = w[1], vt = w[2], vp = w[3], p = w[4];
  const R br = w[5], bt = w[6], bp = w[7];
  const R irc = cm.r(MR_IRC);
  const R cot = cm.t(MT_COT);
  const R ptot = p + R(0.5) * (br * br + bt * bt + bp * bp);
  L[1] += (rho * (vt * vt + vp * vp) - (bt * bt + bp * bp)) * irc + ptot * cm.r(MR_GR);
  L[2] += (-(rho * vr * vt - br * bt) + cot * (rho * vp * vp - bp * bp)) * irc +
          ptot * cm.r(MR_HR) * cot;
  L[3] -= ((rho * vp * vr - bp * br) + cot * (rho * vp * vt - bp * bt)) * irc;
  L[6] += (vr * bt - vt * br) * irc;
  L[7] += ((vr * bp - vp * br) + cot * (vt * bp - vp * bt)) * irc;
  if (gravity) {
    const R g = cm.r(MR_GRAV);
    L[1] += rho * g;
    L[4] += rho * vr * g;
  }
  if (corot) {
    const R sn = cm.t(MT_SNC), cs = cm.t(MT_CSC);
    const R r = cm.r(MR_RC);
    const R cen = rho * omega * omega * r * sn;
    const R cor = R(2) * rho * omega;
    L[1] += cen * sn + cor * vp * sn;
    L[2] += cen * cs + cor * vp * cs;
    L[3] -= cor * (vr * sn + vt * cs);
    L[4] += cen * (vr * sn + vt * cs);
  }
}

template <typename R>
__device__ __forceinline__ void add_sources(const R (&w)[NV], const Metric<R>& m, int i, int j,
                                            R omega, int gravity, int corot, R (&L)[NV]) {
  add_sources_cm<R>(w, CellMetric<R>{m, i, j}, omega, gravity, corot, L);
}

}  // namespace icr
