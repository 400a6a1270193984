// icr_amr.hip -- block-structured adaptive mesh refinement of the
// heliospheric update (the refined runs of Sect. 3.2 and Sect. 4: blocks
// refined where the CME tracer or a compression is present, criteria
// 'tracing', 'shock', 'combined').
//
// Blocks of br x bt x bp cells at every level, each held with two ghost
// layers; a level-(l+1) block is one octant of a level-l block at twice the
// resolution (radial edges split at the geometric mean).  One global dt,
// SSP-RK2 on the leaves.  Per stage:
//   k_amr_ghost   the ghost layers the stage kernel does not take from their
//                 source itself, one block per listed leaf face (a regrid:
//                 all faces): copies from a leaf of the same level,
//                 volume-weighted restriction of finer leaves, physical edges
//                 as in the uniform solver; then, coarse levels first, the
//                 faces next to a coarser leaf: conservative prolongation
//                 (minmod slopes from its padded block, then a constant
//                 correction so the children's volume-weighted mean is the
//                 coarse cell);
//   k_amr_stage_lds (leaves that fit LDS) or k_amr_stage: reconstruct / flux /
//                 divergence / sources / RK combine of every leaf cell, the
//                 fluxes of the faces next to another level kept (k_amr_stage:
//                 of all six faces);
//   k_amr_reflux  a coarse cell next to finer leaves takes the area-weighted
//                 sum of their face fluxes instead of its own on that face.
// After a step: the CFL rate of every leaf cell (one-block finalize), and
// every regrid_every steps the block indicators (max tau, max compression)
// that the host turns into splits (k_amr_prolong) and merges
// (k_amr_restrict), keeping face neighbours within one level.
// The passive CME tracer rho tau rides along as a ninth conserved variable.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include "icarus_hip.h"
#include "icr_kernels.hpp"

namespace icr {

int set_error(int code, const char* msg);  // icr_api.hip

constexpr int AMR_MAXL = 6;
constexpr int NA = 9;   // conserved variables + rho tau
constexpr int AG = 2;   // ghost layers

struct AmrLevel {
  Metric<double> m;
  const double* m64;  // edges and colatitude centres (k_metric layout)
  const int* map;     // [nbp][nbt][nbr] -> block slot, -1 where no block
  int nr, nt, np, nbr, nbt, nbp;
  double dth, dph;
};

struct AmrArgs {
  double* U;   // [slot][9][pp][pt][pr] U^n / U^{n+1}
  double* U1;  // [slot][9][pp][pt][pr] stage-1 state
  double* F;   // [slot][6][9][fmax] fluxes of the block faces r-, r+, t-, t+, p-, p+
  const int* key;  // [slot][4]: level, bi, bj, bk
  const AmrLevel* __restrict__ lv;  // [level], device table
  int nlev, br, bt, bp, pr, pt, pp, fmax;
  long long bvol;  // padded cells per variable of a block
  BndArgs bnd;     // maps and CMEs on the base grid
  DevClock* clock;
  double* partials;
  double gam, gm1, igm1, omega, cfl, r_in;
  int gravity, corot;
};

// What a block needs to know of its leaf, and of one leaf face: built on the
// host with the tree and read through scalar loads, one step from the data
// (walking list -> key -> level map -> leaf flag cost each block that chain
// of dependent loads).
struct LeafDesc {
  int slot, l, bi, bj, bk;
  int other, finer;  // bit f: another level / finer leaves across face f
  int src[6];        // ghosts of face f: LEAF_* | slot << 2
};
// from the padded block's own ghost layers; the same-level leaf's interior;
// the leaf's own cells (zero gradient, mirror rows)
enum { LEAF_POOL, LEAF_COPY, LEAF_SELF };
struct FaceDesc {
  int slot, face, kind, ns;  // face = 2 d + side (d = r, theta, phi); FACE_*
  int l, bi, bj, bk;
};
enum { FACE_COPY, FACE_EDGE, FACE_INNER, FACE_FINE, FACE_COARSE };

__device__ __forceinline__ long long pidx(const AmrArgs& a, int slot, int v, int kk, int jj,
                                          int ii) {
  return (long long)slot * NA * a.bvol + ((long long)(v * a.pp + kk) * a.pt + jj) * a.pr + ii;
}

__device__ __forceinline__ int face_cells(const AmrArgs& a, int d) {
  return d == 0 ? a.bp * a.bt : (d == 1 ? a.bp * a.br : a.bt * a.br);
}

__device__ __forceinline__ long long fidx(const AmrArgs& a, int slot, int face, int v, int q) {
  return (((long long)slot * 6 + face) * NA + v) * a.fmax + q;
}

__device__ __forceinline__ int amr_slot(const AmrArgs& a, int l, int i, int j, int k) {
  const AmrLevel& L = a.lv[l];
  return L.map[((long long)(k / a.bp) * L.nbt + j / a.bt) * L.nbr + i / a.br];
}

// Cell volume without the phi width, and the full volume, at level l.
__device__ __forceinline__ double vol_nophi(const AmrArgs& a, int l, int i, int j) {
  const Metric<double>& m = a.lv[l].m;
  return rcp_fast(m.ivr[i] * m.ict[j]);
}

// Inner-boundary primitive of level-l column (j, k): the map of the base
// column containing it (time interpolated), the cone CME tested at this
// column's centre; *inside = 1 inside an inserted cone.
__device__ void amr_inner_prim(const AmrArgs& a, int l, int j, int k, double t, double (&w)[NV],
                               int* inside) {
  const int f = 1 << (l - 1);
  BndArgs maponly = a.bnd;  // the map of the base column; CMEs tested below
  maponly.n_cme = 0;
  boundary_prim(maponly, t, j / f, k / f, w, nullptr);
  *inside = 0;
  const double th = a.lv[l].m64[OFF_TC64(a.lv[l].nr, a.lv[l].nt) + j];
  const double ph = (k + 0.5) * a.lv[l].dph;
  const double sth = sin(th), cth = cos(th);
  for (int c = 0; c < a.bnd.n_cme; ++c) {
    const double* m = a.bnd.cme + 8 * c;
    if (!(t >= m[0] && t < m[0] + m[1])) continue;
    const double cosd = cth * cos(m[2]) + sth * sin(m[2]) * cos(ph - m[3]);
    if (cosd >= m[4]) {
      *inside = 1;
      w[0] = m[6];
      w[1] = m[5];
      w[2] = 0.0;
      w[3] = -a.omega * a.r_in * sth;
      w[4] = m[7];
    }
  }
}

__device__ __forceinline__ double mm(double x, double y) {
  return x * y <= 0.0 ? 0.0 : (fabs(x) < fabs(y) ? x : y);
}

// Conservative prolongation of a level-l coarse cell (global ic, jc): child
// (c, b, e) = (r, theta, phi half) is c0 + s_r (+-1/4 - f_r) + s_t (+-1/4 -
// f_t) + s_p (+-1/4) with minmod slopes s and f_r, f_t the volume-weighted
// means of the +-1/4 over the 8 children (phi's is zero), so that their
// volume-weighted mean is c0.  The coefficients depend on the cell only and
// serve all its variables.
struct Prolong {
  double cr, ct, cp;
};
__device__ __forceinline__ Prolong prolong_coef(const AmrArgs& a, int l, int ic, int jc, int sub) {
  const double v00 = vol_nophi(a, l + 1, 2 * ic, 2 * jc);
  const double v10 = vol_nophi(a, l + 1, 2 * ic + 1, 2 * jc);
  const double v01 = vol_nophi(a, l + 1, 2 * ic, 2 * jc + 1);
  const double v11 = vol_nophi(a, l + 1, 2 * ic + 1, 2 * jc + 1);
  const double iv = 0.25 * rcp_fast((v00 + v10) + (v01 + v11));
  Prolong p;
  p.cr = (sub & 1 ? 0.25 : -0.25) - ((v10 + v11) - (v00 + v01)) * iv;
  p.ct = (sub & 2 ? 0.25 : -0.25) - ((v01 + v11) - (v00 + v10)) * iv;
  p.cp = sub & 4 ? 0.25 : -0.25;
  return p;
}
// one variable at q = the coarse cell in a padded block
__device__ __forceinline__ double prolong1(const double* q, int pr, int prt, const Prolong& p) {
  const double c0 = q[0];
  const double sr = mm(c0 - q[-1], q[1] - c0);
  const double st = mm(c0 - q[-pr], q[pr] - c0);
  const double sp = mm(c0 - q[-prt], q[prt] - c0);
  return fma_(sp, p.cp, fma_(st, p.ct, fma_(sr, p.cr, c0)));
}

__device__ __forceinline__ void prim_to_cons9(const AmrArgs& a, const double (&w)[NV], double tr,
                                              double (&u)[NA]) {
  double c[NV];
  prim2cons<double>(w, c, a.igm1);
  for (int v = 0; v < NV; ++v) u[v] = c[v];
  u[8] = tr * w[0];
}

// ---------------------------------------------------------------- ghosts --
// One block per listed leaf face: its two ghost layers.  What lies across a
// face is the same for all its cells.  Inside a step only the faces the
// stage kernel does not read from its neighbours itself are filled (at 3800
// leaves in four levels 4800 of 22900: 65 us a stage, where one thread per
// ghost cell of every leaf took 195), and the fill follows the step clock (no
// work once t_end is reached); a regrid fills every face, whatever the clock
// says.
__global__ void __launch_bounds__(256) k_amr_ghost(AmrArgs a, const FaceDesc* __restrict__ list,
                                                   int use_u1, int t_plus_dt, int always) {
  if (!(always || a.clock->active)) return;
  const FaceDesc F = list[blockIdx.x];
  const int slot = F.slot, d = F.face >> 1, side = F.face & 1, ns = F.ns, l = F.l;
  double* buf = use_u1 ? a.U1 : a.U;
  const int n1 = d == 0 ? a.bt : a.br, n2 = d == 2 ? a.bt : a.bp;  // transverse extents
  const int area = n1 * n2, bd = d == 0 ? a.br : (d == 1 ? a.bt : a.bp);
  const int pr = a.pr, prt = a.pr * a.pt;
  const int sd = d == 0 ? 1 : (d == 1 ? pr : prt);    // strides of a padded block
  const int s1 = d == 0 ? pr : 1, s2 = d == 2 ? pr : prt;
  double* own = buf + (long long)slot * NA * a.bvol;
  const int o0 = AG * (1 + pr + prt);  // interior cell (0, 0, 0)
  // ghost layer g = 1, 2 sits at index -g (lower side) or bd - 1 + g along d
  auto ghost = [&](int g) { return (side ? bd - 1 + g : -g) * sd; };
  // plain copies: 256 / (2 area) threads share a ghost cell's variables, all
  // loads before the first store (they could alias it)
  const int ng = 2 * area < 256 ? 256 / (2 * area) : 1;
  const int vg = ng > 1 ? threadIdx.x / (2 * area) : 0, tq = threadIdx.x - vg * 2 * area;
  if (F.kind == FACE_INNER || F.kind == FACE_EDGE) {
    if (F.kind == FACE_INNER) {  // inner boundary: the same value in both layers
      const double t = a.clock->t + (t_plus_dt ? a.clock->dt : 0.0);
      for (int q = threadIdx.x; q < area; q += 256) {
        const int y = q / n1, x = q - y * n1;
        double w[NV], u[NA];
        int inside;
        amr_inner_prim(a, l, F.bj * a.bt + x, F.bk * a.bp + y, t, w, &inside);
        prim_to_cons9(a, w, (double)inside, u);
        const int o = o0 + y * s2 + x * s1;
        for (int v = 0; v < NA; ++v) {
          own[v * a.bvol + o + ghost(1)] = u[v];
          own[v * a.bvol + o + ghost(2)] = u[v];
        }
      }
    } else {  // zero gradient beyond r_out; mirror rows at the colatitude edges
      for (int q0 = tq; q0 < 2 * area && vg < ng; q0 += 256) {
        const int g = q0 < area ? 1 : 2, q = q0 - (g - 1) * area;
        const int y = q / n1, x = q - y * n1;
        const int o = o0 + y * s2 + x * s1;
        const int src = d == 0 ? bd - 1 : (side ? bd - g : g - 1);
        double t[NA];
#pragma unroll
        for (int c = 0; c < NA; ++c) {
          const int v = vg + c * ng;
          if (v < NA) t[c] = own[v * a.bvol + o + src * sd];
          if (d == 1 && (v == 2 || v == 6)) t[c] = -t[c];
        }
#pragma unroll
        for (int c = 0; c < NA; ++c) {
          const int v = vg + c * ng;
          if (v < NA) own[v * a.bvol + o + ghost(g)] = t[c];
        }
      }
    }
    return;
  }
  if (F.kind == FACE_COPY) {  // a leaf of the same level
    const double* from = buf + (long long)ns * NA * a.bvol;
    for (int q0 = tq; q0 < 2 * area && vg < ng; q0 += 256) {
      const int g = q0 < area ? 1 : 2, q = q0 - (g - 1) * area;
      const int y = q / n1, x = q - y * n1;
      const int o = o0 + y * s2 + x * s1;
      const int src = o + (side ? g - 1 : bd - g) * sd;
      double t[NA];
#pragma unroll
      for (int c = 0; c < NA; ++c)
        if (vg + c * ng < NA) t[c] = from[(vg + c * ng) * a.bvol + src];
#pragma unroll
      for (int c = 0; c < NA; ++c)
        if (vg + c * ng < NA) own[(vg + c * ng) * a.bvol + o + ghost(g)] = t[c];
    }
    return;
  }
  for (int q0 = threadIdx.x; q0 < 2 * area; q0 += 256) {
    const int g = q0 < area ? 1 : 2, q = q0 - (g - 1) * area;
    const int y = q / n1, x = q - y * n1;
    const int dst = o0 + y * s2 + x * s1 + ghost(g);
    // global level-l indices of the ghost cell
    const int along = side ? bd - 1 + g : -g;
    const int i = F.bi * a.br + (d == 0 ? along : x);
    const int j = F.bj * a.bt + (d == 0 ? x : (d == 1 ? along : y));
    int k = F.bk * a.bp + (d == 2 ? along : y);
    if (d == 2) k = k < 0 ? k + a.lv[l].np : (k >= a.lv[l].np ? k - a.lv[l].np : k);
    if (F.kind == FACE_FINE) {  // refined: volume-weighted mean of the 8 children
      // (the eight lookups, then the loads, all in flight together)
      long long at[8];
      double vol[8], acc[NA], vs = 0.0;
      bool ok = true;
      int fs[8];
#pragma unroll
      for (int s = 0; s < 8; ++s)
        fs[s] = l < a.nlev ? amr_slot(a, l + 1, 2 * i + (s & 1), 2 * j + ((s >> 1) & 1),
                                      2 * k + (s >> 2))
                           : -1;
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const int fi = 2 * i + (s & 1), fj = 2 * j + ((s >> 1) & 1), fk = 2 * k + (s >> 2);
        ok = ok && fs[s] >= 0;
        const int f0 = fs[s] < 0 ? 0 : fs[s];
        at[s] = pidx(a, f0, 0, AG + fk % a.bp, AG + fj % a.bt, AG + fi % a.br);
        vol[s] = vol_nophi(a, l + 1, fi, fj);
        vs += vol[s];
      }
#pragma unroll
      for (int v = 0; v < NA; ++v) {
        acc[v] = 0.0;
#pragma unroll
        for (int s = 0; s < 8; ++s) acc[v] = fma_(buf[at[s] + v * a.bvol], vol[s], acc[v]);
      }
      // a missing child cannot happen in a valid tree: poison
      const double iv = ok ? rcp_fast(vs) : __builtin_nan("");
#pragma unroll
      for (int v = 0; v < NA; ++v) own[v * a.bvol + dst] = acc[v] * iv;
    } else {  // covered by the coarser leaf
      const int ic = i >> 1, jc = j >> 1, kc = k >> 1;
      const int cs = l > 1 ? amr_slot(a, l - 1, ic, jc, kc) : -1;
      if (cs < 0) {  // cannot happen in a valid tree (levels differ by one)
        for (int v = 0; v < NA; ++v) own[v * a.bvol + dst] = __builtin_nan("");
        continue;
      }
      const int* ckey = a.key + 4 * cs;
      const double* c = buf + pidx(a, cs, 0, AG + kc - ckey[3] * a.bp, AG + jc - ckey[2] * a.bt,
                                   AG + ic - ckey[1] * a.br);
      const Prolong p = prolong_coef(a, l - 1, ic, jc, ((k & 1) << 2) | ((j & 1) << 1) | (i & 1));
      double t[NA];
#pragma unroll
      for (int v = 0; v < NA; ++v) t[v] = prolong1(c + v * a.bvol, pr, prt, p);
#pragma unroll
      for (int v = 0; v < NA; ++v) own[v * a.bvol + dst] = t[v];
    }
  }
}

// ----------------------------------------------------------------- stage --
template <int FLUX, int LIM>
__device__ void amr_face(const AmrArgs& a, const double* buf, int slot, int d, int kk, int jj,
                         int ii, double (&f)[NA]) {
  // face between padded cells (kk, jj, ii) - e_d and (kk, jj, ii): cells
  // -2 .. +1 along d
  const int di = d == 0, dj = d == 1, dk = d == 2;
  double w[4][NV], rho[4], tr[4];
  for (int s = 0; s < 4; ++s) {
    const int o = s - 2;
    double u[NV];
    for (int v = 0; v < NV; ++v)
      u[v] = buf[pidx(a, slot, v, kk + o * dk, jj + o * dj, ii + o * di)];
    cons2prim<double, true>(u, w[s], a.gm1);
    rho[s] = u[0];
    tr[s] = buf[pidx(a, slot, 8, kk + o * dk, jj + o * dj, ii + o * di)];
  }
  double wl[NV], wr[NV], fl[NV];
  reconstruct<double, LIM, true>(w[0], w[1], w[2], w[3], wl, wr);
  if (d == 0)
    face_flux<double, 1, FLUX, true>(wl, wr, a.gam, a.igm1, fl);
  else if (d == 1)
    face_flux<double, 2, FLUX, true>(wl, wr, a.gam, a.igm1, fl);
  else
    face_flux<double, 3, FLUX, true>(wl, wr, a.gam, a.igm1, fl);
  for (int v = 0; v < NV; ++v) f[v] = fl[v];
  // tracer: mass flux times tau of the upwind cell
  f[8] = fl[0] * (fl[0] >= 0.0 ? tr[1] * rcp_fast(rho[1]) : tr[2] * rcp_fast(rho[2]));
}

// One thread per cell of the listed leaves (blocks of 256 threads loop over
// a leaf's cells).  stage 1: U1 = U + dt L(U); stage 2: U = U/2 + (U1 + dt
// L(U1))/2 in place.
template <int FLUX, int LIM>
__global__ void __launch_bounds__(256) k_amr_stage(AmrArgs a, const LeafDesc* __restrict__ list,
                                                   int stage) {
  if (!a.clock->active) return;
  const LeafDesc& D = list[blockIdx.x];
  const int slot = D.slot, l = D.l;
  const AmrLevel& LV = a.lv[l];
  const Metric<double>& m = LV.m;
  const double dt = a.clock->dt;
  const double* in = stage == 1 ? a.U : a.U1;
  double* out = stage == 1 ? a.U1 : a.U;
  const int ncell = a.br * a.bt * a.bp;
  for (int c = threadIdx.x; c < ncell; c += blockDim.x) {
    const int ci = c % a.br, cj = (c / a.br) % a.bt, ck = c / (a.br * a.bt);
    const int ii = AG + ci, jj = AG + cj, kk = AG + ck;
    const int gi = D.bi * a.br + ci, gj = D.bj * a.bt + cj;
    double L[NA];
    for (int v = 0; v < NA; ++v) L[v] = 0.0;
    {  // r
      double fm[NA], fp[NA];
      amr_face<FLUX, LIM>(a, in, slot, 0, kk, jj, ii, fm);
      amr_face<FLUX, LIM>(a, in, slot, 0, kk, jj, ii + 1, fp);
      for (int v = 0; v < NA; ++v) L[v] -= (m.rp2[gi] * fp[v] - m.rm2[gi] * fm[v]) * m.ivr[gi];
      if (ci == 0)
        for (int v = 0; v < NA; ++v) a.F[fidx(a, slot, 0, v, ck * a.bt + cj)] = fm[v];
      if (ci == a.br - 1)
        for (int v = 0; v < NA; ++v) a.F[fidx(a, slot, 1, v, ck * a.bt + cj)] = fp[v];
    }
    {  // theta
      double fm[NA], fp[NA];
      amr_face<FLUX, LIM>(a, in, slot, 1, kk, jj, ii, fm);
      amr_face<FLUX, LIM>(a, in, slot, 1, kk, jj + 1, ii, fp);
      for (int v = 0; v < NA; ++v)
        L[v] -= m.hr[gi] * (m.sp[gj] * fp[v] - m.sm[gj] * fm[v]) * m.ict[gj];
      if (cj == 0)
        for (int v = 0; v < NA; ++v) a.F[fidx(a, slot, 2, v, ck * a.br + ci)] = fm[v];
      if (cj == a.bt - 1)
        for (int v = 0; v < NA; ++v) a.F[fidx(a, slot, 3, v, ck * a.br + ci)] = fp[v];
    }
    {  // phi
      double fm[NA], fp[NA];
      amr_face<FLUX, LIM>(a, in, slot, 2, kk, jj, ii, fm);
      amr_face<FLUX, LIM>(a, in, slot, 2, kk + 1, jj, ii, fp);
      const double fph = m.hr[gi] * m.phf[gj];
      for (int v = 0; v < NA; ++v) L[v] -= fph * (fp[v] - fm[v]);
      if (ck == 0)
        for (int v = 0; v < NA; ++v) a.F[fidx(a, slot, 4, v, cj * a.br + ci)] = fm[v];
      if (ck == a.bp - 1)
        for (int v = 0; v < NA; ++v) a.F[fidx(a, slot, 5, v, cj * a.br + ci)] = fp[v];
    }
    double u[NV], w[NV];
    for (int v = 0; v < NV; ++v) u[v] = in[pidx(a, slot, v, kk, jj, ii)];
    cons2prim<double>(u, w, a.gm1);
    double Ls[NV];
    for (int v = 0; v < NV; ++v) Ls[v] = L[v];
    add_sources<double>(w, m, gi, gj, a.omega, a.gravity, a.corot, Ls);
    for (int v = 0; v < NV; ++v) L[v] = Ls[v];
    for (int v = 0; v < NA; ++v) {
      const long long o = pidx(a, slot, v, kk, jj, ii);
      const double uc = in[o];
      out[o] = stage == 1 ? uc + dt * L[v] : 0.5 * out[o] + 0.5 * (uc + dt * L[v]);
    }
  }
}

// Face-once variant for leaves whose primitives fit LDS.  The padded cells a
// face can read (the interior and two layers beyond each side, no corners)
// are converted once and kept in LDS, one slab of
//   [bp][bt][br + 4]  interior with its r layers,
//   [bp][4][br]       theta layers,  [4][bt][br]  phi layers
// per variable (eight primitives and tau).  Every thread forms up to two
// faces of each direction in registers; then the fluxes take the slabs' place,
// five variables and four, and every thread updates up to two cells.
// 256 threads and 80 KB (two blocks per CU, 10x6x6 cells and below) or 512
// threads and 160 KB; larger leaves take k_amr_stage.  At a mean of 2900
// leaves of 10x6x6 a stage takes 125 us, where every face converting its four
// cells by itself, with IEEE divisions and roots, took 249; it is bound by the
// latency of its phases (two waves per SIMD) and moves 0.35 GB at 3800 leaves.
constexpr int AMR_LDS_S = 80 * 1024, AMR_LDS_L = 160 * 1024;
__host__ __device__ constexpr int amr_slab(int br, int bt, int bp) {
  return (br + 2 * AG) * bt * bp + 2 * AG * br * bp + 2 * AG * br * bt;
}
__host__ __device__ constexpr int amr_faces(int br, int bt, int bp, int d) {
  return d == 0 ? (br + 1) * bt * bp : (d == 1 ? br * (bt + 1) * bp : br * bt * (bp + 1));
}
constexpr int AMR_V0 = 5;  // variables in the first round of fluxes
// doubles of the slabs or of a round of fluxes, then the metric of the
// leaf's rows: MR_N arrays along r, MT_N along theta
__host__ __device__ inline int amr_lds_work(int br, int bt, int bp) {
  const int nf = amr_faces(br, bt, bp, 0) + amr_faces(br, bt, bp, 1) + amr_faces(br, bt, bp, 2);
  const int w = NA * amr_slab(br, bt, bp), f = AMR_V0 * nf;
  return w > f ? w : f;
}
// bytes of LDS, and whether NT threads with two items each cover the leaf
inline int amr_lds_bytes(int br, int bt, int bp) {
  return (int)sizeof(double) * (amr_lds_work(br, bt, bp) + MR_N * br + MT_N * bt);
}
inline bool amr_covers(int nt, int br, int bt, int bp) {
  for (int d = 0; d < 3; ++d)
    if (amr_faces(br, bt, bp, d) > 2 * nt) return false;
  return true;
}

struct AmrCellMetric {  // a cell's metric factors in LDS
  const double *mr, *mt;
  int br, bt;
  __device__ __forceinline__ double r(int arr) const { return mr[arr * br]; }
  __device__ __forceinline__ double t(int arr) const { return mt[arr * bt]; }
};

template <int FLUX, int LIM, int NT, int BYTES>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2)))
k_amr_stage_lds(AmrArgs a, const LeafDesc* __restrict__ list, int stage) {
  __shared__ double sm[BYTES / 8];
  if (!a.clock->active) return;
  const LeafDesc D = list[blockIdx.x];
  const int slot = D.slot, tid = threadIdx.x;
  const Metric<double>& m = a.lv[D.l].m;
  const double dt = a.clock->dt;
  const int br = a.br, bt = a.bt, bp = a.bp, pr = a.pr, prt = a.pr * a.pt;
  const double* pool = stage == 1 ? a.U : a.U1;
  const long long leafsz = NA * a.bvol;
  double* out = (stage == 1 ? a.U1 : a.U) + slot * leafsz;
  const int rw = br + 2 * AG, nW = rw * bt * bp, nT = 2 * AG * br * bp;
  const int S = amr_slab(br, bt, bp), ncell = br * bt * bp;
  double* mr = sm + amr_lds_work(br, bt, bp);
  double* mt = mr + MR_N * br;
  for (int q = tid; q < MR_N * br + MT_N * bt; q += NT) {
    if (q < MR_N * br) {
      const int arr = q / br;
      mr[q] = metric_r(m, arr)[D.bi * br + q - arr * br];
    } else {
      const int t = q - MR_N * br, arr = t / bt;
      mt[t] = metric_t(m, arr)[D.bj * bt + t - arr * bt];
    }
  }
  // (four cells a round: 36 loads in flight per thread; a ghost cell comes
  // straight from the same-level leaf across its face, from the leaf's own
  // edge cells, or from the padded block where k_amr_ghost formed it)
  for (int e0 = tid; e0 < S; e0 += 4 * NT) {
    double raw[4][NA];
    bool flip[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const int e = e0 + h * NT;
      int ii, jj, kk, s, hop;  // source word of the face, cells to its far side
      if (e < nW) {
        const int r = e / rw;
        ii = e - r * rw;
        jj = AG + r % bt;
        kk = AG + r / bt;
        s = ii < AG ? D.src[0] : (ii >= AG + br ? D.src[1] : LEAF_POOL);
        hop = ii < AG ? br : -br;
      } else if (e < nW + nT) {
        const int r = (e - nW) / br;
        const bool lo = (r & 3) < AG;
        ii = AG + (e - nW) - r * br;
        jj = lo ? (r & 3) : bt + (r & 3);
        kk = AG + (r >> 2);
        s = lo ? D.src[2] : D.src[3];
        hop = (lo ? bt : -bt) * pr;
      } else {
        const int r = (e - nW - nT) / br, row = r / bt;
        const bool lo = row < AG;
        ii = AG + (e - nW - nT) - r * br;
        jj = AG + r - row * bt;
        kk = lo ? row : bp + row;
        s = lo ? D.src[4] : D.src[5];
        hop = (lo ? bp : -bp) * prt;
      }
      long long at = (s & 3) == LEAF_COPY ? (s >> 2) * leafsz + hop : slot * leafsz;
      flip[h] = false;
      if ((s & 3) == LEAF_SELF) {
        if (e < nW) {
          ii = AG + br - 1;  // zero gradient beyond r_out
        } else {
          jj = jj < AG ? 2 * AG - 1 - jj : 2 * (AG + bt) - 1 - jj;  // mirror row
          flip[h] = true;
        }
      }
      at += kk * prt + jj * pr + ii;
      if (e < S) {
#pragma unroll
        for (int v = 0; v < NA; ++v) raw[h][v] = pool[at + v * a.bvol];
      }
    }
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const int e = e0 + h * NT;
      if (e < S) {
        double u[NV], w[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) u[v] = raw[h][v];
        cons2prim<double, true>(u, w, a.gm1);
        if (flip[h]) flip_theta(w);
#pragma unroll
        for (int v = 0; v < NV; ++v) sm[v * S + e] = w[v];
        sm[8 * S + e] = raw[h][8] * rcp_fast(u[0]);
      }
    }
  }
  __syncthreads();
  // fluxes: face index along direction d: position p in [0, b_d] (between
  // cells p-1 and p) in place of that direction's cell index, r fastest
  double fl[3][2][NA];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int e0 = d == 0 ? br + 1 : br, e1 = d == 1 ? bt + 1 : bt;
    const int bd = d == 0 ? br : (d == 1 ? bt : bp);
    const int nf = amr_faces(br, bt, bp, d);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int f = tid + q * NT;
      if (f < nf) {
        const int r = f / e0, ci = f - r * e0, ck = r / e1, cj = r - ck * e1;
        const int p = d == 0 ? ci : (d == 1 ? cj : ck);
        int off[4];
#pragma unroll
        for (int o = 0; o < 4; ++o) {
          const int c = p + o - 2;  // cell along d, -2 .. bd + 1
          if (d == 0) {
            off[o] = (ck * bt + cj) * rw + c + AG;
          } else {
            const bool inside = c >= 0 && c < bd;
            const int g = c < 0 ? c + AG : c - bd + AG;
            if (d == 1)
              off[o] = inside ? (ck * bt + c) * rw + ci + AG : nW + (ck * 2 * AG + g) * br + ci;
            else
              off[o] = inside ? (c * bt + cj) * rw + ci + AG : nW + nT + (g * bt + cj) * br + ci;
          }
        }
        double wl[NV], wr[NV], fv[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v)
          face_states<double, LIM, true>(sm[v * S + off[0]], sm[v * S + off[1]],
                                         sm[v * S + off[2]], sm[v * S + off[3]], wl[v], wr[v]);
        if (d == 0)
          face_flux<double, 1, FLUX, true>(wl, wr, a.gam, a.igm1, fv);
        else if (d == 1)
          face_flux<double, 2, FLUX, true>(wl, wr, a.gam, a.igm1, fv);
        else
          face_flux<double, 3, FLUX, true>(wl, wr, a.gam, a.igm1, fv);
#pragma unroll
        for (int v = 0; v < NV; ++v) fl[d][q][v] = fv[v];
        // tracer: mass flux times tau of the upwind cell
        fl[d][q][8] = fv[0] * sm[8 * S + (fv[0] >= 0.0 ? off[1] : off[2])];
        if (p == 0 || p == bd) {  // block face next to another level: kept
          const int face = 2 * d + (p == bd);
          if (D.other >> face & 1) {
            const int fq = d == 0 ? ck * bt + cj : (d == 1 ? ck * br + ci : cj * br + ci);
#pragma unroll
            for (int v = 0; v < NA; ++v) a.F[fidx(a, slot, face, v, fq)] = fl[d][q][v];
          }
        }
      }
    }
  }
  // the cells' own state (from the primitives: the stored values up to
  // rounding, no reload), sources and metric factors
  double uc[2][NA], un[2][NA], src[2][NV], cf[2][5];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int c = tid + q * NT;
    if (c < ncell) {
      const int r = c / br, ci = c - r * br, ck = r / bt, cj = r - ck * bt;
      const int o = (AG + ck) * prt + (AG + cj) * pr + AG + ci;
      if (stage == 2)
#pragma unroll
        for (int v = 0; v < NA; ++v) un[q][v] = out[v * a.bvol + o];
      const int at = (ck * bt + cj) * rw + ci + AG;
      double w[NV], u8[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        w[v] = sm[v * S + at];
        src[q][v] = 0.0;
      }
      prim2cons<double>(w, u8, a.igm1);
#pragma unroll
      for (int v = 0; v < NV; ++v) uc[q][v] = u8[v];
      uc[q][8] = sm[8 * S + at] * w[0];
      const AmrCellMetric cm{mr + ci, mt + cj, br, bt};
      add_sources_cm<double>(w, cm, a.omega, a.gravity, a.corot, src[q]);
      const double ivr = cm.r(MR_IVR), hr = cm.r(MR_HR), hc = hr * cm.t(MT_ICT);
      cf[q][0] = cm.r(MR_RM2) * ivr;
      cf[q][1] = cm.r(MR_RP2) * ivr;
      cf[q][2] = hc * cm.t(MT_SM);
      cf[q][3] = hc * cm.t(MT_SP);
      cf[q][4] = hr * cm.t(MT_PHF);
    }
  }
  const int nf0 = amr_faces(br, bt, bp, 0), nf1 = amr_faces(br, bt, bp, 1);
  const int nfs = nf0 + nf1 + amr_faces(br, bt, bp, 2);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    constexpr int VB[3] = {0, AMR_V0, NA};
    __syncthreads();  // the slabs (or the first fluxes) have been read
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int f = tid + q * NT;
        if (f < amr_faces(br, bt, bp, d)) {
          const int at = (d == 0 ? 0 : (d == 1 ? nf0 : nf0 + nf1)) + f;
#pragma unroll
          for (int v = VB[h]; v < VB[h + 1]; ++v) sm[(v - VB[h]) * nfs + at] = fl[d][q][v];
        }
      }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int c = tid + q * NT;
      if (c < ncell) {
        const int r = c / br, ci = c - r * br, ck = r / bt, cj = r - ck * bt;
        const int o = (AG + ck) * prt + (AG + cj) * pr + AG + ci;
        const int fr = r * (br + 1) + ci, ft = nf0 + (ck * (bt + 1) + cj) * br + ci;
        const int fp = nf0 + nf1 + c;
#pragma unroll
        for (int v = VB[h]; v < VB[h + 1]; ++v) {
          const double* F = sm + (v - VB[h]) * nfs;
          const double dr = fma_(cf[q][0], F[fr], -cf[q][1] * F[fr + 1]);
          const double dth = fma_(cf[q][2], F[ft], -cf[q][3] * F[ft + br]);
          double L = fma_(cf[q][4], F[fp] - F[fp + br * bt], dr + dth);
          if (v < NV) L += src[q][v < NV ? v : 0];
          const double u1 = fma_(dt, L, uc[q][v]);
          out[v * a.bvol + o] = stage == 1 ? u1 : 0.5 * un[q][v] + 0.5 * u1;
        }
      }
    }
  }
}

// --------------------------------------------------------- flux correction --
// One block per listed leaf (those with finer leaves across some face): the
// coarse face's A F is replaced by the sum of the fine faces' A F.  coef: 1
// after stage 1 (U1), 1/2 after stage 2 (U).  An edge or corner cell of a
// block lies on faces of several directions: the directions follow each
// other behind a barrier, so each cell's updates stay ordered (blocks have
// >= 4 cells a side, so the two faces of one direction never share a cell).
__device__ __forceinline__ long long amr_reflux_cell(const AmrArgs& a, const LeafDesc& D, int d,
                                                     int side, int fq, int stage,
                                                     double (&dU)[NA]);

__global__ void __launch_bounds__(128) k_amr_reflux(AmrArgs a, const LeafDesc* __restrict__ list,
                                                    int stage) {
  if (!a.clock->active) return;
  const LeafDesc D = list[blockIdx.x];
  double* tgt = stage == 1 ? a.U1 : a.U;
  const int most = 2 * max(face_cells(a, 0), max(face_cells(a, 1), face_cells(a, 2)));
  for (int q0 = 0; q0 < most; q0 += 128) {
    // the corrections of all three directions (the loads overlap), then
    // their application in order
    double dU[3][NA];
    long long at[3];
    const int q = q0 + threadIdx.x;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int area = face_cells(a, d), side = q >= area;
      at[d] = -1;
      if (q < 2 * area && (D.finer >> (2 * d + side) & 1))
        at[d] = amr_reflux_cell(a, D, d, side, q - side * area, stage, dU[d]);
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      __syncthreads();
      if (at[d] >= 0) {
        double t[NA];
#pragma unroll
        for (int v = 0; v < NA; ++v) t[v] = tgt[at[d] + v * a.bvol];
#pragma unroll
        for (int v = 0; v < NA; ++v) tgt[at[d] + v * a.bvol] = t[v] + dU[d][v];
      }
    }
  }
}

// the correction dt dL of one coarse cell's variables, and its index in the
// padded block of variable 0
__device__ __forceinline__ long long amr_reflux_cell(const AmrArgs& a, const LeafDesc& D, int d,
                                                     int side, int fq, int stage,
                                                     double (&dU)[NA]) {
  const int slot = D.slot, l = D.l;
  const int w2 = d == 0 ? a.bt : a.br;
  const int y = fq / w2, x = fq - y * w2;
  const AmrLevel& L = a.lv[l];
  // coarse cell next to the face (block-local), its global indices
  int ci, cj, ck;
  if (d == 0) {
    ci = side ? a.br - 1 : 0;
    cj = x;
    ck = y;
  } else if (d == 1) {
    ci = x;
    cj = side ? a.bt - 1 : 0;
    ck = y;
  } else {
    ci = x;
    cj = y;
    ck = side ? a.bp - 1 : 0;
  }
  const int gi = D.bi * a.br + ci, gj = D.bj * a.bt + cj;
  const Metric<double>& m = L.m;
  const Metric<double>& mf = a.lv[l + 1].m;
  // coarse face area, and the fine faces (2 x 2) of the finer leaves
  double Ac;
  if (d == 0)
    Ac = (side ? m.rp2[gi] : m.rm2[gi]) / m.ict[gj] * L.dph;
  else if (d == 1)
    Ac = (side ? m.sp[gj] : m.sm[gj]) * m.hr[gi] / m.ivr[gi] * L.dph;
  else
    Ac = m.hr[gi] / m.ivr[gi] * L.dth;
  const double V = vol_nophi(a, l, gi, gj) * L.dph;
  const int face = 2 * d + side, fface = 2 * d + (1 - side);
  const double dt = a.clock->dt * (stage == 1 ? 1.0 : 0.5);
  const int gk = D.bk * a.bp + ck;
  // the 2 x 2 fine faces: slot, face cell and area (s = 2 s2 + s1)
  const AmrLevel& LF = a.lv[l + 1];
  int fsl[4], fqf[4];
  double Af[4];
  bool ok = true;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int s2 = s >> 1, s1 = s & 1;
    // fine cell indices (global, level l+1) on the fine side of the face
    int fi = 2 * gi, fj = 2 * gj, fk = 2 * gk;
    if (d == 0) {
      fi = side ? 2 * gi + 2 : 2 * gi - 1;
      fj += s1;
      fk += s2;
    } else if (d == 1) {
      fj = side ? 2 * gj + 2 : 2 * gj - 1;
      fi += s1;
      fk += s2;
    } else {
      fk = side ? 2 * gk + 2 : 2 * gk - 1;
      fi += s1;
      fj += s2;
    }
    if (d == 2) fk = fk < 0 ? fk + LF.np : (fk >= LF.np ? fk - LF.np : fk);
    fsl[s] = amr_slot(a, l + 1, fi, fj, fk);
    if (fsl[s] < 0) ok = false;  // cannot happen in a valid tree: poison the cell
    const int li = fi % a.br, lj = fj % a.bt, lk = fk % a.bp;
    if (d == 0) {
      fqf[s] = lk * a.bt + lj;
      Af[s] = (side ? mf.rm2[fi] : mf.rp2[fi]) * rcp_fast(mf.ict[fj]) * LF.dph;
    } else if (d == 1) {
      fqf[s] = lk * a.br + li;
      Af[s] = (side ? mf.sm[fj] : mf.sp[fj]) * mf.hr[fi] * rcp_fast(mf.ivr[fi]) * LF.dph;
    } else {
      fqf[s] = lj * a.br + li;
      Af[s] = mf.hr[fi] * rcp_fast(mf.ivr[fi]) * LF.dth;
    }
  }
  const double iV = rcp_fast(V);
#pragma unroll
  for (int v = 0; v < NA; ++v) {
    double sumf = 0.0;
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (fsl[s] >= 0) sumf = fma_(Af[s], a.F[fidx(a, fsl[s], fface, v, fqf[s])], sumf);
    if (!ok) sumf = __builtin_nan("");
    const double delta = sumf - Ac * a.F[fidx(a, slot, face, v, fq)];
    dU[v] = dt * ((side ? -delta : delta) * iV);
  }
  return pidx(a, slot, 0, AG + ck, AG + cj, AG + ci);
}

// ------------------------------------------------------------------- CFL --
__global__ void __launch_bounds__(256) k_amr_cfl(AmrArgs a, const LeafDesc* __restrict__ list) {
  const LeafDesc& D = list[blockIdx.x];
  const int slot = D.slot, l = D.l;
  const Metric<double>& m = a.lv[l].m;
  double lam = 0.0;
  int bad = BAD_NONE;
  const int ncell = a.br * a.bt * a.bp;
  for (int c = threadIdx.x; c < ncell; c += blockDim.x) {
    const int ci = c % a.br, cj = (c / a.br) % a.bt, ck = c / (a.br * a.bt);
    double u[NV], w[NV];
    for (int v = 0; v < NV; ++v) u[v] = a.U[pidx(a, slot, v, AG + ck, AG + cj, AG + ci)];
    cons2prim<double, true>(u, w, a.gm1);
    const int gi = D.bi * a.br + ci, gj = D.bj * a.bt + cj;
    const double rate = cell_rate<double, true>(w, m, gi, gj, a.gam);
    lam = fmax(lam, rate);
    if (bad == BAD_NONE && !cell_valid<double>(u, w)) bad = slot * ncell + c;
  }
  write_partials(a.partials, blockIdx.x, lam, 0.0, 1.0, bad);
}

// ------------------------------------------------------------ indicators --
// Per listed leaf: max tau and max of -div(V) r / (2 |v_r|) (ghosts filled).
__global__ void __launch_bounds__(256) k_amr_indicators(AmrArgs a,
                                                        const LeafDesc* __restrict__ list,
                                                        double* __restrict__ out) {
  __shared__ double sh[2][4];
  const LeafDesc& D = list[blockIdx.x];
  const int slot = D.slot, l = D.l;
  const Metric<double>& m = a.lv[l].m;
  double tmax = -1e300, cmax = -1e300;
  const int ncell = a.br * a.bt * a.bp;
  for (int c = threadIdx.x; c < ncell; c += blockDim.x) {
    const int ci = c % a.br, cj = (c / a.br) % a.bt, ck = c / (a.br * a.bt);
    const int ii = AG + ci, jj = AG + cj, kk = AG + ck;
    const int gi = D.bi * a.br + ci, gj = D.bj * a.bt + cj;
    auto vel = [&](int k2, int j2, int i2, int comp) {
      return a.U[pidx(a, slot, comp, k2, j2, i2)] / a.U[pidx(a, slot, 0, k2, j2, i2)];
    };
    const double v0r = vel(kk, jj, ii, 1), v0t = vel(kk, jj, ii, 2), v0p = vel(kk, jj, ii, 3);
    const double vr0 = 0.5 * (vel(kk, jj, ii - 1, 1) + v0r), vr1 = 0.5 * (v0r + vel(kk, jj, ii + 1, 1));
    const double vt0 = 0.5 * (vel(kk, jj - 1, ii, 2) + v0t), vt1 = 0.5 * (v0t + vel(kk, jj + 1, ii, 2));
    const double vp0 = 0.5 * (vel(kk - 1, jj, ii, 3) + v0p), vp1 = 0.5 * (v0p + vel(kk + 1, jj, ii, 3));
    const double div = (m.rp2[gi] * vr1 - m.rm2[gi] * vr0) * m.ivr[gi] +
                       m.hr[gi] * (m.sp[gj] * vt1 - m.sm[gj] * vt0) * m.ict[gj] +
                       m.hr[gi] * m.phf[gj] * (vp1 - vp0);
    const double comp = -div * m.rc[gi] / (2.0 * fabs(v0r));
    const double tau = a.U[pidx(a, slot, 8, kk, jj, ii)] / a.U[pidx(a, slot, 0, kk, jj, ii)];
    tmax = fmax(tmax, tau);
    cmax = fmax(cmax, comp);
  }
  for (int off = 32; off > 0; off >>= 1) {
    tmax = fmax(tmax, __shfl_xor(tmax, off, 64));
    cmax = fmax(cmax, __shfl_xor(cmax, off, 64));
  }
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    sh[0][wv] = tmax;
    sh[1][wv] = cmax;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < (int)(blockDim.x >> 6); ++q) {
      tmax = fmax(tmax, sh[0][q]);
      cmax = fmax(cmax, sh[1][q]);
    }
    out[2 * blockIdx.x] = tmax;
    out[2 * blockIdx.x + 1] = cmax;
  }
}

// ------------------------------------------------- split, merge, init, io --
// pairs[2q] = parent slot, pairs[2q+1] = child slot: the child's cells from
// the parent's padded U (ghosts filled).
__global__ void __launch_bounds__(256) k_amr_prolong(AmrArgs a, const int* __restrict__ pairs) {
  const int ps = pairs[2 * blockIdx.x], cs = pairs[2 * blockIdx.x + 1];
  const int* pk = a.key + 4 * ps;
  const int* ck = a.key + 4 * cs;
  const int l = pk[0];
  const int ncell = a.br * a.bt * a.bp;
  for (int c = threadIdx.x; c < ncell; c += blockDim.x) {
    const int ci = c % a.br, cj = (c / a.br) % a.bt, cq = c / (a.br * a.bt);
    // global child cell and its coarse parent cell
    const int fi = ck[1] * a.br + ci, fj = ck[2] * a.bt + cj, fk = ck[3] * a.bp + cq;
    const int gi = fi >> 1, gj = fj >> 1, gk = fk >> 1;
    const int ii = AG + gi - pk[1] * a.br, jj = AG + gj - pk[2] * a.bt, kk = AG + gk - pk[3] * a.bp;
    const Prolong p = prolong_coef(a, l, gi, gj,
                                   ((fk & 1) << 2) | ((fj & 1) << 1) | (fi & 1));
    const double* c0 = a.U + pidx(a, ps, 0, kk, jj, ii);
    double t[NA];
#pragma unroll
    for (int v = 0; v < NA; ++v) t[v] = prolong1(c0 + v * a.bvol, a.pr, a.pr * a.pt, p);
#pragma unroll
    for (int v = 0; v < NA; ++v) a.U[pidx(a, cs, v, AG + cq, AG + cj, AG + ci)] = t[v];
  }
}

// parents[q]: the parent's cells from its 8 children (volume-weighted).
__global__ void __launch_bounds__(256) k_amr_restrict(AmrArgs a, const int* __restrict__ parents) {
  const int ps = parents[blockIdx.x];
  const int* pk = a.key + 4 * ps;
  const int l = pk[0];
  const int ncell = a.br * a.bt * a.bp;
  for (int c = threadIdx.x; c < ncell; c += blockDim.x) {
    const int ci = c % a.br, cj = (c / a.br) % a.bt, cq = c / (a.br * a.bt);
    const int gi = pk[1] * a.br + ci, gj = pk[2] * a.bt + cj, gk = pk[3] * a.bp + cq;
    double acc[NA], vs = 0.0;
    for (int v = 0; v < NA; ++v) acc[v] = 0.0;
    for (int s = 0; s < 8; ++s) {
      const int e = s >> 2, b = (s >> 1) & 1, cc = s & 1;
      const int fi = 2 * gi + cc, fj = 2 * gj + b, fk = 2 * gk + e;
      const int fs = l < a.nlev ? amr_slot(a, l + 1, fi, fj, fk) : -1;
      if (fs < 0) {  // cannot happen for a merge of 8 leaves
        vs = __builtin_nan("");
        continue;
      }
      const int* key = a.key + 4 * fs;
      const double vol = vol_nophi(a, l + 1, fi, fj);
      vs += vol;
      for (int v = 0; v < NA; ++v)
        acc[v] += a.U[pidx(a, fs, v, AG + fk - key[3] * a.bp, AG + fj - key[2] * a.bt,
                           AG + fi - key[1] * a.br)] * vol;
    }
    for (int v = 0; v < NA; ++v) a.U[pidx(a, ps, v, AG + cq, AG + cj, AG + ci)] = acc[v] / vs;
  }
}

// Level-1 leaves from the radial expansion of the first map (Sect. 2.1).
__global__ void __launch_bounds__(256) k_amr_init(AmrArgs a, const LeafDesc* __restrict__ list,
                                                  double gam) {
  const LeafDesc& D = list[blockIdx.x];
  const int slot = D.slot;
  const AmrLevel& L = a.lv[1];
  const long long plane = (long long)a.bnd.nt * a.bnd.np;
  const int ncell = a.br * a.bt * a.bp;
  for (int c = threadIdx.x; c < ncell; c += blockDim.x) {
    const int ci = c % a.br, cj = (c / a.br) % a.bt, cq = c / (a.br * a.bt);
    const int i = D.bi * a.br + ci, j = D.bj * a.bt + cj, k = D.bk * a.bp + cq;
    const double rc = L.m.rc[i];
    const double x = a.r_in / rc;
    const double sth = sin(L.m64[OFF_TC64(L.nr, L.nt) + j]);
    const long long q = (long long)k * a.bnd.nt + j;
    double w[NV];
    w[0] = a.bnd.maps[0 * plane + q] * x * x;
    w[1] = a.bnd.maps[1 * plane + q];
    w[2] = 0.0;
    w[3] = -a.omega * rc * sth;
    w[4] = a.bnd.maps[4 * plane + q] * pow(x, 2.0 * gam);
    w[5] = a.bnd.maps[5 * plane + q] * x * x;
    w[6] = 0.0;
    w[7] = a.bnd.maps[7 * plane + q] * x;
    double u[NA];
    prim_to_cons9(a, w, 0.0, u);
    for (int v = 0; v < NA; ++v) a.U[pidx(a, slot, v, AG + cq, AG + cj, AG + ci)] = u[v];
  }
}

// One leaf into host memory; each block then sets its flag to `seq`, which the
// host waits for (see icr_amr_get_block).
constexpr int COPY_BLOCKS = 16;
__global__ void k_amr_copy_out(AmrArgs a, int slot, double* __restrict__ out,
                               unsigned long long* flags, unsigned long long seq) {
  const int ncell = a.br * a.bt * a.bp;
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < NA * ncell; c += gridDim.x * blockDim.x) {
    const int v = c / ncell, q = c - v * ncell;
    const int ci = q % a.br, cj = (q / a.br) % a.bt, cq = q / (a.br * a.bt);
    out[c] = a.U[pidx(a, slot, v, AG + cq, AG + cj, AG + ci)];
  }
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_store(flags + blockIdx.x, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace icr

// ======================================================================
// Host side: the block tree, the step loop and the C-ABI.
// ======================================================================
using namespace icr;

namespace {

constexpr double kAUm = 1.495978707e11;
constexpr double kVu = 1.0e5;
constexpr double kMp = 1.67262192369e-27;
constexpr double kKb = 1.380649e-23;
constexpr double kMu0 = 4.0e-7 * 3.14159265358979323846;
constexpr double kGMs = 1.32712440018e20;
constexpr double kPI = 3.14159265358979323846;

size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

struct Key {
  int l, i, j, k;
  bool operator<(const Key& o) const {
    if (l != o.l) return l < o.l;
    if (i != o.i) return i < o.i;
    if (j != o.j) return j < o.j;
    return k < o.k;
  }
  bool operator==(const Key& o) const { return l == o.l && i == o.i && j == o.j && k == o.k; }
};

int err(int code, const std::string& m) { return set_error(code, m.c_str()); }

#define AMR_TRY(expr)                                                                   \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess) return err(ICR_ERR_HIP, std::string(#expr) + " failed: " +    \
                                                      hipGetErrorString(e_));           \
  } while (0)

struct AmrLayout {
  size_t U, U1, F, key, lv, maps[AMR_MAXL + 1], m64[AMR_MAXL + 1], mr[AMR_MAXL + 1],
      bmaps, tau, cme, clock, partials, ind, lists, leaves, rlist, glist, total;
};

}  // namespace

struct icr_amr {
  icr_grid g;
  icr_phys p;
  icr_amr_params q;
  hipStream_t stream;
  char* ws;
  AmrLayout L;
  int nlev, pr, pt, pp, fmax;
  long long bvol;
  int nb[AMR_MAXL + 1][3];
  double t_unit, len_unit, rho_unit, p_unit, b_unit, v_unit, omega, r_in, gm;
  // tree
  std::map<Key, int> slot_of;      // every block (leaf or not) -> slot
  std::vector<Key> key_of;         // slot -> key
  std::vector<unsigned char> leaf; // slot -> leaf flag
  std::vector<int> hmap[AMR_MAXL + 1];  // level -> [nbp][nbt][nbr] slot or -1 (device copy: maps)
  std::vector<int> free_slots;
  int n_maps = 0, n_cme = 0;
  std::vector<double> tau_h;
  bool have_maps = false, have_state = false;
  long long steps_done = 0;

  char* at(size_t off) { return ws + off; }
  DevClock* clock() { return (DevClock*)at(L.clock); }
  double* pin = nullptr;  // pinned host buffer of one leaf, written by the device
  unsigned long long* pin_flags = nullptr;  // behind it: the call each block last wrote for
  unsigned long long pin_seq = 0;

  // the level table on the device (constant after creation)
  int upload_levels() {
    std::vector<AmrLevel> t(AMR_MAXL + 1);
    std::memset(t.data(), 0, t.size() * sizeof(AmrLevel));
    for (int l = 1; l <= nlev; ++l) {
      AmrLevel& v = t[l];
      v.nr = nb[l][0] * q.block_r;
      v.nt = nb[l][1] * q.block_theta;
      v.np = nb[l][2] * q.block_phi;
      v.nbr = nb[l][0];
      v.nbt = nb[l][1];
      v.nbp = nb[l][2];
      v.dth = (g.th_max - g.th_min) / v.nt;
      v.dph = 2.0 * kPI / v.np;
      v.m = metric_view<double>((const double*)at(L.mr[l]), v.nr, v.nt, v.dth);
      v.m64 = (const double*)at(L.m64[l]);
      v.map = (const int*)at(L.maps[l]);
    }
    AMR_TRY(hipMemcpyAsync(at(L.lv), t.data(), t.size() * sizeof(AmrLevel), hipMemcpyHostToDevice,
                           stream));
    AMR_TRY(hipStreamSynchronize(stream));
    return ICR_OK;
  }

  AmrArgs args() {
    AmrArgs a;
    std::memset(&a, 0, sizeof a);
    a.U = (double*)at(L.U);
    a.U1 = (double*)at(L.U1);
    a.F = (double*)at(L.F);
    a.key = (const int*)at(L.key);
    a.lv = (const AmrLevel*)at(L.lv);
    a.nlev = nlev;
    a.br = q.block_r;
    a.bt = q.block_theta;
    a.bp = q.block_phi;
    a.pr = pr;
    a.pt = pt;
    a.pp = pp;
    a.fmax = fmax;
    a.bvol = bvol;
    a.bnd.nt = g.n_theta;
    a.bnd.np = g.n_phi;
    a.bnd.n_maps = n_maps;
    a.bnd.tau = (const double*)at(L.tau);
    a.bnd.maps = (const double*)at(L.bmaps);
    a.bnd.n_cme = n_cme;
    a.bnd.cme = (const double*)at(L.cme);
    a.bnd.tc = (const double*)at(L.m64[1]) + OFF_TC64(g.n_r, g.n_theta);
    a.bnd.dph = 2.0 * kPI / g.n_phi;
    a.bnd.omega = omega;
    a.bnd.r_in = r_in;
    a.clock = clock();
    a.partials = (double*)at(L.partials);
    a.gam = p.gamma;
    a.gm1 = p.gamma - 1.0;
    a.igm1 = 1.0 / (p.gamma - 1.0);
    a.omega = omega;
    a.cfl = p.cfl;
    a.r_in = r_in;
    a.gravity = p.gravity ? 1 : 0;
    a.corot = p.corotation ? 1 : 0;
    return a;
  }

  std::vector<Key> leaves(int l = 0) const {
    std::vector<Key> out;
    for (const auto& kv : slot_of)
      if (leaf[kv.second] && (l == 0 || kv.first.l == l)) out.push_back(kv.first);
    return out;  // std::map order: level, i, j, k
  }
  size_t map_index(const Key& k) const {
    return ((size_t)k.k * nb[k.l][1] + k.j) * nb[k.l][0] + k.i;
  }
  // slot of a block, -1 where there is none (also outside the levels / grid)
  int slot(const Key& k) const {
    if (k.l < 1 || k.l > nlev || k.i < 0 || k.j < 0 || k.k < 0 || k.i >= nb[k.l][0] ||
        k.j >= nb[k.l][1] || k.k >= nb[k.l][2])
      return -1;
    return hmap[k.l][map_index(k)];
  }
  bool has(const Key& k) const { return slot(k) >= 0; }
  bool is_leaf(const Key& k) const {
    const int s = slot(k);
    return s >= 0 && leaf[s];
  }
  bool neighbour(const Key& k, int d, int side, Key* out) const {
    int b[3] = {k.i, k.j, k.k};
    b[d] += side ? 1 : -1;
    if (d == 2) {
      b[2] = (b[2] % nb[k.l][2] + nb[k.l][2]) % nb[k.l][2];
    } else if (b[d] < 0 || b[d] >= nb[k.l][d]) {
      return false;
    }
    *out = Key{k.l, b[0], b[1], b[2]};
    return true;
  }
  static Key parent(const Key& k) { return Key{k.l - 1, k.i / 2, k.j / 2, k.k / 2}; }
  static std::vector<Key> children(const Key& k) {
    std::vector<Key> c;
    for (int e = 0; e < 2; ++e)
      for (int b = 0; b < 2; ++b)
        for (int a = 0; a < 2; ++a) c.push_back(Key{k.l + 1, 2 * k.i + a, 2 * k.j + b, 2 * k.k + e});
    return c;
  }

  int add_block(const Key& k) {
    if (free_slots.empty()) return -1;
    const int s = free_slots.back();
    free_slots.pop_back();
    slot_of[k] = s;
    hmap[k.l][map_index(k)] = s;
    key_of[s] = k;
    leaf[s] = 1;
    return s;
  }
  void remove_block(const Key& k) {
    const int s = slot_of.at(k);
    slot_of.erase(k);
    hmap[k.l][map_index(k)] = -1;
    leaf[s] = 0;
    free_slots.push_back(s);
  }

  // upload key table and level maps
  int upload_tree() {
    const int mb = q.max_blocks;
    std::vector<int> keys(4 * (size_t)mb, 0);
    for (const auto& kv : slot_of) {
      int* p4 = &keys[4 * (size_t)kv.second];
      p4[0] = kv.first.l;
      p4[1] = kv.first.i;
      p4[2] = kv.first.j;
      p4[3] = kv.first.k;
    }
    AMR_TRY(hipMemcpyAsync(at(L.key), keys.data(), keys.size() * sizeof(int),
                           hipMemcpyHostToDevice, stream));
    for (int l = 1; l <= nlev; ++l)
      AMR_TRY(hipMemcpyAsync(at(L.maps[l]), hmap[l].data(), hmap[l].size() * sizeof(int),
                             hipMemcpyHostToDevice, stream));
    AMR_TRY(hipStreamSynchronize(stream));
    return ICR_OK;
  }

  // device lists: the leaves, their ghost faces and the flux-corrected ones,
  // rebuilt after every change of the tree
  int n_all = 0, n_rl = 0;
  // ghost faces inside a step (0) and of a regrid (1): [0] without
  // prolongation, [l] prolonged to level l
  int g_off[2][AMR_MAXL + 2] = {};
  const LeafDesc* leaf_list() { return (const LeafDesc*)at(L.leaves); }
  int* upload_temp(const std::vector<int>& v) {
    int* d = (int*)at(L.lists);
    if (!v.empty())
      (void)hipMemcpy(d, v.data(), v.size() * sizeof(int), hipMemcpyHostToDevice);
    return d;
  }
  int rebuild_lists() {
    const std::vector<Key> lv = leaves();
    std::vector<LeafDesc> all, rl;
    std::vector<FaceDesc> gl[2][AMR_MAXL + 1];
    all.reserve(lv.size());
    const bool reads_neighbours = lds_stage();
    for (const Key& k : lv) {
      LeafDesc D{slot(k), k.l, k.i, k.j, k.k, 0, 0, {}};
      FaceDesc fd[6];
      for (int f = 0; f < 6; ++f) {
        const int d = f >> 1, side = f & 1;
        Key nk;
        fd[f] = FaceDesc{D.slot, f, FACE_EDGE, -1, k.l, k.i, k.j, k.k};
        D.src[f] = LEAF_SELF;
        if (neighbour(k, d, side, &nk)) {
          const int ns = slot(nk);
          fd[f].ns = ns;
          fd[f].kind = ns < 0 ? FACE_COARSE : (leaf[ns] ? FACE_COPY : FACE_FINE);
          D.src[f] = fd[f].kind == FACE_COPY ? LEAF_COPY | ns << 2 : LEAF_POOL;
          if (fd[f].kind != FACE_COPY) D.other |= 1 << f;
          // refined neighbours' children are leaves, by the one-level rule
          if (fd[f].kind == FACE_FINE) D.finer |= 1 << f;
        } else if (f == 0) {
          fd[f].kind = FACE_INNER;
          D.src[f] = LEAF_POOL;
        }
      }
      all.push_back(D);
      if (D.finer) rl.push_back(D);
      // the stage kernel takes copies and edges from their source; in the
      // padded block they are needed where a finer leaf interpolates from it
      const bool whole = D.finer || !reads_neighbours;
      for (int f = 0; f < 6; ++f) {
        const int to = fd[f].kind == FACE_COARSE ? k.l : 0;
        if (whole || (fd[f].kind != FACE_COPY && fd[f].kind != FACE_EDGE))
          gl[0][to].push_back(fd[f]);
        gl[1][to].push_back(fd[f]);
      }
    }
    n_all = (int)all.size();
    n_rl = (int)rl.size();
    std::vector<FaceDesc> g;
    for (int w = 0; w < 2; ++w)
      for (int l = 0; l <= nlev; ++l) {
        g_off[w][l] = (int)g.size();
        g.insert(g.end(), gl[w][l].begin(), gl[w][l].end());
        g_off[w][l + 1] = (int)g.size();
      }
    AMR_TRY(hipMemcpyAsync(at(L.leaves), all.data(), all.size() * sizeof(LeafDesc),
                           hipMemcpyHostToDevice, stream));
    AMR_TRY(hipMemcpyAsync(at(L.glist), g.data(), g.size() * sizeof(FaceDesc),
                           hipMemcpyHostToDevice, stream));
    if (!rl.empty())
      AMR_TRY(hipMemcpyAsync(at(L.rlist), rl.data(), rl.size() * sizeof(LeafDesc),
                             hipMemcpyHostToDevice, stream));
    AMR_TRY(hipStreamSynchronize(stream));
    return ICR_OK;
  }

  // block size and LDS of the face-once stage kernel: 0 (the leaf does not
  // fit it), 256 or 512 threads
  int lds_stage() const {
    const int br = q.block_r, bt = q.block_theta, bp = q.block_phi;
    const int lds = amr_lds_bytes(br, bt, bp);
    if (lds <= AMR_LDS_S && amr_covers(256, br, bt, bp)) return 256;
    return lds <= AMR_LDS_L && amr_covers(512, br, bt, bp) ? 512 : 0;
  }
  template <int FLUX, int LIM>
  void launch_stage_t(const AmrArgs& a, const LeafDesc* d, int n, int stage) {
    const int nt = lds_stage();
    if (nt == 256)
      hipLaunchKernelGGL((k_amr_stage_lds<FLUX, LIM, 256, AMR_LDS_S>), dim3(n), dim3(256), 0,
                         stream, a, d, stage);
    else if (nt == 512)
      hipLaunchKernelGGL((k_amr_stage_lds<FLUX, LIM, 512, AMR_LDS_L>), dim3(n), dim3(512), 0,
                         stream, a, d, stage);
    else
      hipLaunchKernelGGL((k_amr_stage<FLUX, LIM>), dim3(n), dim3(256), 0, stream, a, d, stage);
  }
  void launch_stage(const AmrArgs& a, const LeafDesc* d, int n, int stage) {
    const int f = p.flux, lm = p.limiter;
    if (f == ICR_FLUX_TVDLF && lm == ICR_LIM_MINMOD) launch_stage_t<FLUX_TVDLF, LIM_MINMOD>(a, d, n, stage);
    else if (f == ICR_FLUX_TVDLF) launch_stage_t<FLUX_TVDLF, LIM_MC>(a, d, n, stage);
    else if (f == ICR_FLUX_HLL && lm == ICR_LIM_MINMOD) launch_stage_t<FLUX_HLL, LIM_MINMOD>(a, d, n, stage);
    else if (f == ICR_FLUX_HLL) launch_stage_t<FLUX_HLL, LIM_MC>(a, d, n, stage);
    else if (lm == ICR_LIM_MINMOD) launch_stage_t<FLUX_HLLD, LIM_MINMOD>(a, d, n, stage);
    else launch_stage_t<FLUX_HLLD, LIM_MC>(a, d, n, stage);
  }

  // stage right-hand sides, updates and flux corrections; CFL of the result
  void enqueue_step() {
    const size_t nl = (size_t)n_all;
    const LeafDesc* d_all = leaf_list();
    for (int stage = 1; stage <= 2; ++stage) {
      fill_ghosts_at(stage == 2, stage == 2, 0);
      AmrArgs a = args();
      launch_stage(a, d_all, (int)nl, stage);
      if (n_rl > 0)
        hipLaunchKernelGGL(k_amr_reflux, dim3((unsigned)n_rl), dim3(128), 0, stream, a,
                           (const LeafDesc*)at(L.rlist), stage);
    }
    AmrArgs a = args();
    hipLaunchKernelGGL(k_amr_cfl, dim3((unsigned)nl), dim3(256), 0, stream, a, d_all);
    ProbeArgs pa;
    std::memset(&pa, 0, sizeof pa);
    launch_finalize<double>(clock(), (const double*)at(L.partials), (int)nl, p.cfl, 1, 0, pa,
                            nullptr, nullptr, stream);
  }

  void fill_ghosts_at(int use_u1, int plus_dt, int always) {
    AmrArgs a = args();
    // the faces without a coarser neighbour first, then the prolonged ones
    // level by level (their source leaves' ghosts are then complete)
    for (int l = 0; l <= nlev; ++l) {
      const int *off = g_off[always ? 1 : 0], n = off[l + 1] - off[l];
      if (n == 0) continue;
      hipLaunchKernelGGL(k_amr_ghost, dim3((unsigned)n), dim3(256), 0, stream, a,
                         (const FaceDesc*)at(L.glist) + off[l], use_u1, plus_dt, always);
    }
  }

  int first_dt() {
    const LeafDesc* d_all = leaf_list();
    AmrArgs a = args();
    hipLaunchKernelGGL(k_amr_cfl, dim3((unsigned)n_all), dim3(256), 0, stream, a, d_all);
    ProbeArgs pa;
    std::memset(&pa, 0, sizeof pa);
    launch_finalize<double>(clock(), (const double*)at(L.partials), n_all, p.cfl, 0, 0, pa,
                            nullptr, nullptr, stream);
    AMR_TRY(hipGetLastError());
    AMR_TRY(hipStreamSynchronize(stream));
    return ICR_OK;
  }

  int read_clock(DevClock* c) {
    AMR_TRY(hipMemcpyAsync(c, clock(), sizeof(DevClock), hipMemcpyDeviceToHost, stream));
    AMR_TRY(hipStreamSynchronize(stream));
    return ICR_OK;
  }
  int write_clock(const DevClock* c) {
    AMR_TRY(hipMemcpyAsync(clock(), c, sizeof(DevClock), hipMemcpyHostToDevice, stream));
    AMR_TRY(hipStreamSynchronize(stream));
    return ICR_OK;
  }

  // --- regrid ------------------------------------------------------------
  void balance(std::set<Key>& refine) const {
    bool changed = true;
    while (changed) {
      changed = false;
      std::vector<Key> cur(refine.begin(), refine.end());
      for (const Key& k : cur)
        for (int d = 0; d < 3; ++d)
          for (int s = 0; s < 2; ++s) {
            Key nk;
            if (!neighbour(k, d, s, &nk) || has(nk)) continue;
            const Key pk = parent(nk);
            if (is_leaf(pk) && !refine.count(pk)) {
              refine.insert(pk);
              changed = true;
            }
          }
    }
  }

  int apply(const std::set<Key>& coarsen, const std::set<Key>& refine) {
    // ghosts of U at the current time for the prolongation slopes
    fill_ghosts_at(0, 0, 1);
    // merges: parents take the volume-weighted mean of their children
    std::vector<int> parents;
    for (const Key& pk : coarsen) parents.push_back(slot_of.at(pk));
    if (!parents.empty()) {
      int* d = upload_temp(parents);
      AmrArgs a = args();
      hipLaunchKernelGGL(k_amr_restrict, dim3((unsigned)parents.size()), dim3(256), 0, stream, a,
                         d);
      AMR_TRY(hipStreamSynchronize(stream));
      for (const Key& pk : coarsen) {
        for (const Key& c : children(pk)) remove_block(c);
        leaf[slot_of.at(pk)] = 1;
      }
    }
    // splits, coarser levels first (std::set order is level-major)
    std::vector<int> pairs;
    for (const Key& k : refine) {
      if (!is_leaf(k)) continue;
      for (const Key& c : children(k)) {
        const int s = add_block(c);
        if (s < 0) return err(ICR_ERR_STATE, "AMR block pool full (raise max_blocks)");
        pairs.push_back(slot_of.at(k));
        pairs.push_back(s);
      }
      leaf[slot_of.at(k)] = 0;
    }
    int rc = upload_tree();
    if (!rc) rc = rebuild_lists();
    if (rc) return rc;
    if (!pairs.empty()) {
      // a split's children read their parent's padded block, which is not
      // touched by any other split of this pass (parents are distinct)
      int* d = upload_temp(pairs);
      AmrArgs a = args();
      hipLaunchKernelGGL(k_amr_prolong, dim3((unsigned)(pairs.size() / 2)), dim3(256), 0, stream,
                         a, d);
      AMR_TRY(hipGetLastError());
      AMR_TRY(hipStreamSynchronize(stream));
    }
    return ICR_OK;
  }

  int regrid() {
    std::vector<Key> lv = leaves();  // the order of the device list
    fill_ghosts_at(0, 0, 1);
    AmrArgs a = args();
    double* ind = (double*)at(L.ind);
    hipLaunchKernelGGL(k_amr_indicators, dim3((unsigned)n_all), dim3(256), 0, stream, a,
                       leaf_list(), ind);
    std::vector<double> h(2 * lv.size());
    AMR_TRY(hipMemcpyAsync(h.data(), ind, h.size() * sizeof(double), hipMemcpyDeviceToHost,
                           stream));
    AMR_TRY(hipStreamSynchronize(stream));
    // per slot: -1 not a leaf of this regrid, else the leaf's criterion
    std::vector<signed char> flag(q.max_blocks, -1);
    std::set<Key> refine;
    for (size_t n = 0; n < lv.size(); ++n) {
      const bool tr = h[2 * n] >= q.tau_threshold;
      const bool sh = h[2 * n + 1] >= q.shock_threshold;
      const bool f = q.criterion == ICR_AMR_TRACING ? tr : (q.criterion == ICR_AMR_SHOCK ? sh : (tr || sh));
      flag[slot(lv[n])] = f ? 1 : 0;
      if (f && lv[n].l < nlev) refine.insert(lv[n]);
    }
    balance(refine);
    std::set<Key> coarsen;
    std::set<Key> parents;
    for (const Key& k : lv)
      if (k.l > 1) parents.insert(parent(k));
    for (const Key& pk : parents) {
      bool all = true;
      for (const Key& c : children(pk)) {
        const int cs = slot(c);
        if (cs < 0 || !leaf[cs] || flag[cs] != 0 || refine.count(c)) all = false;
      }
      if (!all) continue;
      bool ok = true;
      for (int dd = 0; dd < 3; ++dd)
        for (int sd = 0; sd < 2; ++sd) {
          Key nk;
          if (!neighbour(pk, dd, sd, &nk)) continue;
          if (has(nk) && !is_leaf(nk))
            for (const Key& gch : children(nk))
              if (has(gch) && !is_leaf(gch)) ok = false;
          if (refine.count(nk)) ok = false;
          if (has(nk))
            for (const Key& gch : children(nk))
              if (refine.count(gch)) ok = false;
        }
      if (ok) coarsen.insert(pk);
    }
    return apply(coarsen, refine);
  }
};

namespace {

int validate_amr(const icr_grid* g, const icr_phys* p, const icr_amr_params* q) {
  if (!g || !p || !q) return err(ICR_ERR_ARG, "grid, phys and params must not be NULL");
  if (p->precision != ICR_PREC_F64) return err(ICR_ERR_UNSUPPORTED, "AMR runs in FP64 only");
  if (p->limiter == ICR_LIM_WENO5) return err(ICR_ERR_UNSUPPORTED, "AMR has two ghost layers (no WENO5)");
  if (p->bc_transverse != ICR_BCT_MAP) return err(ICR_ERR_UNSUPPORTED, "AMR uses the map transverse rule");
  if (q->block_r < 4 || q->block_theta < 4 || q->block_phi < 4)
    return err(ICR_ERR_ARG, "AMR blocks need at least 4 cells per side");
  if (g->n_r % q->block_r || g->n_theta % q->block_theta || g->n_phi % q->block_phi)
    return err(ICR_ERR_ARG, "the block size must divide the base grid");
  if (q->max_level < 1 || q->max_level > AMR_MAXL)
    return err(ICR_ERR_ARG, "max_level must be in [1, 6]");
  if (q->criterion < ICR_AMR_TRACING || q->criterion > ICR_AMR_COMBINED)
    return err(ICR_ERR_ARG, "unknown AMR criterion");
  if (q->regrid_every < 1) return err(ICR_ERR_ARG, "regrid_every must be >= 1");
  const long long base = (long long)(g->n_r / q->block_r) * (g->n_theta / q->block_theta) *
                         (g->n_phi / q->block_phi);
  if (q->max_blocks < base) return err(ICR_ERR_ARG, "max_blocks below the base grid's blocks");
  if (!(p->gamma > 1.0) || !(p->cfl > 0.0 && p->cfl <= 1.0)) return err(ICR_ERR_ARG, "gamma / cfl");
  if (!(g->r_in > 0 && g->r_out > g->r_in) || !(g->th_min > 0 && g->th_max > g->th_min && g->th_max < kPI))
    return err(ICR_ERR_ARG, "invalid grid extent");
  if (g->max_maps < 1 || g->max_cmes < 0) return err(ICR_ERR_ARG, "invalid capacities");
  return ICR_OK;
}

AmrLayout amr_layout(const icr_grid& g, const icr_amr_params& q) {
  AmrLayout L{};
  const long long pr = q.block_r + 2 * AG, pt = q.block_theta + 2 * AG, pp = q.block_phi + 2 * AG;
  const size_t bvol = (size_t)(pr * pt * pp);
  const int fmax = std::max(q.block_phi * q.block_theta,
                            std::max(q.block_phi * q.block_r, q.block_theta * q.block_r));
  size_t off = 0;
  auto take = [&](size_t b) {
    const size_t o = off;
    off += al256(b);
    return o;
  };
  const size_t mb = (size_t)q.max_blocks;
  L.U = take(sizeof(double) * NA * bvol * mb);
  L.U1 = take(sizeof(double) * NA * bvol * mb);
  L.F = take(sizeof(double) * 6 * NA * (size_t)fmax * mb);
  L.key = take(sizeof(int) * 4 * mb);
  L.lv = take(sizeof(AmrLevel) * (AMR_MAXL + 1));
  for (int l = 1; l <= q.max_level; ++l) {
    const long long f = 1LL << (l - 1);
    const long long nr = g.n_r * f, nt = g.n_theta * f, np = g.n_phi * f;
    L.maps[l] = take(sizeof(int) * (size_t)((nr / q.block_r) * (nt / q.block_theta) *
                                            (np / q.block_phi)));
    L.m64[l] = take(sizeof(double) * (size_t)METRIC64_LEN((int)nr, (int)nt));
    L.mr[l] = take(sizeof(double) * (size_t)METRICR_LEN((int)nr, (int)nt));
  }
  L.bmaps = take(sizeof(double) * (size_t)g.max_maps * NV * g.n_theta * g.n_phi);
  L.tau = take(sizeof(double) * (size_t)g.max_maps);
  L.cme = take(sizeof(double) * 8 * (size_t)std::max(1, g.max_cmes));
  L.clock = take(sizeof(DevClock));
  L.partials = take(sizeof(double) * 4 * mb);
  L.ind = take(sizeof(double) * 2 * mb);
  // temporary slot lists of a regrid [4 mb]; the leaves; those next to finer
  // leaves; the faces to fill inside a step, then those of a regrid
  L.lists = take(sizeof(int) * 4 * mb);
  L.leaves = take(sizeof(LeafDesc) * mb);
  L.rlist = take(sizeof(LeafDesc) * mb);
  L.glist = take(sizeof(FaceDesc) * 12 * mb);
  L.total = off;
  return L;
}

}  // namespace

extern "C" {

int icr_amr_workspace_bytes(const icr_grid* g, const icr_phys* p, const icr_amr_params* q,
                            size_t* bytes) {
  int rc = validate_amr(g, p, q);
  if (rc) return rc;
  if (!bytes) return err(ICR_ERR_ARG, "bytes is NULL");
  *bytes = amr_layout(*g, *q).total;
  return ICR_OK;
}

int icr_amr_create(const icr_grid* g, const icr_phys* p, const icr_amr_params* q, void* ws,
                   size_t bytes, void* stream, icr_amr** out) {
  int rc = validate_amr(g, p, q);
  if (rc) return rc;
  if (!out) return err(ICR_ERR_ARG, "out is NULL");
  *out = nullptr;
  AmrLayout L = amr_layout(*g, *q);
  if (!ws || bytes < L.total) return err(ICR_ERR_ARG, "workspace too small");
  if (((uintptr_t)ws & 255) != 0) return err(ICR_ERR_ARG, "workspace must be 256-byte aligned");
  icr_amr* a = new icr_amr();
  a->g = *g;
  a->p = *p;
  a->q = *q;
  a->stream = (hipStream_t)stream;
  a->ws = (char*)ws;
  a->L = L;
  a->nlev = q->max_level;
  a->pr = q->block_r + 2 * AG;
  a->pt = q->block_theta + 2 * AG;
  a->pp = q->block_phi + 2 * AG;
  a->bvol = (long long)a->pr * a->pt * a->pp;
  a->fmax = std::max(q->block_phi * q->block_theta,
                     std::max(q->block_phi * q->block_r, q->block_theta * q->block_r));
  a->len_unit = kAUm;
  a->v_unit = kVu;
  a->t_unit = kAUm / kVu;
  a->rho_unit = kMp * 1.0e6;
  a->p_unit = a->rho_unit * kVu * kVu;
  a->b_unit = std::sqrt(kMu0 * a->rho_unit) * kVu;
  a->omega = p->corotation ? p->omega * a->t_unit : 0.0;
  a->r_in = g->r_in / a->len_unit;
  a->gm = p->gravity ? kGMs / (a->len_unit * kVu * kVu) : 0.0;
  for (int l = 1; l <= a->nlev; ++l) {
    const int f = 1 << (l - 1);
    a->nb[l][0] = g->n_r * f / q->block_r;
    a->nb[l][1] = g->n_theta * f / q->block_theta;
    a->nb[l][2] = g->n_phi * f / q->block_phi;
    MetricArgs m;
    m.nr = g->n_r * f;
    m.nt = g->n_theta * f;
    m.r_in = a->r_in;
    m.r_out = g->r_out / a->len_unit;
    m.q = std::pow(m.r_out / m.r_in, 1.0 / m.nr);
    m.th_min = g->th_min;
    m.th_max = g->th_max;
    m.dph = 2.0 * kPI / (g->n_phi * f);
    m.gm = a->gm;
    m.m64 = (double*)a->at(L.m64[l]);
    launch_metric(m, a->at(L.mr[l]), false, a->stream);
  }
  for (int l = 1; l <= a->nlev; ++l)
    a->hmap[l].assign((size_t)a->nb[l][0] * a->nb[l][1] * a->nb[l][2], -1);
  a->key_of.assign(q->max_blocks, Key{0, 0, 0, 0});
  a->leaf.assign(q->max_blocks, 0);
  for (int s = q->max_blocks - 1; s >= 0; --s) a->free_slots.push_back(s);
  for (int k = 0; k < a->nb[1][2]; ++k)
    for (int j = 0; j < a->nb[1][1]; ++j)
      for (int i = 0; i < a->nb[1][0]; ++i) a->add_block(Key{1, i, j, k});
  DevClock c;
  std::memset(&c, 0, sizeof c);
  c.bad = BAD_NONE;
  c.t_end = -1.0;
  c.last_sample = -1;
  rc = a->write_clock(&c);
  if (!rc) rc = a->upload_levels();
  if (!rc) rc = a->upload_tree();
  if (!rc) rc = a->rebuild_lists();
  if (!rc) {
    const size_t n = NA * (size_t)q->block_r * q->block_theta * q->block_phi;
    const size_t bytes = sizeof(double) * n + sizeof(unsigned long long) * COPY_BLOCKS;
    const hipError_t e = hipHostMalloc((void**)&a->pin, bytes, hipHostMallocDefault);
    if (e != hipSuccess) {
      rc = err(ICR_ERR_HIP, std::string("hipHostMalloc failed: ") + hipGetErrorString(e));
    } else {
      a->pin_flags = (unsigned long long*)(a->pin + n);
      std::memset(a->pin_flags, 0, sizeof(unsigned long long) * COPY_BLOCKS);
    }
  }
  if (rc) {
    delete a;
    return rc;
  }
  *out = a;
  return ICR_OK;
}

void icr_amr_destroy(icr_amr* a) {
  if (!a) return;
  (void)hipStreamSynchronize(a->stream);
  (void)hipHostFree(a->pin);
  delete a;
}

int icr_amr_set_boundary_maps(icr_amr* a, int n, const double* t_s, const double* maps) {
  if (!a || !t_s || !maps) return err(ICR_ERR_ARG, "NULL argument");
  if (n < 1 || n > a->g.max_maps) return err(ICR_ERR_ARG, "n_maps outside [1, max_maps]");
  for (int m = 1; m < n; ++m)
    if (!(t_s[m] > t_s[m - 1])) return err(ICR_ERR_ARG, "map times must ascend strictly");
  const size_t plane = (size_t)a->g.n_theta * a->g.n_phi;
  std::vector<double> h((size_t)n * NV * plane);
  const double sc[NV] = {a->rho_unit, a->v_unit, a->v_unit, a->v_unit,
                         a->p_unit,   a->b_unit, a->b_unit, a->b_unit};
  const size_t nt = a->g.n_theta, np = a->g.n_phi;
  for (int m = 0; m < n; ++m)
    for (int v = 0; v < NV; ++v) {
      const double* src = maps + ((size_t)m * NV + v) * plane;
      double* dst = h.data() + ((size_t)m * NV + v) * plane;
      for (size_t j = 0; j < nt; ++j)
        for (size_t k = 0; k < np; ++k) {
          const double x = src[j * np + k];
          if ((v == 0 || v == 4) && !(x > 0.0)) return err(ICR_ERR_ARG, "map rho or p <= 0");
          if (!std::isfinite(x)) return err(ICR_ERR_ARG, "map has a non-finite value");
          dst[k * nt + j] = x / sc[v];
        }
    }
  std::vector<double> tau(n);
  for (int m = 0; m < n; ++m) tau[m] = t_s[m] / a->t_unit;
  AMR_TRY(hipMemcpyAsync(a->at(a->L.bmaps), h.data(), h.size() * sizeof(double),
                         hipMemcpyHostToDevice, a->stream));
  AMR_TRY(hipMemcpyAsync(a->at(a->L.tau), tau.data(), n * sizeof(double), hipMemcpyHostToDevice,
                         a->stream));
  AMR_TRY(hipStreamSynchronize(a->stream));
  a->n_maps = n;
  a->have_maps = true;
  return ICR_OK;
}

int icr_amr_set_cmes(icr_amr* a, int n, const double* rows) {
  if (!a) return err(ICR_ERR_ARG, "NULL argument");
  if (n < 0 || n > a->g.max_cmes) return err(ICR_ERR_ARG, "n outside [0, max_cmes]");
  if (n > 0 && !rows) return err(ICR_ERR_ARG, "rows is NULL");
  std::vector<double> c((size_t)8 * std::max(1, n));
  for (int k = 0; k < n; ++k) {
    const double* r = rows + 8 * k;
    if (!(r[1] > 0 && r[4] > 0 && r[5] > 0 && r[6] > 0 && r[7] > 0))
      return err(ICR_ERR_ARG, "CME duration, half-width, speed, density, T must be > 0");
    double* d = c.data() + 8 * k;
    d[0] = r[0] / a->t_unit;
    d[1] = r[1] / a->t_unit;
    d[2] = 0.5 * kPI - r[2];
    d[3] = r[3];
    d[4] = std::cos(r[4]);
    d[5] = r[5] / a->v_unit;
    d[6] = r[6] / a->rho_unit;
    d[7] = 2.0 * (r[6] / kMp) * kKb * r[7] / a->p_unit;
  }
  if (n > 0) {
    AMR_TRY(hipMemcpyAsync(a->at(a->L.cme), c.data(), 8 * n * sizeof(double),
                           hipMemcpyHostToDevice, a->stream));
    AMR_TRY(hipStreamSynchronize(a->stream));
  }
  a->n_cme = n;
  return ICR_OK;
}

int icr_amr_init_radial(icr_amr* a) {
  if (!a) return err(ICR_ERR_ARG, "NULL argument");
  if (!a->have_maps) return err(ICR_ERR_STATE, "set boundary maps first");
  // back to the base blocks
  std::vector<Key> all;
  for (const auto& kv : a->slot_of) all.push_back(kv.first);
  for (const Key& k : all)
    if (k.l > 1) a->remove_block(k);
  for (auto& kv : a->slot_of) a->leaf[kv.second] = 1;
  int rc = a->upload_tree();
  if (!rc) rc = a->rebuild_lists();
  if (rc) return rc;
  AmrArgs args = a->args();
  hipLaunchKernelGGL(k_amr_init, dim3((unsigned)a->n_all), dim3(256), 0, a->stream, args,
                     a->leaf_list(), a->p.gamma);
  AMR_TRY(hipGetLastError());
  DevClock c;
  rc = a->read_clock(&c);
  if (rc) return rc;
  c.t = 0.0;
  c.step = 0;
  c.bad = BAD_NONE;
  c.last_dt = 0.0;
  c.resid = 0.0;
  rc = a->write_clock(&c);
  if (rc) return rc;
  a->have_state = true;
  a->steps_done = 0;
  return a->first_dt();
}

int icr_amr_step(icr_amr* a, int n, double t_end_s, icr_step_info* info) {
  if (!a) return err(ICR_ERR_ARG, "NULL argument");
  if (n < 0) return err(ICR_ERR_ARG, "n_steps must be >= 0");
  if (!a->have_state) return err(ICR_ERR_STATE, "initialise the state first");
  launch_clock_begin(a->clock(), t_end_s > 0.0 ? t_end_s / a->t_unit : -1.0, a->stream);
  DevClock c;
  for (int s = 0; s < n; ++s) {
    a->enqueue_step();
    ++a->steps_done;
    if (a->nlev > 1 && a->steps_done % a->q.regrid_every == 0) {
      int rc = a->read_clock(&c);
      if (rc) return rc;
      if (c.bad != BAD_NONE || !c.active) break;
      rc = a->regrid();
      if (rc) return rc;
      rc = a->first_dt();  // the CFL dt of the new leaves
      if (rc) return rc;
    }
  }
  AMR_TRY(hipGetLastError());
  int rc = a->read_clock(&c);
  if (rc) return rc;
  if (info) {
    info->steps_taken = (int)c.taken;
    info->status = c.bad == BAD_NONE ? ICR_OK : ICR_ERR_NONPHYSICAL;
    info->bad_cell = c.bad == BAD_NONE ? -1 : c.bad;
    info->t = c.t * a->t_unit;
    info->last_dt = c.last_dt * a->t_unit;
    info->residual = 0.0;
  }
  if (c.bad != BAD_NONE) return err(ICR_ERR_NONPHYSICAL, "non-physical cell on the refined grid");
  return ICR_OK;
}

int icr_amr_force_refine(icr_amr* a, int n, const int* keys) {
  if (!a || (n > 0 && !keys)) return err(ICR_ERR_ARG, "NULL argument");
  if (!a->have_state) return err(ICR_ERR_STATE, "initialise the state first");
  std::set<Key> refine;
  for (int q = 0; q < n; ++q) {
    const Key k{keys[4 * q], keys[4 * q + 1], keys[4 * q + 2], keys[4 * q + 3]};
    if (!a->is_leaf(k) || k.l >= a->nlev) return err(ICR_ERR_ARG, "not a leaf below the top level");
    refine.insert(k);
  }
  a->balance(refine);
  int rc = a->apply(std::set<Key>(), refine);
  if (rc) return rc;
  return a->first_dt();
}

int icr_amr_leaves(icr_amr* a, int cap, int* keys, int* n) {
  if (!a || !n) return err(ICR_ERR_ARG, "NULL argument");
  std::vector<Key> lv = a->leaves();
  *n = (int)lv.size();
  for (int q = 0; q < (int)lv.size() && q < cap; ++q) {
    keys[4 * q] = lv[q].l;
    keys[4 * q + 1] = lv[q].i;
    keys[4 * q + 2] = lv[q].j;
    keys[4 * q + 3] = lv[q].k;
  }
  return ICR_OK;
}

int icr_amr_get_block(icr_amr* a, const int* key, double* out) {
  if (!a || !key || !out) return err(ICR_ERR_ARG, "NULL argument");
  const Key k{key[0], key[1], key[2], key[3]};
  if (!a->is_leaf(k)) return err(ICR_ERR_ARG, "no such leaf");
  const int ncell = a->q.block_r * a->q.block_theta * a->q.block_phi;
  // the kernel writes the pinned buffer itself: a device-to-host copy of one
  // leaf into pageable memory cost more than the rest of the call (27 us).
  // It also says when it is done: waiting for its flags takes 10.6 us a call
  // where a stream synchronisation took 14.0.  Not seen within COPY_SPIN (the
  // stream is busy, or failed), the stream is synchronised as ever.
  constexpr auto COPY_SPIN = std::chrono::milliseconds(2);
  AmrArgs args = a->args();
  const unsigned long long seq = ++a->pin_seq;
  hipLaunchKernelGGL(k_amr_copy_out, dim3(COPY_BLOCKS), dim3(256), 0, a->stream, args, a->slot(k),
                     a->pin, a->pin_flags, seq);
  AMR_TRY(hipGetLastError());
  const auto start = std::chrono::steady_clock::now();
  int done = 0;
  for (unsigned n = 1; done < COPY_BLOCKS; ++n) {
    if (__atomic_load_n(a->pin_flags + done, __ATOMIC_ACQUIRE) == seq)
      ++done;
    else if (n % 64 == 0 && std::chrono::steady_clock::now() - start > COPY_SPIN)
      break;
  }
  if (done < COPY_BLOCKS) AMR_TRY(hipStreamSynchronize(a->stream));
  std::memcpy(out, a->pin, sizeof(double) * NA * ncell);
  return ICR_OK;
}

int icr_amr_get_clock(icr_amr* a, icr_clock* out) {
  if (!a || !out) return err(ICR_ERR_ARG, "NULL argument");
  DevClock c;
  int rc = a->read_clock(&c);
  if (rc) return rc;
  out->t = c.t * a->t_unit;
  out->step = c.step;
  out->last_dt = c.last_dt * a->t_unit;
  out->next_dt = c.dt_cfl * a->t_unit;
  out->residual = 0.0;
  out->t_code = c.t;
  return ICR_OK;
}

}  // extern "C"
