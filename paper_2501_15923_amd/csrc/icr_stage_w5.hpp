// icr_stage_w5.hpp -- face-once stage tile for the WENO5 reconstruction
// (three ghost layers, six-cell stencils), the counterpart of stage_tile in
// icr_stage_lds.hpp for the minmod / MC limiters.
//
// A block of 64 x 4 threads marches along phi over a chunk of planes; each
// row of 64 lanes covers 58 cells plus the three-cell r halo on either side.
// Per plane the primitives of the tile's rows plus a three-row theta halo
// sit in LDS; every face flux is computed once and shared by its two cells.
// In every direction each cell forms both of its WENO5 edge values from its
// five-cell stencil (the two mirrored reconstructions share the smoothness
// indicators), and a face pairs the upper value of the cell below with the
// lower value of the cell above: along r the lane below is one lane down in
// the same wave (a wave is one row), along theta the row below is another
// wave and its values pass through LDS, along phi the previous plane's
// value is carried in registers.  Each thread keeps the primitives of
// planes k-1 .. k+2 of its own column (and loads k+3), the upper phi edge
// value of cell k and the flux of face k-1/2 from the previous plane.
// WENO5 works on primitive variables like the slope
// limiters (Jiang & Shu 1996 weights, a face state with rho or p <= 0 falls
// back to its cell value); the weight normalisation multiplies by the
// refined reciprocal, as the fluxes do.  Stage 2 also forms the
// per-block partials of the next CFL dt, of the relaxation residual and of
// the validity flag.
#pragma once
#include "icr_stage_lds.hpp"

namespace icr {

constexpr int W5_TR = 64, W5_TT = 4, W5_H = 3;
constexpr int W5_TI = W5_TR - 2 * W5_H;  // cells along r per tile row

// Both WENO5 edge values of the cell c from the five cells a..e: up = the
// value at the face between c and d (weno5(a, b, c, d, e)), dn = the value
// at the face between b and c (weno5(e, d, c, b, a)).  The mirrored stencil
// has the same three smoothness indicators in reverse order and the same
// eps, so they are formed once.  Reversing the stencil exchanges up and dn up
// to the rounding of the mean square in eps, which is summed in one order.
// Everything is written in the four differences and the three second
// differences, the candidates as offsets from c (times 6), the indicators
// times 4 and the weights times 10: 60 operations and two reciprocals, where
// the textbook sums took 79.  Equal to the two weno5 calls up to rounding.
// At 600 x 60 x 120 in FP64 stage 1 / 2 went from 764 / 874 to 659 / 818 us
// (with the two-wave face flux and the grouped flux reads of the update), and
// with the update at raised priority to 639 / 792 us.
template <typename R, bool FAST = false>
__device__ __forceinline__ void weno5_cell(R a, R b, R c, R d, R e, R& up, R& dn) {
  constexpr R k13 = R(13) / R(3), sixth = R(1) / R(6);
  const R D1 = b - a, D2 = c - b, D3 = d - c, D4 = e - d;
  const R s0 = D2 - D1, s1 = D3 - D2, s2 = D4 - D3;
  const R t0 = fma_(R(2), D2, s0), t1 = D2 + D3, t2 = fma_(R(-2), D3, s2);
  const R sq = fma_(a, a, e * e) + fma_(b, b, fma_(d, d, c * c));
  // 4 eps: 1e-6 of the stencil's mean square and the absolute floor
  const R eps = fma_(R(0.8e-6), sq, sizeof(R) == 8 ? R(4e-40) : R(4e-15));
  const R b0 = fma_(k13, s0 * s0, fma_(t0, t0, eps));
  const R b1 = fma_(k13, s1 * s1, fma_(t1, t1, eps));
  const R b2 = fma_(k13, s2 * s2, fma_(t2, t2, eps));
  const R g0 = b0 * b0, g1 = b1 * b1, g2 = b2 * b2;
  const R P = R(3) * D2, Q = R(3) * D3;
  const R u0 = fma_(R(2), s0, P), u1 = fma_(R(2), D3, D2), u2 = Q - s2;
  const R d0 = fma_(R(-2), s2, Q), d1 = fma_(R(2), D2, D3), d2 = P + s0;
  if constexpr (sizeof(R) == 8) {
    // weights d_k / g_k scaled by 10 g0 g1 g2 (one reciprocal per value)
    const R p12 = g1 * g2, p02 = R(6) * (g0 * g2), p01 = g0 * g1;
    const R q01 = R(3) * p01, q12 = R(3) * p12;
    const R un = fma_(p12, u0, fma_(p02, u1, q01 * u2)), us = (p12 + p02) + q01;
    const R dnn = fma_(p01, d0, fma_(p02, d1, q12 * d2)), ds = (p01 + p02) + q12;
    const R ru = FAST ? rcp_fast(us) : R(1) / us, rd = FAST ? rcp_fast(ds) : R(1) / ds;
    up = fma_(un * ru, sixth, c);
    dn = fma_(dnn * rd, -sixth, c);
  } else {
    const R i0 = FAST ? rcp_fast(g0) : R(1) / g0;
    const R i1 = R(6) * (FAST ? rcp_fast(g1) : R(1) / g1);
    const R i2 = FAST ? rcp_fast(g2) : R(1) / g2;
    const R q0 = R(3) * i0, q2 = R(3) * i2;
    const R un = fma_(i0, u0, fma_(i1, u1, q2 * u2)), us = (i0 + i1) + q2;
    const R dnn = fma_(i2, d0, fma_(i1, d1, q0 * d2)), ds = (i2 + i1) + q0;
    up = fma_(un / us, sixth, c);
    dn = fma_(dnn / ds, -sixth, c);
  }
}

// Both edge values of a variable are complete here: without this the
// compiler forms every variable's upper values first (the shuffle needs
// them) and keeps the inputs of all lower values live, which spills.  The
// empty asm emits no instruction.
template <typename R>
__device__ __forceinline__ void pin(R& x, R& y) {
  asm volatile("" : "+v"(x), "+v"(y));
}

template <typename R>
struct alignas(16) StageW5 {
  R sW[NV][W5_TT + 2 * W5_H][W5_TR];  // primitives, rows j0-3 .. j0+TT+2
  R sFr[NV][W5_TT][W5_TR];            // r face i-1/2 at the lane of cell i
  R sFt[NV][W5_TT + 1][W5_TR];        // theta face j-1/2 at row j (0 .. TT)
};

template <typename R, int FLUX, int STAGE>
__device__ __forceinline__ void stage_tile_w5(const StageArgs<R>& a, int kplanes, int bx, int by,
                                              int bz, int pslot, StageW5<R>& sm) {
  constexpr int TR = W5_TR, TT = W5_TT, H = W5_H, NT = TR * TT, WT = TT + 2 * H;
  auto& sW = sm.sW;
  auto& sFr = sm.sFr;
  auto& sFt = sm.sFt;

  const int ti = threadIdx.x, tj = threadIdx.y, tid = tj * TR + ti;
  const int i0 = bx * W5_TI, j0 = by * TT, k0 = bz * kplanes;
  const int nr = a.nr, nt = a.nt, np = a.np;
  const int kend = k0 + kplanes < np ? k0 + kplanes : np;
  const int i = i0 + ti - H, j = j0 + tj;  // this lane's cell
  const bool inner = ti >= H && ti < TR - H;
  const bool valid = inner && i < nr && j < nt;
  // own column: the cell itself, the last cell beyond r_out; below r_in
  // cell 0, or under the asymm rule the mirror cell -1 - i
  const int ic = i < 0 ? (a.asymm ? (-1 - i < nr ? -1 - i : nr - 1) : 0)
                       : (i < nr ? i : nr - 1);
  const int jc = j < nt ? j : nt - 1;
  const unsigned colbase = (unsigned)(jc * nr + ic);
  bool flipj;
  const int mj = mirror_row(j, nt, flipj);
  const unsigned lbase = (unsigned)(mj * nr + ic);
  const bool lghost = i < 0;
  const unsigned plane_cells = (unsigned)(nt * nr);
  const long long gplane = (long long)nt * np;
  auto load_own = [&](int k, R (&w)[NV]) {
    load_cons_prim<R, true>(a, (unsigned)wrap_phi(k, np) * plane_cells + lbase, w);
    if (flipj) flip_theta(w);
  };

  if (!a.clock->active) {
    if (STAGE == 2 && valid)
      for (int k = k0; k < kend; ++k) {
        const unsigned c = (unsigned)k * plane_cells + colbase;
#pragma unroll
        for (int v = 0; v < NV; ++v) stg(a.uout + v * a.ncell, c, ldg(a.un + v * a.ncell, c));
      }
    return;
  }
  const R dt = (R)a.clock->dt;

  // phi ring: at the top of iteration k, w0 .. w3 = W(k-1) .. W(k+2),
  // ecar = the upper phi edge value of cell k (face k+1/2, left state) and
  // fcar = flux of face k-1/2; iteration k0-2 only forms ecar, k0-1 only
  // ecar and fcar
  R w0[NV], w1[NV], w2[NV], w3[NV], ecar[NV], fcar[NV];
  load_own(k0 - 3, w0);
  load_own(k0 - 2, w1);
  load_own(k0 - 1, w2);
  load_own(k0, w3);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    fcar[v] = R(0);
    ecar[v] = R(0);
  }

  // r edge lane: lane l reads lanes l-2 .. l+2; lanes 2 .. TR-3 give the
  // edge values of the faces the update reads (lanes H .. TR-H); the outer
  // two lanes on either side repeat their neighbour's (never read)
  const int tc = ti < 2 ? 2 : (ti > TR - 3 ? TR - 3 : ti);

  double lam = 0.0, s1 = 0.0, s0 = 0.0;
  int bad = BAD_NONE;

  for (int k = k0 - 2; k < kend; ++k) {
    const bool body = k >= k0;  // uniform over the block
    const unsigned kbase = (unsigned)k * plane_cells;
    if (body) {
      // No barrier here: sW was last read by the previous plane's edge values,
      // all formed before its second barrier, and the fluxes that a slower
      // wave may still read are written again only after this plane's first.
      if (lghost) {  // inner ghost (primitives), the same in every layer
        R w[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) w[v] = ldg(a.ghost + v * gplane, (unsigned)(k * nt + mj));
        if (flipj) flip_theta(w);
        if (a.asymm) {  // w1: the mirror cell's primitives (already flipped)
          w[2] = -w1[2];
          w[3] = -w1[3];
          w[6] = -w1[6];
          w[7] = -w1[7];
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) sW[v][tj + H][ti] = w[v];
      } else {
#pragma unroll
        for (int v = 0; v < NV; ++v) sW[v][tj + H][ti] = w1[v];
      }
      // theta halo: rows -3 .. -1 and TT .. TT+2 over all TR lanes
      for (int h = tid; h < 2 * H * TR; h += NT) {
        const int row = h / TR, l = h - row * TR;
        const int jj = row < H ? row - H : TT + row - H;
        const int gi = i0 + l - H;
        bool flip;
        const int gj = mirror_row(j0 + jj, nt, flip);
        R w[NV];
        if (gi < 0) {
          const unsigned g = (unsigned)(k * nt + gj);
#pragma unroll
          for (int v = 0; v < NV; ++v) w[v] = ldg(a.ghost + v * gplane, g);
        } else {
          load_cons_prim<R, true>(a, kbase + (unsigned)(gj * nr + (gi < nr ? gi : nr - 1)), w);
        }
        if (flip) flip_theta(w);
#pragma unroll
        for (int v = 0; v < NV; ++v) sW[v][jj + H][l] = w[v];
      }
      __builtin_amdgcn_s_setprio(0);
      __syncthreads();
      constexpr int VS = WT * TR;
      {
        // both r edge values of the lane's cell from lanes tc-2 .. tc+2; the
        // face i-1/2 takes the upper value of lane ti-1 (one lane up in the
        // wave, the row being one wave) and the lower value of lane ti
        R eu[NV], ed[NV], f[NV];
        const R* q = &sW[0][tj + H][tc];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          weno5_cell<R, true>(q[v * VS - 2], q[v * VS - 1], q[v * VS], q[v * VS + 1],
                              q[v * VS + 2], eu[v], ed[v]);
          pin(eu[v], ed[v]);
        }
        if (!(eu[0] > R(0) && eu[4] > R(0)))
#pragma unroll
          for (int v = 0; v < NV; ++v) eu[v] = q[v * VS];
        if (!(ed[0] > R(0) && ed[4] > R(0)))
#pragma unroll
          for (int v = 0; v < NV; ++v) ed[v] = q[v * VS];
#pragma unroll
        for (int v = 0; v < NV; ++v) eu[v] = __shfl_up(eu[v], 1, 64);
        face_flux<R, 1, FLUX, true>(eu, ed, a.gam, a.igm1, f);
#pragma unroll
        for (int v = 0; v < NV; ++v) sFr[v][tj][ti] = f[v];
      }
      // theta: both edge values of the lane's cell from sW rows tj+1 ..
      // tj+5; wave 0 also forms the upper value of the row below the tile
      // (cell j0-1) and wave TT-1 the lower value of the row above it (cell
      // j0+TT), with the same expressions as the neighbouring tiles, so a
      // face shared by two tiles gets the same flux in both
      R tu[NV], td[NV], xe[NV];
      {
        const R* q = &sW[0][tj + H][ti];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          weno5_cell<R, true>(q[v * VS - 2 * TR], q[v * VS - TR], q[v * VS], q[v * VS + TR],
                              q[v * VS + 2 * TR], tu[v], td[v]);
          pin(tu[v], td[v]);
        }
        if (!(tu[0] > R(0) && tu[4] > R(0)))
#pragma unroll
          for (int v = 0; v < NV; ++v) tu[v] = q[v * VS];
        if (!(td[0] > R(0) && td[4] > R(0)))
#pragma unroll
          for (int v = 0; v < NV; ++v) td[v] = q[v * VS];
      }
      const bool lo_wave = tj == 0, hi_wave = tj == TT - 1;  // uniform per wave
      if (lo_wave || hi_wave) {
        const R* q = &sW[0][lo_wave ? H - 1 : TT + H][ti];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          R eu, ed;
          weno5_cell<R, true>(q[v * VS - 2 * TR], q[v * VS - TR], q[v * VS], q[v * VS + TR],
                              q[v * VS + 2 * TR], eu, ed);
          xe[v] = lo_wave ? eu : ed;
        }
        if (!(xe[0] > R(0) && xe[4] > R(0)))
#pragma unroll
          for (int v = 0; v < NV; ++v) xe[v] = q[v * VS];
      }
      // the left states of the faces at rows 0 .. TT-1 go through the flux
      // rows (row tj is then read and overwritten by wave tj alone): the
      // upper values of rows 0 .. TT-2 and of the row below the tile; wave
      // TT-1 finishes the tile's upper face (row TT) from its own values
      if (!hi_wave)
#pragma unroll
        for (int v = 0; v < NV; ++v) sFt[v][tj + 1][ti] = tu[v];
      if (lo_wave)
#pragma unroll
        for (int v = 0; v < NV; ++v) sFt[v][0][ti] = xe[v];
      if (hi_wave) {
        R f[NV];
        face_flux<R, 2, FLUX, true>(tu, xe, a.gam, a.igm1, f);
#pragma unroll
        for (int v = 0; v < NV; ++v) sFt[v][TT][ti] = f[v];
      }
      __syncthreads();
      {
        R lft[NV], f[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) lft[v] = sFt[v][tj][ti];
        face_flux<R, 2, FLUX, true>(lft, td, a.gam, a.igm1, f);
#pragma unroll
        for (int v = 0; v < NV; ++v) sFt[v][tj][ti] = f[v];
      }
    }
    // phi edge values of cell k+1 from W(k-1) .. W(k+3); face k+1/2 from
    // the carried upper value of cell k and the lower value of cell k+1
    R fhi[NV];
    {
      R w4[NV], eu[NV], ed[NV];
      load_own(k + 3, w4);
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        weno5_cell<R, true>(w0[v], w1[v], w2[v], w3[v], w4[v], eu[v], ed[v]);
        pin(eu[v], ed[v]);
      }
      if (!(eu[0] > R(0) && eu[4] > R(0)))
#pragma unroll
        for (int v = 0; v < NV; ++v) eu[v] = w2[v];
      if (!(ed[0] > R(0) && ed[4] > R(0)))
#pragma unroll
        for (int v = 0; v < NV; ++v) ed[v] = w2[v];
      if (k >= k0 - 1)
        face_flux<R, 3, FLUX, true>(ecar, ed, a.gam, a.igm1, fhi);
      else
#pragma unroll
        for (int v = 0; v < NV; ++v) fhi[v] = R(0);
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        ecar[v] = eu[v];
        w0[v] = w1[v];
        w1[v] = w2[v];
        w2[v] = w3[v];
        w3[v] = w4[v];
      }
    }
    // now w0 = W(k), w1 = W(k+1)
    // stage 2: the own cell's U^n for the RK combine, in flight across the barrier
    R up[NV];
    if (STAGE == 2 && body && valid) {
      const unsigned c = kbase + colbase;
#pragma unroll
      for (int v = 0; v < NV; ++v) up[v] = ldg(a.un + v * a.ncell, c);
    }
    if (body) {
      __syncthreads();  // r / theta face fluxes are in LDS
      __builtin_amdgcn_s_setprio(2);  // until this block's next rows are in LDS
      if (valid) {
        const R ivr = ldg(a.m.ivr, ic), r0 = ldg(a.m.rm2, ic) * ivr, r1 = ldg(a.m.rp2, ic) * ivr;
        const R hr = ldg(a.m.hr, ic), hc = hr * ldg(a.m.ict, jc);
        const R t0 = hc * ldg(a.m.sm, jc), t1 = hc * ldg(a.m.sp, jc);
        const R fph = hr * ldg(a.m.phf, jc);
        R L[NV];
        // (two variables at a time: with all 32 flux reads in flight at once
        // stage 1 spilled 2 registers and stage 2 28 instead of 24)
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const R dr = fma_(r0, sFr[v][tj][ti], -r1 * sFr[v][tj][ti + 1]);
          const R dth = fma_(t0, sFt[v][tj][ti], -t1 * sFt[v][tj + 1][ti]);
          L[v] = fma_(fph, fcar[v] - fhi[v], dr + dth);
          if (v & 1) __builtin_amdgcn_sched_barrier(0);
        }
        add_sources<R>(w0, a.m, ic, jc, a.omega, a.gravity, a.corot, L);
        R uc[NV];
        prim2cons<R>(w0, uc, a.igm1);
        const unsigned c = kbase + colbase;
        if (STAGE == 1) {
#pragma unroll
          for (int v = 0; v < NV; ++v) stg(a.uout + v * a.ncell, c, uc[v] + dt * L[v]);
        } else {
          R unew[NV], wn[NV];
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            unew[v] = R(0.5) * up[v] + R(0.5) * (uc[v] + dt * L[v]);
            stg(a.uout + v * a.ncell, c, unew[v]);
          }
          __builtin_amdgcn_sched_barrier(0);
          cons2prim<R, true>(unew, wn, a.gm1);
          lam = fmax(lam, cell_rate<R, true>(wn, a.m, ic, jc, a.gam));
          const double d = (double)unew[0] - (double)up[0];
          s1 += d * d;
          s0 += (double)up[0] * (double)up[0];
          if (bad == BAD_NONE && !cell_valid<R>(unew, wn)) bad = (int)c;
        }
      }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) fcar[v] = fhi[v];
  }
  // a block goes on (to its next tile, or to wait at a barrier between lists)
  // no sooner than the others
  __builtin_amdgcn_s_setprio(0);
  if (STAGE == 2) write_partials(a.partials, pslot, lam, s1, s0, bad);
}

}  // namespace icr
