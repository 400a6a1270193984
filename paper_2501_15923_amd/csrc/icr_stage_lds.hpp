// icr_stage_lds.hpp -- device code of the face-once stage (shared by the
// single-run kernels and the ensemble kernels, so that both execute the same
// arithmetic).
//
// One RK2 stage of the finite-volume update (Sect. 2 Eqs. 1-6) with every
// face flux computed exactly once:
//   - a block of TR x TT threads marches along phi over a chunk of planes;
//     each row of TR lanes covers TR - 4 cells of the tile plus the two-cell
//     r halo on either side (the halo lanes load and convert their cells
//     like every other lane, so the r halo costs no extra loads);
//   - per plane the primitives of the tile's rows plus a two-row theta halo
//     sit in LDS; r- and theta-face fluxes go to LDS and are shared by the
//     two cells of each face;
//   - the phi direction is carried in registers: each thread keeps the
//     primitives of planes k .. k+2 of its own column, the state cell k has
//     at its upper face and the flux of face k-1/2.
// Lanes run along r, so global loads and stores are coalesced (state layout
// [8][n_phi][n_theta][n_r]).  Stage 2 also forms the per-block partials of
// the next CFL dt, of the relaxation residual and of the validity flag; the
// kernel that ends the step reduces them in a fixed order.
//
// Bound about equally by FP64 issue and by memory (600 x 60 x 120, minmod and
// TVDLF, stage 1 / 2): without flux arithmetic 213 / 259 us, without loads
// from beyond L2 260 / 290 us, as it is 256 / 291 us (4.73 TB/s is what a large
// copy reaches here; the stages move 0.83 / 1.18 GB).  Against three barriers a
// plane and two slopes a phi face, FP64 272 / 308 us, FP32 (HLL and MC) 143 /
// 178 -> 138 / 167 us.
#pragma once
#include "icr_kernels.hpp"

namespace icr {


template <typename R, bool FAST>
__device__ __forceinline__ void load_cons_prim(const StageArgs<R>& a, unsigned c, R (&w)[NV]) {
  R u[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) u[v] = ldg(a.uin + v * a.ncell, c);
  cons2prim<R, FAST>(u, w, a.gm1);
}

__device__ __forceinline__ int wrap_phi(int k, int np) { return ((k % np) + np) % np; }

// One tile (bx, by, bz) of one run: (TR - 4) x TT columns, planes
// bz*kplanes ..; stage-2 partials go to slot pslot.  Called by the
// single-run kernel and by the ensemble kernels, so both execute the same
// code.
// LDS of one tile, indexed by lane along r (lane l holds cell i0 + l - 2):
// primitives of rows -2 .. TT+1 (StageW), the flux of r face i-1/2 at the
// lane of cell i and the flux of theta face j-1/2 at row j (0 .. TT)
// (StageF).  Two separate LDS objects, declared once per kernel and passed
// to stage_tile: the compiler can then tell that the update's flux reads do
// not touch the rows the stage-2 LDS-DMA copies are landing in, and does not
// wait for those copies before them.
// Rows of G variables lie side by side, G = 16 bytes / sizeof(R) variables
// when a wave's halo copies are 16 bytes a lane (FP64), else 1: a copy
// instruction then fills whole rows of the wave's own halo items.
template <typename R, int TR, int TT>
struct alignas(16) StageW {
  static constexpr int DW = sizeof(R) == 8 ? 16 : 4;  // bytes per lane and halo copy
  static constexpr int G = DW / (int)sizeof(R);
  static constexpr int RS = G * TR;  // values from a row to the next
  R sW[NV / G][TT + 4][G][TR];
  __device__ __forceinline__ R& at(int v, int row, int l) { return sW[v / G][row][v % G][l]; }
  // offset of variable v from variable 0
  static __device__ __forceinline__ constexpr int var(int v) {
    return (v / G) * (TT + 4) * RS + (v % G) * TR;
  }
};
template <typename R, int TR, int TT>
struct alignas(16) StageF {
  R sFr[NV][TT][TR];
  R sFt[NV][TT + 1][TR];
  // the metric factors of the tile's cells, loaded once per block: per-r
  // arrays at each lane's cell, per-theta arrays at each row's cell (the
  // update then reads them from LDS instead of loading them every plane).
  // The face areas (r+-^2, sin t+-) are stored divided by the cell's 1-D
  // volume (times 1/V_r, 1/C_t), as the divergence uses them
  R mr[MR_N][TR];
  R mt[MT_N][TT];
};

// Cell-metric accessor over the tile's LDS copy (lane li, row lj).
template <typename R, int TR, int TT>
struct LdsCellMetric {
  const StageF<R, TR, TT>& f;
  int li, lj;
  R ilth_;
  __device__ __forceinline__ R r(int a) const { return f.mr[a][li]; }
  __device__ __forceinline__ R t(int a) const { return f.mt[a][lj]; }
  __device__ __forceinline__ R ilth() const { return ilth_; }
};

// Face states of face m-1/2 from four LDS values per variable (p0..p3 =
// cells m-2 .. m+1), then the numerical flux.
template <typename R, int N, int FLUX, int LIM, typename W>
__device__ __forceinline__ void lds_face(const R* base, int stride, R gam, R igm1, R (&f)[NV],
                                         const R* own = nullptr) {
  R wl[NV], wr[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const R* q = base + W::var(v);
    const R p0 = q[0], p1 = q[stride], p2 = own ? own[v] : q[2 * stride], p3 = q[3 * stride];
    face_states<R, LIM, true>(p0, p1, p2, p3, wl[v], wr[v]);
  }
  face_flux<R, N, FLUX, true>(wl, wr, gam, igm1, f);
}

// One LDS-DMA copy: every lane moves BYTES bytes from its own global
// address to dst + BYTES * lane (dst is the same for the whole wave).
template <int BYTES>
__device__ __forceinline__ void lds_dma(const char* src, char* dst) {
  static_assert(BYTES == 16 || BYTES == 4, "LDS-DMA copy width");
  auto g = (const __attribute__((address_space(1))) void*)src;
  auto l = (__attribute__((address_space(3))) void*)dst;
  if constexpr (BYTES == 16)
    __builtin_amdgcn_global_load_lds(g, l, 16, 0, 0);
  else
    __builtin_amdgcn_global_load_lds(g, l, 4, 0, 0);
}

template <typename R, int TR, int TT, int FLUX, int LIM, int STAGE, bool FM = false>
__device__ __forceinline__ void stage_tile(const StageArgs<R>& a, int kplanes, int bx, int by,
                                           int bz, int pslot, StageW<R, TR, TT>& smw,
                                           StageF<R, TR, TT>& smf) {
  constexpr int NT = TR * TT;
  constexpr int TI = tile_cells_r(TR);
  using W = StageW<R, TR, TT>;
  auto& sFr = smf.sFr;
  auto& sFt = smf.sFt;

  const int ti = threadIdx.x, tj = threadIdx.y, tid = tj * TR + ti;
  const int i0 = bx * TI, j0 = by * TT, k0 = bz * kplanes;
  const int nr = a.nr, nt = a.nt, np = a.np;
  const int kend = k0 + kplanes < np ? k0 + kplanes : np;
  const int i = i0 + ti - 2, j = j0 + tj;  // this lane's cell
  const bool inner = ti >= 2 && ti < TR - 2;
  const bool valid = inner && i < nr && j < nt;
  // column of the own phi ring: the cell itself, the last cell beyond r_out;
  // below r_in cell 0, or under the asymm rule the mirror cell -1 - i, whose
  // transverse primitives the ghost takes negated
  const int ic = i < 0 ? (a.asymm ? (-1 - i < nr ? -1 - i : nr - 1) : 0)
                       : (i < nr ? i : nr - 1);
  const int jc = j < nt ? j : nt - 1;
  const int active = a.clock->active;
  // cell offsets within one variable's array (32-bit: below 2^29 cells)
  const unsigned colbase = (unsigned)(jc * nr + ic);  // + k * nt * nr
  // own-column loads: rows past the last colatitude mirror it (they serve
  // as ghost rows of the last active row's upper theta face); cells below
  // r_in (halo lanes of the first tile) come from the inner ghost, cells
  // beyond r_out repeat the last cell
  bool flipj;
  const int mj = mirror_row(j, nt, flipj);
  const unsigned lbase = (unsigned)(mj * nr + ic);
  const bool lghost = i < 0;
  const unsigned plane_cells = (unsigned)(nt * nr);
  const long long gplane = (long long)nt * np;
  // The ring of the first tile's two halo lanes below r_in holds cell 0 (or
  // the mirror cell); those lanes put the inner ghost into LDS instead (see
  // below).
  // the next plane's own-column state is loaded one plane ahead (raw
  // conserved values in uring) and converted when the phi face needs it
  auto own_raw = [&](int k, R (&u)[NV]) {
    const unsigned c = (unsigned)wrap_phi(k, np) * plane_cells + lbase;
#pragma unroll
    for (int v = 0; v < NV; ++v) u[v] = ldg(a.uin + v * a.ncell, c);
  };
  auto own_cvt = [&](const R (&u)[NV], R (&w)[NV]) {
    cons2prim<R, true>(u, w, a.gm1);
    if (flipj) flip_theta(w);
  };
  auto load_own = [&](int k, R (&w)[NV]) {
    load_cons_prim<R, true>(a, (unsigned)wrap_phi(k, np) * plane_cells + lbase, w);
    if (flipj) flip_theta(w);
  };

  if (!active) {
    if (STAGE == 2 && valid)
      for (int k = k0; k < kend; ++k) {
        const unsigned c = (unsigned)k * plane_cells + colbase;
#pragma unroll
        for (int v = 0; v < NV; ++v) stg(a.uout + v * a.ncell, c, ldg(a.un + v * a.ncell, c));
      }
    return;
  }

  // metric factors of the tile into LDS (visible after the first plane
  // barrier; the first use is after it).  A block that runs several tiles
  // (ensembles) first waits until every wave has left the previous tile.
  __syncthreads();
  // (array indices are compile-time constants after unrolling, so that the
  // metric pointers stay kernel arguments)
  for (int l = tid; l < TR; l += NT) {
    const int ii = i0 + l - 2;
    const int icl = ii < 0 ? (a.asymm ? (-1 - ii < nr ? -1 - ii : nr - 1) : 0)
                           : (ii < nr ? ii : nr - 1);
#pragma unroll
    for (int arr = 0; arr < MR_N; ++arr) {
      R x = ldg(metric_r(a.m, arr), (unsigned)icl);
      if (arr == MR_RM2 || arr == MR_RP2) x *= ldg(a.m.ivr, (unsigned)icl);
      smf.mr[arr][l] = x;
    }
  }
  for (int row = tid; row < TT; row += NT) {
    const int jr = j0 + row < nt ? j0 + row : nt - 1;
#pragma unroll
    for (int arr = 0; arr < MT_N; ++arr) {
      R x = ldg(metric_t(a.m, arr), (unsigned)jr);
      if (arr == MT_SM || arr == MT_SP) x *= ldg(a.m.ict, (unsigned)jr);
      smf.mt[arr][row] = x;
    }
  }
  const LdsCellMetric<R, TR, TT> cm{smf, ti, tj, a.m.ilth};
  // the stage's dt, read once: a global load inside the update would make
  // it wait for the stage-2 halo copies issued before it
  const R dt = (R)a.clock->dt;

  // phi ring of the own column: at the top of iteration k, wb = W(k),
  // wc = W(k+1), dbc = wc - wb, wup = cell k's state at its upper face and
  // fcar = flux of face k-1/2.  Iteration k0-1 only forms fcar, through the
  // same code as every later phi face.  The slope of a cell gives its states
  // at both its faces, one of them carried to the next plane: 7 operations a
  // variable (minmod, FP64) where forming both slopes of every face took 11,
  // and one array less to move up.
  R wb[NV], wc[NV], dbc[NV], wup[NV], fcar[NV];
  {
    R wa[NV];
    load_own(k0 - 2, wa);
    load_own(k0 - 1, wb);
    load_own(k0, wc);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      R lo;
      dbc[v] = wc[v] - wb[v];
      cell_states<R, LIM>(wb[v], wb[v] - wa[v], dbc[v], lo, wup[v]);
    }
  }
  R uring[NV];
  own_raw(k0 + 1, uring);
#pragma unroll
  for (int v = 0; v < NV; ++v) fcar[v] = R(0);

  // Stage 1 (PF): this thread's theta-halo item is the same (row, lane) of
  // every plane, and the next plane's item is loaded into registers while
  // the current plane is processed.  Stage 2 (DMA) has no registers to
  // spare: the next plane's halo rows are copied global -> LDS by the LDS-DMA
  // loads, issued after the plane's face barrier (nothing reads sW until the
  // next plane), so they travel while the plane is updated; a wave then waits
  // for its own copies and converts its halo cells to primitives in place.  Those copies take, for a halo cell below r_in or beyond
  // r_out, the clamped cell of its row: such cells only feed the theta
  // faces of halo lanes, which the update never reads.
  constexpr bool PF = STAGE == 1;
  constexpr bool DMA = STAGE == 2;
  static_assert(4 * TR <= NT, "at most one theta-halo item per thread");
  const bool hv = tid < 4 * TR;
  const int hrow = tid / TR, hl = tid - hrow * TR;
  const int hjj = hrow < 2 ? hrow - 2 : TT + hrow - 2;
  const int hgi = i0 + hl - 2;
  bool hflip;
  const int hgj = mirror_row(j0 + hjj, nt, hflip);
  const bool hghost = hgi < 0;  // below r_in: inner ghost primitives
  const unsigned hoff = (unsigned)(hgj * nr + (hgi < 0 ? 0 : (hgi < nr ? hgi : nr - 1)));
  auto halo_raw = [&](int k, R (&w)[NV]) {
    if (hghost) {
#pragma unroll
      for (int v = 0; v < NV; ++v) w[v] = ldg(a.ghost + v * gplane, (unsigned)(k * nt + hgj));
    } else {
#pragma unroll
      for (int v = 0; v < NV; ++v) w[v] = ldg(a.uin + v * a.ncell, (unsigned)k * plane_cells + hoff);
    }
  };
  auto halo_put = [&](const R (&raw)[NV]) {
    R w[NV];
    if (hghost) {
#pragma unroll
      for (int v = 0; v < NV; ++v) w[v] = raw[v];
    } else {
      cons2prim<R, true>(raw, w, a.gm1);
    }
    if (hflip) flip_theta(w);
#pragma unroll
    for (int v = 0; v < NV; ++v) smw.at(v, hjj + 2, hl) = w[v];
  };
  R hraw[NV];
  if (PF && hv && k0 < kend) halo_raw(k0, hraw);

  // (the copies need n_r >= 2: a 16-byte copy takes two neighbouring cells
  // of a row; with fewer cells stage 2 loads its halo after the barrier)
  // A wave copies exactly the cells its own lanes convert: an instruction
  // moves G variables of the wave's 64 halo cells, whole rows of StageW.  So
  // the wave's own wait is enough before the conversion, and no barrier.
  constexpr int DW = W::DW, G = W::G;
  static_assert(!DMA || (64 * DW == G * 64 * (int)sizeof(R) && 64 % TR == 0 && TR % 2 == 0 &&
                         tile_cells_r(TR) % 2 == 0 && G <= 2),
                "theta-halo DMA layout");
  const bool dma_on = DMA && nr >= 2;  // uniform
  const int wv = __builtin_amdgcn_readfirstlane(tid) >> 6;  // wave index (uniform)
  const bool dma_wave = dma_on && wv < 4 * TR / 64;
  const int drow = wv * (64 / TR) < 2 ? wv * (64 / TR) : TT + wv * (64 / TR);  // its first sW row
  const char* dsrc = nullptr;  // of plane 0 and the first G variables
  if constexpr (DMA) {
    const int e = (tid & 63) * G;  // first value of this lane's copies
    const int l = e % TR;
    bool fl;
    const int gj = mirror_row(j0 + drow + e / W::RS - 2, nt, fl);
    // clamped into the row; a two-cell copy keeps both cells in the row
    int gi = i0 + l - 2;
    gi = gi < 0 ? 0 : (gi <= nr - G ? gi : nr - G);
    dsrc = reinterpret_cast<const char*>(a.uin + (size_t)(e / TR % G) * a.ncell) +
           (size_t)(unsigned)(gj * nr + gi) * sizeof(R);
  }
  auto dma_halo = [&](int k) {
    const char* src = dsrc + (size_t)((unsigned)k * plane_cells) * sizeof(R);
#pragma unroll
    for (int m = 0; m < NV / G; ++m)
      lds_dma<DW>(src + (size_t)(m * G) * a.ncell * sizeof(R),
                  reinterpret_cast<char*>(&smw.at(m * G, drow, 0)));
  };
  if constexpr (DMA) {
    if (dma_wave && k0 < kend) dma_halo(k0);
  }

  double lam = 0.0, s1 = 0.0, s0 = 0.0;
  int bad = BAD_NONE;

  for (int k = k0 - 1; k < kend; ++k) {
    const bool body = k >= k0;  // uniform over the block
    const unsigned kbase = (unsigned)k * plane_cells;
    if (body) {
      // No barrier here: sW was last read by the previous plane's faces, all
      // done before its second barrier, and the fluxes that a slower wave may
      // still read are written again only after this plane's first barrier.
      // stage 2: this wave's halo copies have landed (s_waitcnt vmcnt(0))
      if constexpr (DMA) {
        if (dma_on) __builtin_amdgcn_s_waitcnt(0x3f70);
        asm volatile("" ::: "memory");
      }
      if (lghost) {  // inner ghost (primitives) at this lane's row
        R w[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) w[v] = ldg(a.ghost + v * gplane, (unsigned)(k * nt + mj));
        if (flipj) flip_theta(w);
        if (a.asymm) {  // wb: the mirror cell's primitives (already flipped)
          w[2] = -wb[2];
          w[3] = -wb[3];
          w[6] = -wb[6];
          w[7] = -wb[7];
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) smw.at(v, tj + 2, ti) = w[v];
      } else {
#pragma unroll
        for (int v = 0; v < NV; ++v) smw.at(v, tj + 2, ti) = wb[v];
      }
      // theta halo: rows -2, -1, TT, TT + 1 over all TR lanes
      if constexpr (PF) {
        if (hv) {
          halo_put(hraw);
          if (k + 1 < kend) halo_raw(k + 1, hraw);  // in flight during this plane
        }
      } else if (dma_on) {
        if (hv) {  // conserved -> primitive in place
          R u[NV], w[NV];
          // a two-cell copy starts at an even lane (an even cell, the tile
          // start being even): at the end of a row of odd length it was
          // shifted back into the row, so the even lane of the last cell got
          // its left neighbour; reload that one cell
          if (G == 2 && hgi == nr - 1 && (hl & 1) == 0 && hl >= 2 && hl < TR - 2) {
#pragma unroll
            for (int v = 0; v < NV; ++v)
              u[v] = ldg(a.uin + v * a.ncell, kbase + (unsigned)(hgj * nr + hgi));
          } else {
#pragma unroll
            for (int v = 0; v < NV; ++v) u[v] = smw.at(v, hjj + 2, hl);
          }
          cons2prim<R, true>(u, w, a.gm1);
          if (hflip) flip_theta(w);
#pragma unroll
          for (int v = 0; v < NV; ++v) smw.at(v, hjj + 2, hl) = w[v];
        }
      } else {
        for (int h = tid; h < 4 * TR; h += NT) {
          const int row = h / TR, l = h - row * TR;
          const int jj = row < 2 ? row - 2 : TT + row - 2;
          const int gi = i0 + l - 2;
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
          for (int v = 0; v < NV; ++v) smw.at(v, jj + 2, l) = w[v];
        }
      }
      __builtin_amdgcn_s_setprio(0);
      __syncthreads();
      // r face i-1/2 and theta face j-1/2 at every lane (the update reads
      // the r faces of lanes 2 .. TR-2, the last being the tile's upper r
      // face, and the theta faces of the inner lanes; the others are never
      // read, and lanes 0, 1 and TR-1 read neighbouring LDS rows for their
      // r face), then the tile's upper theta face of every inner lane
      {
        R f[NV];
        lds_face<R, 1, FLUX, LIM, W>(&smw.at(0, tj + 2, ti) - 2, 1, a.gam, a.igm1, f, wb);
#pragma unroll
        for (int v = 0; v < NV; ++v) sFr[v][tj][ti] = f[v];
      }
      {
        R f[NV];
        lds_face<R, 2, FLUX, LIM, W>(&smw.at(0, tj, ti), W::RS, a.gam, a.igm1, f, wb);
#pragma unroll
        for (int v = 0; v < NV; ++v) sFt[v][tj][ti] = f[v];
      }
      {
        // one wave a plane, in turn: always the same one would load its SIMD
        // with four faces a plane where the others have three
        const int q = tid - 64 * (k & (NT / 64 - 1));
        if (q >= 2 && q < TR - 2) {
          R f[NV];
          lds_face<R, 2, FLUX, LIM, W>(&smw.at(0, TT, q), W::RS, a.gam, a.igm1, f);
#pragma unroll
          for (int v = 0; v < NV; ++v) sFt[v][TT][q] = f[v];
        }
      }
    }
    // Stage 2: the own cell's U^n for the RK combine is loaded here, before
    // the phi face and the barrier, so that its latency overlaps that work
    // instead of stalling the update.
    R up[NV];
    if (STAGE == 2 && body && valid) {
      const unsigned c = kbase + colbase;
#pragma unroll
      for (int v = 0; v < NV; ++v) up[v] = ldg(a.un + v * a.ncell, c);
    }
    // phi face k+1/2 from the register ring (and the next plane's load)
    R fhi[NV], wa[NV];
    {
      R wd[NV], wl[NV], wr[NV];
      own_cvt(uring, wd);      // W(k + 2), loaded one plane ago
      own_raw(k + 3, uring);   // in flight until the next plane's phi face
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const R d = wd[v] - wc[v];
        wl[v] = wup[v];
        cell_states<R, LIM>(wc[v], dbc[v], d, wr[v], wup[v]);
        dbc[v] = d;
      }
      face_flux<R, 3, FLUX, true>(wl, wr, a.gam, a.igm1, fhi);
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        wa[v] = wb[v];
        wb[v] = wc[v];
        wc[v] = wd[v];
      }
    }
    // now wa = W(k), wb = W(k+1), wc = W(k+2)
    if (body) {
      __syncthreads();  // r / theta face fluxes are in LDS
      // from here to the next rows' barrier a wave goes before the other
      // block's waves: all four of this block wait there for the slowest
      __builtin_amdgcn_s_setprio(2);
      if constexpr (DMA) {
        if (dma_wave && k + 1 < kend) dma_halo(k + 1);  // in flight during this update
      }
      if (valid) {
        const R r0 = cm.r(MR_RM2), r1 = cm.r(MR_RP2), hr = cm.r(MR_HR);
        const R t0 = hr * cm.t(MT_SM), t1 = hr * cm.t(MT_SP);
        const R fph = hr * cm.t(MT_PHF);
        R L[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const R dr = fma_(r0, sFr[v][tj][ti], -r1 * sFr[v][tj][ti + 1]);
          const R dth = fma_(t0, sFt[v][tj][ti], -t1 * sFt[v][tj + 1][ti]);
          L[v] = fma_(fph, fcar[v] - fhi[v], dr + dth);
        }
        add_sources_cm<R>(wa, cm, a.omega, a.gravity, a.corot, L);
        // the stage's own conserved state, rebuilt from the ring's primitives
        // (equal to the stored values up to rounding; no reload)
        R uc[NV];
        prim2cons<R>(wa, uc, a.igm1);
        const unsigned c = kbase + colbase;
        if constexpr (FM) {  // passive tracer on: keep this stage's mass fluxes
          stg(a.fmass, c, sFr[0][tj][ti]);
          stg(a.fmass + a.ncell, c, sFt[0][tj][ti]);
          stg(a.fmass + 2 * a.ncell, c, fcar[0]);
          if (i == nr - 1) stg(a.fmass_rout, (unsigned)(k * nt + j), sFr[0][tj][ti + 1]);
          if (j == nt - 1) stg(a.fmass_tend, (unsigned)(k * nr + i), sFt[0][tj + 1][ti]);
        }
        if (STAGE == 1) {
#pragma unroll
          for (int v = 0; v < NV; ++v) stg(a.uout + v * a.ncell, c, uc[v] + dt * L[v]);
        } else {
          R un[NV], unew[NV], wn[NV];
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            un[v] = up[v];
            unew[v] = R(0.5) * un[v] + R(0.5) * (uc[v] + dt * L[v]);
            stg(a.uout + v * a.ncell, c, unew[v]);
          }
          cons2prim<R, true>(unew, wn, a.gm1);
          lam = fmax(lam, cell_rate_cm<R, true>(wn, cm, a.gam));
          const double d = (double)unew[0] - (double)un[0];
          s1 += d * d;
          s0 += (double)un[0] * (double)un[0];
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


// ------------------------------------------------------------ finalize --
// Reduce the stage-2 (or CFL) block partials in a fixed order (a block of 256
// threads; the result is thread 0's).
__device__ __forceinline__ void reduce_partials(const double* __restrict__ part, int nblocks,
                                                double& l, double& a1, double& a0, int& b,
                                                double (*sh)[4]) {
  const int tid = threadIdx.y * blockDim.x + threadIdx.x;
  const int nthr = blockDim.x * blockDim.y;
  l = a1 = a0 = 0.0;
  b = BAD_NONE;
  for (int q = tid; q < nblocks; q += nthr) {
    l = fmax(l, part[4 * q + 0]);
    a1 += part[4 * q + 1];
    a0 += part[4 * q + 2];
    const int qb = (int)part[4 * q + 3];
    b = qb < b ? qb : b;
  }
  block_reduce(l, a1, a0, b, sh);
}

// Advance the clock by the step the partials belong to (advance = 1) and set
// the next dt; *idx is the cadence index of the new time and the result says
// whether a probe record is due.
__device__ __forceinline__ bool advance_clock(DevClock& c, double l, double a1, double a0, int b,
                                              double cfl, int advance, int log_on,
                                              const ProbeArgs& pa) {
  if (advance) {
    c.t = c.clip ? c.t_end : c.t + c.dt;
    c.step += 1;
    c.taken += 1;
    c.last_dt = c.dt;
    c.resid = sqrt(a1) / sqrt(a0);
    if (b != BAD_NONE) {
      if (c.bad == BAD_NONE || b < c.bad) c.bad = b;
    }
  }
  set_next_dt(&c, cfl / l);
  if (c.bad != BAD_NONE) c.active = 0;
  // probe cadence decision on the new time
  bool rec = advance && log_on;
  long long idx = 0;
  if (rec && pa.cadence > 0.0) {
    idx = (long long)floor(c.t * pa.sc.t / pa.cadence);
    rec = idx > c.last_sample;
  }
  if (rec) {
    c.n_log += 1;
    if (pa.cadence > 0.0) c.last_sample = idx;
  }
  return rec;
}

// One block: the reduction, the clock and, if probes are logged, a record.
// reset: what a new state clears first (see RESET_*).
template <typename R>
__device__ __forceinline__ void finalize_run(DevClock* ck, const double* __restrict__ part,
                                             int nblocks, double cfl, int advance, int log_on,
                                             const ProbeArgs& pa, const R* __restrict__ u,
                                             double* __restrict__ log, int reset = RESET_NONE) {
  __shared__ double sh[4][4];
  __shared__ int s_rec;
  __shared__ long long s_row;
  __shared__ double s_t;
  const int tid = threadIdx.y * blockDim.x + threadIdx.x;
  if (!ck->active && advance) return;  // the stage kernels did not run
  double l, a1, a0;
  int b;
  reduce_partials(part, nblocks, l, a1, a0, b, sh);
  if (tid == 0) {
    DevClock c = *ck;
    if (reset != RESET_NONE) {
      c.bad = BAD_NONE;
      c.counter = 0;
    }
    if (reset == RESET_RUN) {
      c.t = 0.0;
      c.step = 0;
      c.last_dt = 0.0;
      c.resid = 0.0;
    }
    s_row = c.n_log;
    s_rec = advance_clock(c, l, a1, a0, b, cfl, advance, log_on, pa);
    s_t = c.t;
    *ck = c;
  }
  __syncthreads();
  if (s_rec && s_row < pa.log_rows && tid < pa.n)
    probe_eval<R>(pa, u, tid, s_t, log + (s_row * pa.max_probes + tid) * 12);
}

// The end of a step and the boundary of the next one in a launch: every
// block reduces the partials for itself (the same order, so the same clock)
// from the clock as it was when the step began (ck[1], written by stage 1),
// then forms its columns' inner-boundary primitives at the new times; block 0
// of a run also writes the clock and the probe record.
// (Single runs of more columns than one round of blocks use finalize_run and
// k_boundary instead.)
template <typename R>
__device__ __forceinline__ void end_step(int blk, DevClock* ck, const double* __restrict__ part,
                                         int nblocks,
                                         double cfl, int log_on, const ProbeArgs& pa,
                                         const R* __restrict__ u, double* __restrict__ log,
                                         const BndArgs& bnd, R* __restrict__ g1,
                                         R* __restrict__ g2, R* __restrict__ tg1,
                                         R* __restrict__ tg2) {
  __shared__ double sh[4][4];
  __shared__ int s_rec, s_active;
  __shared__ long long s_row;
  __shared__ double s_t, s_dt;
  const int tid = threadIdx.y * blockDim.x + threadIdx.x;
  if (!ck[1].active) return;  // the stage kernels did not run
  double l, a1, a0;
  int b;
  reduce_partials(part, nblocks, l, a1, a0, b, sh);
  if (tid == 0) {
    DevClock c = ck[1];
    s_row = c.n_log;
    s_rec = advance_clock(c, l, a1, a0, b, cfl, 1, log_on, pa);
    s_t = c.t;
    s_dt = c.dt;
    s_active = c.active;
    if (blk == 0) ck[0] = c;
  }
  __syncthreads();
  if (s_active)
    boundary_block<R>(bnd, s_t, s_dt, blk, tid, g1, g2, tg1, tg2);
  if (blk == 0 && s_rec && s_row < pa.log_rows && tid < pa.n)
    probe_eval<R>(pa, u, tid, s_t, log + (s_row * pa.max_probes + tid) * 12);
}

}  // namespace icr
