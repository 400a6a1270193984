// icr_nn.hip -- warm-start network for the relaxation phase (not in the
// paper; it shortens the relaxation that the paper runs for 8 days before
// the period of interest, Sect. 3).
//
// Network (per sample): boundary map features X [n_theta][n_phi][8]
//   conv 3 x (phi_hi - phi_lo + 1) (periodic in phi, edge-clamped in theta) 8 -> C1, SiLU
//   conv 3x3 C1 -> C2, SiLU                              = latent z per column
//   per-column decoder: Linear C2 -> H, SiLU; Linear H -> n_r * 8
// output: normalised residual of the state over the radial expansion of the
// map.  All products run on BF16 MFMA (v_mfma_f32_32x32x16_bf16) with FP32
// accumulation; weights have FP32 masters updated by Adam and BF16 copies.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "icarus_nn.h"

namespace icrnn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// float -> bf16 bits, round to nearest even (NaN kept quiet)
__device__ __forceinline__ uint16_t f2bf(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu)) return (uint16_t)((u >> 16) | 0x40);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// ------------------------------------------------------------------ GEMM --
// C[m][n] = sum_k A(m,k) B(k,n) on v_mfma_f32_32x32x16_bf16, FP32
// accumulation with k ascending in groups of 16.
// A(m,k) = TA ? a[k*lda + m] : a[m*lda + k];  B(k,n) = TB ? b[n*ldb + k] : b[k*ldb + n].
// A may also be the neighbourhood matrix of a convolution, gathered from the
// channel array while its tile is loaded instead of being stored (Conv).
//
// Block tile TM x TN x 64 on 4 waves, two shapes: 128 x 128 (waves of 64 x
// 64) and 64 x 64 (waves of 32 x 32).  The next k-tile travels into
// registers while the current one is multiplied out of LDS.  LDS rows hold
// 64 k values (128 bytes, eight 16-byte chunks), the chunk of row r stored
// at chunk ^ swz(r): a wave reads one chunk of 32 consecutive rows, and the
// eight rows that share a 128-byte LDS cycle land on eight different chunks
// (padding the rows instead would misalign the 16-byte reads).  An operand
// stored with its row index fastest is loaded as 4 (k) x 8 (row) patches and
// transposed by v_perm_b32, one per output dword, on the way to LDS.
//
// What bounds it: the output layer's products (57600 x 4800 x 384 at 600 x
// 60 x 120, batch 8) read the targets and write dY (1.7 GB), 0.63 ms; its two
// gradients run at 0.6 and 0.5 PFLOP/s, limited by the load latency of a
// k-tile.  A training step of that size went from 9.0 to 2.2 ms (batch 8 at
// 150 x 30 x 60: 1.15 -> 0.40 ms) over the kernels that stored the
// neighbourhood matrices, Y and every pre-activation gradient in FP32 and
// summed them in passes of their own.  The products and what follows from them
// element by element round as before, bit by bit; the loss and the bias
// gradients, sums in FP64, are grouped by tile (so by the tile's shape).
constexpr int BK = 64;
__device__ __forceinline__ int swz(int r) { return (r & 7) ^ ((r & 8) >> 1); }
__device__ __forceinline__ int lds_chunk(int r, int c) { return r * BK + ((c ^ swz(r)) << 3); }

// The neighbourhood matrix of a convolution over 3 colatitude rows and nk
// longitudes starting at offset dk0: row m = (b, j, k), column
// tap * C + c = h[b][clamp(j + dj)][(k + dk) mod np][c],
// tap = (dj + 1) * nk + (dk - dk0).
struct Conv {
  int nt, np, C, dk0, nk;
};

struct Operand {
  const uint16_t* p;
  int ld;
  int vec;  // rows may be read 16 bytes at a time (base and stride aligned)
  Conv cv;
};

struct ConvRow {  // one row of the neighbourhood matrix
  int b, j, k;
};
__device__ __forceinline__ ConvRow conv_row(const Conv& cv, int m) {
  ConvRow r;
  const int q = m / cv.np;
  r.k = m - q * cv.np;
  r.b = q / cv.nt;
  r.j = q - r.b * cv.nt;
  return r;
}
__device__ __forceinline__ void conv_next(const Conv& cv, ConvRow& r) {  // row m + 1
  if (++r.k == cv.np) {
    r.k = 0;
    if (++r.j == cv.nt) {
      r.j = 0;
      ++r.b;
    }
  }
}
struct ConvCol {  // one column: neighbour offsets and channel
  int dj, dk, c;
};
__device__ __forceinline__ ConvCol conv_col(const Conv& cv, int col) {
  const int tap = col / cv.C, d = tap / cv.nk;
  return ConvCol{d - 1, tap - d * cv.nk + cv.dk0, col - tap * cv.C};
}
__device__ __forceinline__ long long conv_at(const Conv& cv, const ConvRow& r, const ConvCol& q) {
  int j = r.j + q.dj, k = r.k + q.dk;
  j = j < 0 ? 0 : (j >= cv.nt ? cv.nt - 1 : j);
  k = k < 0 ? k + cv.np : (k >= cv.np ? k - cv.np : k);  // |dk| < np
  return ((long long)(r.b * cv.nt + j) * cv.np + k) * cv.C + q.c;
}
// How eight columns of the neighbourhood matrix are read: 16 bytes at once
// where 8 channels never straddle two taps, else by channel pairs (even C),
// else one by one.
enum { CONV_NONE, CONV_VEC, CONV_PAIR, CONV_ONE };

// 8 consecutive elements (r, c .. c+7) of a matrix with rows of ld elements,
// zero outside R x C.
__device__ __forceinline__ uint4 fetch8(const Operand& o, int r, int c, int R, int C) {
  uint4 q = make_uint4(0, 0, 0, 0);
  if (r >= R || c >= C) return q;
  const uint16_t* g = o.p + (long long)r * o.ld + c;
  if (o.vec && c + 8 <= C) return *reinterpret_cast<const uint4*>(g);
  uint16_t v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = c + i < C ? g[i] : (uint16_t)0;
  memcpy(&q, v, 16);
  return q;
}

// The same of the neighbourhood matrix: columns c .. c+7 of K, whose offsets
// (for every first, second or single column, by CM) are in `col`.
template <int CM, int NC>
__device__ __forceinline__ uint4 fetch8_conv(const Operand& o, const ConvRow& row,
                                             const ConvCol (&col)[NC], int c, int K) {
  uint4 q = make_uint4(0, 0, 0, 0);
  if (c >= K) return q;
  if constexpr (CM == CONV_VEC) {
    q = *reinterpret_cast<const uint4*>(o.p + conv_at(o.cv, row, col[0]));
  } else {
    constexpr int W = 8 / NC;
    uint16_t v[8];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      uint32_t w = 0;
      if (c + W * i < K) {
        const uint16_t* g = o.p + conv_at(o.cv, row, col[i]);
        if (W == 2) w = *reinterpret_cast<const uint32_t*>(g); else w = *g;
      }
      memcpy(v + W * i, &w, 2 * W);
    }
    memcpy(&q, v, 16);
  }
  return q;
}

// One operand's k-tile, T rows x 64 k, in registers.
// KR = 0: stored k-contiguous; piece q is chunk tid % 8 of row tid / 8 + 32 q.
// KR = 1: stored row-contiguous; a 4 (k) x 8 (row) patch, 8 k-groups and 8
// row-groups per wave (64 rows: two waves hold all the patches).
template <int T, int KR>
struct Piece {
  uint4 v[KR ? 4 : T / 32];
};
// A convolution's rows and columns that a thread keeps for the whole product:
// its rows (KR = 0) or its columns (KR = 1); the other index moves with k.
template <int T, int KR, int CM>
struct Tile {
  static constexpr int NP = KR ? 4 : T / 32;
  static constexpr int NC = CM == CONV_PAIR ? 4 : (CM == CONV_ONE ? 8 : 1);
  ConvRow row[CM && !KR ? NP : 1];
  ConvCol col[CM && KR ? NC : 1];

  __device__ __forceinline__ static int patch_k() {
    return 4 * ((threadIdx.x & 7) + 8 * ((threadIdx.x >> 6) & 1));
  }
  __device__ __forceinline__ static int patch_r() {
    return 8 * (((threadIdx.x & 63) >> 3) + 8 * (threadIdx.x >> 7));
  }
  __device__ __forceinline__ static bool idle() { return KR && T < 128 && threadIdx.x >= 128; }

  __device__ __forceinline__ void init(const Operand& o, int r0, int R) {
    if constexpr (CM && !KR) {
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const int r = r0 + (threadIdx.x >> 3) + 32 * q;
        row[q] = conv_row(o.cv, r < R ? r : R - 1);
      }
    } else if constexpr (CM) {
#pragma unroll
      for (int i = 0; i < NC; ++i) col[i] = conv_col(o.cv, r0 + patch_r() + (8 / NC) * i);
    }
  }
  // rows r0 .. of R, k0 .. of K
  __device__ __forceinline__ void load(Piece<T, KR>& p, const Operand& o, int r0, int k0, int R,
                                       int K) const {
    const int tid = threadIdx.x;
    if constexpr (!KR) {
      const int k = k0 + (tid & 7) * 8;
      if constexpr (CM) {
        ConvCol cc[NC];
#pragma unroll
        for (int i = 0; i < NC; ++i) cc[i] = conv_col(o.cv, k + (8 / NC) * i);
#pragma unroll
        for (int q = 0; q < NP; ++q)
          p.v[q] = r0 + (tid >> 3) + 32 * q < R ? fetch8_conv<CM>(o, row[q], cc, k, K)
                                                : make_uint4(0, 0, 0, 0);
      } else {
#pragma unroll
        for (int q = 0; q < NP; ++q) p.v[q] = fetch8(o, r0 + (tid >> 3) + 32 * q, k, R, K);
      }
    } else {
      if (idle()) return;
      const int r = r0 + patch_r(), k = k0 + patch_k();
      if constexpr (CM) {
        ConvRow rw = conv_row(o.cv, k);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          p.v[q] = k + q < K ? fetch8_conv<CM>(o, rw, col, r, R) : make_uint4(0, 0, 0, 0);
          conv_next(o.cv, rw);
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) p.v[q] = fetch8(o, k + q, r, K, R);
      }
    }
  }
  __device__ __forceinline__ static void store(const Piece<T, KR>& p, uint16_t* s) {
    const int tid = threadIdx.x;
    if constexpr (!KR) {
#pragma unroll
      for (int q = 0; q < NP; ++q)
        *reinterpret_cast<uint4*>(s + lds_chunk((tid >> 3) + 32 * q, tid & 7)) = p.v[q];
    } else {
      if (idle()) return;
      const int r = patch_r(), k = patch_k();
      const uint32_t a0[4] = {p.v[0].x, p.v[0].y, p.v[0].z, p.v[0].w};
      const uint32_t a1[4] = {p.v[1].x, p.v[1].y, p.v[1].z, p.v[1].w};
      const uint32_t a2[4] = {p.v[2].x, p.v[2].y, p.v[2].z, p.v[2].w};
      const uint32_t a3[4] = {p.v[3].x, p.v[3].y, p.v[3].z, p.v[3].w};
#pragma unroll
      for (int i = 0; i < 8; ++i) {  // row r + i: its four k values
        const uint32_t sel = i & 1 ? 0x07060302u : 0x05040100u;
        const uint2 d = make_uint2(__builtin_amdgcn_perm(a1[i >> 1], a0[i >> 1], sel),
                                   __builtin_amdgcn_perm(a3[i >> 1], a2[i >> 1], sel));
        *reinterpret_cast<uint2*>(s + lds_chunk(r + i, k >> 3) + (k & 4)) = d;
      }
    }
  }
};

// What happens to a finished tile.
//   EP_OUT   C = acc (+ bias)
//   EP_SILU  h = SiLU(acc + bias) in BF16; z = acc + bias kept where z is set
//   EP_MSE   d = acc + bias - t: dY = 2 d scale in BF16, the block's sum of
//            d^2, and the column sums of d over the block's rows
//   EP_BACK  d = acc * SiLU'(z) in BF16 and its column sums
enum { EP_OUT, EP_SILU, EP_MSE, EP_BACK };
struct Epi {
  float* c;           // EP_OUT: C; EP_SILU: z or NULL
  const float* bias;  // or NULL
  uint16_t* h;        // BF16 result
  const float* t;     // EP_MSE: targets; EP_BACK: z
  double* loss;       // EP_MSE: one per block
  double* col;        // EP_MSE, EP_BACK: [row tiles][N]
  float scale;
  int ldc;            // row length of C (the other arrays: N)
  int wide;           // every array given allows 16- (BF16: 8-) byte access
};

// h = SiLU(z) = z / (1 + exp(-z));  SiLU'(z) = s (1 + z (1 - s)), s = 1 / (1 + exp(-z))
__device__ __forceinline__ float silu(float v) { return v / (1.f + expf(-v)); }
__device__ __forceinline__ float silu_back(float dh, float v) {
  const float s = 1.f / (1.f + expf(-v));
  return dh * s * (1.f + v * (1.f - s));
}

// Tile order: workgroups go to the 8 XCDs in turn, each with its own L2, so
// XCD x takes a contiguous range of the list; the list walks groups of 8 row
// tiles column by column, so that a group's rows of A and one column panel
// of B stay in that L2 while they are used.
__device__ __forceinline__ void tile_of(int b, int nm, int nn, int& tm, int& tn) {
  const int nb = nm * nn, x = b % 8, per = nb / 8, rem = nb % 8;
  const int t = x * per + (x < rem ? x : rem) + b / 8;
  const int g = t / (8 * nn), m0 = g * 8, h = nm - m0 < 8 ? nm - m0 : 8;
  const int u = t - g * 8 * nn;
  tm = m0 + u % h;
  tn = u / h;
}

template <int TM, int TN, int TA, int TB, int CONV, int EP>
__global__ void __launch_bounds__(256) k_gemm(Operand A, Operand B, Epi ep, int M, int N,
                                              int Kfull, int kchunk) {
  constexpr int FM = TM / 64, FN = TN / 64;  // 32 x 32 fragments of a wave
  __shared__ __attribute__((aligned(16))) uint16_t sAB[(TM + TN) * BK];
  uint16_t *sA = sAB, *sB = sAB + TM * BK;
  const int nm = (M + TM - 1) / TM, nn = (N + TN - 1) / TN;
  int tm, tn;
  tile_of(blockIdx.x, nm, nn, tm, tn);
  const int m0 = tm * TM, n0 = tn * TN;
  // split K: slab z covers k in [z kchunk, min(K, (z + 1) kchunk)) and writes
  // its partial product to slab z of C (slabs M x ldc apart)
  const int kbeg = blockIdx.y * kchunk;
  const int K = Kfull < kbeg + kchunk ? Kfull : kbeg + kchunk;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int wm = (w >> 1) * (TM / 2), wn = (w & 1) * (TN / 2);
  f32x16 acc[FM][FN];
#pragma unroll
  for (int a = 0; a < FM; ++a)
#pragma unroll
    for (int b = 0; b < FN; ++b)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[a][b][q] = 0.f;
  // PF k-tiles in flight in registers: a small product has few blocks and
  // little to do per k-tile, so that only the depth hides the load latency
  // (1800 rows: the first layers' products 19.7 -> 15.7 us).  A second k-tile
  // of the large shape costs a block per CU and more than it gains (57600 x
  // 4800 x 384 with the loss: 634 -> 759 us).
  constexpr int PF = TM == 64 ? 3 : 1;
  Tile<TM, TA, CONV> ta;
  Tile<TN, !TB, CONV_NONE> tb;
  Piece<TM, TA> pa[PF];
  Piece<TN, !TB> pb[PF];
  ta.init(A, m0, M);
#pragma unroll
  for (int s = 0; s < PF; ++s)
    if (kbeg + s * BK < K) {
      ta.load(pa[s], A, m0, kbeg + s * BK, M, K);
      tb.load(pb[s], B, n0, kbeg + s * BK, N, K);
    }
  for (int kg = kbeg; kg < K; kg += PF * BK) {
#pragma unroll
    for (int s = 0; s < PF; ++s) {
      const int k0 = kg + s * BK;
      if (k0 >= K) break;
      __syncthreads();  // the previous k-tile has been read
      ta.store(pa[s], sA);
      tb.store(pb[s], sB);
      __syncthreads();
      if (k0 + PF * BK < K) {
        ta.load(pa[s], A, m0, k0 + PF * BK, M, K);
        tb.load(pb[s], B, n0, k0 + PF * BK, N, K);
      }
#pragma unroll
      for (int ks = 0; ks < BK / 16; ++ks) {
        const int ch = 2 * ks + (lane >> 5);
        bf16x8 fa[FM], fb[FN];
#pragma unroll
        for (int t = 0; t < FM; ++t)
          memcpy(&fa[t], sA + lds_chunk(wm + t * 32 + (lane & 31), ch), 16);
#pragma unroll
        for (int t = 0; t < FN; ++t)
          memcpy(&fb[t], sB + lds_chunk(wn + t * 32 + (lane & 31), ch), 16);
#pragma unroll
        for (int a = 0; a < FM; ++a)
#pragma unroll
          for (int b = 0; b < FN; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a], fb[b], acc[a][b], 0, 0, 0);
      }
    }
  }
  // The finished tile goes through LDS, 64 rows at a time, so that each
  // thread holds four neighbouring columns: the epilogue's loads and stores
  // are then 16 (FP32) or 8 (BF16) bytes a lane over whole rows.
  // (accumulator element q = 4 i + j of a 32x32 fragment holds row
  // 8 i + 4 (lane / 32) + j, column lane % 32)
  float* sC = reinterpret_cast<float*>(sAB);  // [64][TN]: as large as the operand tiles
  constexpr int TC = TN / 4, RP = 256 / TC, RN = 64 / RP;  // column groups, row phases, rows
  float* C = ep.c ? ep.c + (EP == EP_OUT ? (long long)blockIdx.y * M * ep.ldc : 0) : nullptr;
  const int cq = threadIdx.x % TC, rp = threadIdx.x / TC;
  const int n = n0 + 4 * cq;
  const int ldc = EP == EP_OUT ? ep.ldc : N;
  const bool wide = n + 4 <= N && (N & 3) == 0 && (ldc & 3) == 0 && ep.wide;
  float bn[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) bn[i] = ep.bias && n + i < N ? ep.bias[n + i] : 0.f;
  double e2 = 0.0, cs[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int half = 0; half < TM / 64; ++half) {
    float4 src[RN];
    if constexpr (EP == EP_MSE || EP == EP_BACK) {
#pragma unroll
      for (int q = 0; q < RN; ++q) {
        const int m = m0 + 64 * half + rp + RP * q;
        src[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (m < M && wide) {
          src[q] = *reinterpret_cast<const float4*>(ep.t + (long long)m * N + n);
        } else if (m < M) {
          float v[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) v[i] = n + i < N ? ep.t[(long long)m * N + n + i] : 0.f;
          src[q] = make_float4(v[0], v[1], v[2], v[3]);
        }
      }
    }
    __syncthreads();
    if (TM == 64 || (w >> 1) == half) {
      const int wr = TM == 64 ? wm : 0;
#pragma unroll
      for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b)
#pragma unroll
          for (int q = 0; q < 16; ++q)
            sC[(wr + a * 32 + 8 * (q >> 2) + 4 * (lane >> 5) + (q & 3)) * TN + wn + b * 32 +
               (lane & 31)] = acc[a][b][q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < RN; ++q) {
      const int r = rp + RP * q, m = m0 + 64 * half + r;
      if (m >= M) continue;
      const float4 c4 = *reinterpret_cast<const float4*>(sC + r * TN + 4 * cq);
      const float v[4] = {c4.x, c4.y, c4.z, c4.w};
      const float s4[4] = {src[q].x, src[q].y, src[q].z, src[q].w};
      float out[4];
      uint16_t hb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (EP == EP_OUT) {
          out[i] = v[i] + bn[i];
        } else if constexpr (EP == EP_SILU) {
          out[i] = v[i] + bn[i];
          hb[i] = f2bf(silu(out[i]));
        } else {
          float d;
          if constexpr (EP == EP_MSE) {
            const float y = v[i] + bn[i];
            d = y - s4[i];
            hb[i] = f2bf(2.f * d * ep.scale);
          } else {
            d = silu_back(v[i], s4[i]);
            hb[i] = f2bf(d);
          }
          if (n + i < N) {
            if (EP == EP_MSE) e2 += (double)d * d;
            cs[i] += (double)d;
          }
        }
      }
      const long long o = (long long)m * ldc + n;
      if (wide) {
        if ((EP == EP_OUT || EP == EP_SILU) && C)
          *reinterpret_cast<float4*>(C + o) = make_float4(out[0], out[1], out[2], out[3]);
        if constexpr (EP != EP_OUT)
          *reinterpret_cast<ushort4*>(ep.h + o) = make_ushort4(hb[0], hb[1], hb[2], hb[3]);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n + i < N) {
            if ((EP == EP_OUT || EP == EP_SILU) && C) C[o + i] = out[i];
            if constexpr (EP != EP_OUT) ep.h[o + i] = hb[i];
          }
      }
    }
  }
  if constexpr (EP == EP_MSE || EP == EP_BACK) {
    // column sums over the tile's rows: the row phases in a fixed order
    __syncthreads();
    double* sc = reinterpret_cast<double*>(sAB);  // [RP][TN], then 4 wave sums
#pragma unroll
    for (int i = 0; i < 4; ++i) sc[rp * TN + 4 * cq + i] = cs[i];
    if (EP == EP_MSE) {
      for (int o = 32; o > 0; o >>= 1) e2 += __shfl_xor(e2, o, 64);
      if (lane == 0) sc[RP * TN + w] = e2;
    }
    __syncthreads();
    if (threadIdx.x < TN && n0 + (int)threadIdx.x < N) {
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < RP; ++q) s += sc[q * TN + threadIdx.x];
      ep.col[(long long)tm * N + n0 + threadIdx.x] = s;
    }
    if (EP == EP_MSE && threadIdx.x == 0) {
      const double* se = sc + RP * TN;
      ep.loss[blockIdx.x] = ((se[0] + se[1]) + se[2]) + se[3];
    }
  }
}

// Tile shape: 128 x 128 where that fills the chip (256 CUs, two blocks each)
// and the output is wider than one 64-column tile, else 64 x 64: with fewer
// tiles CUs stay empty, and 64 output columns would leave half of a 128-wide
// tile to padding.
constexpr int TBIG = 128, TSMALL = 64;
inline long long tiles(int t, int M, int N) {
  return (long long)((M + t - 1) / t) * ((N + t - 1) / t);
}
inline int tile_for(int M, int N, int splits) {
  return N > TSMALL && tiles(TBIG, M, N) * splits >= 512 ? TBIG : TSMALL;
}

Operand operand(const uint16_t* p, int ld) {
  Operand o{};
  o.p = p;
  o.ld = ld;
  o.vec = (ld & 7) == 0 && ((uintptr_t)p & 15) == 0;
  return o;
}
Operand conv_operand(const uint16_t* p, const Conv& cv) {
  Operand o{};
  o.p = p;
  o.cv = cv;
  o.vec = (cv.C & 7) == 0 && ((uintptr_t)p & 15) == 0;
  return o;
}

template <int TA, int TB, int CONV, int EP>
void gemm_launch_as(const Operand& A, const Operand& B, Epi ep, int M, int N, int K, int splits,
                    int kchunk, hipStream_t s) {
  ep.wide = ((((uintptr_t)ep.c | (uintptr_t)ep.t) & 15) | ((uintptr_t)ep.h & 7)) == 0;
  const int t = tile_for(M, N, splits);
  const dim3 grid((unsigned)tiles(t, M, N), splits), blk(256);
  if (t == TBIG)
    hipLaunchKernelGGL((k_gemm<TBIG, TBIG, TA, TB, CONV, EP>), grid, blk, 0, s, A, B, ep, M, N, K,
                       kchunk);
  else
    hipLaunchKernelGGL((k_gemm<TSMALL, TSMALL, TA, TB, CONV, EP>), grid, blk, 0, s, A, B, ep, M,
                       N, K, kchunk);
}

// CONV = 1: A is a neighbourhood matrix, read as its channel count allows
template <int TA, int TB, int CONV, int EP>
void gemm_launch(const Operand& A, const Operand& B, const Epi& ep, int M, int N, int K,
                 int splits, int kchunk, hipStream_t s) {
  if constexpr (!CONV)
    gemm_launch_as<TA, TB, CONV_NONE, EP>(A, B, ep, M, N, K, splits, kchunk, s);
  else if (A.vec)
    gemm_launch_as<TA, TB, CONV_VEC, EP>(A, B, ep, M, N, K, splits, kchunk, s);
  else if ((A.cv.C & 1) == 0)
    gemm_launch_as<TA, TB, CONV_PAIR, EP>(A, B, ep, M, N, K, splits, kchunk, s);
  else
    gemm_launch_as<TA, TB, CONV_ONE, EP>(A, B, ep, M, N, K, splits, kchunk, s);
}

template <int TA, int TB, int CONV, int EP>
void gemm(const Operand& A, const Operand& B, const Epi& ep, int M, int N, int K, hipStream_t s) {
  gemm_launch<TA, TB, CONV, EP>(A, B, ep, M, N, K, 1, (K + BK - 1) / BK * BK, s);
}

// Split of the reduction dimension for products whose output has few tiles
// and whose K is long (the weight gradients, K = rows of the batch): about
// 1024 (128 x 128 tile, slab) blocks, each slab a multiple of 32 rows and at
// least 256.  The slab sums are rounded to FP32 before they are added, so
// this partition fixes the gradients' rounding: it does not follow BK or the
// tile shape.
struct Split {
  int slabs, kchunk;
};
int split_most(int M, int N) { return (int)((1024 + tiles(TBIG, M, N) - 1) / tiles(TBIG, M, N)); }
Split ksplit(int M, int N, int K) {
  int want = split_most(M, N);
  const int most = (K + 255) / 256;
  want = want < 1 ? 1 : (want > most ? most : want);
  const int kchunk = ((K + want - 1) / want + 31) / 32 * 32;
  return Split{(K + kchunk - 1) / kchunk, kchunk};
}

// C[i] = sum over slabs z (in order) of P[z][i]
__global__ void k_sum_slabs(const float* __restrict__ part, int slabs, long long n,
                            float* __restrict__ C) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float acc = 0.f;
#pragma unroll 8
  for (int z = 0; z < slabs; ++z) acc += part[(long long)z * n + i];
  C[i] = acc;
}

// weight gradient C [M][N] (contiguous) = A^T B from a product over a long K
template <int CONV>
void gemm_wgrad(const Operand& A, const Operand& B, float* C, int M, int N, int K,
                float* scratch, hipStream_t s) {
  const Split sp = ksplit(M, N, K);
  Epi ep{};
  ep.ldc = N;
  ep.c = sp.slabs == 1 ? C : scratch;
  gemm_launch<1, 0, CONV, EP_OUT>(A, B, ep, M, N, K, sp.slabs, sp.kchunk, s);
  if (sp.slabs == 1) return;
  const long long n = (long long)M * N;
  hipLaunchKernelGGL(k_sum_slabs, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, scratch,
                     sp.slabs, n, C);
}

// ------------------------------------------------------------ elementwise --
__global__ void k_to_bf16(const float* __restrict__ x, uint16_t* __restrict__ y, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = f2bf(x[i]);
}

// Backward of the neighbourhood gather and of the SiLU before it: dH[b, j,
// k][c] = sum of dA over every (row, tap) that gathered (j, k) (dA stored
// [row][tap * C + c]), dZ = dH SiLU'(Z) in BF16, and the column sums of dZ
// over the block's rows.  Blocks of CI_ROWS rows x 64 channels, 4 row phases.
constexpr int CI_ROWS = 32;
__global__ void __launch_bounds__(256) k_col2im_back(const float* __restrict__ da,
                                                     const float* __restrict__ z,
                                                     uint16_t* __restrict__ dzb,
                                                     double* __restrict__ col, int M, Conv cv) {
  __shared__ double sh[4][64];
  const int nt = cv.nt, np = cv.np, C = cv.C, nk = cv.nk, taps = 3 * nk;
  const int c = blockIdx.y * 64 + (threadIdx.x & 63), ph = threadIdx.x >> 6;
  const int r0 = blockIdx.x * CI_ROWS, r1 = r0 + CI_ROWS < M ? r0 + CI_ROWS : M;
  double acc = 0.0;
  if (c < C)
    for (int m = r0 + ph; m < r1; m += 4) {
      const ConvRow r = conv_row(cv, m);
      float s = 0.f;
      for (int dj = -1; dj <= 1; ++dj) {
        // source rows jsrc whose clamp(jsrc + dj) == j
        int js[2], ns = 0;
        const int j0 = r.j - dj;
        if (j0 >= 0 && j0 < nt) js[ns++] = j0;
        if (dj == -1 && r.j == 0) js[ns++] = 0;            // clamp(0 - 1) = 0
        if (dj == 1 && r.j == nt - 1) js[ns++] = nt - 1;  // clamp(nt - 1 + 1) = nt - 1
        for (int q = 0; q < ns; ++q)
          for (int t = 0; t < nk; ++t) {
            int ks = (r.k - (t + cv.dk0)) % np;
            if (ks < 0) ks += np;
            const int tap = (dj + 1) * nk + t;
            s += da[((((long long)r.b * nt + js[q]) * np + ks) * taps + tap) * C + c];
          }
      }
      const long long o = (long long)m * C + c;
      const float d = silu_back(s, z[o]);
      dzb[o] = f2bf(d);
      acc += (double)d;
    }
  sh[ph][threadIdx.x & 63] = acc;
  __syncthreads();
  if (ph == 0 && c < C)
    col[(long long)blockIdx.x * C + c] =
        ((sh[0][threadIdx.x] + sh[1][threadIdx.x]) + sh[2][threadIdx.x]) + sh[3][threadIdx.x];
}

// Bias gradients of the four layers in one launch: db[n] = scale times the
// column sums added over the row tiles, 16 row phases combined in order.
struct ColJob {
  const double* part;
  float* db;
  int rows, N, blk0;  // first block of this job
  double scale;
};
struct ColJobs {
  ColJob j[4];
};
__global__ void __launch_bounds__(1024) k_colsum_fin(ColJobs jobs) {
  __shared__ double sh[16][64];
  int q = 0;
  while (q < 3 && (int)blockIdx.x >= jobs.j[q + 1].blk0) ++q;
  const ColJob& J = jobs.j[q];
  const int n = (blockIdx.x - J.blk0) * 64 + (threadIdx.x & 63), ph = threadIdx.x >> 6;
  double acc = 0.0;
  if (n < J.N) {
#pragma unroll 8
    for (int r = ph; r < J.rows; r += 16) acc += J.part[(long long)r * J.N + n];
  }
  sh[ph][threadIdx.x & 63] = acc;
  __syncthreads();
  if (ph == 0 && n < J.N) {
    double s = 0.0;
#pragma unroll
    for (int p = 0; p < 16; ++p) s += sh[p][threadIdx.x];
    J.db[n] = (float)(s * J.scale);
  }
}

// out = sum of part[0..n): one block of 1024, strided partial sums, then a
// fixed tree
__global__ void __launch_bounds__(1024) k_sum(const double* __restrict__ part, int n,
                                              double* __restrict__ out) {
  __shared__ double sh[1024];
  double acc = 0.0;
  for (int i = threadIdx.x; i < n; i += 1024) acc += part[i];
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = sh[0];
}

// Adam on FP32 masters, BF16 copies refreshed
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, uint16_t* __restrict__ pb, long long n, float lr,
                       float b1, float b2, float eps, float c1, float c2) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  p[i] = pi;
  pb[i] = f2bf(pi);
}

// ------------------------------------------------------ feature transforms --
struct Norm {
  double rho_ref, v_ref, p_ref, b_ref;
};

// X[b][j][k][f] from SI maps [b][8][nt][np] (cin = 8, or 10 with the two
// colatitude channels)
__global__ void k_encode_map(const double* __restrict__ maps, float* __restrict__ x, int B, int nt,
                             int np, double omega, double r_in, const double* __restrict__ thc,
                             Norm nz, int cin) {
  const long long n = (long long)B * nt * np;
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  const int k = (int)(q % np);
  const int j = (int)((q / np) % nt);
  const int b = (int)(q / ((long long)nt * np));
  const long long plane = (long long)nt * np;
  const double* m = maps + (long long)b * 8 * plane + (long long)j * np + k;
  float* o = x + q * cin;
  if (cin > 8) {
    const double t = nt > 1 ? (2.0 * thc[j] - thc[0] - thc[nt - 1]) / (thc[nt - 1] - thc[0]) : 0.0;
    o[8] = (float)t;
    o[9] = (float)(2.0 * t * t - 1.0);
  }
  o[0] = (float)log(m[0] / nz.rho_ref);
  o[1] = (float)(m[1 * plane] / nz.v_ref - 5.0);
  o[2] = (float)(m[2 * plane] / nz.v_ref);
  o[3] = (float)((m[3 * plane] + omega * r_in * sin(thc[j])) / nz.v_ref);
  o[4] = (float)log(m[4 * plane] / nz.p_ref);
  o[5] = (float)(m[5 * plane] / nz.b_ref);
  o[6] = (float)(m[6 * plane] / nz.b_ref);
  o[7] = (float)(m[7 * plane] / nz.b_ref);
}

// radial expansion of the map column at r (same laws as the initial state)
__device__ __forceinline__ void radial_base(const double* m, long long plane, double r, double r_in,
                                            double omega, double sth, double gam, double (&w)[8]) {
  const double x = r_in / r;
  w[0] = m[0] * x * x;
  w[1] = m[plane];
  w[2] = 0.0;
  w[3] = -omega * r * sth;
  w[4] = m[4 * plane] * pow(x, 2.0 * gam);
  w[5] = m[5 * plane] * x * x;
  w[6] = 0.0;
  w[7] = m[7 * plane] * x;
}

// T[col][i*8 + v] (col = j*np + k) from a primitive SI state [8][np][nt][nr] and its map
__global__ void k_encode_target(const double* __restrict__ map, const double* __restrict__ st,
                                const double* __restrict__ rc, const double* __restrict__ thc,
                                float* __restrict__ t, int nr, int nt, int np, double omega,
                                double r_in, double gam, double v_ref) {
  const long long n = (long long)nr * nt * np;
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  const int i = (int)(q % nr);
  const int j = (int)((q / nr) % nt);
  const int k = (int)(q / ((long long)nr * nt));
  const long long plane = (long long)nt * np;
  double w[8];
  radial_base(map + (long long)j * np + k, plane, rc[i], r_in, omega, sin(thc[j]), gam, w);
  const long long cell = ((long long)k * nt + j) * nr + i;
  double s[8];
  for (int v = 0; v < 8; ++v) s[v] = st[v * n + cell];
  const double bs = fabs(w[5]) + fabs(w[7]) + 1e-30;
  float* o = t + (((long long)j * np + k) * nr + i) * 8;
  o[0] = (float)log(s[0] / w[0]);
  o[1] = (float)((s[1] - w[1]) / v_ref);
  o[2] = (float)(s[2] / v_ref);
  o[3] = (float)((s[3] - w[3]) / v_ref);
  o[4] = (float)log(s[4] / w[4]);
  o[5] = (float)((s[5] - w[5]) / bs);
  o[6] = (float)(s[6] / bs);
  o[7] = (float)((s[7] - w[7]) / bs);
}

// inverse of k_encode_target: primitive SI state from the network output
__global__ void k_decode_state(const double* __restrict__ map, const float* __restrict__ y,
                               const double* __restrict__ rc, const double* __restrict__ thc,
                               double* __restrict__ st, int nr, int nt, int np, double omega,
                               double r_in, double gam, double v_ref) {
  const long long n = (long long)nr * nt * np;
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  const int i = (int)(q % nr);
  const int j = (int)((q / nr) % nt);
  const int k = (int)(q / ((long long)nr * nt));
  const long long plane = (long long)nt * np;
  double w[8];
  radial_base(map + (long long)j * np + k, plane, rc[i], r_in, omega, sin(thc[j]), gam, w);
  const double bs = fabs(w[5]) + fabs(w[7]) + 1e-30;
  const float* o = y + (((long long)j * np + k) * nr + i) * 8;
  double s[8];
  s[0] = w[0] * exp((double)o[0]);
  s[1] = w[1] + v_ref * o[1];
  s[2] = v_ref * o[2];
  s[3] = w[3] + v_ref * o[3];
  s[4] = w[4] * exp((double)o[4]);
  s[5] = w[5] + bs * o[5];
  s[6] = bs * o[6];
  s[7] = w[7] + bs * o[7];
  const long long cell = ((long long)k * nt + j) * nr + i;
  for (int v = 0; v < 8; ++v) st[v * n + cell] = s[v];
}

}  // namespace icrnn

using namespace icrnn;

namespace {
thread_local std::string g_nn_err;
int nfail(int code, const char* fmt, ...) {
  char buf[400];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_nn_err = buf;
  return code;
}
#define NN_TRY(expr)                                                                   \
  do {                                                                                 \
    hipError_t e_ = (expr);                                                            \
    if (e_ != hipSuccess) return nfail(ICR_NN_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

size_t al(size_t x) { return (x + 255) & ~size_t(255); }

struct Sizes {
  long long ncol, M;           // columns per sample, rows of a batch
  long long w1, w2, w3, w4;    // weight counts
  long long nparam;
  int cin, c1, c2, h, no, k1, k2;  // input features, channels, hidden, outputs, conv K
};

Sizes sizes(const icr_nn_shape& s) {
  Sizes z;
  z.ncol = (long long)s.n_theta * s.n_phi;
  z.M = z.ncol * s.batch_max;
  z.c1 = s.c1;
  z.c2 = s.c2;
  z.h = s.hidden;
  z.no = s.n_r * 8;
  z.cin = s.coord ? 10 : 8;
  z.k1 = 3 * (s.phi_hi - s.phi_lo + 1) * z.cin;
  z.k2 = 9 * s.c1;
  z.w1 = (long long)z.k1 * z.c1;
  z.w2 = (long long)z.k2 * z.c2;
  z.w3 = (long long)z.c2 * z.h;
  z.w4 = (long long)z.h * z.no;
  z.nparam = z.w1 + z.c1 + z.w2 + z.c2 + z.w3 + z.h + z.w4 + z.no;
  return z;
}

int check_shape(const icr_nn_shape* s) {
  if (!s) return nfail(ICR_NN_ERR_ARG, "shape is NULL");
  if (s->n_theta < 1 || s->n_phi < 3 || s->n_r < 1 || s->c1 < 1 || s->c2 < 1 || s->hidden < 1 ||
      s->batch_max < 1 || (s->coord != 0 && s->coord != 1))
    return nfail(ICR_NN_ERR_ARG, "invalid network shape");
  if (s->phi_lo > 0 || s->phi_hi < 0 || s->phi_hi - s->phi_lo + 1 > s->n_phi)
    return nfail(ICR_NN_ERR_ARG, "first-layer longitude window must hold offset 0 and fit n_phi");
  return ICR_NN_OK;
}

}  // namespace

struct icr_nn {
  icr_nn_shape s;
  Sizes z;
  hipStream_t stream;
  char* ws;
  // parameters: fp32 master, bf16 copy, grads, Adam moments (same layout)
  float *p, *g, *m, *v;
  uint16_t* pb;
  long long step;
  // activations (batch_max rows)
  uint16_t *xb, *h1, *h2, *h3;             // bf16 operands
  float *z1, *z2, *z3, *y;                 // pre-activations and output
  uint16_t *dyb, *dz3b, *dz2b, *dz1b;
  float* da2;
  double *part, *loss;
  float* split;     // split-K partial products of the weight gradients
  double* cpart[4]; // column-sum partials of each layer [row tiles][width]
  // parameter views
  float *W1, *b1, *W2, *b2, *W3, *b3, *W4, *b4;
  uint16_t *W1b, *W2b, *W3b, *W4b;
  float *gW1, *gb1, *gW2, *gb2, *gW3, *gb3, *gW4, *gb4;
};

namespace {

size_t layout(const icr_nn_shape& s, icr_nn* n) {
  const Sizes z = sizes(s);
  size_t off = 0;
  char* base = n ? n->ws : nullptr;
  auto take = [&](size_t b) {
    char* p = base ? base + off : nullptr;
    off += al(b);
    return p;
  };
  const long long P = z.nparam, M = z.M;
  float* p = (float*)take(4 * P);
  float* g = (float*)take(4 * P);
  float* m = (float*)take(4 * P);
  float* v = (float*)take(4 * P);
  uint16_t* pb = (uint16_t*)take(2 * P);
  uint16_t* xb = (uint16_t*)take(2 * M * z.cin);
  float* z1 = (float*)take(4 * M * z.c1);
  uint16_t* h1 = (uint16_t*)take(2 * M * z.c1);
  float* z2 = (float*)take(4 * M * z.c2);
  uint16_t* h2 = (uint16_t*)take(2 * M * z.c2);
  float* z3 = (float*)take(4 * M * z.h);
  uint16_t* h3 = (uint16_t*)take(2 * M * z.h);
  float* y = (float*)take(4 * M * z.no);
  uint16_t* dyb = (uint16_t*)take(2 * M * z.no);
  uint16_t* dz3b = (uint16_t*)take(2 * M * z.h);
  uint16_t* dz2b = (uint16_t*)take(2 * M * z.c2);
  float* da2 = (float*)take(4 * M * z.k2);
  uint16_t* dz1b = (uint16_t*)take(2 * M * z.c1);
  // one loss partial per tile of the output layer, column sums per row tile
  // (sized for the smaller tile)
  double* part = (double*)take(8 * tiles(TSMALL, (int)M, z.no));
  double* loss = (double*)take(8);
  // (a smaller batch may be split differently, but never into more slabs)
  long long nsplit = 1;
  {
    const int dims[4][2] = {{z.h, z.no}, {z.c2, z.h}, {z.k2, z.c2}, {z.k1, z.c1}};
    for (const auto& d : dims) {
      const long long most = split_most(d[0], d[1]);
      if (most > 1 && most * d[0] * d[1] > nsplit) nsplit = most * d[0] * d[1];
    }
  }
  float* split = (float*)take(4 * nsplit);
  const long long rt = (M + TSMALL - 1) / TSMALL;
  const int width[4] = {z.c1, z.c2, z.h, z.no};
  double* cpart[4];
  for (int q = 0; q < 4; ++q)
    cpart[q] = (double*)take(8 * width[q] * (q == 0 ? (M + CI_ROWS - 1) / CI_ROWS : rt));
  if (n) {
    n->z = z;
    n->p = p; n->g = g; n->m = m; n->v = v; n->pb = pb;
    n->xb = xb; n->z1 = z1; n->h1 = h1; n->z2 = z2; n->h2 = h2; n->z3 = z3; n->h3 = h3;
    n->y = y; n->dyb = dyb; n->dz3b = dz3b; n->dz2b = dz2b; n->da2 = da2; n->dz1b = dz1b;
    n->part = part; n->loss = loss; n->split = split;
    for (int q = 0; q < 4; ++q) n->cpart[q] = cpart[q];
    long long o = 0;
    auto view = [&](long long cnt, float*& fp, float*& gp, uint16_t** bp) {
      fp = p + o;
      gp = g + o;
      if (bp) *bp = pb + o;
      o += cnt;
    };
    view(z.w1, n->W1, n->gW1, &n->W1b);
    view(z.c1, n->b1, n->gb1, nullptr);
    view(z.w2, n->W2, n->gW2, &n->W2b);
    view(z.c2, n->b2, n->gb2, nullptr);
    view(z.w3, n->W3, n->gW3, &n->W3b);
    view(z.h, n->b3, n->gb3, nullptr);
    view(z.w4, n->W4, n->gW4, &n->W4b);
    view(z.no, n->b4, n->gb4, nullptr);
  }
  return off;
}

inline dim3 g1(long long n) { return dim3((unsigned)((n + 255) / 256)); }

Conv conv1(const icr_nn* n) {
  return Conv{n->s.n_theta, n->s.n_phi, n->z.cin, n->s.phi_lo, n->s.phi_hi - n->s.phi_lo + 1};
}
Conv conv2(const icr_nn* n) { return Conv{n->s.n_theta, n->s.n_phi, n->z.c1, -1, 3}; }

Epi silu_epi(float* z, const float* bias, uint16_t* h) {
  Epi e{};
  e.c = z;
  e.bias = bias;
  e.h = h;
  return e;
}

// The layers before the output layer; the pre-activations are kept for a
// backward pass only.
void encode(icr_nn* n, int B, const float* x_dev, bool keep) {
  const Sizes& z = n->z;
  const int M = (int)((long long)B * z.ncol);
  hipStream_t s = n->stream;
  hipLaunchKernelGGL(k_to_bf16, g1((long long)M * z.cin), dim3(256), 0, s, x_dev, n->xb,
                     (long long)M * z.cin);
  gemm<0, 0, 1, EP_SILU>(conv_operand(n->xb, conv1(n)), operand(n->W1b, z.c1),
                         silu_epi(keep ? n->z1 : nullptr, n->b1, n->h1), M, z.c1, z.k1, s);
  gemm<0, 0, 1, EP_SILU>(conv_operand(n->h1, conv2(n)), operand(n->W2b, z.c2),
                         silu_epi(keep ? n->z2 : nullptr, n->b2, n->h2), M, z.c2, z.k2, s);
  gemm<0, 0, 0, EP_SILU>(operand(n->h2, z.c2), operand(n->W3b, z.h),
                         silu_epi(keep ? n->z3 : nullptr, n->b3, n->h3), M, z.h, z.c2, s);
}

void forward(icr_nn* n, int B, const float* x_dev, float* y) {
  const Sizes& z = n->z;
  encode(n, B, x_dev, false);
  Epi e{};
  e.c = y;
  e.ldc = z.no;
  e.bias = n->b4;
  gemm<0, 0, 0, EP_OUT>(operand(n->h3, z.h), operand(n->W4b, z.no), e, (int)(B * z.ncol), z.no,
                        z.h, n->stream);
}

Epi back_epi(const float* z, uint16_t* dzb, double* col) {
  Epi e{};
  e.t = z;
  e.h = dzb;
  e.col = col;
  return e;
}

// Loss and gradients.  The output layer's tiles go straight to dY and the
// loss; Y itself is not stored.
void loss_grad(icr_nn* n, int B, const float* x_dev, const float* t_dev) {
  const Sizes& z = n->z;
  const int M = (int)((long long)B * z.ncol);
  const long long ny = (long long)M * z.no;
  hipStream_t s = n->stream;
  auto row_tiles = [&](int N) {
    const int t = tile_for(M, N, 1);
    return (M + t - 1) / t;
  };
  encode(n, B, x_dev, true);
  Epi e{};
  e.bias = n->b4;
  e.t = t_dev;
  e.h = n->dyb;
  e.loss = n->part;
  e.col = n->cpart[3];
  e.scale = 1.f / (float)ny;
  gemm<0, 0, 0, EP_MSE>(operand(n->h3, z.h), operand(n->W4b, z.no), e, M, z.no, z.h, s);
  hipLaunchKernelGGL(k_sum, dim3(1), dim3(1024), 0, s, n->part,
                     (int)tiles(tile_for(M, z.no, 1), M, z.no), n->loss);
  // decoder layer 2: Y = H3 W4 + b4
  gemm_wgrad<0>(operand(n->h3, z.h), operand(n->dyb, z.no), n->gW4, z.h, z.no, M, n->split, s);
  gemm<0, 1, 0, EP_BACK>(operand(n->dyb, z.no), operand(n->W4b, z.no),
                         back_epi(n->z3, n->dz3b, n->cpart[2]), M, z.h, z.no, s);
  gemm_wgrad<0>(operand(n->h2, z.c2), operand(n->dz3b, z.h), n->gW3, z.c2, z.h, M, n->split, s);
  gemm<0, 1, 0, EP_BACK>(operand(n->dz3b, z.h), operand(n->W3b, z.h),
                         back_epi(n->z2, n->dz2b, n->cpart[1]), M, z.c2, z.h, s);
  gemm_wgrad<1>(conv_operand(n->h1, conv2(n)), operand(n->dz2b, z.c2), n->gW2, z.k2, z.c2, M,
                n->split, s);
  Epi da{};
  da.c = n->da2;
  da.ldc = z.k2;
  gemm<0, 1, 0, EP_OUT>(operand(n->dz2b, z.c2), operand(n->W2b, z.c2), da, M, z.k2, z.c2, s);
  const int ci = (M + CI_ROWS - 1) / CI_ROWS;
  hipLaunchKernelGGL(k_col2im_back, dim3(ci, (z.c1 + 63) / 64), dim3(256), 0, s, n->da2, n->z1,
                     n->dz1b, n->cpart[0], M, conv2(n));
  gemm_wgrad<1>(conv_operand(n->xb, conv1(n)), operand(n->dz1b, z.c1), n->gW1, z.k1, z.c1, M,
                n->split, s);
  ColJobs jobs;
  float* db[4] = {n->gb1, n->gb2, n->gb3, n->gb4};
  const int width[4] = {z.c1, z.c2, z.h, z.no};
  int blk = 0;
  for (int q = 0; q < 4; ++q) {
    jobs.j[q] = ColJob{n->cpart[q], db[q], q == 0 ? ci : row_tiles(width[q]), width[q], blk,
                       q == 3 ? 2.0 / (double)ny : 1.0};
    blk += (width[q] + 63) / 64;
  }
  hipLaunchKernelGGL(k_colsum_fin, dim3(blk), dim3(1024), 0, s, jobs);
}

}  // namespace


extern "C" {

const char* icr_nn_last_error(void) { return g_nn_err.c_str(); }

int icr_nn_param_count(const icr_nn_shape* s, long long* n) {
  int rc = check_shape(s);
  if (rc) return rc;
  if (!n) return nfail(ICR_NN_ERR_ARG, "n is NULL");
  *n = sizes(*s).nparam;
  return ICR_NN_OK;
}

int icr_nn_workspace_bytes(const icr_nn_shape* s, size_t* bytes) {
  int rc = check_shape(s);
  if (rc) return rc;
  if (!bytes) return nfail(ICR_NN_ERR_ARG, "bytes is NULL");
  *bytes = layout(*s, nullptr);
  return ICR_NN_OK;
}

int icr_nn_create(const icr_nn_shape* s, void* ws, size_t bytes, void* stream, icr_nn** out) {
  int rc = check_shape(s);
  if (rc) return rc;
  if (!out) return nfail(ICR_NN_ERR_ARG, "out is NULL");
  const size_t need = layout(*s, nullptr);
  if (!ws || bytes < need) return nfail(ICR_NN_ERR_ARG, "workspace too small (%zu < %zu)", bytes, need);
  if (((uintptr_t)ws & 255) != 0) return nfail(ICR_NN_ERR_ARG, "workspace must be 256-byte aligned");
  icr_nn* n = new icr_nn();
  n->s = *s;
  n->stream = (hipStream_t)stream;
  n->ws = (char*)ws;
  n->step = 0;
  layout(*s, n);
  *out = n;
  return ICR_NN_OK;
}

void icr_nn_destroy(icr_nn* n) { delete n; }

int icr_nn_set_params(icr_nn* n, const float* host) {
  if (!n || !host) return nfail(ICR_NN_ERR_ARG, "NULL argument");
  const long long P = n->z.nparam;
  NN_TRY(hipMemcpyAsync(n->p, host, 4 * P, hipMemcpyHostToDevice, n->stream));
  NN_TRY(hipMemsetAsync(n->m, 0, 4 * P, n->stream));
  NN_TRY(hipMemsetAsync(n->v, 0, 4 * P, n->stream));
  hipLaunchKernelGGL(k_to_bf16, g1(P), dim3(256), 0, n->stream, n->p, n->pb, P);
  NN_TRY(hipStreamSynchronize(n->stream));
  n->step = 0;
  return ICR_NN_OK;
}

int icr_nn_get_params(icr_nn* n, float* host) {
  if (!n || !host) return nfail(ICR_NN_ERR_ARG, "NULL argument");
  NN_TRY(hipMemcpyAsync(host, n->p, 4 * n->z.nparam, hipMemcpyDeviceToHost, n->stream));
  NN_TRY(hipStreamSynchronize(n->stream));
  return ICR_NN_OK;
}

int icr_nn_forward(icr_nn* n, int batch, const float* x_dev, float* y_dev) {
  if (!n || !x_dev) return nfail(ICR_NN_ERR_ARG, "NULL argument");
  if (batch < 1 || batch > n->s.batch_max) return nfail(ICR_NN_ERR_ARG, "batch outside [1, %d]", n->s.batch_max);
  forward(n, batch, x_dev, y_dev ? y_dev : n->y);
  NN_TRY(hipGetLastError());
  return ICR_NN_OK;
}

int icr_nn_loss_grad(icr_nn* n, int batch, const float* x_dev, const float* t_dev, double* loss,
                     float* grad_host) {
  if (!n || !x_dev || !t_dev) return nfail(ICR_NN_ERR_ARG, "NULL argument");
  if (batch < 1 || batch > n->s.batch_max) return nfail(ICR_NN_ERR_ARG, "batch outside [1, %d]", n->s.batch_max);
  loss_grad(n, batch, x_dev, t_dev);
  const long long ny = (long long)batch * n->z.ncol * n->z.no;
  NN_TRY(hipGetLastError());
  double l = 0.0;
  NN_TRY(hipMemcpyAsync(&l, n->loss, 8, hipMemcpyDeviceToHost, n->stream));
  if (grad_host)
    NN_TRY(hipMemcpyAsync(grad_host, n->g, 4 * n->z.nparam, hipMemcpyDeviceToHost, n->stream));
  NN_TRY(hipStreamSynchronize(n->stream));
  if (loss) *loss = l / (double)ny;
  return ICR_NN_OK;
}

int icr_nn_adam_step(icr_nn* n, float lr, float beta1, float beta2, float eps) {
  if (!n) return nfail(ICR_NN_ERR_ARG, "NULL argument");
  n->step += 1;
  const float c1 = 1.f - powf(beta1, (float)n->step), c2 = 1.f - powf(beta2, (float)n->step);
  hipLaunchKernelGGL(k_adam, g1(n->z.nparam), dim3(256), 0, n->stream, n->p, n->g, n->m, n->v,
                     n->pb, n->z.nparam, lr, beta1, beta2, eps, c1, c2);
  NN_TRY(hipGetLastError());
  return ICR_NN_OK;
}

int icr_nn_encode_map(icr_nn* n, int batch, const double* maps_dev, const double* thc_dev,
                      double omega, double r_in, float* x_dev) {
  if (!n || !maps_dev || !thc_dev || !x_dev) return nfail(ICR_NN_ERR_ARG, "NULL argument");
  const Norm nz{1.67262192369e-27 * 1e8, 1e5, 2.0 * 1e8 * 1.380649e-23 * 1e6, 250e-9};
  const long long q = (long long)batch * n->z.ncol;
  hipLaunchKernelGGL(k_encode_map, g1(q), dim3(256), 0, n->stream, maps_dev, x_dev, batch,
                     n->s.n_theta, n->s.n_phi, omega, r_in, thc_dev, nz, n->z.cin);
  NN_TRY(hipGetLastError());
  return ICR_NN_OK;
}

int icr_nn_encode_target(icr_nn* n, const double* map_dev, const double* state_dev,
                         const double* rc_dev, const double* thc_dev, double omega, double r_in,
                         double gamma, float* t_dev) {
  if (!n || !map_dev || !state_dev || !rc_dev || !thc_dev || !t_dev)
    return nfail(ICR_NN_ERR_ARG, "NULL argument");
  const long long c = (long long)n->s.n_r * n->z.ncol;
  hipLaunchKernelGGL(k_encode_target, g1(c), dim3(256), 0, n->stream, map_dev, state_dev, rc_dev,
                     thc_dev, t_dev, n->s.n_r, n->s.n_theta, n->s.n_phi, omega, r_in, gamma, 1e5);
  NN_TRY(hipGetLastError());
  return ICR_NN_OK;
}

int icr_nn_decode_state(icr_nn* n, const double* map_dev, const float* y_dev, const double* rc_dev,
                        const double* thc_dev, double omega, double r_in, double gamma,
                        double* state_dev) {
  if (!n || !map_dev || !y_dev || !rc_dev || !thc_dev || !state_dev)
    return nfail(ICR_NN_ERR_ARG, "NULL argument");
  const long long c = (long long)n->s.n_r * n->z.ncol;
  hipLaunchKernelGGL(k_decode_state, g1(c), dim3(256), 0, n->stream, map_dev, y_dev, rc_dev,
                     thc_dev, state_dev, n->s.n_r, n->s.n_theta, n->s.n_phi, omega, r_in, gamma,
                     1e5);
  NN_TRY(hipGetLastError());
  return ICR_NN_OK;
}

int icr_nn_gemm_bf16(int trans_a, int trans_b, int M, int N, int K, const void* A, int lda,
                     const void* B, int ldb, float* C, int ldc, const float* bias, void* stream) {
  if (M < 1 || N < 1 || K < 1 || !A || !B || !C) return nfail(ICR_NN_ERR_ARG, "invalid GEMM");
  const Operand a = operand((const uint16_t*)A, lda), b = operand((const uint16_t*)B, ldb);
  Epi e{};
  e.c = C;
  e.ldc = ldc;
  e.bias = bias;
  hipStream_t s = (hipStream_t)stream;
  if (!trans_a && !trans_b) gemm<0, 0, 0, EP_OUT>(a, b, e, M, N, K, s);
  else if (!trans_a) gemm<0, 1, 0, EP_OUT>(a, b, e, M, N, K, s);
  else if (!trans_b) gemm<1, 0, 0, EP_OUT>(a, b, e, M, N, K, s);
  else gemm<1, 1, 0, EP_OUT>(a, b, e, M, N, K, s);
  NN_TRY(hipGetLastError());
  return ICR_NN_OK;
}

}  // extern "C"
