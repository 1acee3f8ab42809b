// The device side of the SARA operator (Sec. 5.1), one workgroup's work at a
// time, so that a launch can hold it beside other work: see sara.hip for the
// form and what bounds it.
#pragma once

#include <type_traits>

#include "ppd_internal.h"

namespace ppd {
namespace {

constexpr int TX = 64;                        // analysis tile per sub-band: columns
constexpr int DS = 2 * TX + FILT_STRIDE;      // row stride of its filtered columns in LDS (2 TX + 14, 16-byte rows)
constexpr int DWT_THREADS = 320;              // 2 runs of at most 2 TX + 14 columns
constexpr int SX = 64, SY = 16;               // synthesis tile
constexpr int SP = SY / 2;                    // its coefficient rows per band, without the filter's reach
constexpr int SS = SX / 2 + 8;                // row stride in LDS (SX / 2 + 7 columns, 16-byte rows)
// Window of a low-pass band that a synthesis tile reads, with one row and
// column for its alignment.
constexpr int WROWS = SP + 8, WCOLS = SX / 2 + 8;

// Workgroups a launch must have for analysis tiles of 16 rows; below it tiles
// of 8 rows keep more compute units busy (128 tall tiles: 5.7 us against 5.0;
// 512 tall tiles: 8.6 against 10.4; level 1 at 2048^2, 9216: 82 against 91).
constexpr int DWT_TALL_MIN = 400;

__device__ __host__ inline size_t lvl_size(const SaraGeom& g, int l) { return g.N >> (2 * l); }

enum { A_PLAIN = 0, A_DUAL = 1 };

// The tile (x, y) and basis (z) of workgroup lin of gx gy gz.  Consecutive workgroups
// go round-robin to the XCDs; the tiles are handed out so that each XCD
// takes a contiguous band of them instead, and neighbouring tiles, whose
// staged windows overlap, meet in one L2.  INNER: the bases of a tile are
// consecutive too, so that an XCD reads its band of the image once for all
// of them (level 1 at 2048^2: 97 -> 83 us, at 512^2 11.9 -> 10.5 us).
struct TileId {
  int x, y, z;
  int gx;   // tiles in a row, a power of two
};
template <bool INNER>
__device__ inline TileId sara_tile(int lin, int gx, int gy, int gz) {
  const int total = gx * gy * gz;
  if (total % MAX_XCD == 0) lin = xcd_remap(lin, total);
  if (INNER) return TileId{(lin / gz) % gx, lin / (gz * gx), lin % gz, gx};
  return TileId{lin % gx, (lin / gx) % gy, lin / (gx * gy), gx};
}

// Filters of db-Q: 2Q taps each, low-pass h and high-pass g, in registers
// (the addresses are wave-uniform, so the compiler uses scalar loads).
template <int Q>
__device__ __forceinline__ void load_filt(const float* __restrict__ filt, float (&h)[2 * Q], float (&g)[2 * Q]) {
  const float* b = filt + (Q - 1) * 2 * FILT_STRIDE;
#pragma unroll
  for (int n = 0; n < 2 * Q; ++n) {
    h[n] = b[n];
    g[n] = b[FILT_STRIDE + n];
  }
}

__device__ __forceinline__ float clip_dual(float u, float c, float alpha, float lambda) {
  const float cl = fminf(fmaxf(u + c, -alpha), alpha);
  return u + lambda * (cl - u);
}

// 4 consecutive floats, of which the first n exist; one 16-byte access if vec
// (the address is 16-byte aligned and all 4 exist).
__device__ __forceinline__ void load4(const float* __restrict__ p, bool vec, int n, float (&v)[4]) {
  if (vec) {
    const float4 q = *reinterpret_cast<const float4*>(p);
    v[0] = q.x;
    v[1] = q.y;
    v[2] = q.z;
    v[3] = q.w;
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = i < n ? p[i] : 0.f;
  }
}
__device__ __forceinline__ void store4(float* __restrict__ p, bool vec, int n, const float (&v)[4]) {
  if (vec) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < n) p[i] = v[i];
  }
}

// One analysis level of basis db-Q on one output tile: columns (axis 0), then
// rows (axis 1).  a[k] = sum_n h[n] s[(2k + n) mod L], d[k] likewise with g.
// A column run makes RB outputs of either filter.  HW: there are weights.
template <int Q, int MODE, int RB, bool HW>
__device__ __forceinline__ void dwt_tile(const float* __restrict__ src, int sstride, float scale, int hh, int ww,
                                         int k0y, int k0x, int toy, int tox, const float* __restrict__ filt,
                                         float* s_lo, float* s_hi, float* __restrict__ ub,
                                         const float* __restrict__ wb, int nx, int oh, int ow,
                                         float* __restrict__ llout, float alpha, float lambda, bool vec) {
  constexpr int TAPS = 2 * Q;
  float h[TAPS], g[TAPS];
  load_filt<Q>(filt, h, g);
  const int tid = threadIdx.x;
  // This thread's 4 outputs per sub-band in the row pass: its weights and, in
  // the dual mode, its u values are loaded first, so that they are in flight
  // beside the columns.
  const int G = (tox + 3) >> 2;
  const bool mine = tid < toy * G;
  const int k = mine ? tid / G : 0, m0 = mine ? 4 * (tid - k * G) : 0;
  const int r = k0y + k, c = k0x + m0, nv = tox - m0;
  const size_t pos[4] = {size_t(r) * nx + (ow + c), size_t(oh + r) * nx + c, size_t(oh + r) * nx + (ow + c),
                         size_t(r) * nx + c};
  const int nout = llout ? 3 : 4;
  float uo[4][4], wo[4][4];
  // The weights too, where their latency is not hidden (low tiles are few waves)
  // or where the registers are there (the dual mode's four waves per SIMD: a
  // weighted dual step at 2048^2 293 -> 267 us, 1024^2 77.8 -> 75.1; plain
  // analysis, seven waves before, 115 -> 127).
  constexpr bool AHEAD = HW && (RB == 4 || MODE == A_DUAL);
  if (AHEAD && mine) {
#pragma unroll
    for (int b = 0; b < 4; ++b)
      if (b < nout) load4(wb + pos[b], vec, nv, wo[b]);
  }
  if (MODE == A_DUAL && mine) {
#pragma unroll
    for (int b = 0; b < 4; ++b)
      if (b < nout) load4(ub + pos[b], vec, nv, uo[b]);
  }
  const int IC = 2 * tox + TAPS - 2;
  const int groups = (toy + RB - 1) / RB;
  for (int i = tid; i < IC * groups; i += DWT_THREADS) {
    const int gr = i / IC, cx = i - gr * IC;
    const int col = (2 * k0x + cx) & (ww - 1), r0 = 2 * (k0y + gr * RB);
    float v[2 * RB + TAPS - 2];
#pragma unroll
    for (int a = 0; a < 2 * RB + TAPS - 2; ++a) v[a] = src[size_t((r0 + a) & (hh - 1)) * sstride + col];
#pragma unroll
    for (int a = 0; a < 2 * RB + TAPS - 2; ++a) v[a] *= scale;
#pragma unroll
    for (int q = 0; q < RB; ++q) {
      float lo = 0.f, hi = 0.f;
#pragma unroll
      for (int n = 0; n < TAPS; ++n) {
        lo = fmaf(h[n], v[2 * q + n], lo);
        hi = fmaf(g[n], v[2 * q + n], hi);
      }
      s_lo[(gr * RB + q) * DS + cx] = lo;
      s_hi[(gr * RB + q) * DS + cx] = hi;
    }
  }
  __syncthreads();
  if (!mine) return;
  float cv[4][4];   // lh, hl, hh, ll of the 4 outputs
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    constexpr int NF = (TAPS + 6 + 3) / 4;
    float v[4 * NF];
    const float4* row = reinterpret_cast<const float4*>((half ? s_hi : s_lo) + k * DS + 2 * m0);
#pragma unroll
    for (int n = 0; n < NF; ++n) {
      const float4 q = row[n];
      v[4 * n] = q.x;
      v[4 * n + 1] = q.y;
      v[4 * n + 2] = q.z;
      v[4 * n + 3] = q.w;
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      float a = 0.f, d = 0.f;
#pragma unroll
      for (int n = 0; n < TAPS; ++n) {
        a = fmaf(h[n], v[2 * m + n], a);
        d = fmaf(g[n], v[2 * m + n], d);
      }
      cv[half ? 1 : 3][m] = a;
      cv[half ? 2 : 0][m] = d;
    }
  }
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    if (b >= nout) break;
    float o[4];
    if (HW) {
      if (!AHEAD) load4(wb + pos[b], vec, nv, wo[b]);
#pragma unroll
      for (int m = 0; m < 4; ++m) o[m] = cv[b][m] * wo[b][m];
    } else {
#pragma unroll
      for (int m = 0; m < 4; ++m) o[m] = cv[b][m];
    }
    if (MODE == A_DUAL) {   // the sparsity dual update of Algorithm 3 on the coefficient of Psi^H x~
#pragma unroll
      for (int m = 0; m < 4; ++m) o[m] = clip_dual(uo[b][m], o[m], alpha, lambda);
    }
    store4(ub + pos[b], vec, nv, o);
  }
  if (llout) store4(llout + size_t(r) * ow + c, vec, nv, cv[3]);
}

// Level l of the 8 wavelet bases (tile z = basis - 1); at level 1 the
// Dirac basis is z = 8.  `active` (dual mode, may be NULL) masks
// the bases updated this iteration.  Level 1 reads the image scaled by 1/3,
// deeper levels the low-pass band of the previous level.  vec: every array is
// 16-byte aligned and a level's rows are whole float4s.
template <int MODE, int RB, bool HW>
__device__ __forceinline__ void dwt_block(TileId tl, const float* __restrict__ x, float* __restrict__ tmp,
                                          float* __restrict__ out, const float* __restrict__ filt,
                                          const float* __restrict__ W, const SaraGeom& g, int l, float alpha,
                                          float lambda, const uint8_t* __restrict__ active, int vec) {
  constexpr int TY = 2 * RB;
  static_assert(TY * (TX / 4) <= DWT_THREADS, "one thread per 4 outputs of the tile");
  __shared__ __align__(16) float s_lo[TY * DS];
  __shared__ __align__(16) float s_hi[TY * DS];
  const int hh = g.ny >> (l - 1), ww = g.nx >> (l - 1);
  const int oh = hh >> 1, ow = ww >> 1;
  const int toy = min(TY, oh), tox = min(TX, ow);
  const int k0y = tl.y * toy, k0x = tl.x * tox;
  const int q = tl.z + 1;   // 1..8 wavelets, 9 = Dirac (level 1 only)
  const float third = 1.0f / 3.0f;
  // randomised updates (Algorithm 3 with a random set of bases): an inactive basis keeps
  // its u_i (basis index 0 is the Dirac basis)
  if (active && !active[q == 9 ? 0 : q]) return;
  if (q == 9) {
    // Dirac basis: coefficient x / 3 at every pixel of this tile's footprint,
    // 4 pixels at a time (its rows are 2 tox >= 4 wide: images are at least 16)
    const int F = tox >> 1;
    for (int i = threadIdx.x; i < 2 * toy * F; i += DWT_THREADS) {
      const int a = i / F;
      const size_t P = size_t(2 * k0y + a) * g.nx + (2 * k0x + 4 * (i - a * F));
      float xv[4], wv[4] = {1.f, 1.f, 1.f, 1.f}, uo[4], o[4];
      load4(x + P, vec, 4, xv);
      if (HW) load4(W + P, vec, 4, wv);
      if (MODE == A_DUAL) load4(out + P, vec, 4, uo);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const float c = xv[m] * third * wv[m];
        o[m] = MODE == A_DUAL ? clip_dual(uo[m], c, alpha, lambda) : c;
      }
      store4(out + P, vec, 4, o);
    }
    return;
  }
  const float* src = l == 1 ? x : tmp + g.off[l - 1] + size_t(q - 1) * lvl_size(g, l - 1);
  const int sstride = l == 1 ? g.nx : ww;
  const float scale = l == 1 ? third : 1.0f;
  float* ub = out + size_t(q) * g.N;
  const float* wb = HW ? W + size_t(q) * g.N : nullptr;
  float* llout = l == g.L ? nullptr : tmp + g.off[l] + size_t(q - 1) * lvl_size(g, l);
#define PPD_DWT_CASE(Q)                                                                                       \
  case Q:                                                                                                     \
    dwt_tile<Q, MODE, RB, HW>(src, sstride, scale, hh, ww, k0y, k0x, toy, tox, filt, s_lo, s_hi, ub, wb, g.nx, oh, \
                          ow, llout, alpha, lambda, vec != 0);                                                \
    break;
  switch (q) {
    PPD_DWT_CASE(1) PPD_DWT_CASE(2) PPD_DWT_CASE(3) PPD_DWT_CASE(4)
    PPD_DWT_CASE(5) PPD_DWT_CASE(6) PPD_DWT_CASE(7) PPD_DWT_CASE(8)
  }
#undef PPD_DWT_CASE
}

// Orders the LDS accesses of one wave's lanes (LDS operations of a wave take
// effect in program order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int tile_width(int ww, int gx) { return ww >> (31 - __builtin_clz(gx)); }

// The four sub-bands of one level of one basis in the Mallat layout, periodic,
// with optional weights, and where the low-pass band is read instead if it is
// not LL of u (row stride lls, unweighted).
struct Bands {
  const float* u;    // coefficients of the basis (stride nx)
  const float* w;    // weights or NULL
  const float* ll;   // low-pass band of the level below, or NULL
  int nx, oh, ow, lls;
};

// How a synthesis kernel takes the weights: none, loaded after the values, or
// ahead of them (in flight beside them; weighted synthesis at 2048^2 122 -> 119
// us, 1024 x 512 22.7 -> 21.9).
enum { W_NONE, W_AFTER, W_AHEAD };

// Inverse of one level for basis db-Q on one tile by one wave.  Transposing
// the analysis gives s[2j + e] = sum_t h[2t + e] a[j - t] + g[2t + e] d[j - t],
// e in {0, 1}.  Column pass: the axis-1 low band (from LL, HL) and high band
// (from LH, HH) of 2 SP output rows, at coefficient columns c0 - (Q - 1) + b,
// b < hx + Q - 1, to s_x[band][row][b].  WIN: the low-pass entry at
// coefficient row j0 - (Q - 1) + a, column index b is win[a WCOLS + b].
template <int Q, bool WIN, int WM>
__device__ __forceinline__ void synth_cols(const float (&h)[2 * Q], const float (&g)[2 * Q], const Bands& bd, int j0,
                                           int c0, int hx, const float* win, float* s_x) {
  constexpr int NR = SP + Q - 1;
  const int nb = hx + Q - 1;
  for (int i = threadIdx.x & 63; i < 2 * nb; i += 64) {
    const int band = i >= nb ? 1 : 0, b = i - band * nb;
    const int c = (c0 - (Q - 1) + b) & (bd.ow - 1);
    // row indices in vector registers: as scalars they would take more than there are
    int r0 = j0 - (Q - 1);
    asm volatile("" : "+v"(r0));
    float av[NR], dv[NR];
    int off[NR];
#pragma unroll
    for (int a = 0; a < NR; ++a) off[a] = (r0 + a) & (bd.oh - 1);
    const int cd = bd.oh * bd.nx + band * bd.ow + c, ca = band * bd.ow + c;
    float wd[WM == W_NONE ? 1 : NR], wa[WM == W_NONE ? 1 : NR];
    auto load_weights = [&]() {
      if constexpr (WM != W_NONE) {
#pragma unroll
        for (int a = 0; a < NR; ++a) {
          wd[a] = bd.w[off[a] * bd.nx + cd];
          wa[a] = bd.w[off[a] * bd.nx + ca];
        }
      }
    };
    if (WM == W_AHEAD) load_weights();
#pragma unroll
    for (int a = 0; a < NR; ++a) dv[a] = bd.u[off[a] * bd.nx + cd];
    if constexpr (WIN) {
      if (band) {
#pragma unroll
        for (int a = 0; a < NR; ++a) av[a] = bd.u[off[a] * bd.nx + ca];
      } else {
#pragma unroll
        for (int a = 0; a < NR; ++a) av[a] = win[a * WCOLS + b];
      }
    } else {
      const bool low = bd.ll && !band;
      const float* pa = low ? bd.ll + c : bd.u + ca;
      const int sa = low ? bd.lls : bd.nx;
#pragma unroll
      for (int a = 0; a < NR; ++a) av[a] = pa[off[a] * sa];
    }
    if (WM == W_AFTER) load_weights();
    if constexpr (WM != W_NONE) {
      const bool low = (WIN || bd.ll) && !band;   // an unweighted low-pass band
#pragma unroll
      for (int a = 0; a < NR; ++a) {
        dv[a] *= wd[a];
        av[a] = low ? av[a] : av[a] * wa[a];
      }
    }
    float* dst = s_x + band * (SY * SS) + b;
#pragma unroll
    for (int j = 0; j < SP; ++j) {
      float s0 = 0.f, s1 = 0.f;
#pragma unroll
      for (int t = 0; t < Q; ++t) {
        const float a = av[j - t + Q - 1], d = dv[j - t + Q - 1];
        s0 = fmaf(h[2 * t], a, fmaf(g[2 * t], d, s0));
        s1 = fmaf(h[2 * t + 1], a, fmaf(g[2 * t + 1], d, s1));
      }
      dst[(2 * j) * SS] = s0;
      dst[(2 * j + 1) * SS] = s1;
    }
  }
}

// Row pass: 8 outputs (columns 8 mg ..) of tile row `row`, added to o.
template <int Q>
__device__ __forceinline__ void synth_row8(const float (&h)[2 * Q], const float (&g)[2 * Q], const float* s_x, int row,
                                           int mg, float (&o)[8]) {
  constexpr int NF = (Q + 3 + 3) / 4;
  float lv[4 * NF], hv[4 * NF];
  const float4* lr = reinterpret_cast<const float4*>(s_x + row * SS + 4 * mg);
  const float4* hr = reinterpret_cast<const float4*>(s_x + (SY + row) * SS + 4 * mg);
#pragma unroll
  for (int n = 0; n < NF; ++n) {
    const float4 a = lr[n], d = hr[n];
    lv[4 * n] = a.x;
    lv[4 * n + 1] = a.y;
    lv[4 * n + 2] = a.z;
    lv[4 * n + 3] = a.w;
    hv[4 * n] = d.x;
    hv[4 * n + 1] = d.y;
    hv[4 * n + 2] = d.z;
    hv[4 * n + 3] = d.w;
  }
#pragma unroll
  for (int m = 0; m < 4; ++m)
#pragma unroll
    for (int t = 0; t < Q; ++t) {
      const float a = lv[m - t + Q - 1], d = hv[m - t + Q - 1];
      o[2 * m] = fmaf(h[2 * t], a, fmaf(g[2 * t], d, o[2 * m]));
      o[2 * m + 1] = fmaf(h[2 * t + 1], a, fmaf(g[2 * t + 1], d, o[2 * m + 1]));
    }
}

// 8 floats at p, of which n exist.
__device__ __forceinline__ void store8(float* __restrict__ p, bool vec, int n, const float (&o)[8]) {
  const float a[4] = {o[0], o[1], o[2], o[3]}, b[4] = {o[4], o[5], o[6], o[7]};
  store4(p, vec, n, a);
  store4(p + 4, vec, n - 4, b);
}

// Calls fn(std::integral_constant<int, q>) for basis db-q (wave-uniform).
template <typename Fn>
__device__ __forceinline__ void with_basis(int q, Fn fn) {
  switch (q) {
    case 1: fn(std::integral_constant<int, 1>()); break;
    case 2: fn(std::integral_constant<int, 2>()); break;
    case 3: fn(std::integral_constant<int, 3>()); break;
    case 4: fn(std::integral_constant<int, 4>()); break;
    case 5: fn(std::integral_constant<int, 5>()); break;
    case 6: fn(std::integral_constant<int, 6>()); break;
    case 7: fn(std::integral_constant<int, 7>()); break;
    default: fn(std::integral_constant<int, 8>()); break;
  }
}

// The basis of a wave of the per-basis synthesis launches (workgroup z = 0, 1):
// 1, 8, 3, 6 and 2, 7, 4, 5, the same number of taps in both.
__device__ __forceinline__ int wave_basis(int z) {
  const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  return w == 0 ? 1 + z : w == 1 ? 8 - z : w == 2 ? 3 + z : 6 - z;
}

// Intermediate synthesis level l >= 2 (output = low-pass band of level l-1).
template <int WM>
__device__ __forceinline__ void idwt_block(TileId tl, const float* __restrict__ u, float* __restrict__ rec,
                                           const float* __restrict__ filt, const float* __restrict__ W,
                                           const SaraGeom& g, int l) {
  __shared__ __align__(16) float s_all[4][2 * SY * SS];
  const int hh = g.ny >> (l - 1), ww = g.nx >> (l - 1);
  const int tsy = min(SY, hh), tsx = tile_width(ww, tl.gx), hx = tsx >> 1;
  const int y0 = tl.y * tsy, x0 = tl.x * tsx;
  const int q = wave_basis(tl.z), lane = threadIdx.x & 63;
  float* s_x = s_all[threadIdx.x >> 6];
  const Bands bd{u + size_t(q) * g.N, W ? W + size_t(q) * g.N : nullptr,
                 l == g.L ? nullptr : rec + g.off[l] + size_t(q - 1) * lvl_size(g, l), g.nx, hh >> 1, ww >> 1, ww >> 1};
  float* dst = rec + g.off[l - 1] + size_t(q - 1) * lvl_size(g, l - 1);
  const bool vec = (tsx & 7) == 0;
  with_basis(q, [&](auto ql) {
    constexpr int Q = decltype(ql)::value;
    float h[2 * Q], gf[2 * Q];
    load_filt<Q>(filt, h, gf);
    synth_cols<Q, false, WM>(h, gf, bd, y0 >> 1, x0 >> 1, hx, nullptr, s_x);
    wave_sync();
    const int G = (hx + 3) >> 2;
    for (int i = lane; i < tsy * G; i += 64) {
      const int row = i / G, mg = i - row * G;
      float o[8] = {};
      synth_row8<Q>(h, gf, s_x, row, mg, o);
      store8(dst + size_t(y0 + row) * ww + (x0 + 8 * mg), vec, tsx - 8 * mg, o);
    }
  });
}

// The two coarsest synthesis levels L and L-1 (L >= 3) in one launch: a wave
// first rebuilds, from the level-L coefficients, the window of the level-(L-1)
// low-pass band its level-(L-1) tile reads (periodic, even aligned;
// neighbouring tiles recompute the overlap), keeps it in LDS, then
// synthesises its tile of the level-(L-2) low-pass band.  One launch fewer on
// SARA's chain of dependent launches.
static_assert(WROWS <= SY && WCOLS <= SS && WCOLS / 2 + 7 <= SS, "the window is an inner tile of its own");

template <int WM>
__device__ __forceinline__ void idwt2_block(TileId tl, const float* __restrict__ u, float* __restrict__ rec,
                                            const float* __restrict__ filt, const float* __restrict__ W,
                                            const SaraGeom& g) {
  __shared__ __align__(16) float s_all[4][2 * SY * SS];
  __shared__ __align__(16) float w_all[4][WROWS * WCOLS];
  const int l = g.L - 1;                                      // outer level
  const int hh = g.ny >> (l - 1), ww = g.nx >> (l - 1);
  const int tsy = min(SY, hh), tsx = tile_width(ww, tl.gx), hx = tsx >> 1;
  const int y0 = tl.y * tsy, x0 = tl.x * tsx;
  const int q = wave_basis(tl.z), lane = threadIdx.x & 63;
  float* s_x = s_all[threadIdx.x >> 6];
  float* s_w = w_all[threadIdx.x >> 6];
  const Bands bo{u + size_t(q) * g.N, W ? W + size_t(q) * g.N : nullptr, nullptr, g.nx, hh >> 1, ww >> 1, 0};
  const Bands bi{bo.u, bo.w, nullptr, g.nx, hh >> 2, ww >> 2, 0};
  float* dst = rec + g.off[l - 1] + size_t(q - 1) * lvl_size(g, l - 1);
  const bool vec = (tsx & 7) == 0;
  with_basis(q, [&](auto ql) {
    constexpr int Q = decltype(ql)::value;
    float h[2 * Q], gf[2 * Q];
    load_filt<Q>(filt, h, gf);
    const int j0 = y0 >> 1, c0 = x0 >> 1;
    const int wy0 = j0 - (Q - 1), wx0 = c0 - (Q - 1);         // outer window origin
    const int ya = wy0 - (wy0 & 1), xa = wx0 - (wx0 & 1);     // even-aligned inner tile origin
    const int offy = wy0 - ya, offx = wx0 - xa;
    const int hxi = (hx + Q - 1 + offx + 1) >> 1;             // inner coefficient columns
    // level L: its low-pass band and details are coefficients (in u, weighted)
    synth_cols<Q, false, WM>(h, gf, bi, ya >> 1, xa >> 1, hxi, nullptr, s_x);
    wave_sync();
    const int Gi = (hxi + 3) >> 2;
    for (int i = lane; i < WROWS * Gi; i += 64) {
      const int row = i / Gi, mg = i - row * Gi;
      float o[8] = {};
      synth_row8<Q>(h, gf, s_x, row, mg, o);
      *reinterpret_cast<float4*>(s_w + row * WCOLS + 8 * mg) = make_float4(o[0], o[1], o[2], o[3]);
      *reinterpret_cast<float4*>(s_w + row * WCOLS + 8 * mg + 4) = make_float4(o[4], o[5], o[6], o[7]);
    }
    wave_sync();
    synth_cols<Q, true, WM>(h, gf, bo, j0, c0, hx, s_w + offy * WCOLS + offx, s_x);
    wave_sync();
    const int G = (hx + 3) >> 2;
    for (int i = lane; i < tsy * G; i += 64) {
      const int row = i / G, mg = i - row * G;
      float o[8] = {};
      synth_row8<Q>(h, gf, s_x, row, mg, o);
      store8(dst + size_t(y0 + row) * ww + (x0 + 8 * mg), vec, tsx - 8 * mg, o);
    }
  });
}

// Level 1 for all 8 wavelet bases, plus the Dirac part, times 1/3.  Wave w of
// the workgroup takes bases 8 - w and 1 + w (the same number of taps in every
// wave) on the same tile; their sums are added in wave order.
template <int WM>
__device__ __forceinline__ void idwt_final_block(TileId tl, const float* __restrict__ u, const float* __restrict__ rec,
                                                 const float* __restrict__ filt, const float* __restrict__ W,
                                                 const SaraGeom& g, float* __restrict__ out, int vec) {
  __shared__ __align__(16) float s_all[4][2 * SY * SS];
  static_assert(SY * SX <= 2 * SY * SS, "a wave's sums take the place of its columns");
  constexpr int IPL = SY * (SX / 8) / 64;   // runs of 8 outputs per lane
  const int nx = g.nx, tsx = tile_width(nx, tl.gx), hx = tsx >> 1;   // images are at least 16 x 16
  const int y0 = tl.y * SY, x0 = tl.x * tsx;
  const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), lane = threadIdx.x & 63;
  float* s_x = s_all[w];
  const int j0 = y0 >> 1, c0 = x0 >> 1, G = tsx >> 3;
  float o[IPL][8] = {};
#pragma unroll 1
  for (int part = 0; part < 2; ++part) {
    const int q = part == 0 ? 8 - w : 1 + w;
    const Bands bd{u + size_t(q) * g.N, W ? W + size_t(q) * g.N : nullptr,
                   g.L == 1 ? nullptr : rec + g.off[1] + size_t(q - 1) * lvl_size(g, 1), nx, g.ny >> 1, nx >> 1,
                   nx >> 1};
    with_basis(q, [&](auto ql) {
      constexpr int Q = decltype(ql)::value;
      float h[2 * Q], gf[2 * Q];
      load_filt<Q>(filt, h, gf);
      synth_cols<Q, false, WM>(h, gf, bd, j0, c0, hx, nullptr, s_x);
      wave_sync();
#pragma unroll
      for (int n = 0; n < IPL; ++n) {
        const int i = lane + 64 * n;
        if (i < SY * G) synth_row8<Q>(h, gf, s_x, i / G, i % G, o[n]);
      }
      wave_sync();
    });
  }
  // run i of 8 outputs of every wave at s_x[n][i], n-th of 8 words apart: conflict-free
#pragma unroll
  for (int n = 0; n < IPL; ++n)
#pragma unroll
    for (int k = 0; k < 8; ++k) s_x[k * (64 * IPL) + lane + 64 * n] = o[n][k];
  __syncthreads();
  const float third = 1.0f / 3.0f;
  for (int i = threadIdx.x; i < SY * G * 2; i += 256) {   // 4 outputs each
    const int run = i >> 1, k0 = 4 * (i & 1);
    const size_t P = size_t(y0 + run / G) * nx + (x0 + 8 * (run % G) + k0);
    float d[4], v[4];
    load4(u + P, vec, 4, d);
    if (WM != W_NONE) {
      float wv[4];
      load4(W + P, vec, 4, wv);
#pragma unroll
      for (int k = 0; k < 4; ++k) d[k] *= wv[k];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int a = (k0 + k) * (64 * IPL) + run;
      v[k] = ((((s_all[0][a] + s_all[1][a]) + s_all[2][a]) + s_all[3][a]) + d[k]) * third;
    }
    store4(out + P, vec, 4, v);
  }
}

// A SARA launch as a part of a launch of other work, which never depends on
// it: its workgroups, which take longer, come first.  With small
// images an iteration is two chains of launches that each leave the chip
// nearly empty; run on two streams they cost a captured graph 45 to 50 us of
// host time per iteration (every node of a forked graph is enqueued by
// itself; of a chain, 8 us), so the launches of the two chains are paired
// instead.  Waves beyond the workgroup size of their part end at once.
// HW: the job has weights.
template <bool HW>
__device__ __forceinline__ void sara_dwt_part(const SaraJob& j, int lin) {
  if (threadIdx.x >= DWT_THREADS) return;
  dwt_block<A_DUAL, 4, HW>(sara_tile<true>(lin, j.gx, j.gy, j.gz), j.in, j.tmp, j.out, j.filt, j.W, j.g, j.l, j.alpha,
                           j.lambda, j.active, j.vec);
}
// One synthesis launch: the two coarsest levels, one level, or the last one.
template <int KIND, bool HW>
__device__ __forceinline__ void sara_synth_part(const SaraJob& j, int lin) {
  if (threadIdx.x >= 256) return;
  constexpr int WM = HW ? W_AHEAD : W_NONE;
  const TileId tl = sara_tile<false>(lin, j.gx, j.gy, j.gz);
  if constexpr (KIND == SARA_IDWT2) idwt2_block<WM>(tl, j.in, j.tmp, j.filt, j.W, j.g);
  else if constexpr (KIND == SARA_IDWT) idwt_block<WM>(tl, j.in, j.tmp, j.filt, j.W, j.g, j.l);
  else idwt_final_block<WM>(tl, j.in, j.tmp, j.filt, j.W, j.g, j.out, j.vec);
}

}  // namespace
}  // namespace ppd
