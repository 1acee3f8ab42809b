// Interpolation G and its adjoint (Sec. 2; Sec. 5: 8x8 Kaiser-Bessel
// kernels), with the data-block dual update of Algorithm 3 fused in.
//
// Work item: up to chunk_max visibilities whose first tap lies in one
// T x T grid tile, as per-block segments (at most 64), flattened into one
// range and taken in batches of 64.  The workgroup works on the tile plus
// its 7-cell halo, (T+7)^2 complex cells, in LDS:
//   degrid: the forward spectrum region is copied in, each thread then
//           interpolates its visibilities from LDS (64 taps each);
//   grid:   8 x 8 tiles (the default): the region is one 16 x 16 matrix
//           tile and gridding a product of the separable weights, done on
//           the matrix cores (k_grid_mfma).  Larger tiles: each wave owns
//           private copies of the region; a batch of 64 visibilities is
//           prepared one per lane (weights to LDS), then applied one
//           visibility at a time with lane (a, b) owning tap (a, b), so a
//           wave's 64 read-modify-writes never collide and no atomics are
//           needed (k_grid).  Either way the item's region is stored to a
//           per-item scratch slot; a fold pass then sums, for every grid
//           cell, the slots of the owning tile and the halos of its left /
//           upper / upper-left neighbours.  No global atomics, no zeroing
//           pass, and a fixed summation order across items.
// The 8 per-axis weights are evaluated on the fly from the even and odd
// parts of four degree-9 polynomials (the kernel is even), so only the two
// float32 frequencies are read per visibility.
// Items are launched in spatial order through an XCD-aware remap.
#include <type_traits>

#include "sara_device.h"

namespace ppd {
namespace {

struct Taps {
  int ou, ov;         // first tap relative to the staged region
  bool conj;          // gridded at its mirror frequency: the grid holds the conjugate
  float wx[KB_TAPS];  // u-axis weights
  float wy[KB_TAPS];  // v-axis weights
};

template <int T>
__device__ __forceinline__ void taps_for(float omu, float omv, double su, double sv, int Ky,
                                         int c0, int r0, const float* coef, Taps& t) {
  double tu = double(omu) * su, tv = double(omv) * sv;
  t.conj = mirrored(tu);
  tu = t.conj ? -tu : tu;
  tv = t.conj ? -tv : tv;
  const double fu = floor(tu), fv = floor(tv);
  const int pu0 = int(fu) - 3 + GRID_PAD;
  const int cv0 = (int(fv) - 3) & (Ky - 1);
  t.ou = min(max(pu0 - c0, 0), T - 1);
  t.ov = min(max(cv0 - r0, 0), T - 1);
  kb_weights(float(tu - fu), coef, t.wx);
  kb_weights(float(tv - fv), coef, t.wy);
}

// The coefficients kb_weights reads (taps 0..3), loaded with uniform
// addresses so that they stay in scalar registers (an LDS copy would be
// re-read by every lane for every batch).
struct KbCoef {
  float c[KB_TAPS / 2 * KB_NC];
};
__device__ __forceinline__ void load_kb(const float* __restrict__ kbc, KbCoef& k) {
#pragma unroll
  for (int i = 0; i < KB_TAPS / 2 * KB_NC; ++i) k.c[i] = kbc[i];
}

#ifndef PPD_DEGRID_WAVES
#define PPD_DEGRID_WAVES 4
#endif

// Degridding: one workgroup per item, the region staged in LDS; the item's
// visibilities (all its segments, flattened) are taken in batches of 64, a
// batch per wave in turn, one visibility per lane.  In the dual mode the
// per-segment partials of ||q - y||^2 and ||G a - y||^2 are wave sums over
// the lanes of each segment, added per wave in batch order and summed over
// the waves in a fixed order at the end: deterministic.  (Wave sums by
// permuted operands instead of LDS shuffles: 25.9 -> 22.5 us per dual launch
// at 512^2, 1.3M points.)
// 8 x 8 tiles: the 15 x 15 region is staged twice in LDS with a row stride
// of G8_RS float2 (16-byte aligned rows), copy E holding cell (r, c) at
// r G8_RS + c and copy O holding cell (r, c + 1) there, so that a lane's 8
// consecutive cells of a tap row start at an even float2 of one copy and
// are read as four 16-byte loads (half the LDS instructions of 8-byte
// loads).  The weighted sums run in the same order as the 8-byte form.
constexpr int G8_RS = 18;
constexpr int G8_COPY = 15 * G8_RS;   // float2 per copy

// The 16 x 15 cells a region's 4 column blocks hold are staged two columns at
// a time (16-byte loads, consecutive within a block); pair e is block e / 30,
// row (e mod 30) / 2.  The 16th column is beyond every tap.
constexpr int G8_PAIRS = 4 * 15 * 2;
static_assert(FFT_CB == 4 && GRID_PAD == 8, "a tile's region starts on a column block");

__device__ __forceinline__ float4 load_pair8(const float2* __restrict__ grid, int e, int c0, int r0, int Ky) {
  const int blk = e / 30, w = e - blk * 30;
  return *reinterpret_cast<const float4*>(grid + grid_index(c0 + 4 * blk + 2 * (w & 1), (r0 + (w >> 1)) & (Ky - 1), Ky));
}

__device__ __forceinline__ void stage8(float2* reg2, int e, float4 g) {
  const int blk = e / 30, w = e - blk * 30;
  const int b = 4 * blk + 2 * (w & 1), o = (w >> 1) * G8_RS + b;
  *reinterpret_cast<float4*>(reg2 + o) = g;
  if (b > 0) reg2[G8_COPY + o - 1] = make_float2(g.x, g.y);
  reg2[G8_COPY + o] = make_float2(g.z, g.w);
}

__device__ __forceinline__ float2 gather8(const float2* reg2, const Taps& t) {
  const float2* base = (t.ou & 1) ? reg2 + G8_COPY + t.ov * G8_RS + (t.ou - 1) : reg2 + t.ov * G8_RS + t.ou;
  float ax = 0.f, ay = 0.f;
#pragma unroll
  for (int a = 0; a < KB_TAPS; ++a) {
    const float4* row = reinterpret_cast<const float4*>(base + a * G8_RS);
    const float4 q0 = row[0], q1 = row[1], q2 = row[2], q3 = row[3];
    float sx = 0.f, sy = 0.f;
    sx = fmaf(t.wx[0], q0.x, sx);
    sy = fmaf(t.wx[0], q0.y, sy);
    sx = fmaf(t.wx[1], q0.z, sx);
    sy = fmaf(t.wx[1], q0.w, sy);
    sx = fmaf(t.wx[2], q1.x, sx);
    sy = fmaf(t.wx[2], q1.y, sy);
    sx = fmaf(t.wx[3], q1.z, sx);
    sy = fmaf(t.wx[3], q1.w, sy);
    sx = fmaf(t.wx[4], q2.x, sx);
    sy = fmaf(t.wx[4], q2.y, sy);
    sx = fmaf(t.wx[5], q2.z, sx);
    sy = fmaf(t.wx[5], q2.w, sy);
    sx = fmaf(t.wx[6], q3.x, sx);
    sy = fmaf(t.wx[6], q3.y, sy);
    sx = fmaf(t.wx[7], q3.z, sx);
    sy = fmaf(t.wx[7], q3.w, sy);
    const float wya = a == 0 ? t.wy[0] : a == 1 ? t.wy[1] : a == 2 ? t.wy[2] : a == 3 ? t.wy[3]
                    : a == 4 ? t.wy[4] : a == 5 ? t.wy[5] : a == 6 ? t.wy[6] : t.wy[7];
    ax = fmaf(wya, sx, ax);
    ay = fmaf(wya, sy, ay);
  }
  return make_float2(ax, ay);
}

// NW: waves per workgroup.  8 x 8 tiles hold about two batches, so there an
// item is one wave's work; where the items are too few to fill the chip
// (SHARE_ITEMS) two waves share it.
// MODE: plain (out = Theta G a), the dual update, or the residual
// (out = Theta G a - y, with the item's part of its squared norm: the whole's
// is all that is asked for, and wave sums per segment took 110 us instead of
// the plain mode's 50 at 512^2, 1.3M points in 20000 blocks).
enum { DEGRID_PLAIN = 0, DEGRID_DUAL = 1, DEGRID_RES = 2 };
template <int T, int MODE, int NW>
__device__ __forceinline__ void degrid_block(
    int block, const float2* __restrict__ grid, int PW, int Ky, const Item* __restrict__ items, int n_items,
    const Seg* __restrict__ segs, const float* __restrict__ wu, const float* __restrict__ wv,
    const float* __restrict__ theta, double su, double sv, const float* __restrict__ kbc,
    float2* __restrict__ out, const int32_t* __restrict__ uperm, const float2* __restrict__ y,
    const double* __restrict__ U, const float2* __restrict__ v, const double2* __restrict__ z,
    float2* __restrict__ gout, double mu, double* __restrict__ part, double* __restrict__ rpart, const XcdSplit& xs) {
  constexpr int R = T + 7;
  constexpr bool DUAL = MODE == DEGRID_DUAL, RES = MODE == DEGRID_RES;
  constexpr bool B128 = T == 8;
  __shared__ __align__(16) float2 reg[B128 ? 2 * G8_COPY : R * R];
  __shared__ ItemTab tab;
  __shared__ double s_q[NW][DUAL ? MAX_ITEM_SEGS : 1], s_r[NW][DUAL ? MAX_ITEM_SEGS : 1];
  const int ii = xcd_item(block, xs);
  if (ii < 0 || ii >= n_items) return;
  const Item it = items[ii];
  const int r0 = it.ty * T, c0 = it.tx * T;
  const int lane = threadIdx.x & 63;
  const int uwid = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  // staging: all of the thread's loads are issued before its LDS stores
  constexpr int CELLS = B128 ? G8_PAIRS : R * R;
  constexpr int RPT = (CELLS + 64 * NW - 1) / (64 * NW);
  using Cell = std::conditional_t<B128, float4, float2>;
  Cell gv[RPT];
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int i = threadIdx.x + k * 64 * NW;
    if (i < CELLS) {
      if constexpr (B128) {
        gv[k] = load_pair8(grid, i, c0, r0, Ky);
      } else {
        const int a = i / R, b = i - a * R;
        gv[k] = c0 + b < PW ? grid[grid_index(c0 + b, (r0 + a) & (Ky - 1), Ky)] : make_float2(0.f, 0.f);
      }
    }
  }
  const int nseg = it.seg1 - it.seg0;
  const bool one = nseg == 1;   // uniform
  const int total = it.total;
  if (!one) load_item_tab(it, segs, tab);
  KbCoef kbw;
  load_kb(kbc, kbw);
  if (DUAL)
    for (int i = threadIdx.x; i < NW * MAX_ITEM_SEGS; i += 64 * NW) {
      (&s_q[0][0])[i] = 0.0;
      (&s_r[0][0])[i] = 0.0;
    }
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int i = threadIdx.x + k * 64 * NW;
    if (i < CELLS) {
      if constexpr (B128) stage8(reg, i, gv[k]);
      else reg[i] = gv[k];
    }
  }
  __syncthreads();
  // Batch k of 64 flattened visibilities goes to wave k mod NW; a wave
  // loads its next batch's operands before working on the current one.
  struct Batch {
    float ou, ov, th;
    float2 v, y;
    double2 z;
    double U;
    int pi, sg, sb, po;
  };
  auto load = [&](int bt, int& sb, Batch& b) {
    if (!one)
      while (bt * 64 >= tab.pre[sb + 1]) ++sb;
    b.sb = sb;
    const int li = bt * 64 + lane;
    b.sg = sb;
    if (li < total) {
      if (one) {
        b.pi = it.start + li;
      } else {
        b.sg = seg_of(li, sb, tab.pre);
        b.pi = tab.start[b.sg] + (li - tab.pre[b.sg]);
      }
      b.ou = wu[b.pi];
      b.ov = wv[b.pi];
      b.th = theta ? theta[b.pi] : 1.0f;
      if (DUAL) {
        b.v = v[b.pi];
        b.U = U[b.pi];
        b.z = z[b.pi];
        b.y = y[b.pi];
      } else {
        b.po = uperm ? uperm[b.pi] : b.pi;   // where the caller's order has it
        if (RES) b.y = y[b.pi];
      }
    }
  };
  int sbl = 0;
  double racc = 0.0;   // RES: this lane's squares
  Batch bn{};
  if (uwid * 64 < total) load(uwid, sbl, bn);
  for (int bt = uwid; bt * 64 < total; bt += NW) {
    const Batch cb = bn;
    if ((bt + NW) * 64 < total) load(bt + NW, sbl, bn);
    const int li = bt * 64 + lane;
    const bool act = li < total;
    const int sb = __builtin_amdgcn_readfirstlane(cb.sb), sg = cb.sg, pi = cb.pi;
    double qn = 0.0, rn = 0.0;
    if (act) {
      const float omu = cb.ou, omv = cb.ov, th = cb.th;
      const float2 ve = cb.v, ye = cb.y;
      const double Ue = DUAL ? cb.U : 1.0;
      const double2 ze = cb.z;
      Taps t;
      taps_for<T>(omu, omv, su, sv, Ky, c0, r0, kbw.c, t);
      float ax = 0.f, ay = 0.f;
      if constexpr (B128) {
        const float2 s2 = gather8(reg, t);
        ax = s2.x;
        ay = s2.y;
      } else {
#pragma unroll
        for (int a = 0; a < KB_TAPS; ++a) {
          const float2* row = reg + (t.ov + a) * R + t.ou;
          float sx = 0.f, sy = 0.f;
#pragma unroll
          for (int b = 0; b < KB_TAPS; ++b) {
            const float2 g = row[b];
            sx = fmaf(t.wx[b], g.x, sx);
            sy = fmaf(t.wx[b], g.y, sy);
          }
          const float wya = a == 0 ? t.wy[0] : a == 1 ? t.wy[1] : a == 2 ? t.wy[2] : a == 3 ? t.wy[3]
                          : a == 4 ? t.wy[4] : a == 5 ? t.wy[5] : a == 6 ? t.wy[6] : t.wy[7];
          ax = fmaf(wya, sx, ax);
          ay = fmaf(wya, sy, ay);
        }
      }
      const float2 g = make_float2(ax * th, (t.conj ? -ay : ay) * th);
      if (RES) {
        out[cb.po] = make_float2(g.x - ye.x, g.y - ye.y);
        const double ex = double(g.x) - double(ye.x), ey = double(g.y) - double(ye.y);
        racc += ex * ex + ey * ey;
      } else if (!DUAL) {
        out[cb.po] = g;
      } else {
        // argument of the data-dual update of Algorithm 3: w = U^-1 v + Theta G a (Theta G a kept for the
        // gridding pass, which rebuilds w); first Algorithm 2 step
        gout[pi] = g;
        const double2 we = dual_arg(ve, Ue, g);
        const double wx = we.x, wy = we.y;
        const double mU = mu * Ue;
        const double dx = (ze.x - mU * (ze.x - wx)) - double(ye.x);
        const double dy = (ze.y - mU * (ze.y - wy)) - double(ye.y);
        qn = dx * dx + dy * dy;
        const double ex = double(g.x) - double(ye.x), ey = double(g.y) - double(ye.y);
        rn = ex * ex + ey * ey;
      }
    }
    if (DUAL) {
      const int slast = __builtin_amdgcn_readlane(sg, min(63, total - 1 - bt * 64));
      for (int ss = sb; ss <= slast; ++ss) {
        const double a = part ? wave_sum(act && sg == ss ? qn : 0.0) : 0.0;
        const double r = rpart ? wave_sum(act && sg == ss ? rn : 0.0) : 0.0;
        if (lane == 0) {
          s_q[uwid][ss] += a;
          s_r[uwid][ss] += r;
        }
      }
    }
  }
  if (DUAL) {
    __syncthreads();
    for (int k = threadIdx.x; k < nseg; k += 64 * NW) {
      double q = 0.0, r = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        q += s_q[w][k];
        r += s_r[w][k];
      }
      if (part) part[it.seg0 + k] = q;
      if (rpart) rpart[it.seg0 + k] = r;
    }
  }
  if (RES) {
    racc = wave_sum(racc);
    if (lane == 0) s_r[uwid][0] = racc;
    __syncthreads();
    if (threadIdx.x == 0) {
      double r = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) r += s_r[w][0];
      rpart[ii] = r;
    }
  }
}

template <int T, int MODE, int NW>
__global__ __launch_bounds__(64 * NW) void k_degrid(
    const float2* __restrict__ grid, int PW, int Ky, const Item* __restrict__ items, int n_items,
    const Seg* __restrict__ segs, const float* __restrict__ wu, const float* __restrict__ wv,
    const float* __restrict__ theta, double su, double sv, const float* __restrict__ kbc,
    float2* __restrict__ out, const int32_t* __restrict__ uperm, const float2* __restrict__ y,
    const double* __restrict__ U, const float2* __restrict__ v, const double2* __restrict__ z,
    float2* __restrict__ gout, double mu, double* __restrict__ part, double* __restrict__ rpart, XcdSplit xs) {
  degrid_block<T, MODE, NW>(blockIdx.x, grid, PW, Ky, items, n_items, segs, wu, wv, theta, su, sv, kbc, out, uperm, y, U, v, z, gout, mu, part, rpart, xs);
}

// The shared 8 x 8 items in the dual mode, after an analysis level of SARA in
// the first workgroups.
template <bool HW>
__global__ __launch_bounds__(DWT_THREADS) void k_degrid_dwt(
    const float2* __restrict__ grid, int PW, int Ky, const Item* __restrict__ items, int n_items,
    const Seg* __restrict__ segs, const float* __restrict__ wu, const float* __restrict__ wv,
    const float* __restrict__ theta, double su, double sv, const float* __restrict__ kbc, const float2* __restrict__ y,
    const double* __restrict__ U, const float2* __restrict__ v, const double2* __restrict__ z,
    float2* __restrict__ gout, double mu, double* __restrict__ part, double* __restrict__ rpart, XcdSplit xs,
    SaraJob j) {
  const int b = int(blockIdx.x) - j.blocks();
  if (b < 0)
    sara_dwt_part<HW>(j, blockIdx.x);
  else if (threadIdx.x < 128)
    degrid_block<8, DEGRID_DUAL, 2>(b, grid, PW, Ky, items, n_items, segs, wu, wv, theta, su, sv, kbc,
                                    nullptr, nullptr, y, U, v, z, gout, mu, part, rpart, xs);
}

// Operands of one gridding batch (one visibility per lane), loaded a batch
// ahead of use.
struct GridBatch {
  float ou, ov, th;
  float2 vin, y, v, ga;
  double2 z, bf;
  double U;
  int pi;
  bool act;
};

struct GridSrc {
  const float* wu; const float* wv; const float* theta;
  const float2* vin; const float2* y; const double* U; const float2* v; const double2* z;
  const float2* ga; const double2* bfac; const uint8_t* active;
  const int32_t* uperm;   // plain: vin is in the caller's order (plan -> caller), NULL: in plan order
};

// Loads batch bt (64 flattened visibilities of the item) for this lane;
// sb tracks the segment of the batch's first visibility.  An item of one
// segment (uniform) is found without the table: from `start`, in `block`.
template <bool DUAL>
__device__ __forceinline__ void grid_load(const GridSrc& g, const ItemTab& tab, bool one, int start, int block,
                                          int total, int lane, int bt, int& sb, GridBatch& b) {
  if (!one)
    while (bt * 64 >= tab.pre[sb + 1]) ++sb;
  const int li = bt * 64 + lane;
  if (li < total) {
    int pi = start + li, bk = block;
    if (!one) {
      const int sg = seg_of(li, sb, tab.pre);
      pi = tab.start[sg] + (li - tab.pre[sg]);
      bk = tab.block[sg];
    }
    b.pi = pi;
    b.ou = g.wu[pi];
    b.ov = g.wv[pi];
    b.th = g.theta ? g.theta[pi] : 1.0f;
    if (!DUAL) {
      b.vin = g.vin[g.uperm ? g.uperm[pi] : pi];
    } else {
      b.ga = g.ga[pi];
      b.z = g.z[pi];
      b.U = g.U[pi];
      b.y = g.y[pi];
      b.v = g.v[pi];
      b.bf = g.bfac[bk];
      b.act = !g.active || g.active[bk];
    }
  }
}

// The value a visibility spreads onto the grid (before Theta).  In the dual
// mode: the last Algorithm 2 projection z = P_B(q) with the block's factor
// (or the exact prox with the block's nu), then the dual finish and relaxation; an inactive
// block (randomised updates of Algorithm 3) keeps v and z and spreads its v.
template <bool DUAL>
__device__ __forceinline__ float2 grid_value(const GridBatch& bt, double mu, double lambda, int exact,
                                             double2& znew, float2& vnew) {
  if (!DUAL) return bt.vin;
  if (!bt.act) return bt.v;
  const double2 bw = dual_arg(bt.v, bt.U, bt.ga);   // w of the data-dual update
  double zx, zy;
  if (exact) {
    // exact prox: (U w + nu y) / (U + nu) with the block's nu, w if nu = 0
    const double nu = bt.bf.x, inv = 1.0 / (bt.U + nu);
    zx = nu == 0.0 ? bw.x : (bt.U * bw.x + nu * double(bt.y.x)) * inv;
    zy = nu == 0.0 ? bw.y : (bt.U * bw.y + nu * double(bt.y.y)) * inv;
  } else {
    const double fac = bt.bf.x;
    const bool inside = bt.bf.y != 0.0;
    const double mU = mu * bt.U;
    const double qx = bt.z.x - mU * (bt.z.x - bw.x), qy = bt.z.y - mU * (bt.z.y - bw.y);
    zx = inside ? qx : double(bt.y.x) + (qx - double(bt.y.x)) * fac;
    zy = inside ? qy : double(bt.y.y) + (qy - double(bt.y.y)) * fac;
  }
  znew = make_double2(zx, zy);
  const double vbx = bt.U * (bw.x - zx), vby = bt.U * (bw.y - zy);
  vnew = make_float2(float(double(bt.v.x) + lambda * (vbx - double(bt.v.x))),
                     float(double(bt.v.y) + lambda * (vby - double(bt.v.y))));
  return vnew;
}

// Gridding workgroup shape: NW waves, each owning C private copies of the
// (T+7)^2 region in LDS (rows padded to T+8 cells, so the 8 tap rows of a
// footprint fall in distinct LDS banks).  Visibility k of a batch goes to
// copy k mod C: C independent read-modify-write chains per wave that the
// compiler interleaves (distinct LDS arrays cannot alias).
#ifndef PPD_GRID_CHAINS
#define PPD_GRID_CHAINS 2
#endif
#ifndef PPD_GRID_WAVES16
#define PPD_GRID_WAVES16 2
#endif
template <int T>
struct GridCfg {
  static constexpr int R = T + 7;
  static constexpr int RS = T + 8;
  static constexpr int C = (T <= 32) ? PPD_GRID_CHAINS : 2;
  static constexpr int NW = (T <= 16) ? PPD_GRID_WAVES16 : (T <= 32 ? 2 : 1);
  static constexpr int THREADS = NW * 64;
};

template <int T, bool DUAL>
__global__ __launch_bounds__(GridCfg<T>::THREADS) void k_grid(
    float2* __restrict__ scratch, int Ky, const Item* __restrict__ items, int n_items,
    const Seg* __restrict__ segs, const float* __restrict__ wu, const float* __restrict__ wv,
    const float* __restrict__ theta, double su, double sv, const float* __restrict__ kbc,
    const float2* __restrict__ vin, const int32_t* __restrict__ uperm, const float2* __restrict__ y,
    const double* __restrict__ U,
    float2* __restrict__ v, double2* __restrict__ z, const double2* zin, const float2* __restrict__ ga, double mu,
    double lambda, const double2* __restrict__ bfac, int exact, const uint8_t* __restrict__ active,
    XcdSplit xs) {
  constexpr int R = GridCfg<T>::R;
  constexpr int RS = GridCfg<T>::RS;
  constexpr int C = GridCfg<T>::C;
  constexpr int NW = GridCfg<T>::NW;
  __shared__ float2 acc[NW][C][R * RS];
  constexpr int WXS = KB_TAPS + 1;             // staging stride per visibility (bank spread)
  __shared__ float2 wxv[NW][64 * WXS];         // wx[b] * value, per visibility of the batch
  __shared__ float wyb[NW][64 * WXS];          // wy[a]
  __shared__ ItemTab tab;
  const int ii = xcd_item(blockIdx.x, xs);
  if (ii < 0 || ii >= n_items) return;
  const Item it = items[ii];
  const int r0 = it.ty * T, c0 = it.tx * T;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int uwid = __builtin_amdgcn_readfirstlane(wid);   // wave-uniform
  load_item_tab(it, segs, tab);
  for (int i = threadIdx.x; i < NW * C * R * RS; i += blockDim.x) (&acc[0][0][0])[i] = make_float2(0.f, 0.f);
  KbCoef kbw;
  load_kb(kbc, kbw);
  __syncthreads();
  float2 (*myacc)[R * RS] = acc[wid];
  float2* mywxv = wxv[wid];
  float* mywy = wyb[wid];
  const int ta = lane >> 3, tb = lane & 7;   // tap of this lane in the apply phase
  const int lofs = ta * RS + tb;
  // The item's visibilities (all segments, flattened) are taken in batches
  // of 64, batch k by wave k mod NW.  The global operands of a wave's next
  // batch are loaded before its current batch is prepared and applied, so
  // their latency overlaps the LDS work.
  const GridSrc src{wu, wv, theta, vin, y, U, v, zin ? zin : z, ga, bfac, active, uperm};
  const int nseg = it.seg1 - it.seg0;
  const int total = tab.pre[nseg];
  int sb = 0;
  GridBatch bn{};
  if (uwid * 64 < total) grid_load<DUAL>(src, tab, false, 0, 0, total, lane, uwid, sb, bn);
  for (int k = uwid; k * 64 < total; k += NW) {
    const GridBatch bt = bn;
    if ((k + NW) * 64 < total) grid_load<DUAL>(src, tab, false, 0, 0, total, lane, k + NW, sb, bn);
    const int nb = min(64, total - k * 64);
    // prepare: one visibility per lane (lanes past nb carry zero weight).
    // The new z and v are stored after the apply loop, so that no store is
    // in flight (and waited for) while the loop runs.
    double2 znew{};
    float2 vnew{};
    int pos = 0;
    float vx = 0.f, vy = 0.f;
    Taps t;
    if (lane < nb) {
      taps_for<T>(bt.ou, bt.ov, su, sv, Ky, c0, r0, kbw.c, t);
      const float2 val = grid_value<DUAL>(bt, mu, lambda, exact, znew, vnew);
      vx = val.x * bt.th;
      vy = (t.conj ? -val.y : val.y) * bt.th;
      pos = t.ov * RS + t.ou;
    } else {
#pragma unroll
      for (int m = 0; m < KB_TAPS; ++m) {
        t.wx[m] = 0.f;
        t.wy[m] = 0.f;
      }
    }
#pragma unroll
    for (int m = 0; m < KB_TAPS; ++m) {
      mywxv[lane * WXS + m] = make_float2(t.wx[m] * vx, t.wx[m] * vy);
      mywy[lane * WXS + m] = t.wy[m];
    }
    __builtin_amdgcn_wave_barrier();
    // apply: lane (a, b) owns tap (a, b) of one visibility at a time, so
    // the wave's 64 read-modify-writes touch distinct cells (LDS float
    // atomics are far slower on this part, collisions or not).
    // C visibilities per step, visibility k into copy k mod C: C independent
    // read-modify-write chains.  (Summing runs of visibilities that share a
    // first-tap cell in registers before one read-modify-write per run was
    // measured slower: the data-dependent loop costs more than it saves.)
    const int nbc = (nb + C - 1) / C * C;
    for (int k = 0; k < nbc; k += C) {
      int pc[C];
      float2 xc[C], cc[C];
      float gc[C];
#pragma unroll
      for (int j = 0; j < C; ++j) {
        pc[j] = __builtin_amdgcn_readlane(pos, k + j) + lofs;
        xc[j] = mywxv[(k + j) * WXS + tb];
        gc[j] = mywy[(k + j) * WXS + ta];
        cc[j] = myacc[j][pc[j]];
      }
#pragma unroll
      for (int j = 0; j < C; ++j) {
        cc[j].x = fmaf(gc[j], xc[j].x, cc[j].x);
        cc[j].y = fmaf(gc[j], xc[j].y, cc[j].y);
        myacc[j][pc[j]] = cc[j];
      }
    }
    __builtin_amdgcn_wave_barrier();
    if (DUAL && lane < nb && bt.act) {
      z[bt.pi] = znew;
      v[bt.pi] = vnew;
    }
  }
  __syncthreads();
  float2* dst = scratch + size_t(ii) * (R * R);
  for (int i = threadIdx.x; i < R * R; i += blockDim.x) {
    const int ra = i / R, li = ra * RS + (i - ra * R);
    float sx = 0.f, sy = 0.f;
#pragma unroll
    for (int q2 = 0; q2 < NW; ++q2)
#pragma unroll
      for (int j = 0; j < C; ++j) {
        sx += acc[q2][j][li].x;
        sy += acc[q2][j][li].y;
      }
    dst[i] = make_float2(sx, sy);
  }
}

// Gridding of 8 x 8 tiles as a matrix product on the matrix cores.  The
// item's region (15 x 15 cells, padded to 16 x 16) receives
//     G[i][j] = sum_k wy_k(i) * (wx_k(j) * theta_k * val_k),
// wy_k(i) the v-axis weight of visibility k at region row i (zero outside
// its 8 taps), wx_k(j) likewise along u: a 16 x 16 x K product of the
// separable weights, accumulated over the item's visibilities 4 at a time by
// v_mfma_f32_16x16x4_f32 (real and imaginary parts), in FP32 registers.  A
// batch of 64 visibilities is prepared one per lane, as in k_grid, and its
// taps are written into 16-entry LDS rows that are zero elsewhere: weight
// rows (the A operand) and value-scaled weight rows (B), 32 rows at a time;
// lane l of a product step then reads row 4 g + l / 16, entry l mod 16, of
// each.  No read-modify-write of LDS.
//
// A single-wave workgroup takes one item; the operands of its next batch are
// loaded before the current batch is prepared and applied.  (Runs of 2 items
// per wave in one pipeline were 37.5 against 36.6 us at 512^2, 1.3M points,
// and 12.2 against 8.6 at 256^2, 65536: with the items' first segments in
// their records there is little left to hide, and fewer waves.)  Where the
// items are too few to fill the chip (SHARE_ITEMS), two waves alternate an
// item's batches and their partial regions are added at the end.
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int GM_T = 8;
constexpr int GM_AS = 17;   // A row stride (floats): spreads the prepare writes over banks
constexpr int GM_BS = 17;   // B row stride (float2)

// Lane l holds rows 4 (l / 16) + e, e = 0..3, of column l mod 16 (row 15 and
// column 15 stay zero: no footprint reaches them).
__device__ __forceinline__ void store_region(f32x4 sr, f32x4 si, float2* __restrict__ dst, int gq, int gc) {
  constexpr int R = GM_T + 7;
  if (gc < R)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (4 * gq + e < R) dst[(4 * gq + e) * R + gc] = make_float2(sr[e], si[e]);
}

template <bool DUAL, int NW>
__device__ __forceinline__ void grid_mfma_block(
    int block, float2* __restrict__ scratch, int Ky, const Item* __restrict__ items, int n_items,
    const Seg* __restrict__ segs, const float* __restrict__ wu, const float* __restrict__ wv,
    const float* __restrict__ theta, double su, double sv, const float* __restrict__ kbc,
    const float2* __restrict__ vin, const int32_t* __restrict__ uperm, const float2* __restrict__ y,
    const double* __restrict__ U,
    float2* __restrict__ v, double2* __restrict__ z, const double2* zin, const float2* __restrict__ ga, double mu,
    double lambda, const double2* __restrict__ bfac, int exact, const uint8_t* __restrict__ active,
    const XcdSplit& xs) {
  constexpr int T = GM_T, R = T + 7;
  static_assert(R <= 16, "the region must fit one 16 x 16 product tile");
  __shared__ float sAw[NW][32 * GM_AS];
  __shared__ __align__(16) float2 sBw[NW][32 * GM_BS];
  __shared__ ItemTab tab;
  const int ii = xcd_item(block, xs);
  if (ii < 0 || ii >= n_items) return;
  const Item it = items[ii];
  const int wid = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), lane = threadIdx.x & 63;
  const int c0 = it.tx * T, r0 = it.ty * T, total = it.total;
  float* sA = sAw[wid];
  float2* sB = sBw[wid];
  const int gq = lane >> 4, gc = lane & 15;   // row-in-group and entry read in a product step
  const GridSrc src{wu, wv, theta, vin, y, U, v, zin ? zin : z, ga, bfac, active, uperm};
  const bool one = it.seg1 - it.seg0 == 1;
  if (!one) {
    load_item_tab(it, segs, tab);
    __syncthreads();
  }
  int sb = 0;
  GridBatch bn{};
  if (wid * 64 < total) grid_load<DUAL>(src, tab, one, it.start, it.block, total, lane, wid, sb, bn);
  KbCoef kbw;
  load_kb(kbc, kbw);
  f32x4 accr = {0.f, 0.f, 0.f, 0.f}, acci = {0.f, 0.f, 0.f, 0.f};
  f32x4 accr2 = {0.f, 0.f, 0.f, 0.f}, acci2 = {0.f, 0.f, 0.f, 0.f};
  float* arow = sA + (lane & 31) * GM_AS;
  float2* brow = sB + (lane & 31) * GM_BS;
  const float* aq = sA + gq * GM_AS + gc;    // entry read by this lane in product step 0
  const float2* bq = sB + gq * GM_BS + gc;
  // the staging rows start zero; each batch writes its taps and clears them
  for (int e = lane; e < 32 * GM_AS; e += 64) sA[e] = 0.f;
  for (int e = lane; e < 32 * GM_BS; e += 64) sB[e] = make_float2(0.f, 0.f);
  __builtin_amdgcn_wave_barrier();
  for (int kb = wid; kb * 64 < total; kb += NW) {
    const int nb = min(64, total - kb * 64);
    // this batch's taps and values, from the operands loaded during the
    // previous one; bn is free again afterwards
    double2 znew{};
    float2 vnew{};
    float vx = 0.f, vy = 0.f;
    Taps t;
    t.ou = 0;
    t.ov = 0;
    const bool has = lane < nb;
    const int pi = bn.pi;
    const bool zst = DUAL && has && bn.act;
    if (has) {
      taps_for<T>(bn.ou, bn.ov, su, sv, Ky, c0, r0, kbw.c, t);
      const float2 val = grid_value<DUAL>(bn, mu, lambda, exact, znew, vnew);
      vx = val.x * bn.th;
      vy = (t.conj ? -val.y : val.y) * bn.th;
    }
    // stores before the next batch's loads: vector memory operations
    // complete in issue order, so the wait for those loads does not add a
    // wait for stores issued after them
    if (zst) {
      z[pi] = znew;
      v[pi] = vnew;
    }
    if ((kb + NW) * 64 < total)
      grid_load<DUAL>(src, tab, one, it.start, it.block, total, lane, kb + NW, sb, bn);
    // The batch goes through LDS in two halves of 32 rows (half the staging
    // memory: more waves per CU): lanes 0-31 write their 8 taps into rows
    // that are otherwise zero and the first 8 product steps read them, the
    // lanes put the zeros back, then the same for lanes 32-63.  Rows of
    // lanes past the batch end are never written.  The tap stores go to a
    // per-lane base with constant offsets; LDS operations of one wave take
    // effect in program order, so the zeros land after the product reads.
    float* pa = arow + t.ov;
    float2* pb = brow + t.ou;
    for (int h = 0; h * 32 < nb; ++h) {
      const bool mine = has && (lane >> 5) == h;
      if (mine) {
#pragma unroll
        for (int m = 0; m < KB_TAPS; ++m) {
          pa[m] = t.wy[m];
          pb[m] = make_float2(t.wx[m] * vx, t.wx[m] * vy);
        }
      }
      __builtin_amdgcn_wave_barrier();
      // the operands of RA product steps are read before their first product
      // (rows past the batch end read as zero; 4 or 8 steps cost 1.5 us at
      // 512^2 and 15 at 2048^2 in registers and so in waves); two accumulator
      // pairs (even / odd steps) make independent chains
      constexpr int RA = 2;
      const int ng = (min(32, nb - 32 * h) + 3) >> 2;
#pragma unroll
      for (int g0 = 0; g0 < 8; g0 += RA) {
        float a8[RA];
        float2 b8[RA];
#pragma unroll
        for (int g = 0; g < RA; ++g) {
          a8[g] = aq[4 * (g0 + g) * GM_AS];
          b8[g] = bq[4 * (g0 + g) * GM_BS];
        }
#pragma unroll
        for (int g = 0; g < RA; g += 2) {
          if (g0 + g < ng) {
            accr = __builtin_amdgcn_mfma_f32_16x16x4f32(a8[g], b8[g].x, accr, 0, 0, 0);
            acci = __builtin_amdgcn_mfma_f32_16x16x4f32(a8[g], b8[g].y, acci, 0, 0, 0);
          }
          if (g0 + g + 1 < ng) {
            accr2 = __builtin_amdgcn_mfma_f32_16x16x4f32(a8[g + 1], b8[g + 1].x, accr2, 0, 0, 0);
            acci2 = __builtin_amdgcn_mfma_f32_16x16x4f32(a8[g + 1], b8[g + 1].y, acci2, 0, 0, 0);
          }
        }
      }
      __builtin_amdgcn_wave_barrier();
      if (mine) {
#pragma unroll
        for (int m = 0; m < KB_TAPS; ++m) {
          pa[m] = 0.f;
          pb[m] = make_float2(0.f, 0.f);
        }
      }
    }
  }
  float2* dst = scratch + size_t(ii) * (R * R);
  f32x4 sr = accr + accr2, si = acci + acci2;
  if constexpr (NW == 2) {
    // the second wave's region through its staging memory, whose products are done
    f32x4* s = reinterpret_cast<f32x4*>(sBw[1]);
    static_assert(sizeof(sBw[1]) >= 128 * sizeof(f32x4), "room for two accumulators");
    if (wid == 1) {
      s[lane] = sr;
      s[64 + lane] = si;
    }
    __syncthreads();
    if (wid == 1) return;
    sr += s[lane];
    si += s[64 + lane];
  }
  store_region(sr, si, dst, gq, gc);
}

// ZIN: the dual mode's iterate is read from zin (two scalar registers that cost the
// plain iteration 0.4 us in 34 at 512^2, 1.3M points).
template <bool DUAL, int NW, bool ZIN = false>
__global__ __launch_bounds__(64 * NW) void k_grid_mfma(
    float2* __restrict__ scratch, int Ky, const Item* __restrict__ items, int n_items,
    const Seg* __restrict__ segs, const float* __restrict__ wu, const float* __restrict__ wv,
    const float* __restrict__ theta, double su, double sv, const float* __restrict__ kbc,
    const float2* __restrict__ vin, const int32_t* __restrict__ uperm, const float2* __restrict__ y,
    const double* __restrict__ U,
    float2* __restrict__ v, double2* __restrict__ z, const double2* zin, const float2* __restrict__ ga, double mu,
    double lambda, const double2* __restrict__ bfac, int exact, const uint8_t* __restrict__ active,
    XcdSplit xs) {
  grid_mfma_block<DUAL, NW>(blockIdx.x, scratch, Ky, items, n_items, segs, wu, wv, theta, su, sv, kbc, vin, uperm, y, U,
                            v, z, ZIN ? zin : nullptr, ga, mu, lambda, bfac, exact, active, xs);
}

// The shared items in the dual mode, after a synthesis launch of SARA in the
// first workgroups.
template <int KIND, bool HW>
__global__ __launch_bounds__(256) void k_grid_synth(
    float2* __restrict__ scratch, int Ky, const Item* __restrict__ items, int n_items, const Seg* __restrict__ segs,
    const float* __restrict__ wu, const float* __restrict__ wv, const float* __restrict__ theta, double su, double sv,
    const float* __restrict__ kbc, const float2* __restrict__ y, const double* __restrict__ U, float2* __restrict__ v,
    double2* __restrict__ z, const double2* zin, const float2* __restrict__ ga, double mu, double lambda,
    const double2* __restrict__ bfac, int exact, const uint8_t* __restrict__ active, XcdSplit xs, SaraJob j) {
  const int b = int(blockIdx.x) - j.blocks();
  if (b < 0)
    sara_synth_part<KIND, HW>(j, blockIdx.x);
  else if (threadIdx.x < 128)
    grid_mfma_block<true, 2>(b, scratch, Ky, items, n_items, segs, wu, wv, theta, su, sv, kbc, nullptr,
                             nullptr, y, U, v, z, zin, ga, mu, lambda, bfac, exact, active, xs);
}

// One thread per grid cell (FOLD_CELLS cells per workgroup, T*T/FOLD_CELLS
// workgroups per tile); the item loops are unrolled so their independent
// loads overlap.
constexpr int FOLD_CELLS = 256;

// Sums of the regions of up to FOLD_GROUP consecutive items of a tile, into the
// first one's: a dense centre puts thousands of items into a few tiles, and a
// fold's threads would add them up one after the other.  Bound by the loads'
// latency, all of a thread's at once.  Phi^H at 512^2, 1.3M points normal about
// the centre, with and without groups, us: standard deviation 0.06 rad (1359
// items in a tile) 52 and 129, 0.02 rad (5858) 56 and 232; tiles of 16 at 0.06
// rad (993) 88 and 227, of 32 (1562) 123 and 304, of 64 (1575) 428 and 601.
// Cells are independent, so the sums take their first region's place.
template <int T>
__global__ __launch_bounds__(FOLD_CELLS) void k_fold_groups(float2* __restrict__ scratch,
                                                            const int2* __restrict__ groups) {
  constexpr int R2 = (T + 7) * (T + 7), PARTS = (R2 + FOLD_CELLS - 1) / FOLD_CELLS;
  const int g = blockIdx.x / PARTS, c = (blockIdx.x - g * PARTS) * FOLD_CELLS + threadIdx.x;
  if (c >= R2) return;
  const int2 e = groups[g];
  float2* r = scratch + size_t(e.x) * R2 + c;
  float2 v[FOLD_GROUP];
#pragma unroll
  for (int k = 0; k < FOLD_GROUP; ++k) v[k] = k < e.y ? r[k * R2] : make_float2(0.f, 0.f);
#pragma unroll
  for (int w = FOLD_GROUP / 2; w > 0; w >>= 1)
#pragma unroll
    for (int k = 0; k < w; ++k) v[k] = make_float2(v[k].x + v[k + w].x, v[k].y + v[k + w].y);
  r[0] = v[0];
}

// Items between the regions that a tile of n items is summed from.
template <bool GROUPED>
__device__ __forceinline__ int fold_step(int n) {
  return GROUPED && n > FOLD_GROUP ? FOLD_GROUP : 1;
}

template <bool GROUPED>
__device__ __forceinline__ void fold_items(const float2* __restrict__ scratch, int R2, int off, int i0,
                                           int i1, float& sx, float& sy) {
  const int st = fold_step<GROUPED>(i1 - i0);
  int i = i0;
  for (; i + 3 * st < i1; i += 4 * st) {
    const float2 g0 = scratch[size_t(i) * R2 + off];
    const float2 g1 = scratch[size_t(i + st) * R2 + off];
    const float2 g2 = scratch[size_t(i + 2 * st) * R2 + off];
    const float2 g3 = scratch[size_t(i + 3 * st) * R2 + off];
    sx += (g0.x + g1.x) + (g2.x + g3.x);
    sy += (g0.y + g1.y) + (g2.y + g3.y);
  }
  for (; i < i1; i += st) {
    const float2 g = scratch[size_t(i) * R2 + off];
    sx += g.x;
    sy += g.y;
  }
}

template <int T, bool GROUPED>
__global__ __launch_bounds__(FOLD_CELLS) void k_fold(const float2* __restrict__ scratch,
                                                     const int32_t* __restrict__ tio, int tiles_x,
                                                     int tiles_y, int PW, int Ky, float2* __restrict__ grid) {
  constexpr int R = T + 7;
  constexpr int PARTS = (T * T) / FOLD_CELLS;
  static_assert(PARTS >= 1 && T > 7, "whole workgroups per tile; a cell lies in at most 4 tile regions");
  const int wg = xcd_remap(blockIdx.x, gridDim.x);
  if (wg >= tiles_x * tiles_y * PARTS) return;
  const int t = wg / PARTS, part = wg - t * PARTS;
  const int tx = t % tiles_x, ty = t / tiles_x;
  const int lx = (tx + tiles_x - 1) % tiles_x, uy = (ty + tiles_y - 1) % tiles_y;
  const int tl = ty * tiles_x + lx, tu = uy * tiles_x + tx, tul = uy * tiles_x + lx;
  const int c = part * FOLD_CELLS + threadIdx.x;
  const int a = c / T, b = c - a * T;
  float sx = 0.f, sy = 0.f;
  fold_items<GROUPED>(scratch, R * R, a * R + b, tio[t], tio[t + 1], sx, sy);
  if (b < 7) fold_items<GROUPED>(scratch, R * R, a * R + T + b, tio[tl], tio[tl + 1], sx, sy);
  if (a < 7) {
    fold_items<GROUPED>(scratch, R * R, (T + a) * R + b, tio[tu], tio[tu + 1], sx, sy);
    if (b < 7) fold_items<GROUPED>(scratch, R * R, (T + a) * R + T + b, tio[tul], tio[tul + 1], sx, sy);
  }
  if (tx * T + b < PW) grid[grid_index(tx * T + b, ty * T + a, Ky)] = make_float2(sx, sy);
}

// What one cell receives from its four source tiles: the regions i0[q],
// i0[q] + STRIDE st[q], .. < i1[q] (wave-uniform; st: fold_step) at off[q] where
// ok[q], four at a time and the rest one by one.  All that remains of a source after whole fours
// is loaded before anything is added: most tiles have one to three regions, and
// their four sources together then cost one load's latency, not four to twelve.
// Bound by that latency at small sizes and by the regions' bytes at large ones:
// 64^2 .. 256^2 5.2 -> 3.9 us; 512^2, 1.3M points 10.7 -> 9.6; 2048^2, 6M points,
// beside SARA 117 -> 76 (236 MB of regions in, 67 MB out).  Regions stored as
// four 512-byte quadrants, so that both sides move whole lines, were no faster
// (10.0 and 78), nor eight loads in flight for the heavy tiles.
template <int STRIDE, bool GROUPED>
__device__ __forceinline__ float2 fold_sources(const float2* __restrict__ scratch, int R2, const int (&off)[4],
                                               const bool (&ok)[4], const int (&i0)[4], const int (&i1)[4],
                                               const int (&st)[4]) {
  float2 g[4][3];
  int n[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int step = GROUPED ? STRIDE * st[q] : STRIDE;
    n[q] = max(0, (i1[q] - i0[q] + step - 1) / step);
    const int i = i0[q] + step * (n[q] & ~3);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      g[q][k] = make_float2(0.f, 0.f);
      if ((n[q] & 3) > k && ok[q]) g[q][k] = scratch[size_t(i + step * k) * R2 + off[q]];
    }
  }
  float sx = 0.f, sy = 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (n[q] >= 4 && ok[q]) {
      const int step = GROUPED ? STRIDE * st[q] : STRIDE;
      for (int k = 0; k + 4 <= n[q]; k += 4) {
        const float2* r = scratch + size_t(i0[q] + step * k) * R2 + off[q];
        const float2 g0 = r[0], g1 = r[step * R2], g2 = r[2 * step * R2], g3 = r[3 * step * R2];
        sx += (g0.x + g1.x) + (g2.x + g3.x);
        sy += (g0.y + g1.y) + (g2.y + g3.y);
      }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if ((n[q] & 3) > k && ok[q]) {
        sx += g[q][k].x;
        sy += g[q][k].y;
      }
  }
  return make_float2(sx, sy);
}

// 8 x 8 tiles, 4-wave workgroups in the plan's fold order (tile rows spread
// over the XCDs, on each XCD the tiles with the most item regions first).
// Entry {t0, t1, t2, t3} folds up to four light tiles, one per wave, one
// thread per cell; entry {t, -2, -2, -2} folds one heavy tile (more than
// FOLD_HEAVY regions to sum: the dense centre of the coverage), wave w
// summing every fourth item region of each source tile from the w-th, the
// four partial sums then added in wave order.
template <bool GROUPED>
__device__ __forceinline__ void fold8_block(int block, int nblocks, const float2* __restrict__ scratch,
                                            const int32_t* __restrict__ tio, const int4* __restrict__ wgs,
                                            int tiles_x, int tiles_y, int Ky, float2* __restrict__ grid) {
  constexpr int T = 8, R = T + 7;
  __shared__ float2 part[4][64];
  const int4 e = wgs[xcd_remap(block, nblocks)];
  const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), c = threadIdx.x & 63;
  const int a = c / T, b = c - a * T;
  const bool heavy = e.y == -2;   // uniform over the workgroup
  const int t = heavy ? e.x : (w == 0 ? e.x : w == 1 ? e.y : w == 2 ? e.z : e.w);
  if (t < 0) return;              // never taken by a heavy workgroup
  const int tx = t % tiles_x, ty = t / tiles_x;
  const int lx = (tx + tiles_x - 1) % tiles_x, uy = (ty + tiles_y - 1) % tiles_y;
  const int src[4] = {t, ty * tiles_x + lx, uy * tiles_x + tx, uy * tiles_x + lx};
  const int off[4] = {a * R + b, a * R + T + b, (T + a) * R + b, (T + a) * R + T + b};
  const bool ok[4] = {true, b < 7, a < 7, a < 7 && b < 7};
  int i0[4], i1[4], st[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    i0[q] = tio[src[q]];
    i1[q] = tio[src[q] + 1];
    st[q] = fold_step<GROUPED>(i1[q] - i0[q]);
    i0[q] += heavy ? w * st[q] : 0;
  }
  if (!heavy) {
    grid[grid_index(tx * T + b, ty * T + a, Ky)] = fold_sources<1, GROUPED>(scratch, R * R, off, ok, i0, i1, st);
    return;
  }
  part[w][c] = fold_sources<4, GROUPED>(scratch, R * R, off, ok, i0, i1, st);
  __syncthreads();
  if (w == 0) {
    const float2 p0 = part[0][c], p1 = part[1][c], p2 = part[2][c], p3 = part[3][c];
    grid[grid_index(tx * T + b, ty * T + a, Ky)] =
        make_float2(((p0.x + p1.x) + p2.x) + p3.x, ((p0.y + p1.y) + p2.y) + p3.y);
  }
}

__global__ __launch_bounds__(256) void k_fold8(const float2* __restrict__ scratch, const int32_t* __restrict__ tio,
                                                const int4* __restrict__ wgs, int tiles_x, int tiles_y, int Ky,
                                                float2* __restrict__ grid) {
  fold8_block<false>(blockIdx.x, gridDim.x, scratch, tio, wgs, tiles_x, tiles_y, Ky, grid);
}
__global__ __launch_bounds__(256) void k_fold8_grouped(const float2* __restrict__ scratch,
                                                       const int32_t* __restrict__ tio,
                                                       const int4* __restrict__ wgs, int tiles_x, int tiles_y, int Ky,
                                                       float2* __restrict__ grid) {
  fold8_block<true>(blockIdx.x, gridDim.x, scratch, tio, wgs, tiles_x, tiles_y, Ky, grid);
}

// The same after a synthesis launch of SARA in the first workgroups.
template <int KIND, bool HW, bool GROUPED>
__global__ __launch_bounds__(256) void k_fold8_synth(int nblocks, const float2* __restrict__ scratch,
                                                     const int32_t* __restrict__ tio, const int4* __restrict__ wgs,
                                                     int tiles_x, int tiles_y, int Ky, float2* __restrict__ grid,
                                                     SaraJob j) {
  const int b = int(blockIdx.x) - j.blocks();
  if (b < 0) sara_synth_part<KIND, HW>(j, blockIdx.x);
  else fold8_block<GROUPED>(b, nblocks, scratch, tio, wgs, tiles_x, tiles_y, Ky, grid);
}

template <typename E>
__global__ void k_permute(const int32_t* __restrict__ perm, int64_t M, int to_user,
                          const E* __restrict__ in, E* __restrict__ out) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < M; i += int64_t(gridDim.x) * blockDim.x) {
    if (to_user) out[perm[i]] = in[i];
    else out[i] = in[perm[i]];
  }
}


template <int T, int NW>
int launch_degrid(ppd_plan* p, int mode, float2* out, const int32_t* uperm, const float2* y, const DualArgs* a,
                  double* part_out) {
  if (mode == DEGRID_RES) {
    hipLaunchKernelGGL((k_degrid<T, DEGRID_RES, NW>), dim3(p->split1.launch), dim3(64 * NW), 0, p->stream, p->grid_f,
                       p->PW, p->Ky, p->items, p->n_items, p->segs, p->wu, p->wv, p->theta, p->su_scale, p->sv_scale,
                       p->kbc, out, nullptr, y, nullptr, nullptr, nullptr, nullptr, 0.0, nullptr, p->rpart, p->split1);
  } else if (mode == DEGRID_PLAIN) {
    hipLaunchKernelGGL((k_degrid<T, DEGRID_PLAIN, NW>), dim3(p->split1.launch), dim3(64 * NW), 0, p->stream, p->grid_f, p->PW,
                       p->Ky, p->items, p->n_items, p->segs, p->wu, p->wv, p->theta, p->su_scale, p->sv_scale, p->kbc,
                       out, uperm, nullptr, nullptr, nullptr, nullptr, nullptr, 0.0, nullptr, nullptr, p->split1);
  } else {
    hipLaunchKernelGGL((k_degrid<T, DEGRID_DUAL, NW>), dim3(p->split1.launch), dim3(64 * NW), 0, p->stream, p->grid_f, p->PW,
                       p->Ky, p->items, p->n_items, p->segs, p->wu, p->wv, p->theta, p->su_scale, p->sv_scale, p->kbc,
                       nullptr, nullptr, a->y, a->U, a->v, a->z, p->gabuf, a->mu, part_out, a->rpart, p->split1);
  }
  PPD_HIP(hipGetLastError());
  return PPD_OK;
}

template <int NW>
int launch_grid_mfma(ppd_plan* p, bool dual, const float2* vin, const int32_t* uperm, const DualArgs* a, int exact) {
  const XcdSplit& xs = p->split1;
  if (!dual) {
    hipLaunchKernelGGL((k_grid_mfma<false, NW>), dim3(xs.launch), dim3(64 * NW), 0, p->stream, p->gscratch, p->Ky,
                       p->items, p->n_items, p->segs, p->wu, p->wv, p->theta, p->su_scale, p->sv_scale, p->kbc, vin,
                       uperm, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0.0, 0.0, nullptr, 0, nullptr, xs);
  } else {
    hipLaunchKernelGGL((a->zin ? k_grid_mfma<true, NW, true> : k_grid_mfma<true, NW>), dim3(xs.launch), dim3(64 * NW), 0, p->stream, p->gscratch, p->Ky,
                       p->items, p->n_items, p->segs, p->wu, p->wv, p->theta, p->su_scale, p->sv_scale, p->kbc,
                       nullptr, nullptr, a->y, a->U, a->v, a->z, a->zin, p->gabuf, a->mu, a->lambda, p->bfac,
                       exact, a->active, xs);
  }
  PPD_HIP(hipGetLastError());
  return PPD_OK;
}

template <int T>
int launch_grid(ppd_plan* p, bool dual, const float2* vin, const int32_t* uperm, const DualArgs* a, int exact) {
  if (!dual) {
    hipLaunchKernelGGL((k_grid<T, false>), dim3(p->split1.launch), dim3(GridCfg<T>::THREADS), 0, p->stream,
                       p->gscratch, p->Ky, p->items, p->n_items, p->segs, p->wu, p->wv, p->theta, p->su_scale,
                       p->sv_scale, p->kbc, vin, uperm, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0.0,
                       0.0, nullptr, 0, nullptr, p->split1);
  } else {
    hipLaunchKernelGGL((k_grid<T, true>), dim3(p->split1.launch), dim3(GridCfg<T>::THREADS), 0, p->stream,
                       p->gscratch, p->Ky, p->items, p->n_items, p->segs, p->wu, p->wv, p->theta, p->su_scale,
                       p->sv_scale, p->kbc, nullptr, nullptr, a->y, a->U, a->v, a->z, a->zin, p->gabuf,
                       a->mu, a->lambda, p->bfac, exact, a->active, p->split1);
  }
  PPD_HIP(hipGetLastError());
  return PPD_OK;
}

// The sums of the groups, where the plan has any.
int fold_groups(ppd_plan* p) {
  if (!p->n_fold_groups) return PPD_OK;
  auto launch = [&](auto kernel, int T) {
    const int parts = ((T + 7) * (T + 7) + FOLD_CELLS - 1) / FOLD_CELLS;
    hipLaunchKernelGGL(kernel, dim3(p->n_fold_groups * parts), dim3(FOLD_CELLS), 0, p->stream, p->gscratch,
                       reinterpret_cast<const int2*>(p->fold_groups));
  };
  switch (p->T) {
    case 8: launch(k_fold_groups<8>, 8); break;
    case 16: launch(k_fold_groups<16>, 16); break;
    case 32: launch(k_fold_groups<32>, 32); break;
    default: launch(k_fold_groups<64>, 64); break;
  }
  PPD_HIP(hipGetLastError());
  return PPD_OK;
}

template <int T>
int launch_fold(ppd_plan* p) {
  const int n = p->n_tiles * ((T * T) / FOLD_CELLS);
  const int nl = ((n + MAX_XCD - 1) / MAX_XCD) * MAX_XCD;
  hipLaunchKernelGGL((p->n_fold_groups ? k_fold<T, true> : k_fold<T, false>), dim3(nl), dim3(FOLD_CELLS), 0, p->stream, p->gscratch,
                     p->tile_item_off, p->tiles_x, p->tiles_y, p->PW, p->Ky, p->grid_a);
  PPD_HIP(hipGetLastError());
  return PPD_OK;
}

int launch_fold8(ppd_plan* p) {
  hipLaunchKernelGGL(p->n_fold_groups ? k_fold8_grouped : k_fold8, dim3(p->n_fold_wg), dim3(256), 0, p->stream, p->gscratch, p->tile_item_off,
                     reinterpret_cast<const int4*>(p->fold_wg), p->tiles_x, p->tiles_y, p->Ky, p->grid_a);
  PPD_HIP(hipGetLastError());
  return PPD_OK;
}

int dispatch_degrid(ppd_plan* p, int mode, float2* out, const int32_t* uperm, const float2* y, const DualArgs* a,
                    double* part_out) {
  int slot;
  PPD_TRY(timer_begin(p, KK_DEGRID, &slot));
  int st;
  switch (p->T) {
    case 8:
      st = p->n_items <= SHARE_ITEMS ? launch_degrid<8, 2>(p, mode, out, uperm, y, a, part_out)
                                     : launch_degrid<8, 1>(p, mode, out, uperm, y, a, part_out);
      break;
    case 16: st = launch_degrid<16, PPD_DEGRID_WAVES>(p, mode, out, uperm, y, a, part_out); break;
    case 32: st = launch_degrid<32, PPD_DEGRID_WAVES>(p, mode, out, uperm, y, a, part_out); break;
    default: st = launch_degrid<64, PPD_DEGRID_WAVES>(p, mode, out, uperm, y, a, part_out); break;
  }
  PPD_TRY(st);
  return timer_end(p, slot);
}

int dispatch_grid(ppd_plan* p, bool dual, const float2* vin, const int32_t* uperm, const DualArgs* a, int exact) {
  int slot;
  PPD_TRY(timer_begin(p, KK_GRID, &slot));
  int st;
  switch (p->T) {
    case 8:
      st = p->n_items <= SHARE_ITEMS ? launch_grid_mfma<2>(p, dual, vin, uperm, a, exact)
                                     : launch_grid_mfma<1>(p, dual, vin, uperm, a, exact);
      break;
    case 16: st = launch_grid<16>(p, dual, vin, uperm, a, exact); break;
    case 32: st = launch_grid<32>(p, dual, vin, uperm, a, exact); break;
    default: st = launch_grid<64>(p, dual, vin, uperm, a, exact); break;
  }
  PPD_TRY(st);
  return timer_end(p, slot);
}

}  // namespace

int degrid_plain(ppd_plan* p, float2* out, const int32_t* uperm) {
  return dispatch_degrid(p, DEGRID_PLAIN, out, uperm, nullptr, nullptr, nullptr);
}
int degrid_dual(ppd_plan* p, const DualArgs& a, double* part_out, const SaraJob* with) {
  if (with) {
    hipLaunchKernelGGL((with->W ? k_degrid_dwt<true> : k_degrid_dwt<false>), dim3(p->split1.launch + with->blocks()), dim3(DWT_THREADS), 0, p->stream,
                       p->grid_f, p->PW, p->Ky, p->items, p->n_items, p->segs, p->wu, p->wv, p->theta, p->su_scale,
                       p->sv_scale, p->kbc, a.y, a.U, a.v, a.z, p->gabuf, a.mu, part_out, a.rpart, p->split1, *with);
    PPD_HIP(hipGetLastError());
    return PPD_OK;
  }
  return dispatch_degrid(p, DEGRID_DUAL, nullptr, nullptr, nullptr, &a, part_out);
}
int degrid_residual(ppd_plan* p, const float2* y, float2* out) {
  return dispatch_degrid(p, DEGRID_RES, out, nullptr, y, nullptr, nullptr);
}

int grid_plain(ppd_plan* p, const float2* v, const int32_t* uperm) {
  PPD_TRY(dispatch_grid(p, false, v, uperm, nullptr, 0));
  return fold_grid(p);
}

int grid_dual(ppd_plan* p, const DualArgs& a, const double* part_in) {
  PPD_TRY(block_factors(p, part_in));
  PPD_TRY(dispatch_grid(p, true, nullptr, nullptr, &a, 0));
  return fold_grid(p);
}

int grid_dual_paired(ppd_plan* p, const DualArgs& a, int exact, const SaraJob* with, const SaraJob* with_fold) {
  if (!with) {
    PPD_TRY(dispatch_grid(p, true, nullptr, nullptr, &a, exact));
    return fold_grid(p, with_fold);
  }
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(p->split1.launch + with->blocks()), dim3(256), 0, p->stream, p->gscratch, p->Ky,
                       p->items, p->n_items, p->segs, p->wu, p->wv, p->theta, p->su_scale, p->sv_scale, p->kbc, a.y,
                       a.U, a.v, a.z, a.zin, p->gabuf, a.mu, a.lambda, p->bfac, exact, a.active, p->split1,
                       *with);
  };
  if (with->kind == SARA_IDWT2) launch(with->W ? k_grid_synth<SARA_IDWT2, true> : k_grid_synth<SARA_IDWT2, false>);
  else launch(with->W ? k_grid_synth<SARA_IDWT, true> : k_grid_synth<SARA_IDWT, false>);
  PPD_HIP(hipGetLastError());
  return fold_grid(p, with_fold);
}

int grid_dual_factored(ppd_plan* p, const DualArgs& a) {
  PPD_TRY(dispatch_grid(p, true, nullptr, nullptr, &a, 0));
  return fold_grid(p);
}

int grid_dual_exact(ppd_plan* p, const DualArgs& a) {
  PPD_TRY(dispatch_grid(p, true, nullptr, nullptr, &a, 1));
  return fold_grid(p);
}

int fold_grid(ppd_plan* p, const SaraJob* with) {
  if (with) {
    PPD_TRY(fold_groups(p));
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(p->n_fold_wg + with->blocks()), dim3(256), 0, p->stream, p->n_fold_wg,
                         p->gscratch, p->tile_item_off, reinterpret_cast<const int4*>(p->fold_wg), p->tiles_x,
                         p->tiles_y, p->Ky, p->grid_a, *with);
    };
    auto choose = [&](auto grouped) {
      constexpr bool G = decltype(grouped)::value;
      if (with->kind == SARA_IDWT)
        launch(with->W ? k_fold8_synth<SARA_IDWT, true, G> : k_fold8_synth<SARA_IDWT, false, G>);
      else
        launch(with->W ? k_fold8_synth<SARA_FINAL, true, G> : k_fold8_synth<SARA_FINAL, false, G>);
    };
    if (p->n_fold_groups) choose(std::true_type());
    else choose(std::false_type());
    PPD_HIP(hipGetLastError());
    return PPD_OK;
  }
  int slot;
  PPD_TRY(timer_begin(p, KK_FOLD, &slot));
  PPD_TRY(fold_groups(p));
  int st;
  switch (p->T) {
    case 8: st = launch_fold8(p); break;
    case 16: st = launch_fold<16>(p); break;
    case 32: st = launch_fold<32>(p); break;
    default: st = launch_fold<64>(p); break;
  }
  PPD_TRY(st);
  return timer_end(p, slot);
}

int permute(ppd_plan* p, int direction, const void* in, void* out, int elem_bytes) {
  int slot;
  PPD_TRY(timer_begin(p, KK_PERMUTE, &slot));
  const int to_user = direction == PPD_PLAN_TO_USER;
  const int blocks = int(std::min<int64_t>((p->M + 255) / 256, 4096));
  switch (elem_bytes) {
    case 4:
      hipLaunchKernelGGL(k_permute<float>, dim3(blocks), dim3(256), 0, p->stream, p->perm, p->M,
                         to_user, static_cast<const float*>(in), static_cast<float*>(out));
      break;
    case 8:
      hipLaunchKernelGGL(k_permute<float2>, dim3(blocks), dim3(256), 0, p->stream, p->perm, p->M,
                         to_user, static_cast<const float2*>(in), static_cast<float2*>(out));
      break;
    default:
      hipLaunchKernelGGL(k_permute<double2>, dim3(blocks), dim3(256), 0, p->stream, p->perm, p->M,
                         to_user, static_cast<const double2*>(in), static_cast<double2*>(out));
      break;
  }
  PPD_HIP(hipGetLastError());
  return timer_end(p, slot);
}

}  // namespace ppd

using namespace ppd;

// Whether the caller's order takes a permutation pass of its own.  A tile's
// points come from up to d blocks, a cache line of each per-visibility array from
// each block; neighbouring tiles use the lines again while they are in an XCD's
// 4 MB of L2.  With more than 8192 blocks the operator's arrays, the permutation
// and the scattered values no longer fit.  Phi and Phi^H through the permutation
// and with the pass, us: 512^2, 1.3M points in 8192 blocks 46 and 47, 73 and 74
// (sorted by radius), in 16384 55 and 50, 81 and 78, interleaved 76 and 63, 106 and
// 93; 1024^2, 3M in 32768 142 and 111, 198 and 173.  At 600000 points 35 and 36, 53
// and 53, interleaved 44 and 39, 64 and 59; fewer points than that are so few a
// block that the lines stay: 250000 in 16384 26 and 28, 40 and 41.
static bool permutes_apart(const ppd_plan* p) { return p->d > 8192 && p->M > (int64_t(1) << 19); }

extern "C" int ppd_phi(ppd_plan* p, const float* x, float* y, int order) {
  if (!p || !x || !y) return fail(PPD_EINVAL, "ppd_phi: NULL argument");
  if (order != PPD_ORDER_PLAN && order != PPD_ORDER_USER) return fail(PPD_EINVAL, "ppd_phi: bad order");
  PPD_TRY(fft_forward(p, x));
  if (order == PPD_ORDER_USER && permutes_apart(p)) {
    PPD_TRY(degrid_plain(p, p->ybuf));
    return permute(p, PPD_PLAN_TO_USER, p->ybuf, y, sizeof(float2));
  }
  // in the caller's order the degridding stores through the permutation
  return degrid_plain(p, reinterpret_cast<float2*>(y), order == PPD_ORDER_USER ? p->perm : nullptr);
}

extern "C" int ppd_phit(ppd_plan* p, const float* y, float* x, int order) {
  if (!p || !x || !y) return fail(PPD_EINVAL, "ppd_phit: NULL argument");
  if (order != PPD_ORDER_PLAN && order != PPD_ORDER_USER) return fail(PPD_EINVAL, "ppd_phit: bad order");
  if (order == PPD_ORDER_USER && permutes_apart(p)) {
    PPD_TRY(permute(p, PPD_USER_TO_PLAN, y, p->ybuf, sizeof(float2)));
    PPD_TRY(grid_plain(p, p->ybuf));
  } else {
    PPD_TRY(grid_plain(p, reinterpret_cast<const float2*>(y), order == PPD_ORDER_USER ? p->perm : nullptr));
  }
  return fft_adjoint(p, x);
}
