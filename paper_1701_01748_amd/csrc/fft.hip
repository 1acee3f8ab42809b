// Oversampled 2D FFT of the measurement operator (Sec. 2: F Z and
// Z^H F^H), complex float32, one row or column per group of threads with the
// sequence in registers.
//
// The image is real, so its spectrum is Hermitian and only the grid columns
// c = 0 .. Kx/2 are transformed (half the transforms and half the bytes of a
// complex transform).  Forward: two image rows, deapodised and zero-padded
// into their wrapped position, are the real and imaginary part of one
// sequence of length Kx; the two spectra are separated and the columns
// c < Kx/2 stored.  Columns 0 and Kx/2 of a real row are real, so they share
// one stored column (real part: column 0, imaginary part: column Kx/2).
// Every stored column is then transformed from its ny non-zero entries; the
// grid keeps 8 more columns on either side (see GRID_PAD), copies of their
// mirror images.  Adjoint: the mirrored columns are added back as the columns
// are loaded, full inverse column transforms keep the ny rows the image
// needs, then two rows at a time are transformed back, the deapodisation
// undone and the real part kept -- in iterations fused with the primal update
// of Algorithm 3 and the next forward row pass.
//
// A transform of length L runs on P = L / E threads with E elements each:
// thread t holds elements t + P n.  A DFT over n in registers, twiddles, an
// exchange through LDS, and more such stages leave thread t with outputs
// t + P m: the input's distribution, so global accesses of consecutive threads
// are consecutive on both sides and an inverse transform is followed by a
// forward one without another exchange.  The padding half of an input or
// output is never computed: it is a fixed set of a thread's elements.
// Twiddles are computed in float64 on the host, in the order the threads read
// them (fft_twiddles).
//
// What bounds the passes is the latency of their load - exchange - store chain
// at small sizes and HBM, beside the SARA launches, at large ones.  Measured in
// the iteration against the earlier radix-2 pairs in LDS over the full complex
// grid (rocprofv3, median us per launch; rows: inverse, primal update and
// forward): 64^2 columns 4.7 -> 3.6 and 5.4 -> 3.0, rows 6.9 -> 4.2; 512^2
// columns 9.0 -> 4.8 and 8.7 -> 4.8, rows 9.8 -> 6.8; 2048^2 columns
// 343 -> 151 and 160 -> 103, rows 92 -> 40.
#include "sara_device.h"

namespace ppd {
namespace {

// Which product is fused is written out, so that a transform rounds the same
// in every kernel it is compiled into.
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(fmaf(a.x, b.x, -(a.y * b.y)), fmaf(a.y, b.x, a.x * b.y));
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 conjf2(float2 a) { return make_float2(a.x, -a.y); }
// a times W_4 = -i (forward) or +i (inverse)
template <bool INV>
__device__ __forceinline__ float2 rot4(float2 a) {
  return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}
template <bool INV>
__device__ __forceinline__ float2 twmul(float2 a, float2 w) {
  return cmul(a, INV ? conjf2(w) : w);
}

template <bool INV>
__device__ __forceinline__ void dft4(float2& a0, float2& a1, float2& a2, float2& a3) {
  const float2 s0 = cadd(a0, a2), s1 = csub(a0, a2), s2 = cadd(a1, a3), s3 = rot4<INV>(csub(a1, a3));
  a0 = cadd(s0, s2);
  a1 = cadd(s1, s3);
  a2 = csub(s0, s2);
  a3 = csub(s1, s3);
}

// W_16^k for the k = j s that occur (j, s <= 3)
template <int K>
__device__ __forceinline__ float2 w16() {
  constexpr float C1 = 0.92387953251128675613f, S1 = 0.38268343236508977173f, H = 0.70710678118654752440f;
  if constexpr (K == 0) return make_float2(1.f, 0.f);
  else if constexpr (K == 1) return make_float2(C1, -S1);
  else if constexpr (K == 2) return make_float2(H, -H);
  else if constexpr (K == 3) return make_float2(S1, -C1);
  else if constexpr (K == 4) return make_float2(0.f, -1.f);
  else if constexpr (K == 6) return make_float2(-H, -H);
  else return make_float2(-C1, S1);   // 9
}

// DFT of N = 2, 4, 8 or 16 registers, natural order in and out.  HALF: the
// middle half of the input (indices N/4 .. 3N/4) is zero and not read.
template <int N, bool INV, bool HALF>
__device__ __forceinline__ void dft(float2* x) {
  if constexpr (N == 2) {
    const float2 a = x[0], b = x[1];
    x[0] = cadd(a, b);
    x[1] = csub(a, b);
  } else if constexpr (N == 4 && !HALF) {
    dft4<INV>(x[0], x[1], x[2], x[3]);
  } else {
    // x[j + R s] -> X[s' + 4 j']: 4-point DFTs over s, twiddles, R-point DFTs over j
    constexpr int R = N / 4;
    float2 y[4][R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if constexpr (HALF) {
        const float2 a = x[j], b = rot4<INV>(x[j + 3 * R]);   // the two others are zero
        y[0][j] = cadd(x[j], x[j + 3 * R]);
        y[1][j] = csub(a, b);
        y[2][j] = csub(x[j], x[j + 3 * R]);
        y[3][j] = cadd(a, b);
      } else {
        float2 a0 = x[j], a1 = x[j + R], a2 = x[j + 2 * R], a3 = x[j + 3 * R];
        dft4<INV>(a0, a1, a2, a3);
        y[0][j] = a0;
        y[1][j] = a1;
        y[2][j] = a2;
        y[3][j] = a3;
      }
    }
    if constexpr (R == 2) {
      y[1][1] = twmul<INV>(y[1][1], w16<2>());
      y[2][1] = rot4<INV>(y[2][1]);
      y[3][1] = twmul<INV>(y[3][1], w16<6>());
    } else if constexpr (R == 4) {
      y[1][1] = twmul<INV>(y[1][1], w16<1>());
      y[1][2] = twmul<INV>(y[1][2], w16<2>());
      y[1][3] = twmul<INV>(y[1][3], w16<3>());
      y[2][1] = twmul<INV>(y[2][1], w16<2>());
      y[2][2] = rot4<INV>(y[2][2]);
      y[2][3] = twmul<INV>(y[2][3], w16<6>());
      y[3][1] = twmul<INV>(y[3][1], w16<3>());
      y[3][2] = twmul<INV>(y[3][2], w16<6>());
      y[3][3] = twmul<INV>(y[3][3], w16<9>());
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if constexpr (R > 1) dft<R, INV, false>(y[s]);
#pragma unroll
      for (int j = 0; j < R; ++j) x[s + 4 * j] = y[s][j];
    }
  }
}

// A transform of length L with E elements per thread and S sequences
// interleaved element by element in LDS (columns; 1 for rows).  Stage i turns
// A[k][n], k < K, n < M (K M = L), into A[k + K k1][n2]: DFTs of radix R over
// n1, n = n2 + (M / R) n1, times exp(-2 pi i n2 k1 / M).  All radices are E but
// the last, L's remainder.  Thread t takes the DFTs (k, n2) numbered t + P a
// with n2 fastest, so its first inputs and last outputs are elements t + P m.
template <int L, int E_, int S>
struct Fft {
  static constexpr int E = E_, P = L / E;
  static constexpr int radix(int M) { return M > E ? E : M; }
  // Exchange before the stage at (K, M): A[k][n] at k (M + pad) + n, before the
  // last stage at n (K + pad) + k; the padding (elements) spreads the strided
  // side over the 16 8-byte words a cycle of LDS serves.
  static constexpr bool last(int M) { return M <= E; }
  static constexpr int pad(int M) {
    if (last(M)) return M * S < 16 ? 16 / (M * S) : 1;
    const int run = M / radix(M);   // consecutive elements a stage's threads read
    return run * S < 16 ? run : 0;
  }
  static constexpr int stride(int M) { return last(M) ? L / M + pad(M) : M + pad(M); }
  static constexpr int lds_from(int M) {   // largest exchange from the one before the stage at M on
    const int n = last(M) ? M * stride(M) : (L / M) * stride(M);
    const int rest = last(M) ? 0 : lds_from(M / radix(M));
    return n > rest ? n : rest;
  }
  static constexpr int ONE = lds_from(L / E);
  // Two buffers in turn save the barrier between an exchange's reads and the
  // next one's writes, where they leave room for a second workgroup.
  static constexpr bool TWO = !last(L / E) && 2 * ONE * S * int(sizeof(float2)) <= FFT_TWO_LDS;
  static constexpr int LDS = (TWO ? 2 : 1) * ONE;   // elements per sequence
  static_assert(E >= 4 && L >= 2 * E, "at least two stages, a first radix of 4 or more");
  static_assert(LDS * S >= L, "room for the mirror exchanges");
  static constexpr int twiddles_from(int M) { return last(M) ? 0 : (radix(M) - 1) * (M / radix(M)) + twiddles_from(M / radix(M)); }
  static constexpr int stages_from(int M) { return last(M) ? 1 : 1 + stages_from(M / radix(M)); }
  static constexpr int NW = (E - 1) * (stages_from(L) - 1);

  float2 w[NW];   // this thread's twiddles (forward sign), stage by stage

  template <int M, int I>
  __device__ __forceinline__ void load_from(const float2* __restrict__ tw, int t) {
    if constexpr (!last(M)) {
      constexpr int Q = M / E;
#pragma unroll
      for (int k = 0; k < E - 1; ++k) w[I + k] = tw[k * Q + t % Q];
      load_from<Q, I + E - 1>(tw + (E - 1) * Q, t);
    }
  }
  __device__ __forceinline__ void load_twiddles(const float2* __restrict__ tw, int t) { load_from<L, 0>(tw, t); }

  template <bool INV, bool HALF, int M, int I, int B>
  __device__ __forceinline__ void stage(float2 (&x)[E], int t, float2* s) const {
    constexpr int R = radix(M), K = L / M, SETS = E / R;
    float2* buf = s + (TWO ? B * ONE * S : 0);
    if constexpr (last(M)) {
      float2 y[R];
#pragma unroll
      for (int a = 0; a < SETS; ++a) {
#pragma unroll
        for (int q = 0; q < R; ++q) y[q] = buf[(q * stride(M) + t + P * a) * S];
        dft<R, INV, false>(y);
#pragma unroll
        for (int q = 0; q < R; ++q) x[a + SETS * q] = y[q];
      }
    } else {
      constexpr int Q = M / E;   // the next stage's M
      const int k0 = t / Q, n2 = t % Q;
      if constexpr (M < L) {
#pragma unroll
        for (int q = 0; q < E; ++q) x[q] = buf[(k0 * stride(M) + n2 + Q * q) * S];
      }
      dft<E, INV, HALF && M == L>(x);
#pragma unroll
      for (int k = 1; k < E; ++k) x[k] = twmul<INV>(x[k], w[I + k - 1]);
      constexpr int NB = M < L ? 1 - B : 0;
      float2* out = s + (TWO ? NB * ONE * S : 0);
      if constexpr (M < L && !TWO) __syncthreads();
#pragma unroll
      for (int k = 0; k < E; ++k) {
        const int kk = k0 + K * k;
        out[(last(Q) ? n2 * stride(Q) + kk : kk * stride(Q) + n2) * S] = x[k];
      }
      __syncthreads();
      stage<INV, HALF, Q, I + E - 1, NB>(x, t, s);
    }
  }

  // x[n] = element t + P n in; x[m] = output t + P m out.  s: this
  // sequence's first LDS element (stride S); every thread of the workgroup
  // calls it, and the LDS may be overwritten only after a barrier.
  template <bool INV, bool HALF>
  __device__ __forceinline__ void run(float2 (&x)[E], int t, float2* s) const {
    stage<INV, HALF, L, 0, 0>(x, t, s);
  }
};

// Rows: pairs of image rows per workgroup (one wave's worth of threads, or
// one pair where a pair takes more).
template <int L>
struct RowCfg {
  using F = Fft<L, FftShape<L>::ROW_E, 1>;
  static constexpr int NS = F::P < 64 ? 64 / F::P : 1;
  static constexpr int THREADS = NS * F::P;
};

// Columns: FFT_CB columns per workgroup, more where they take less than a wave.
template <int L>
struct ColCfg {
  static constexpr int E = FftShape<L>::COL_E;
  static constexpr int C = FftShape<L>::COL_C * (L / E) < 64 ? 64 / (L / E) : FftShape<L>::COL_C;
  using F = Fft<L, E, C>;
  static constexpr int THREADS = C * F::P;
  static_assert(C >= 2 && C <= 16, "a workgroup's columns divide Kx / 2 >= 16; two hold the staged mirror column");
};

// Spectra of the two rows of a packed sequence: x[m] = Z(t + P m), the rows'
// entries k < L/2 to the row-pass buffer (columns 0 and L/2 share column 0).
template <int L>
__device__ __forceinline__ void store_pair(const float2* x, int t, float2* s, int row, int ny, bool ok,
                                           float2* __restrict__ half) {
  using F = typename RowCfg<L>::F;
  constexpr int E = F::E, P = F::P, H = L / 2;
  __syncthreads();
#pragma unroll
  for (int m = E / 2; m < E; ++m) s[t + P * m - H] = x[m];
  __syncthreads();
  if (!ok) return;
#pragma unroll
  for (int m = 0; m < E / 2; ++m) {
    const int k = t + P * m;
    const float2 z = x[m], w = s[k == 0 ? 0 : H - k];   // Z(k), Z(L - k); Z(L/2) for k = 0
    float2 a, b;
    if (m == 0 && k == 0) {
      a = make_float2(z.x, w.x);
      b = make_float2(z.y, w.y);
    } else {
      a = make_float2(0.5f * (z.x + w.x), 0.5f * (z.y - w.y));
      b = make_float2(0.5f * (z.y + w.y), 0.5f * (w.x - z.x));
    }
    float2* dst = half + half_index(k, row, ny);
    dst[0] = a;
    dst[FFT_CB] = b;
  }
}

// Image column of sequence index n = t + P m for the elements m outside the
// padding (the middle half): c = (n + nx / 2) mod L, nx = L / 2.
template <int L>
__device__ __forceinline__ int pixel_of(int n) {
  return (n + L / 4) & (L - 1);
}

// Forward rows: image rows 2 i, 2 i + 1 -> row-pass buffer.
template <int L>
__global__ __launch_bounds__(RowCfg<L>::THREADS) void k_fft_rows_fwd(const float* __restrict__ x,
                                                                     const float* __restrict__ dpx,
                                                                     const float* __restrict__ dpy,
                                                                     const float2* __restrict__ tw, int ny,
                                                                     float2* __restrict__ half) {
  using F = typename RowCfg<L>::F;
  constexpr int E = F::E, P = F::P, NX = L / 2;
  __shared__ float2 sm[RowCfg<L>::NS * F::LDS];
  const int t = threadIdx.x % P, q = threadIdx.x / P;
  const int row = 2 * (blockIdx.x * RowCfg<L>::NS + q);
  const bool ok = row < ny;
  F f;
  f.load_twiddles(tw, t);
  float2 z[E];
#pragma unroll
  for (int m = 0; m < E; ++m) {
    if (m >= E / 4 && m < 3 * E / 4) continue;
    const int c = pixel_of<L>(t + P * m);
    z[m] = make_float2(0.f, 0.f);
    if (ok) {
      const float d = dpx[c];
      z[m] = make_float2(x[size_t(row) * NX + c] * d * dpy[row], x[size_t(row + 1) * NX + c] * d * dpy[row + 1]);
    }
  }
  float2* s = sm + q * F::LDS;
  f.template run<false, true>(z, t, s);
  store_pair<L>(z, t, s, row, ny, ok, half);
}

// Forward columns: stored columns 4 g .. -> grid, with the mirror images that
// the padding columns hold.
template <int L>
__device__ __forceinline__ void cols_fwd_block(int block, int nblocks, const float2* __restrict__ half,
                                               const float2* __restrict__ tw, int Hx, int ngroups,
                                               float2* __restrict__ grid) {
  using F = typename ColCfg<L>::F;
  constexpr int E = F::E, P = F::P, C = ColCfg<L>::C, NY = L / 2;
  __shared__ float2 sm[C * F::LDS];
  const int grp = xcd_remap(block, nblocks);
  if (grp >= ngroups) return;
  const int cc = threadIdx.x % C, t = threadIdx.x / C;
  const int c = grp * C + cc;
  F f;
  float2 z[E];
#pragma unroll
  for (int m = 0; m < E; ++m) {
    if (m >= E / 4 && m < 3 * E / 4) continue;
    z[m] = half[half_index(c, pixel_of<L>(t + P * m), NY)];
  }
  f.load_twiddles(tw, t);
  float2* s = sm + cc;
  f.template run<false, true>(z, t, s);
  if (grp == 0) {   // column 0 carries columns 0 and Hx: Z(k) = F_0(k) + i F_Hx(k), both Hermitian in k
    __syncthreads();
    if (cc == 0) {
#pragma unroll
      for (int m = 0; m < E; ++m) sm[t + P * m] = z[m];
    }
    __syncthreads();
    if (cc == 0) {
#pragma unroll
      for (int m = 0; m < E; ++m) {
        const int k = t + P * m;
        const float2 a = z[m], b = sm[(L - k) & (L - 1)];
        z[m] = make_float2(0.5f * (a.x + b.x), 0.5f * (a.y - b.y));
        grid[grid_index(GRID_PAD + Hx, k, L)] = make_float2(0.5f * (a.y + b.y), 0.5f * (b.x - a.x));
      }
    }
  }
#pragma unroll
  for (int m = 0; m < E; ++m) grid[grid_index(GRID_PAD + c, t + P * m, L)] = z[m];
  // mirror images: column -c at row -k (left padding), column 2 Hx - c (right padding)
  if (c >= 1 && c <= GRID_PAD) {
#pragma unroll
    for (int m = 0; m < E; ++m)
      grid[grid_index(GRID_PAD - c, (L - (t + P * m)) & (L - 1), L)] = conjf2(z[m]);
  }
  if (c > Hx - GRID_PAD) {
#pragma unroll
    for (int m = 0; m < E; ++m)
      grid[grid_index(GRID_PAD + 2 * Hx - c, (L - (t + P * m)) & (L - 1), L)] = conjf2(z[m]);
  }
}

template <int L>
__global__ __launch_bounds__(ColCfg<L>::THREADS) void k_fft_cols_fwd(const float2* __restrict__ half,
                                                                     const float2* __restrict__ tw, int Hx,
                                                                     int ngroups, float2* __restrict__ grid) {
  cols_fwd_block<L>(blockIdx.x, gridDim.x, half, tw, Hx, ngroups, grid);
}

// The same after an analysis level of SARA in the first workgroups.
template <int L, bool HW>
__global__ __launch_bounds__(std::max(ColCfg<L>::THREADS, DWT_THREADS)) void k_fft_cols_fwd_dwt(
    int nblocks, const float2* __restrict__ half, const float2* __restrict__ tw, int Hx, int ngroups,
    float2* __restrict__ grid, SaraJob j) {
  const int b = int(blockIdx.x) - j.blocks();
  if (b < 0) sara_dwt_part<HW>(j, blockIdx.x);
  else if (threadIdx.x < ColCfg<L>::THREADS) cols_fwd_block<L>(b, nblocks, half, tw, Hx, ngroups, grid);
}

// Inverse columns of the accumulated grid, keeping the ny rows that map to
// image rows.  The image takes the real part, so what the padding columns
// hold is added to their mirror images, and columns 0 and Hx, of which only
// the Hermitian part counts, go through one transform.
template <int L>
__global__ __launch_bounds__(ColCfg<L>::THREADS) void k_fft_cols_inv(const float2* __restrict__ grid,
                                                                     const float2* __restrict__ tw, int Hx,
                                                                     int ngroups, float2* __restrict__ half) {
  using F = typename ColCfg<L>::F;
  constexpr int E = F::E, P = F::P, C = ColCfg<L>::C, NY = L / 2;
  __shared__ float2 sm[C * F::LDS];
  const int grp = xcd_remap(blockIdx.x, gridDim.x);
  if (grp >= ngroups) return;
  const int cc = threadIdx.x % C, t = threadIdx.x / C;
  const int c = grp * C + cc;
  F f;
  float2 z[E];
#pragma unroll
  for (int m = 0; m < E; ++m) z[m] = grid[grid_index(GRID_PAD + c, t + P * m, L)];
  f.load_twiddles(tw, t);
  // the padding column that mirrors c, at row -k; for c = 0 column Hx, at row k
  const int pm = c == 0 ? GRID_PAD + Hx : c <= GRID_PAD ? GRID_PAD - c : c > Hx - GRID_PAD ? GRID_PAD + 2 * Hx - c : -1;
  if (pm >= 0) {
    // (8 elements at a time: all 16 at once would spill)
    constexpr int B = E < 8 ? E : 8;
#pragma unroll
    for (int m0 = 0; m0 < E; m0 += B) {
      float2 e[B];
#pragma unroll
      for (int i = 0; i < B; ++i) {
        const int k = t + P * (m0 + i);
        e[i] = grid[grid_index(pm, c == 0 ? k : (L - k) & (L - 1), L)];
      }
#pragma unroll
      for (int i = 0; i < B; ++i) {
        const int m = m0 + i;
        if (c == 0) {   // staged for the rows -k, as columns sm[0 .. L) and sm[L .. 2 L)
          sm[t + P * m] = z[m];
          sm[L + t + P * m] = e[i];
        } else {
          z[m] = cadd(z[m], conjf2(e[i]));
        }
      }
    }
  }
  if (grp == 0) {
    __syncthreads();
    if (c == 0) {
#pragma unroll
      for (int m = 0; m < E; ++m) {
        const int k = t + P * m, kn = (L - k) & (L - 1);
        const float2 a = sm[k], b = sm[kn], p = sm[L + k], q = sm[L + kn];
        z[m] = make_float2(0.5f * (a.x + b.x) - 0.5f * (p.y - q.y), 0.5f * (a.y - b.y) + 0.5f * (p.x + q.x));
      }
    }
    __syncthreads();
  }
  f.template run<true, false>(z, t, sm + cc);
#pragma unroll
  for (int m = 0; m < E; ++m) {
    if (m >= E / 4 && m < 3 * E / 4) continue;
    half[half_index(c, pixel_of<L>(t + P * m), NY)] = z[m];
  }
}

__device__ inline double block_sum(double v, double* red) {
  // wave reduction then across waves through LDS (red: >= 16 doubles)
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if (lane == 0) red[wid] = v;
  __syncthreads();
  double s = 0.0;
  for (int w = 0; w < nw; ++w) s += red[w];
  return s;
}

// Inverse rows: row-pass buffer -> image rows 2 i, 2 i + 1 (add: added to
// them).  PRIMAL fuses the
// primal update of Algorithm 3 (gradient step, projection onto the positive
// orthant, relaxation and the extrapolated iterate), the FP64 statistics
// partials of the new iterate, and the forward row pass of the new x~ (the
// first transform of the next iteration's F Z x~) on the rows just updated,
// into half_next.
template <int L, bool PRIMAL>
__global__ __launch_bounds__(RowCfg<L>::THREADS) void k_fft_rows_inv(
    const float2* __restrict__ half, const float2* __restrict__ tw, const float* __restrict__ dpx,
    const float* __restrict__ dpy, int ny, float* __restrict__ x, float* __restrict__ xt,
    const float* __restrict__ ut, const float* __restrict__ x_true, double tau, double eta, double zeta,
    double lambda, double* __restrict__ part, float2* __restrict__ half_next, int add) {
  using F = typename RowCfg<L>::F;
  constexpr int E = F::E, P = F::P, NX = L / 2, H = L / 2;
  __shared__ float2 sm[RowCfg<L>::NS * F::LDS];
  __shared__ double red[16];
  const int t = threadIdx.x % P, q = threadIdx.x / P;
  const int row = 2 * (blockIdx.x * RowCfg<L>::NS + q);
  const bool ok = row < ny;
  // Z = S_a + i S_b of the two rows' Hermitian spectra, twice their value
  // (the factor is taken out with the deapodisation)
  float2 z[E];
#pragma unroll
  for (int m = 0; m < E; ++m) {
    z[m] = make_float2(0.f, 0.f);
    if (ok) {
      const int k = t + P * m;
      const int kk = m < E / 2 ? k : (L - k) & (H - 1);   // stored column; 0 for k = H too
      const float2* src = half + half_index(kk, row, ny);
      const float2 a = src[0], b = src[FFT_CB];
      if (m < E / 2) z[m] = m == 0 && k == 0 ? make_float2(2.f * a.x, 2.f * b.x) : make_float2(a.x - b.y, a.y + b.x);
      else z[m] = m == E / 2 && k == H ? make_float2(2.f * a.y, 2.f * b.y) : make_float2(a.x + b.y, b.x - a.y);
    }
  }
  F f;
  f.load_twiddles(tw, t);
  // the update's operands are loaded before the transform
  constexpr int NV = PRIMAL ? E / 2 : 1;
  float xo_a[NV], xo_b[NV], ut_a[NV], ut_b[NV];
  if (PRIMAL && ok) {
#pragma unroll
    for (int i = 0; i < E / 2; ++i) {
      const int m = i < E / 4 ? i : i + E / 2;
      const size_t idx = size_t(row) * NX + pixel_of<L>(t + P * m);
      xo_a[i] = x[idx];
      xo_b[i] = x[idx + NX];
      ut_a[i] = ut[idx];
      ut_b[i] = ut[idx + NX];
    }
  }
  float2* s = sm + q * F::LDS;
  f.template run<true, false>(z, t, s);
  double dx2 = 0.0, xx = 0.0, ee = 0.0, tt = 0.0;
  const float dy_a = ok ? 0.5f * dpy[row] : 0.f, dy_b = ok ? 0.5f * dpy[row + 1] : 0.f;
#pragma unroll
  for (int i = 0; i < E / 2; ++i) {
    const int m = i < E / 4 ? i : i + E / 2;
    const int c = pixel_of<L>(t + P * m);
    const float dx = dpx[c];
    const float val[2] = {z[m].x * dx * dy_a, z[m].y * dx * dy_b};
    float nxt[2] = {0.f, 0.f};
    if (ok) {
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const size_t idx = size_t(row + r) * NX + c;
        if constexpr (!PRIMAL) {
          x[idx] = add ? x[idx] + val[r] : val[r];
        } else {
          const double xo = r ? xo_b[i] : xo_a[i];
          double xb = xo - tau * (eta * double(val[r]) + zeta * double(r ? ut_b[i] : ut_a[i]));   // primal step, then P_C
          xb = xb > 0.0 ? xb : 0.0;
          const double xn = xo + lambda * (xb - xo);                              // relaxation
          const float xnf = float(xn);
          x[idx] = xnf;
          const float xtf = float(2.0 * xb - xo);                                 // x~ = 2 xbar - x
          xt[idx] = xtf;
          nxt[r] = xtf * dx * dpy[row + r];
          if (part) {   // statistics partials only when the call reads them (uniform branch)
            const double dn = double(xnf) - xo;
            dx2 += dn * dn;
            xx += double(xnf) * double(xnf);
            if (x_true) {
              const double tv = x_true[idx];
              ee += (tv - double(xnf)) * (tv - double(xnf));
              tt += tv * tv;
            }
          }
        }
      }
    }
    z[m] = make_float2(nxt[0], nxt[1]);
  }
  if constexpr (PRIMAL) {
    if (part) {
      dx2 = block_sum(dx2, red);
      xx = block_sum(xx, red);
      ee = block_sum(ee, red);
      tt = block_sum(tt, red);
      if (threadIdx.x == 0) {
        part[4 * blockIdx.x + 0] = dx2;
        part[4 * blockIdx.x + 1] = xx;
        part[4 * blockIdx.x + 2] = ee;
        part[4 * blockIdx.x + 3] = tt;
      }
    }
    // the forward row pass of the new x~, already in the input's distribution
    __syncthreads();
    f.template run<false, true>(z, t, s);
    store_pair<L>(z, t, s, row, ny, ok, half_next);
  }
}

// Calls fn(std::integral_constant<int, L>) for the transform length L.
template <typename Fn>
int with_length(int L, Fn fn) {
  switch (L) {
    case 32: return fn(std::integral_constant<int, 32>());
    case 64: return fn(std::integral_constant<int, 64>());
    case 128: return fn(std::integral_constant<int, 128>());
    case 256: return fn(std::integral_constant<int, 256>());
    case 512: return fn(std::integral_constant<int, 512>());
    case 1024: return fn(std::integral_constant<int, 1024>());
    case 2048: return fn(std::integral_constant<int, 2048>());
    case 4096: return fn(std::integral_constant<int, 4096>());
    default: return fail(PPD_EUNSUPPORTED, "fft: transform length must be a power of two in [32, 4096]");
  }
}

template <int L>
int row_blocks(const ppd_plan* p) {
  return (p->ny / 2 + RowCfg<L>::NS - 1) / RowCfg<L>::NS;
}

template <int L>
struct ColLaunch {
  int groups, blocks;
  explicit ColLaunch(const ppd_plan* p) {
    groups = (p->Kx / 2) / ColCfg<L>::C;
    blocks = (groups + MAX_XCD - 1) / MAX_XCD * MAX_XCD;
  }
};

}  // namespace

int fft_rows_forward(ppd_plan* p, const float* x, float2* dst) {
  int slot;
  PPD_TRY(timer_begin(p, KK_FFT_ROWS_FWD, &slot));
  PPD_TRY(with_length(p->Kx, [&](auto l) {
    constexpr int L = decltype(l)::value;
    hipLaunchKernelGGL(k_fft_rows_fwd<L>, dim3(row_blocks<L>(p)), dim3(RowCfg<L>::THREADS), 0, p->stream, x, p->dpx,
                       p->dpy, p->twx, p->ny, dst);
    PPD_HIP(hipGetLastError());
    return PPD_OK;
  }));
  return timer_end(p, slot);
}

int fft_cols_forward(ppd_plan* p, const float2* src, const SaraJob* with) {
  int slot;
  PPD_TRY(timer_begin(p, KK_FFT_COLS_FWD, &slot));
  PPD_TRY(with_length(p->Ky, [&](auto l) {
    constexpr int L = decltype(l)::value;
    const ColLaunch<L> c(p);
    if (with) {
      if constexpr (L <= PAIR_MAX_KY) {
        auto kernel = with->W ? k_fft_cols_fwd_dwt<L, true> : k_fft_cols_fwd_dwt<L, false>;
        hipLaunchKernelGGL(kernel, dim3(c.blocks + with->blocks()),
                           dim3(std::max(ColCfg<L>::THREADS, DWT_THREADS)), 0, p->stream, c.blocks, src, p->twy,
                           p->Kx / 2, c.groups, p->grid_f, *with);
      } else {
        return fail(PPD_EUNSUPPORTED, "fft: no launch with an analysis level at this length");
      }
    } else {
      hipLaunchKernelGGL(k_fft_cols_fwd<L>, dim3(c.blocks), dim3(ColCfg<L>::THREADS), 0, p->stream, src, p->twy,
                         p->Kx / 2, c.groups, p->grid_f);
    }
    PPD_HIP(hipGetLastError());
    return PPD_OK;
  }));
  return timer_end(p, slot);
}

int fft_forward(ppd_plan* p, const float* x) {
  PPD_TRY(fft_rows_forward(p, x, p->half));
  return fft_cols_forward(p, p->half);
}

int fft_cols_inverse(ppd_plan* p) {
  int slot;
  PPD_TRY(timer_begin(p, KK_FFT_COLS_INV, &slot));
  PPD_TRY(with_length(p->Ky, [&](auto l) {
    constexpr int L = decltype(l)::value;
    const ColLaunch<L> c(p);
    hipLaunchKernelGGL(k_fft_cols_inv<L>, dim3(c.blocks), dim3(ColCfg<L>::THREADS), 0, p->stream, p->grid_a, p->twy,
                       p->Kx / 2, c.groups, p->half);
    PPD_HIP(hipGetLastError());
    return PPD_OK;
  }));
  return timer_end(p, slot);
}

int fft_adjoint(ppd_plan* p, float* x, bool add) {
  PPD_TRY(fft_cols_inverse(p));
  int slot;
  PPD_TRY(timer_begin(p, KK_FFT_ROWS_INV, &slot));
  PPD_TRY(with_length(p->Kx, [&](auto l) {
    constexpr int L = decltype(l)::value;
    hipLaunchKernelGGL((k_fft_rows_inv<L, false>), dim3(row_blocks<L>(p)), dim3(RowCfg<L>::THREADS), 0, p->stream,
                       p->half, p->twx, p->dpx, p->dpy, p->ny, x, nullptr, nullptr, nullptr, 0.0, 0.0, 0.0, 0.0,
                       nullptr, nullptr, add ? 1 : 0);
    PPD_HIP(hipGetLastError());
    return PPD_OK;
  }));
  return timer_end(p, slot);
}

int fft_rows_inverse_primal(ppd_plan* p, const PrimalArgs& a, float2* next) {
  int slot;
  PPD_TRY(timer_begin(p, KK_FFT_ROWS_INV, &slot));
  PPD_TRY(with_length(p->Kx, [&](auto l) {
    constexpr int L = decltype(l)::value;
    hipLaunchKernelGGL((k_fft_rows_inv<L, true>), dim3(row_blocks<L>(p)), dim3(RowCfg<L>::THREADS), 0, p->stream,
                       p->half, p->twx, p->dpx, p->dpy, p->ny, a.x, a.xt, a.ut, a.x_true, a.tau, a.eta, a.zeta,
                       a.lambda, a.part, next, 0);
    PPD_HIP(hipGetLastError());
    return PPD_OK;
  }));
  return timer_end(p, slot);
}

int primal_partial_count(ppd_plan* p) {
  return with_length(p->Kx, [&](auto l) { return row_blocks<decltype(l)::value>(p); });
}

FftTwiddles fft_twiddles(int L) {
  FftTwiddles out;
  (void)with_length(L, [&](auto l) {
    constexpr int N = decltype(l)::value;
    auto fill = [](std::vector<float2>& tw, int E) {
      for (int M = N; M > E; M /= E)
        for (int k = 1; k < E; ++k)
          for (int n = 0; n < M / E; ++n) {
            const double a = -2.0 * M_PI * double(n * k) / double(M);
            tw.push_back(make_float2(float(std::cos(a)), float(std::sin(a))));
          }
    };
    fill(out.row, FftShape<N>::ROW_E);
    fill(out.col, FftShape<N>::COL_E);
    return PPD_OK;
  });
  return out;
}

}  // namespace ppd
