// SARA sparsity operator (Sec. 5.1): Psi = (1/3)[I, W_1, .., W_8], W_p the
// orthonormal periodised 2D Daubechies-p wavelet transform, coefficients in
// the Mallat layout of the image.  Float32.
//
// Analysis runs one launch per level for the 8 wavelet bases at once
// (one grid dimension per basis; the Dirac basis rides in the first launch).
// In the dual mode (the sparsity dual update of Algorithm 3) every final
// coefficient c is consumed in place: u <- u + lambda (clip(u + c, +-alpha) - u).
// Synthesis is the transpose, one launch per level, the two coarsest in one;
// the last level sums the 8 reconstructions and the Dirac part (no atomics)
// and applies the 1/3.
//
// Both directions filter along the columns first, straight from memory: a
// thread owns one column of the tile, loads a run of it into registers
// (consecutive threads read consecutive addresses) and makes all outputs of
// the run from them, so that a value is read once for a run's outputs and not
// once for each.  The results go to LDS, and the row pass makes 4 consecutive
// output pairs per thread from 16-byte LDS reads in the same way: 3 to 6
// reads for 8 or 16 outputs instead of 2 per tap and output.  Tiles are 64
// columns wide (256-byte runs of the duals).  A synthesis tile is one wave's
// work, so its two passes need no workgroup barrier.
//
// Bound by HBM at large sizes (302 MB of duals in and out per dual step at
// 2048^2) and by the latency of five dependent launches at small ones.  One
// dual step alone, against the earlier form that staged a tile's window in
// LDS and read LDS once per tap and output: 2048^2 332 -> 183 us, 1024^2
// 108 -> 65 us, 512^2 44 -> 33 us, 64^2 31 -> 27 us.
#include <cmath>
#include "sara_device.h"

namespace ppd {
namespace {

// Workgroup number of a three-dimensional launch.
__device__ __forceinline__ int linear_block() {
  return int(blockIdx.x) + int(gridDim.x) * (int(blockIdx.y) + int(gridDim.y) * int(blockIdx.z));
}

template <int MODE, int RB, bool HW>
__global__ __launch_bounds__(DWT_THREADS) void k_dwt(const float* __restrict__ x, float* __restrict__ tmp,
                                                     float* __restrict__ out, const float* __restrict__ filt,
                                                     const float* __restrict__ W, SaraGeom g, int l, float alpha,
                                                     float lambda, const uint8_t* __restrict__ active, int vec) {
  dwt_block<MODE, RB, HW>(sara_tile<true>(linear_block(), gridDim.x, gridDim.y, gridDim.z), x, tmp, out, filt, W, g, l,
                      alpha, lambda, active, vec);
}

template <int WM>
__global__ __launch_bounds__(256) void k_idwt(const float* __restrict__ u, float* __restrict__ rec,
                                              const float* __restrict__ filt, const float* __restrict__ W,
                                              SaraGeom g, int l) {
  idwt_block<WM>(sara_tile<false>(linear_block(), gridDim.x, gridDim.y, gridDim.z), u, rec, filt, W, g, l);
}

template <int WM>
__global__ __launch_bounds__(256) void k_idwt2(const float* __restrict__ u, float* __restrict__ rec,
                                               const float* __restrict__ filt, const float* __restrict__ W,
                                               SaraGeom g) {
  idwt2_block<WM>(sara_tile<false>(linear_block(), gridDim.x, gridDim.y, gridDim.z), u, rec, filt, W, g);
}

template <int WM>
__global__ __launch_bounds__(256) void k_idwt_final(const float* __restrict__ u, const float* __restrict__ rec,
                                                    const float* __restrict__ filt, const float* __restrict__ W,
                                                    SaraGeom g, float* __restrict__ out, int vec) {
  idwt_final_block<WM>(sara_tile<false>(linear_block(), gridDim.x, gridDim.y, gridDim.z), u, rec, filt, W, g, out, vec);
}

// Algorithm 1 weights (eq. reweighting): W = omega / (omega + |c|), in
// place over the analysis coefficients c.
__global__ void k_reweight(float* __restrict__ w, size_t n, float omega) {
  for (size_t i = blockIdx.x * size_t(blockDim.x) + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x)
    w[i] = omega / (omega + fabsf(w[i]));
}

SaraGeom geom(const ppd_plan* p) {
  SaraGeom g{};
  g.nx = p->nx;
  g.ny = p->ny;
  g.L = p->levels;
  g.N = size_t(p->nx) * p->ny;
  size_t o = 0;
  for (int l = 1; l < g.L; ++l) {
    g.off[l] = o;
    o += 8 * (g.N >> (2 * l));
  }
  return g;
}

// Analysis tiles of 16 rows while they fill the chip, else of 8.
bool tall_tiles(const SaraGeom& g, int l) {
  const int oh = g.ny >> l, ow = g.nx >> l;
  return int64_t(ow / std::min(TX, ow)) * (oh / std::min(16, oh)) * (l == 1 ? 9 : 8) >= DWT_TALL_MIN;
}

// Columns of the synthesis tiles of an output of hh x ww: 64, or 32 where that
// makes fewer than `most` waves.  A wave of 64 columns loads its two bands in
// two rounds, one of 32 in one: shorter where waves are few, more columns
// loaded twice where they are many.  A dual step of 3 levels, 64 and 32 columns:
// 128 x 64 30.3 and 27.3 us, 256^2 32.7 and 29.0, 512^2 38.2 and 34.9.  Last
// level: 512^2 (2048 waves) 15.0 and 13.9 with the others at 32, 1024 x 512 (4096)
// 18.8 and 21.3.  The levels before it: 512 x 256 (1024 waves) 20.2 and 18.8
// for the whole synthesis, 512^2 (2048) 28.7 and 30.1.
constexpr int64_t NARROW_LAST = 4096, NARROW_LEVEL = 2048;
int synth_width(int hh, int ww, int64_t most) {
  const int sx = int64_t(8) * std::max(1, ww / SX) * std::max(1, hh / SY) < most ? SX / 2 : SX;
  return std::min(sx, ww);
}

bool aligned16(const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

template <int MODE, int RB>
void launch_dwt(ppd_plan* p, dim3 grid, const float* x, float* out, const float* W, const SaraGeom& g, int l,
                float alpha, float lambda, const uint8_t* active, int vec) {
  auto kernel = W ? k_dwt<MODE, RB, true> : k_dwt<MODE, RB, false>;
  hipLaunchKernelGGL(kernel, grid, dim3(DWT_THREADS), 0, p->stream, x, p->sara_ll, out, p->filt, W, g, l, alpha, lambda,
                     active, vec);
}

int analysis_launch(ppd_plan* p, const float* x, float* out, const float* W, bool dual, float alpha,
                    float lambda, const uint8_t* active) {
  const SaraGeom g = geom(p);
  for (int l = 1; l <= g.L; ++l) {
    const int oh = (g.ny >> l), ow = (g.nx >> l);
    const int tox = std::min(TX, ow), nz = l == 1 ? 9 : 8;
    const int vec = ow % 4 == 0 && aligned16(out) && aligned16(W) && aligned16(x);
    const bool tall = tall_tiles(g, l);
    const dim3 grid(ow / tox, oh / std::min(tall ? 16 : 8, oh), nz);
    int slot;
    PPD_TRY(timer_begin(p, KK_DWT, &slot));
    if (dual && tall) launch_dwt<A_DUAL, 8>(p, grid, x, out, W, g, l, alpha, lambda, active, vec);
    else if (dual) launch_dwt<A_DUAL, 4>(p, grid, x, out, W, g, l, alpha, lambda, active, vec);
    else if (tall) launch_dwt<A_PLAIN, 8>(p, grid, x, out, W, g, l, alpha, lambda, nullptr, vec);
    else launch_dwt<A_PLAIN, 4>(p, grid, x, out, W, g, l, alpha, lambda, nullptr, vec);
    PPD_HIP(hipGetLastError());
    PPD_TRY(timer_end(p, slot));
  }
  return PPD_OK;
}

}  // namespace

int sara_analysis(ppd_plan* p, const float* x, float* coef, const float* W) {
  return analysis_launch(p, x, coef, W, false, 0.f, 0.f, nullptr);
}

int sara_dual(ppd_plan* p, const float* x, float* u, float alpha, float lambda, const float* W,
              const uint8_t* active) {
  return analysis_launch(p, x, u, W, true, alpha, lambda, active);
}

// The synthesis launches: the two coarsest levels in one (from three levels
// on), the others one by one, the last one into out.
struct SynthJobs {
  SaraJob job[8];
  int n = 0;
};
static SynthJobs synth_jobs(ppd_plan* p, const float* u, const float* W, float* out) {
  SynthJobs js;
  const SaraGeom g = geom(p);
  auto level = [&](int kind, int l) {
    const int hh = g.ny >> (l - 1), ww = g.nx >> (l - 1);
    js.job[js.n++] = SaraJob{kind, u, p->sara_rec, nullptr, p->filt, W, g, l, 0.f, 0.f, nullptr, 0,
                             ww / synth_width(hh, ww, NARROW_LEVEL), hh / std::min(SY, hh), 2};
  };
  int top = g.L;
  if (g.L >= 3) {
    level(SARA_IDWT2, g.L - 1);
    top = g.L - 2;
  }
  for (int l = top; l >= 2; --l) level(SARA_IDWT, l);
  js.job[js.n++] = SaraJob{SARA_FINAL, u, p->sara_rec, out, p->filt, W, g, 1, 0.f, 0.f, nullptr,
                           aligned16(u) && aligned16(W) && aligned16(out),
                           g.nx / synth_width(g.ny, g.nx, NARROW_LAST), g.ny / SY, 1};
  return js;
}

bool sara_pairs(const ppd_plan* p) { return p->levels <= SARA_PAIR_LEVELS && !tall_tiles(geom(p), 1); }

SaraJobs sara_jobs(ppd_plan* p, const float* x, float* u, float alpha, float lambda, const float* W,
                   const uint8_t* active, float* out) {
  SaraJobs js{};
  const SaraGeom g = geom(p);
  for (int l = 1; l <= g.L; ++l) {
    const int oh = g.ny >> l, ow = g.nx >> l;
    js.dwt[js.n_dwt++] = SaraJob{SARA_DWT, x, p->sara_ll, u, p->filt, W, g, l, alpha, lambda, active,
                                 ow % 4 == 0 && aligned16(u) && aligned16(W) && aligned16(x),
                                 ow / std::min(TX, ow), oh / std::min(8, oh), l == 1 ? 9 : 8};
  }
  const SynthJobs sy = synth_jobs(p, u, W, out);
  for (; js.n_synth < sy.n; ++js.n_synth) js.synth[js.n_synth] = sy.job[js.n_synth];
  return js;
}

int sara_launch(ppd_plan* p, const SaraJob& j) {
  const dim3 grid(j.gx, j.gy, j.gz);
  auto synth = [&](auto plain, auto weighted, auto... args) {
    hipLaunchKernelGGL(j.W ? weighted : plain, grid, dim3(256), 0, p->stream, args...);
  };
  if (j.kind == SARA_DWT)
    launch_dwt<A_DUAL, 4>(p, grid, j.in, j.out, j.W, j.g, j.l, j.alpha, j.lambda, j.active, j.vec);
  else if (j.kind == SARA_IDWT2)
    synth(k_idwt2<W_NONE>, k_idwt2<W_AHEAD>, j.in, j.tmp, j.filt, j.W, j.g);
  else if (j.kind == SARA_IDWT)
    // a single level's weights ahead cost a wave per SIMD: only where waves are few, in tiles below 64 columns
    synth(k_idwt<W_NONE>, (j.g.nx >> (j.l - 1)) / j.gx < SX ? k_idwt<W_AHEAD> : k_idwt<W_AFTER>, j.in, j.tmp, j.filt,
          j.W, j.g, j.l);
  else
    synth(k_idwt_final<W_NONE>, k_idwt_final<W_AHEAD>, j.in, j.tmp, j.filt, j.W, j.g, j.out, j.vec);
  PPD_HIP(hipGetLastError());
  return PPD_OK;
}

int sara_synthesis(ppd_plan* p, const float* u, float* out, const float* W) {
  const SynthJobs js = synth_jobs(p, u, W, out);
  for (int k = 0; k < js.n; ++k) {
    int slot;
    PPD_TRY(timer_begin(p, KK_IDWT, &slot));
    PPD_TRY(sara_launch(p, js.job[k]));
    PPD_TRY(timer_end(p, slot));
  }
  return PPD_OK;
}

}  // namespace ppd

using namespace ppd;

extern "C" int ppd_sara_w(ppd_plan* p, int op, const float* in, float* out, float* u, const float* W,
                          float alpha, float lambda) {
  if (!p || !in || !out) return fail(PPD_EINVAL, "ppd_sara: NULL argument");
  switch (op) {
    case PPD_SARA_ANALYSIS:
      return sara_analysis(p, in, out, W);
    case PPD_SARA_SYNTHESIS:
      return sara_synthesis(p, in, out, W);
    case PPD_SARA_DUAL:
      if (!u) return fail(PPD_EINVAL, "ppd_sara: dual mode needs u_inout");
      if (!(alpha >= 0.0f)) return fail(PPD_EINVAL, "ppd_sara: alpha must be >= 0");
      PPD_TRY(sara_dual(p, in, u, alpha, lambda, W));
      return sara_synthesis(p, u, out, W);
    default:
      return fail(PPD_EINVAL, "ppd_sara: unknown op");
  }
}

extern "C" int ppd_sara(ppd_plan* p, int op, const float* in, float* out, float* u, float alpha,
                        float lambda) {
  return ppd_sara_w(p, op, in, out, u, nullptr, alpha, lambda);
}

extern "C" int ppd_reweight(ppd_plan* p, const float* x, float omega, float* W) {
  if (!p || !x || !W) return fail(PPD_EINVAL, "ppd_reweight: NULL argument");
  if (!(omega > 0.0f) || !std::isfinite(omega)) return fail(PPD_EINVAL, "ppd_reweight: omega must be > 0");
  PPD_TRY(sara_analysis(p, x, W, nullptr));
  const size_t n = size_t(N_BASES) * p->nx * p->ny;
  int slot;
  PPD_TRY(timer_begin(p, KK_MISC, &slot));
  hipLaunchKernelGGL(k_reweight, dim3(int(std::min<size_t>((n + 255) / 256, 4096))), dim3(256), 0, p->stream, W,
                     n, omega);
  PPD_HIP(hipGetLastError());
  return timer_end(p, slot);
}
