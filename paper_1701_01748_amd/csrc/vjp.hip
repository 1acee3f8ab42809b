// Differentiable pieces of Algorithm 3 for unrolled iterations: the
// data-dual update (Algorithm 2 inside the generalised Moreau step), the
// sparsity dual update (the clip (I - S_alpha) and relaxation) and the
// primal update (P_C, relaxation and x~), each as a forward kernel and a
// vector-Jacobian product (VJP) kernel.  Gradients follow torch's
// convention for complex tensors (dL/dRe + i dL/dIm of a real loss L).
//
// The data-dual update works on plan-order vectors, block by block, in
// chunks of consecutive points of one block (the chunk table of the exact
// prox); every block norm or block inner product is a sum of
// chunk partials in chunk order (deterministic).
#include <cmath>

#include "ppd_internal.h"

namespace ppd {
namespace {

constexpr int DU_THREADS = 256;

__device__ __forceinline__ double du_block_sum(double v, double* red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < DU_THREADS / 64; ++k) s += red[k];
  __syncthreads();
  return s;
}

struct DuIn {
  const float2* g; const float2* y; const double* U; const float2* v;
  double mu;
};

// w = U^-1 v + g in FP64 (the argument of the generalised Moreau step)
__device__ __forceinline__ double2 du_w(const DuIn& a, int64_t i, double Ue) {
  const float2 ve = a.v[i], ge = a.g[i];
  return dual_arg(ve, Ue, ge);
}

// q - y for q = z - mu U (z - w).
__device__ __forceinline__ double2 du_offset(double2 ze, double2 we, float2 ye, double mU) {
  return make_double2((ze.x - mU * (ze.x - we.x)) - double(ye.x), (ze.y - mU * (ze.y - we.y)) - double(ye.y));
}

// A block's coefficients from r^2 = ||q - y||^2 and (VJP) sd = Re <q - y, gz>:
// (eps / r or 1, eps sd / r^3 or 0, inside, r).  Forward uses the factor; the
// transposed Jacobian of P_B outside the ball is gq = (eps / r) gz - (eps
// <d, gz> / r^3) d.
__device__ __forceinline__ double4 du_coef(double s2, double sd, double e) {
  const double r = sqrt(s2);
  return r <= e ? make_double4(1.0, 0.0, 1.0, r) : make_double4(e / r, e * sd / (r * r * r), 0.0, r);
}

// The coefficients of block j: blk[j], else from its chunk partials, which
// every workgroup of the block adds up in the same order (pd: VJP).  Every
// thread calls it.
__device__ __forceinline__ double4 du_block(const double4* __restrict__ blk, const int32_t* __restrict__ coff,
                                            const double* __restrict__ eps, const double* __restrict__ p2,
                                            const double* __restrict__ pd, int j, double* red) {
  if (blk) return blk[j];
  double s2 = 0.0, sd = 0.0;
  for (int c = coff[j] + int(threadIdx.x); c < coff[j + 1]; c += DU_THREADS) {
    s2 += p2[c];
    if (pd) sd += pd[c];
  }
  s2 = du_block_sum(s2, red);
  if (pd) sd = du_block_sum(sd, red);
  return du_coef(s2, sd, eps[j]);
}

__global__ __launch_bounds__(DU_THREADS) void k_du_blocks(const int32_t* __restrict__ coff,
                                                          const double* __restrict__ eps,
                                                          const double* __restrict__ p2,
                                                          const double* __restrict__ pd,
                                                          double4* __restrict__ blk) {
  __shared__ double red[DU_THREADS / 64];
  const int j = blockIdx.x;
  const double4 b = du_block(nullptr, coff, eps, p2, pd, j, red);
  if (threadIdx.x == 0) blk[j] = b;
}

struct DuChunks {
  const int32_t* cstart; const int32_t* cblock; const int32_t* coff;
  const double* eps;
};

// Forward.  FIRST: the chunk's partial of ||q_1 - y||^2 from z_0 = zprev.
// Else step s: z_s = P_B(q_s) with the factor of the partials p_in (or blk),
// then the partial of the next step's, or after the last step (v_out)
// v' = v + lambda (U (w - z_n) - v).  A step is one launch: 72 bytes of inputs
// and 16 of z per point; five steps and the finish take 6 launches instead of
// the 16 that separate partials, factors and updates took.
template <bool FIRST>
__global__ __launch_bounds__(DU_THREADS) void k_du_step(DuIn a, DuChunks t, const double4* __restrict__ blk,
                                                        const double* __restrict__ p_in, double* __restrict__ p_out,
                                                        const double2* zprev, double2* znext, double lambda,
                                                        float2* __restrict__ v_out, double2* __restrict__ z_out) {
  __shared__ double red[DU_THREADS / 64];
  const int c = blockIdx.x;
  double4 b = make_double4(1.0, 0.0, 1.0, 0.0);
  if (!FIRST) b = du_block(blk, t.coff, t.eps, p_in, nullptr, t.cblock[c], red);
  double s2 = 0.0;
#pragma unroll 2
  for (int64_t i = t.cstart[c] + threadIdx.x; i < t.cstart[c + 1]; i += DU_THREADS) {
    const double Ue = a.U[i], mU = a.mu * Ue;
    const double2 we = du_w(a, i, Ue);
    const float2 ye = a.y[i];
    double2 ze = zprev[i];
    if (!FIRST) {
      const double qx = ze.x - mU * (ze.x - we.x), qy = ze.y - mU * (ze.y - we.y);
      ze = b.z != 0.0 ? make_double2(qx, qy)
                      : make_double2(double(ye.x) + (qx - double(ye.x)) * b.x,
                                     double(ye.y) + (qy - double(ye.y)) * b.x);
      znext[i] = ze;
    }
    if (p_out) {
      const double2 d = du_offset(ze, we, ye, mU);
      s2 += d.x * d.x + d.y * d.y;
    } else {
      const float2 ve = a.v[i];
      const double vbx = Ue * (we.x - ze.x), vby = Ue * (we.y - ze.y);
      v_out[i] = make_float2(float(double(ve.x) + lambda * (vbx - double(ve.x))),
                             float(double(ve.y) + lambda * (vby - double(ve.y))));
      if (z_out != znext) z_out[i] = ze;
    }
  }
  if (p_out) {
    s2 = du_block_sum(s2, red);
    if (threadIdx.x == 0) p_out[c] = s2;
  }
}

// VJP.  FIRST: gz_n = gz' - lambda U gv', gw = lambda U gv', gy = 0.  Else the
// VJP of step s: gq = P_B Jacobian^T gz_s (block coefficients of p2 / pd or
// blk; zprev = z_{s-1}); gy += gz_s - gq; gz_{s-1} = (1 - mu U) gq;
// gw += mu U gq.  Then the partials of step s - 1 (zprev2 = z_{s-2}), or after
// step 1 the outputs: gg = gw, gv = (1 - lambda) gv' + gw / U, gy.
struct DuGrad {
  const float2* gv_out; const float2* gv_more;   // added, each NULL = 0
  const double2* gz_out;
  double2* gzc; double2* gw; double2* gy;
  float2* g_g; float2* g_v; float2* g_y;
  double lambda;
};
__device__ __forceinline__ float2 du_gv(const DuGrad& o, int64_t i) {
  float2 g = o.gv_out ? o.gv_out[i] : make_float2(0.f, 0.f);
  if (o.gv_more) {
    const float2 m = o.gv_more[i];
    g.x += m.x;
    g.y += m.y;
  }
  return g;
}
template <bool FIRST>
__global__ __launch_bounds__(DU_THREADS) void k_du_vjp_step(DuIn a, DuChunks t, DuGrad o,
                                                            const double4* __restrict__ blk,
                                                            const double* __restrict__ p2,
                                                            const double* __restrict__ pd, double* __restrict__ p2n,
                                                            double* __restrict__ pdn,
                                                            const double2* __restrict__ zprev,
                                                            const double2* __restrict__ zprev2) {
  __shared__ double red[DU_THREADS / 64];
  const int c = blockIdx.x;
  double4 b = make_double4(1.0, 0.0, 1.0, 0.0);
  if (!FIRST) b = du_block(blk, t.coff, t.eps, p2, pd, t.cblock[c], red);
  double s2 = 0.0, sd = 0.0;
#pragma unroll 2
  for (int64_t i = t.cstart[c] + threadIdx.x; i < t.cstart[c + 1]; i += DU_THREADS) {
    const double Ue = a.U[i], mU = a.mu * Ue;
    const double2 we = du_w(a, i, Ue);
    const float2 ye = a.y[i];
    double2 g, gw, gy;
    if (FIRST) {
      const double lU = o.lambda * Ue;
      const float2 gv = du_gv(o, i);
      const double2 z = o.gz_out ? o.gz_out[i] : make_double2(0.0, 0.0);
      g = make_double2(z.x - lU * double(gv.x), z.y - lU * double(gv.y));
      gw = make_double2(lU * double(gv.x), lU * double(gv.y));
      gy = make_double2(0.0, 0.0);
    } else {
      g = o.gzc[i];
      gw = o.gw[i];
      gy = o.gy[i];
      double2 gq = g;
      if (b.z == 0.0) {
        const double2 d = du_offset(zprev[i], we, ye, mU);
        gq = make_double2(b.x * g.x - b.y * d.x, b.x * g.y - b.y * d.y);
      }
      gy = make_double2(gy.x + (g.x - gq.x), gy.y + (g.y - gq.y));
      g = make_double2((1.0 - mU) * gq.x, (1.0 - mU) * gq.y);
      gw = make_double2(gw.x + mU * gq.x, gw.y + mU * gq.y);
    }
    o.gzc[i] = g;
    if (p2n) {
      o.gw[i] = gw;
      o.gy[i] = gy;
      const double2 d = du_offset(zprev2[i], we, ye, mU);
      s2 += d.x * d.x + d.y * d.y;
      sd += d.x * g.x + d.y * g.y;
    } else {
      const float2 gv = du_gv(o, i);
      if (o.g_g) o.g_g[i] = make_float2(float(gw.x), float(gw.y));
      if (o.g_v)
        o.g_v[i] = make_float2(float((1.0 - o.lambda) * double(gv.x) + gw.x / Ue),
                               float((1.0 - o.lambda) * double(gv.y) + gw.y / Ue));
      if (o.g_y) o.g_y[i] = make_float2(float(gy.x), float(gy.y));
    }
  }
  if (p2n) {
    s2 = du_block_sum(s2, red);
    sd = du_block_sum(sd, red);
    if (threadIdx.x == 0) {
      p2n[c] = s2;
      pdn[c] = sd;
    }
  }
}

// Sparsity dual update, per coefficient: u' = u + lambda (clip(u + c) - u);
// VJP: g_u = (1 - lambda) g + lambda m g, g_c = lambda m g, m = [|u + c| < alpha].
__global__ void k_su(int64_t n, const float* __restrict__ u, const float* __restrict__ c, float alpha, float lambda,
                     float* __restrict__ u_out) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) {
    const float s = u[i] + c[i];
    const float ub = fminf(fmaxf(s, -alpha), alpha);
    u_out[i] = u[i] + lambda * (ub - u[i]);
  }
}

__global__ void k_su_vjp(int64_t n, const float* __restrict__ u, const float* __restrict__ c, float alpha,
                         float lambda, const float* __restrict__ g, const float* __restrict__ g_more,
                         float* __restrict__ g_u, float* __restrict__ g_c) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) {
    const float s = u[i] + c[i];
    const float m = fabsf(s) < alpha ? 1.0f : 0.0f;
    const float gi = g_more ? g[i] + g_more[i] : g[i];
    if (g_u) g_u[i] = (1.0f - lambda) * gi + lambda * m * gi;
    if (g_c) g_c[i] = lambda * m * gi;
  }
}

// Primal update, per pixel (FP64 as in the fused kernel):
// xbar = P_C(x - tau (eta a + zeta b)), x' = x + lambda (xbar - x), x~' = 2 xbar - x.
// VJP: gxbar = lambda gx' + 2 gx~', m = [x - tau (eta a + zeta b) > 0],
// g_x = (1 - lambda) gx' - gx~' + m gxbar, g_a = -tau eta m gxbar, g_b = -tau zeta m gxbar.
__global__ void k_pu(int64_t n, const float* __restrict__ x, const float* __restrict__ a, const float* __restrict__ b,
                     double tau, double eta, double zeta, double lambda, float* __restrict__ x_out,
                     float* __restrict__ xt_out) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) {
    const double xo = x[i];
    double xb = xo - tau * (eta * double(a[i]) + zeta * double(b[i]));
    xb = xb > 0.0 ? xb : 0.0;
    x_out[i] = float(xo + lambda * (xb - xo));
    xt_out[i] = float(2.0 * xb - xo);
  }
}

__global__ void k_pu_vjp(int64_t n, const float* __restrict__ x, const float* __restrict__ a,
                         const float* __restrict__ b, double tau, double eta, double zeta, double lambda,
                         const float* __restrict__ gx, const float* __restrict__ gxt, float* __restrict__ g_x,
                         float* __restrict__ g_a, float* __restrict__ g_b) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) {
    const double arg = double(x[i]) - tau * (eta * double(a[i]) + zeta * double(b[i]));
    const double g1 = gx ? double(gx[i]) : 0.0, g2 = gxt ? double(gxt[i]) : 0.0;
    const double gb = arg > 0.0 ? lambda * g1 + 2.0 * g2 : 0.0;
    if (g_x) g_x[i] = float((1.0 - lambda) * g1 - g2 + gb);
    if (g_a) g_a[i] = float(-tau * eta * gb);
    if (g_b) g_b[i] = float(-tau * zeta * gb);
  }
}

int ew_blocks(int64_t n) { return int(std::min<int64_t>((n + 255) / 256, 4096)); }

// The block coefficients of partials p2 (and pd), for plans with a block of
// too many chunks for every workgroup to add up; else NULL.
int du_blocks(ppd_plan* p, const double* p2, const double* pd, const double4** blk) {
  *blk = nullptr;
  if (p->own_sums) return PPD_OK;
  hipLaunchKernelGGL(k_du_blocks, dim3(p->d), dim3(DU_THREADS), 0, p->stream, p->sec_coff, p->eps_d, p2, pd,
                     p->du_blk);
  PPD_HIP(hipGetLastError());
  *blk = p->du_blk;
  return PPD_OK;
}

}  // namespace
}  // namespace ppd

using namespace ppd;

extern "C" int ppd_dual_update(ppd_plan* p, const float* g, const float* y, const double* U, const double* eps,
                               const float* v, const double* z, int n_itr, double mu, double lambda, float* v_out,
                               double* z_out, double* zs) {
  if (!p || !g || !y || !U || !eps || !v || !z || !v_out || !z_out)
    return fail(PPD_EINVAL, "ppd_dual_update: NULL argument");
  if (n_itr < 1) return fail(PPD_EINVAL, "ppd_dual_update: n_itr must be >= 1");
  if (!(mu > 0.0) || !std::isfinite(mu) || !(lambda > 0.0 && lambda <= 1.0))
    return fail(PPD_EINVAL, "ppd_dual_update: need mu > 0 and 0 < lambda <= 1");
  if (z_out == z) return fail(PPD_EINVAL, "ppd_dual_update: z_out must not alias z");
  PPD_TRY(upload_eps(p, eps));
  const DuIn in{reinterpret_cast<const float2*>(g), reinterpret_cast<const float2*>(y), U,
                reinterpret_cast<const float2*>(v), mu};
  double2* zo = reinterpret_cast<double2*>(z_out);
  float2* vo = reinterpret_cast<float2*>(v_out);
  double2* hist = reinterpret_cast<double2*>(zs);
  const double2* zprev = reinterpret_cast<const double2*>(z);
  const DuChunks t{p->sec_cstart, p->sec_cblock, p->sec_coff, p->eps_d};
  const dim3 grid(p->n_sec_chunks), block(DU_THREADS);
  double* part[2] = {p->sec_part, p->sec_part + p->n_sec_chunks};
  hipLaunchKernelGGL(k_du_step<true>, grid, block, 0, p->stream, in, t, nullptr, nullptr, part[0], zprev, nullptr,
                     lambda, nullptr, nullptr);
  for (int s = 1; s <= n_itr; ++s) {
    // z_s goes to zs[s - 1] when a history is kept, else to z_out
    double2* znext = hist ? hist + size_t(s - 1) * p->M : zo;
    const double* pin = part[(s - 1) & 1];
    const double4* blk;
    PPD_TRY(du_blocks(p, pin, nullptr, &blk));
    hipLaunchKernelGGL(k_du_step<false>, grid, block, 0, p->stream, in, t, blk, pin, s < n_itr ? part[s & 1] : nullptr,
                       zprev, znext, lambda, vo, zo);
    zprev = znext;
  }
  PPD_HIP(hipGetLastError());
  return PPD_OK;
}

static int dual_update_vjp(ppd_plan* p, const float* g, const float* y, const double* U, const double* eps,
                           const float* v, const double* z, int n_itr, double mu, double lambda, const double* zs,
                           const float* gv_out, const float* gv_more, const double* gz_out, float* g_g, float* g_v,
                           double* g_z, float* g_y) {
  if (!p || !g || !y || !U || !eps || !v || !z || !zs || !g_z)
    return fail(PPD_EINVAL, "ppd_dual_update_vjp: NULL argument");
  if (n_itr < 1) return fail(PPD_EINVAL, "ppd_dual_update_vjp: n_itr must be >= 1");
  if (!(mu > 0.0) || !std::isfinite(mu) || !(lambda > 0.0 && lambda <= 1.0))
    return fail(PPD_EINVAL, "ppd_dual_update_vjp: need mu > 0 and 0 < lambda <= 1");
  if (static_cast<const void*>(gz_out) == static_cast<const void*>(g_z))
    return fail(PPD_EINVAL, "ppd_dual_update_vjp: g_z must not alias gz_out");
  PPD_TRY(upload_eps(p, eps));
  const DuIn in{reinterpret_cast<const float2*>(g), reinterpret_cast<const float2*>(y), U,
                reinterpret_cast<const float2*>(v), mu};
  // gzc: the running gradient of z_s
  const DuGrad o{reinterpret_cast<const float2*>(gv_out), reinterpret_cast<const float2*>(gv_more),
                 reinterpret_cast<const double2*>(gz_out),
                 reinterpret_cast<double2*>(g_z), p->wbuf, p->qbuf, reinterpret_cast<float2*>(g_g),
                 reinterpret_cast<float2*>(g_v), reinterpret_cast<float2*>(g_y), lambda};
  const double2* z0 = reinterpret_cast<const double2*>(z);
  const double2* hist = reinterpret_cast<const double2*>(zs);
  auto z_at = [&](int s) { return s == 0 ? z0 : hist + size_t(s - 1) * p->M; };
  const DuChunks t{p->sec_cstart, p->sec_cblock, p->sec_coff, p->eps_d};
  const dim3 grid(p->n_sec_chunks), block(DU_THREADS);
  const int nc = p->n_sec_chunks;
  double* part[2] = {p->sec_part, p->sec_part + 2 * nc};
  hipLaunchKernelGGL(k_du_vjp_step<true>, grid, block, 0, p->stream, in, t, o, nullptr, nullptr, nullptr,
                     part[n_itr & 1], part[n_itr & 1] + nc, nullptr, z_at(n_itr - 1));
  for (int s = n_itr; s >= 1; --s) {
    const double* p2 = part[s & 1];
    double* p2n = s > 1 ? part[(s - 1) & 1] : nullptr;
    const double4* blk;
    PPD_TRY(du_blocks(p, p2, p2 + nc, &blk));
    hipLaunchKernelGGL(k_du_vjp_step<false>, grid, block, 0, p->stream, in, t, o, blk, p2, p2 + nc, p2n,
                       p2n ? p2n + nc : nullptr, z_at(s - 1), s > 1 ? z_at(s - 2) : nullptr);
  }
  PPD_HIP(hipGetLastError());
  return PPD_OK;
}

extern "C" int ppd_dual_update_vjp(ppd_plan* p, const float* g, const float* y, const double* U, const double* eps,
                                   const float* v, const double* z, int n_itr, double mu, double lambda,
                                   const double* zs, const float* gv_out, const double* gz_out, float* g_g,
                                   float* g_v, double* g_z, float* g_y) {
  return dual_update_vjp(p, g, y, U, eps, v, z, n_itr, mu, lambda, zs, gv_out, nullptr, gz_out, g_g, g_v, g_z, g_y);
}

extern "C" int ppd_sparsity_update(ppd_plan* p, const float* u, const float* c, float alpha, float lambda,
                                   float* u_out) {
  if (!p || !u || !c || !u_out) return fail(PPD_EINVAL, "ppd_sparsity_update: NULL argument");
  if (!(alpha >= 0.0f) || !(lambda > 0.0f && lambda <= 1.0f))
    return fail(PPD_EINVAL, "ppd_sparsity_update: need alpha >= 0 and 0 < lambda <= 1");
  const int64_t n = int64_t(N_BASES) * p->nx * p->ny;
  hipLaunchKernelGGL(k_su, dim3(ew_blocks(n)), dim3(256), 0, p->stream, n, u, c, alpha, lambda, u_out);
  PPD_HIP(hipGetLastError());
  return PPD_OK;
}

static int sparsity_update_vjp(ppd_plan* p, const float* u, const float* c, float alpha, float lambda,
                               const float* g_out, const float* g_more, float* g_u, float* g_c) {
  if (!p || !u || !c || !g_out) return fail(PPD_EINVAL, "ppd_sparsity_update_vjp: NULL argument");
  if (!(alpha >= 0.0f) || !(lambda > 0.0f && lambda <= 1.0f))
    return fail(PPD_EINVAL, "ppd_sparsity_update_vjp: need alpha >= 0 and 0 < lambda <= 1");
  const int64_t n = int64_t(N_BASES) * p->nx * p->ny;
  hipLaunchKernelGGL(k_su_vjp, dim3(ew_blocks(n)), dim3(256), 0, p->stream, n, u, c, alpha, lambda, g_out,
                     g_more, g_u, g_c);
  PPD_HIP(hipGetLastError());
  return PPD_OK;
}

extern "C" int ppd_sparsity_update_vjp(ppd_plan* p, const float* u, const float* c, float alpha, float lambda,
                                       const float* g_out, float* g_u, float* g_c) {
  return sparsity_update_vjp(p, u, c, alpha, lambda, g_out, nullptr, g_u, g_c);
}

extern "C" int ppd_primal_update(ppd_plan* p, const float* x, const float* a, const float* b, double tau, double eta,
                                 double zeta, double lambda, float* x_out, float* xt_out) {
  if (!p || !x || !a || !b || !x_out || !xt_out) return fail(PPD_EINVAL, "ppd_primal_update: NULL argument");
  if (!std::isfinite(tau) || !std::isfinite(eta) || !std::isfinite(zeta) || !(lambda > 0.0 && lambda <= 1.0))
    return fail(PPD_EINVAL, "ppd_primal_update: non-finite step or lambda outside (0, 1]");
  const int64_t n = int64_t(p->nx) * p->ny;
  hipLaunchKernelGGL(k_pu, dim3(ew_blocks(n)), dim3(256), 0, p->stream, n, x, a, b, tau, eta, zeta, lambda, x_out,
                     xt_out);
  PPD_HIP(hipGetLastError());
  return PPD_OK;
}

extern "C" int ppd_primal_update_vjp(ppd_plan* p, const float* x, const float* a, const float* b, double tau,
                                     double eta, double zeta, double lambda, const float* gx_out,
                                     const float* gxt_out, float* g_x, float* g_a, float* g_b) {
  if (!p || !x || !a || !b) return fail(PPD_EINVAL, "ppd_primal_update_vjp: NULL argument");
  if (!std::isfinite(tau) || !std::isfinite(eta) || !std::isfinite(zeta) || !(lambda > 0.0 && lambda <= 1.0))
    return fail(PPD_EINVAL, "ppd_primal_update_vjp: non-finite step or lambda outside (0, 1]");
  const int64_t n = int64_t(p->nx) * p->ny;
  hipLaunchKernelGGL(k_pu_vjp, dim3(ew_blocks(n)), dim3(256), 0, p->stream, n, x, a, b, tau, eta, zeta, lambda,
                     gx_out, gxt_out, g_x, g_a, g_b);
  PPD_HIP(hipGetLastError());
  return PPD_OK;
}

// The scalars of an iteration and, for the data dual, its radii, checked before
// anything is launched: as the pieces check theirs.
static int step_check(ppd_plan* p, const ppd_step_args* s, bool dual, const char* fn) {
  const std::string f(fn);
  if (s->n_itr < 1) return fail(PPD_EINVAL, f + ": n_itr must be >= 1");
  if (!(s->mu > 0.0) || !std::isfinite(s->mu) || !(s->lambda <= 1.0 && float(s->lambda) > 0.0f))
    return fail(PPD_EINVAL, f + ": need mu > 0 and 0 < lambda <= 1");
  if (!(float(s->alpha) >= 0.0f)) return fail(PPD_EINVAL, f + ": need alpha >= 0");
  if (!std::isfinite(s->tau) || !std::isfinite(s->eta) || !std::isfinite(s->zeta))
    return fail(PPD_EINVAL, f + ": non-finite step");
  return dual ? upload_eps(p, s->eps) : PPD_OK;
}

// One differentiable iteration as one call, on one stream: at 256^2 with
// 65536 points, three levels and one Algorithm 2 step its 16 launches, and the
// 16 of its VJP with all gradients, take less time on the GPU (150 us together)
// than on the host, and a fork to the second stream and back cost 40 us of host
// time each (450 us per forward and backward against 365).
extern "C" int ppd_step(ppd_plan* p, const ppd_step_args* s) {
  if (!p || !s || !s->x || !s->xt || !s->v || !s->u || !s->z || !s->y || !s->U || !s->eps || !s->g || !s->c || !s->a ||
      !s->b || !s->zs || !s->x_out || !s->xt_out || !s->v_out || !s->u_out || !s->z_out)
    return fail(PPD_EINVAL, "ppd_step: NULL argument");
  if (s->z_out == s->z) return fail(PPD_EINVAL, "ppd_step: z_out must not alias z");
  PPD_TRY(step_check(p, s, true, "ppd_step"));
  PPD_TRY(ppd_sara_w(p, PPD_SARA_ANALYSIS, s->xt, s->c, nullptr, nullptr, 0.f, 0.f));
  PPD_TRY(ppd_sparsity_update(p, s->u, s->c, float(s->alpha), float(s->lambda), s->u_out));
  PPD_TRY(ppd_sara_w(p, PPD_SARA_SYNTHESIS, s->u_out, s->b, nullptr, nullptr, 0.f, 0.f));
  PPD_TRY(ppd_phi(p, s->xt, s->g, PPD_ORDER_PLAN));
  PPD_TRY(ppd_dual_update(p, s->g, s->y, s->U, s->eps, s->v, s->z, s->n_itr, s->mu, s->lambda, s->v_out, s->z_out,
                          s->zs));
  PPD_TRY(ppd_phit(p, s->v_out, s->a, PPD_ORDER_PLAN));
  return ppd_primal_update(p, s->x, s->a, s->b, s->tau, s->eta, s->zeta, s->lambda, s->x_out, s->xt_out);
}

extern "C" int ppd_step_vjp(ppd_plan* p, const ppd_step_args* s, const ppd_step_grads* q) {
  if (!p || !s || !q || !s->x || !s->v || !s->u || !s->z || !s->y || !s->U || !s->eps || !s->g || !s->c || !s->a ||
      !s->b || !s->zs)
    return fail(PPD_EINVAL, "ppd_step_vjp: NULL argument");
  // what flows back through the primal update, the data dual, the sparsity dual
  const bool prim = q->gx_out || q->gxt_out, dual = q->g_z != nullptr, sparse = q->g_u || q->g_c;
  if (prim && (!q->g_a || !q->g_b)) return fail(PPD_EINVAL, "ppd_step_vjp: g_a and g_b are needed");
  if (dual && prim && !q->t_v) return fail(PPD_EINVAL, "ppd_step_vjp: t_v is needed");
  if (!dual && (q->g_v || q->g_y || q->g_g)) return fail(PPD_EINVAL, "ppd_step_vjp: the data dual's gradients need g_z");
  if (sparse && (prim ? !q->t_u : !q->gu_out)) return fail(PPD_EINVAL, "ppd_step_vjp: t_u (or gu_out) is needed");
  if (q->g_xt && ((!dual && !sparse) || (dual && !q->g_g) || (sparse && !q->g_c)))
    return fail(PPD_EINVAL, "ppd_step_vjp: g_xt needs g_g and g_c");
  if (dual && q->gz_out == q->g_z) return fail(PPD_EINVAL, "ppd_step_vjp: g_z must not alias gz_out");
  PPD_TRY(step_check(p, s, dual, "ppd_step_vjp"));
  if (prim)
    PPD_TRY(ppd_primal_update_vjp(p, s->x, s->a, s->b, s->tau, s->eta, s->zeta, s->lambda, q->gx_out, q->gxt_out,
                                  q->g_x, q->g_a, q->g_b));
  if (sparse) {
    if (prim) PPD_TRY(ppd_sara_w(p, PPD_SARA_ANALYSIS, q->g_b, q->t_u, nullptr, nullptr, 0.f, 0.f));
    PPD_TRY(sparsity_update_vjp(p, s->u, s->c, float(s->alpha), float(s->lambda), prim ? q->t_u : q->gu_out,
                                prim ? q->gu_out : nullptr, q->g_u, q->g_c));
    if (q->g_xt) PPD_TRY(ppd_sara_w(p, PPD_SARA_SYNTHESIS, q->g_c, q->g_xt, nullptr, nullptr, 0.f, 0.f));
  }
  if (dual) {
    if (prim) PPD_TRY(ppd_phi(p, q->g_a, q->t_v, PPD_ORDER_PLAN));
    PPD_TRY(dual_update_vjp(p, s->g, s->y, s->U, s->eps, s->v, s->z, s->n_itr, s->mu, s->lambda, s->zs,
                            prim ? q->t_v : nullptr, q->gv_out, q->gz_out, q->g_g, q->g_v, q->g_z, q->g_y));
    if (q->g_xt) PPD_TRY(sparse ? ppd_phit_add(p, q->g_g, q->g_xt) : ppd_phit(p, q->g_g, q->g_xt, PPD_ORDER_PLAN));
  }
  return PPD_OK;
}
