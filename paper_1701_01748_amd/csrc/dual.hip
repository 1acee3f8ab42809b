// Data-fidelity dual update of Algorithm 3 and Algorithm 2,
// FP64: the standalone ellipsoid projection entry point, the unfused
// per-block ("plain") form of the dual update, and the uniform-weighting
// preconditioner (inverse local sampling density, Sec. 4.3).
#include <cmath>

#include "sara_device.h"

namespace ppd {
namespace {

__device__ inline double block_sum(double v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if (lane == 0) red[wid] = v;
  __syncthreads();
  double s = 0.0;
  for (int w = 0; w < nw; ++w) s += red[w];
  return s;
}

// Sum of v over a 256-thread workgroup in a fixed order, in every thread.
// Every thread must call it; red is free again after the next barrier.
__device__ __forceinline__ double sum256(double v, double* red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return ((red[0] + red[1]) + red[2]) + red[3];
}

// P_B factor of a block from its squared norm (Sec. 3.3, eq. proj-L2):
// (eps_j / r, 0) outside the ball, (1, 1) inside.
__device__ __forceinline__ double2 ball_factor(double r2, double eps) {
  const double r = sqrt(r2);
  return r > eps ? make_double2(eps / r, 0.0) : make_double2(1.0, 1.0);
}

// One Algorithm 2 step on a chunk of consecutive plan-order points of one
// block: z <- P_B(q), q = z - mu U (z - w), then the chunk's partial of
// ||q - y||^2 of the next q.  Every workgroup of a block adds up the previous
// step's partials itself, in the same order (pin), so that a step is one
// launch; the partials alternate between two buffers.  APPLY: there is a
// factor; NEXT: there is a next step.  HBM carries 80 bytes per point and
// step; a step of 65536 points is bound by the launch's latency.
template <bool APPLY, bool NEXT>
__global__ __launch_bounds__(256) void k_ball_step(BallIn in, const int32_t* __restrict__ cstart,
                                                   const int32_t* __restrict__ cblock,
                                                   const int32_t* __restrict__ coff, const double* __restrict__ eps,
                                                   const double2* __restrict__ fac, const double* __restrict__ pin,
                                                   double2* __restrict__ z, double* __restrict__ pout) {
  __shared__ double red[8];
  const int c = blockIdx.x, j = cblock[c];
  const int i0 = cstart[c], i1 = cstart[c + 1];
  double2 bf = make_double2(1.0, 1.0);
  if (APPLY) {
    if (fac) {
      bf = fac[j];
    } else {
      double t = 0.0;
      for (int k = coff[j] + int(threadIdx.x); k < coff[j + 1]; k += 256) t += pin[k];
      bf = ball_factor(sum256(t, red), eps[j]);
    }
  }
  // randomised updates of Algorithm 3: an inactive block keeps z
  const bool act = !in.active || in.active[j];
  double acc = 0.0;
#pragma unroll 2
  for (int i = i0 + int(threadIdx.x); i < i1; i += 256) {
    const double Ue = in.U[i], mU = in.mu * Ue;
    const double2 we = in.w ? in.w[i] : dual_arg(in.v[i], Ue, in.ga[i]);
    const float2 ye = in.y[i];
    double2 ze = z[i];
    if (APPLY && act) {
      const double qx = ze.x - mU * (ze.x - we.x), qy = ze.y - mU * (ze.y - we.y);
      ze.x = bf.y != 0.0 ? qx : double(ye.x) + (qx - double(ye.x)) * bf.x;
      ze.y = bf.y != 0.0 ? qy : double(ye.y) + (qy - double(ye.y)) * bf.x;
      z[i] = ze;
    }
    if (NEXT) {
      const double dx = (ze.x - mU * (ze.x - we.x)) - double(ye.x);
      const double dy = (ze.y - mU * (ze.y - we.y)) - double(ye.y);
      acc += dx * dx + dy * dy;
    }
  }
  if (NEXT) {
    acc = sum256(acc, red + 4);
    if (threadIdx.x == 0) pout[c] = acc;
  }
}

// bfac[j] from block j's chunk partials.
__global__ __launch_bounds__(256) void k_ball_factors(const int32_t* __restrict__ coff, const double* __restrict__ eps,
                                                      const double* __restrict__ pin, double2* __restrict__ bfac) {
  __shared__ double red[4];
  const int j = blockIdx.x;
  double t = 0.0;
  for (int k = coff[j] + int(threadIdx.x); k < coff[j + 1]; k += 256) t += pin[k];
  t = sum256(t, red);
  if (threadIdx.x == 0) bfac[j] = ball_factor(t, eps[j]);
}

// Projection factor of a data block for P_B (Sec. 3.3, eq. proj-L2):
// a workgroup sums the segment partials of ||q - y_j||^2 in a fixed order
// and stores (eps_j / r, 0) if r > eps_j, else (1, 1).
constexpr int BF_PER = 8;
// One pass of 1024 threads covers up to 8192 segments (the largest block of
// the 512^2, 1.3M workload has ~3k); 256 threads took two passes there.
constexpr int BF_THREADS = 1024;
__device__ __forceinline__ void block_factor(int j, const double* __restrict__ part, const int32_t* __restrict__ bids,
                                             const int32_t* __restrict__ boff, const double* __restrict__ eps,
                                             double2* __restrict__ bfac) {
  __shared__ double red[BF_THREADS / 64];
  const int c0 = boff[j], c1 = boff[j + 1];
  double s = 0.0;
  for (int base = c0; base < c1; base += BF_THREADS * BF_PER) {
    int id[BF_PER];
#pragma unroll
    for (int k = 0; k < BF_PER; ++k) {
      const int c = base + int(threadIdx.x) + k * BF_THREADS;
      id[k] = c < c1 ? bids[c] : -1;
    }
    double v[BF_PER];
#pragma unroll
    for (int k = 0; k < BF_PER; ++k) v[k] = id[k] >= 0 ? part[id[k]] : 0.0;
#pragma unroll
    for (int k = 0; k < BF_PER; ++k) s += v[k];
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int q = 0; q < BF_THREADS / 64; ++q) t += red[q];
    bfac[j] = ball_factor(t, eps[j]);
  }
}

__global__ __launch_bounds__(BF_THREADS) void k_block_factors(const double* __restrict__ part,
                                                              const int32_t* __restrict__ bids,
                                                              const int32_t* __restrict__ boff,
                                                              const double* __restrict__ eps,
                                                              double2* __restrict__ bfac) {
  block_factor(blockIdx.x, part, bids, boff, eps, bfac);
}

// The same after an analysis level of SARA in the first workgroups.
template <bool HW>
__global__ __launch_bounds__(BF_THREADS) void k_block_factors_dwt(const double* __restrict__ part,
                                                                  const int32_t* __restrict__ bids,
                                                                  const int32_t* __restrict__ boff,
                                                                  const double* __restrict__ eps,
                                                                  double2* __restrict__ bfac, SaraJob job) {
  const int b = int(blockIdx.x) - job.blocks();
  if (b < 0) sara_dwt_part<HW>(job, blockIdx.x);
  else block_factor(b, part, bids, boff, eps, bfac);
}

// ---- persistent middle steps of Algorithm 2 ---------------------------------
// One launch runs the n_itr - 1 middle forward-backward steps of every block
// with the per-point state (w, z, U, y) held in registers: workgroup g owns
// PER PA_THREADS consecutive plan-order points (blocks are contiguous in
// plan order, so these span at most PA_MAXB blocks; the plan checks it).  A
// step applies z <- P_B(q) with the block factors and forms the workgroup's
// partial ||q - y_j||^2 of the next q per block it touches; every workgroup
// of block j then sums the block's workgroup partials in the same fixed
// order, so all of them get the same factor.  The grid is launched only when
// all its workgroups fit the device at once.
//
// There is no grid-wide barrier: a step of block j waits only for the
// partials of block j's workgroups.  Each partial is published in a slot of
// its own with one device-scope atomic exchange and carries its step in the
// sign bit (the partials are sums of squares, so the sign is free): slot
// s mod 2 of step s holds +p when bit 1 of s is clear and -p when it is set.
// A reader of step s finds in that slot either step s's partial (ready),
// step s - 2's (the writer is behind; it can never be ahead, because its
// step s + 1 needs the reader's own step s + 1 partial) or a NaN left by the
// previous launch's reset (step 0 and 1), so the sign tells them apart.  The
// wait is bounded: a thread that has polled spin_limit times sets a give-up
// flag that every other waiter checks, all workgroups run to the end, and the
// last one out forms the steps of all blocks alone, from memory.  So the
// iterate goes to an array of its own, which the gridding then reads, and z
// stays what it was: a workgroup that has every factor stores its points (they
// are what the last one out forms, too), one that gave up stores nothing.  Other
// work on the device, and workgroups that are not resident at once, thus cost
// time only.  The last workgroup out puts NaN back into
// every slot for the next launch (the plan starts them at NaN).
#ifndef PPD_PA_SLEEP
#define PPD_PA_SLEEP 1   // s_sleep argument between polls (units of 64 clocks)
#endif
struct PaArgs {
  int steps, G, d, spin_limit, report;   // report: a give-up is told to the host
  int64_t M;
  double mu;
  const float2* v; const float2* ga; const float2* y; const double* U;
  const double2* z; double2* zout;
  const uint8_t* active;
  const int32_t* voff; const int32_t* wgb0; const int32_t* gfirst; const int32_t* glast;
  const double* eps;
  double2* bfac;
  uint64_t* part;   // [2][G][PA_MAXB] tagged partials
  uint32_t* sync;   // [1] exits, [2] give-up to report, [3] give-up flag, [4] solves by one workgroup
};

// Waits for the tagged partial in *slot; returns its value, or -1 after a
// give-up (polls exceeded here, or the flag raised elsewhere).
__device__ double pa_wait(uint64_t* slot, uint64_t tag, uint32_t* flag, int spin_limit) {
  int polls = 0;
  while (true) {
    const uint64_t b = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (b != PA_EMPTY && (b & PA_SIGN) == tag) return __longlong_as_double(int64_t(b & ~PA_SIGN));
    if ((polls & 31) == 31 && __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u)
      return -1.0;
    if (++polls > spin_limit) {
      __hip_atomic_store(flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return -1.0;
    }
#if PPD_PA_SLEEP > 0
    __builtin_amdgcn_s_sleep(PPD_PA_SLEEP);
#endif
  }
}

// All blocks' steps by one workgroup, from memory; red: 4 doubles.
__device__ __forceinline__ void pa_alone(const PaArgs& a, double* red) {
  for (int j = 0; j < a.d; ++j) {
    if (a.active && !a.active[j]) continue;   // keeps z
    double2 f = make_double2(1.0, 1.0);
    for (int s = 0; s <= a.steps; ++s) {   // 0: the first step's factor only
      double acc = 0.0;
      for (int64_t i = a.voff[j] + threadIdx.x; i < a.voff[j + 1]; i += PA_THREADS) {
        const double Ue = a.U[i], mU = a.mu * Ue;
        const double2 we = dual_arg(a.v[i], Ue, a.ga[i]);
        const float2 ye = a.y[i];
        double2 ze = s <= 1 ? a.z[i] : a.zout[i];
        if (s > 0) {
          const double qx = ze.x - mU * (ze.x - we.x), qy = ze.y - mU * (ze.y - we.y);
          ze.x = f.y != 0.0 ? qx : double(ye.x) + (qx - double(ye.x)) * f.x;
          ze.y = f.y != 0.0 ? qy : double(ye.y) + (qy - double(ye.y)) * f.x;
          a.zout[i] = ze;
        }
        const double dx = (ze.x - mU * (ze.x - we.x)) - double(ye.x);
        const double dy = (ze.y - mU * (ze.y - we.y)) - double(ye.y);
        acc += dx * dx + dy * dy;
      }
      __syncthreads();   // red is free again
      f = ball_factor(sum256(acc, red), a.eps[j]);
    }
    if (threadIdx.x == 0) a.bfac[j] = f;
  }
}

template <int PER>
__global__ __launch_bounds__(PA_THREADS) void k_alg2_persistent(PaArgs a) {
  static_assert(PA_PER_MAX % PER == 0, "shorter chunks divide the longest");
  static_assert(PA_THREADS == 256, "partials are summed over exactly 4 waves");
  __shared__ double red[PA_THREADS / 64][PA_MAXB];
  __shared__ double2 fac[PA_MAXB];
  __shared__ int act[PA_MAXB];
  __shared__ int quit;
  const int g = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & 63, wid = tid >> 6;
  const int64_t i0 = int64_t(g) * PER * PA_THREADS;
  const int64_t i1 = min(i0 + int64_t(PER) * PA_THREADS, a.M);
  const int b0 = a.wgb0[g];
  int nb = 1;
  while (nb < PA_MAXB && b0 + nb < a.d && a.voff[b0 + nb] < i1) ++nb;
  double2 w[PER], z[PER];
  double U[PER];
  float2 y[PER];
  int sl[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int64_t i = i0 + int64_t(k) * PA_THREADS + tid;
    sl[k] = -1;
    if (i < i1) {
      U[k] = a.U[i];
      w[k] = dual_arg(a.v[i], U[k], a.ga[i]);
      z[k] = a.z[i];
      y[k] = a.y[i];
      int b = 0;
      while (b + 1 < nb && i >= a.voff[b0 + b + 1]) ++b;
      sl[k] = b;
    }
  }
  // factors of the first middle step (from the degridding's partials)
  if (tid < nb) {
    fac[tid] = a.bfac[b0 + tid];
    act[tid] = !a.active || a.active[b0 + tid];
  }
  if (tid == 0) quit = 0;
  __syncthreads();
  for (int s = 0; s < a.steps; ++s) {
    double acc[PA_MAXB];
#pragma unroll
    for (int b = 0; b < PA_MAXB; ++b) acc[b] = 0.0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      if (sl[k] < 0) continue;
      const int b = sl[k];
      const double mU = a.mu * U[k];
      if (act[b]) {
        const double2 f = fac[b];
        const double qx = z[k].x - mU * (z[k].x - w[k].x), qy = z[k].y - mU * (z[k].y - w[k].y);
        z[k].x = f.y != 0.0 ? qx : double(y[k].x) + (qx - double(y[k].x)) * f.x;
        z[k].y = f.y != 0.0 ? qy : double(y[k].y) + (qy - double(y[k].y)) * f.x;
      }
      const double dx = (z[k].x - mU * (z[k].x - w[k].x)) - double(y[k].x);
      const double dy = (z[k].y - mU * (z[k].y - w[k].y)) - double(y[k].y);
      const double q2 = dx * dx + dy * dy;
#pragma unroll
      for (int bb = 0; bb < PA_MAXB; ++bb) acc[bb] += bb == b ? q2 : 0.0;
    }
    // the workgroup's partial per block, summed in a fixed order
#pragma unroll
    for (int b = 0; b < PA_MAXB; ++b) {
      const double t = wave_sum(acc[b]);
      if (lane == 0) red[wid][b] = t;
    }
    __syncthreads();
    uint64_t* part = a.part + size_t(s & 1) * size_t(a.G) * PA_MAXB;
    const uint64_t tag = (s & 2) ? PA_SIGN : 0ull;
    if (wid == 0) {
      // this wave's earlier exchanges (steps s - 1, s - 2) are acknowledged
      // before the slot of step s - 2 is overwritten
      __builtin_amdgcn_s_waitcnt(0);
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
    }
    if (tid < nb) {
      const double p = ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
      // a NaN partial (diverged data) must not read as an empty slot
      uint64_t bits = uint64_t(__double_as_longlong(p)) & ~PA_SIGN;
      if (bits == PA_EMPTY) bits |= 1ull;
      (void)__hip_atomic_exchange(&part[size_t(g) * PA_MAXB + tid], bits | tag, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
    }
    // the factors of this workgroup's blocks from all their workgroups' partials
    for (int b = 0; b < nb; ++b) {
      const int j = b0 + b;
      double t = 0.0;
      int bad = 0;
      for (int gg = a.gfirst[j] + tid; gg <= a.glast[j]; gg += PA_THREADS) {
        const double v = pa_wait(&part[size_t(gg) * PA_MAXB + (j - a.wgb0[gg])], tag, &a.sync[3], a.spin_limit);
        if (v < 0.0) bad = 1;
        else t += v;
      }
      t = wave_sum(t);
      __syncthreads();   // red is free again
      if (lane == 0) red[wid][0] = t;
      if (bad) quit = 1;
      __syncthreads();
      if (tid == 0) {
        const double r = sqrt(((red[0][0] + red[1][0]) + red[2][0]) + red[3][0]), e = a.eps[j];
        fac[b] = r > e ? make_double2(e / r, 0.0) : make_double2(1.0, 1.0);
      }
    }
    __syncthreads();
    if (quit) break;   // uniform: read after the barrier
  }
  const bool whole = !quit;   // every factor came from all workgroups of its block
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int64_t i = i0 + int64_t(k) * PA_THREADS + tid;
    if (whole && sl[k] >= 0 && act[sl[k]]) a.zout[i] = z[k];
  }
  // the last step's factors, for the final projection in the gridding:
  // stored by the first workgroup of each block (all others hold the same)
  if (whole && tid < nb && a.gfirst[b0 + tid] == g) a.bfac[b0 + tid] = fac[tid];
  // what each wave stored (partials, the flag) is acknowledged before the exit
  // is counted, so that neither the reset nor the reading of the flag can be
  // overtaken by one of them
  __shared__ int last_out, gave_up;
  __builtin_amdgcn_s_waitcnt(0);
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __syncthreads();
  if (tid == 0) {
    const uint32_t out = __hip_atomic_fetch_add(&a.sync[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last_out = out == uint32_t(a.G) - 1u;
  }
  __syncthreads();
  if (!last_out) return;
  // the last workgroup out empties every slot for the next launch and clears
  // the exit count and the flag
  for (size_t e = tid; e < 2 * size_t(a.G) * PA_MAXB; e += PA_THREADS)
    __hip_atomic_store(&a.part[e], PA_EMPTY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (tid == 0) {
    __hip_atomic_store(&a.sync[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    gave_up = int(__hip_atomic_exchange(&a.sync[3], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    if (gave_up) {
      (void)__hip_atomic_fetch_add(&a.sync[4], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (a.report) __hip_atomic_store(&a.sync[2], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __syncthreads();
  if (gave_up) pa_alone(a, &red[0][0]);
}

// ---- exact prox of eq. elip-proj-1: Newton on the secular equation ------
// With a = U |w - y| and r(nu)^2 = sum a^2 / (U + nu)^2 per block, the prox
// is (U w + nu y) / (U + nu) at the root of g(nu) = 1 / r(nu) - 1 / eps
// (nu = 0 when r(0) <= eps).  g is concave and increasing, so Newton from
// nu = 0 climbs to the root without overshooting; g'(nu) = S3 / r^3 with
// S3 = sum a^2 / (U + nu)^3.  bfac[j].x carries nu between the passes.

// A pass runs over chunks of consecutive plan-order points (newton_chunk) inside
// one block (blocks are contiguous in plan order).  The first pass forms
// a^2 = U^2 |w - y|^2 and keeps (a^2, U) per point, the later ones read only
// that (16 bytes per point); each workgroup writes its chunk's S2, S3 at the
// block's current nu, summed in a fixed order (deterministic).  A later
// pass first takes the Newton step from the previous pass's partials
// itself (every workgroup of a block computes the same value in the same
// order), so one launch per step remains; partials and nu alternate
// between two buffers, and a last k_sec_update takes the final step.
constexpr int SEC_THREADS = 256;

// nu = max(0, nu0 - g / g'), g = 1 / r - 1 / eps; 0 if nothing is left to move.
__device__ __forceinline__ double newton_step(double S2, double S3, double eps, double nu0) {
  if (!(S2 > 0.0 && S3 > 0.0)) return 0.0;
  const double r = sqrt(S2);
  const double g = 1.0 / r - 1.0 / eps, gp = S3 / (r * r * r);
  return fmax(0.0, nu0 - g / gp);
}

// Newton step of block j from its chunk partials [c0, c1).  All SEC_THREADS
// threads take part; the result is returned to every thread.
__device__ double newton_nu(const double* __restrict__ p2, const double* __restrict__ p3, int c0, int c1,
                            double eps, double nu0, double* red2, double* red3, double* out) {
  double a = 0.0, b = 0.0;
  for (int c = c0 + int(threadIdx.x); c < c1; c += SEC_THREADS) {
    a += p2[c];
    b += p3[c];
  }
  a = wave_sum(a);
  b = wave_sum(b);
  if ((threadIdx.x & 63) == 0) {
    red2[threadIdx.x >> 6] = a;
    red3[threadIdx.x >> 6] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double S2 = 0.0, S3 = 0.0;
#pragma unroll
    for (int k = 0; k < SEC_THREADS / 64; ++k) {
      S2 += red2[k];
      S3 += red3[k];
    }
    *out = newton_step(S2, S3, eps, nu0);
  }
  __syncthreads();
  return *out;
}

// FIRST: nu = 0.  Else the step from the previous partials (pp2, pp3) and
// the previous nu (pnu, NULL after the first pass); the chunk that starts
// its block stores the new nu to nnu.
template <bool FIRST>
__global__ __launch_bounds__(SEC_THREADS) void k_sec_chunk(
    const int32_t* __restrict__ cstart, const int32_t* __restrict__ cblock, const int32_t* __restrict__ coff,
    const double* __restrict__ eps, const double2* __restrict__ w, const float2* __restrict__ v,
    const float2* __restrict__ ga, const float2* __restrict__ y, const double* __restrict__ U,
    double2* __restrict__ aq, const double* __restrict__ pp2, const double* __restrict__ pp3,
    const double* __restrict__ pnu, double* __restrict__ nnu, double* __restrict__ p2, double* __restrict__ p3) {
  __shared__ double red2[SEC_THREADS / 64], red3[SEC_THREADS / 64], s_nu;
  const int c = blockIdx.x;
  const int i0 = cstart[c], i1 = cstart[c + 1];
  double nu = 0.0;
  if (!FIRST) {
    const int j = cblock[c];
    nu = newton_nu(pp2, pp3, coff[j], coff[j + 1], eps[j], pnu ? pnu[j] : 0.0, red2, red3, &s_nu);
    if (c == coff[j] && threadIdx.x == 0) nnu[j] = nu;
  }
  double t2 = 0.0, t3 = 0.0;
#pragma unroll 4
  for (int i = i0 + int(threadIdx.x); i < i1; i += SEC_THREADS) {
    double a2, Ue;
    if (FIRST) {
      Ue = U[i];
      const double2 we = w ? w[i] : dual_arg(v[i], Ue, ga[i]);
      const float2 ye = y[i];
      const double dx = we.x - double(ye.x), dy = we.y - double(ye.y);
      a2 = Ue * Ue * (dx * dx + dy * dy);
      aq[i] = make_double2(a2, Ue);
    } else {
      const double2 q = aq[i];
      a2 = q.x;
      Ue = q.y;
    }
    const double inv = 1.0 / (Ue + nu);
    const double s2 = a2 * inv * inv;
    t2 += s2;
    t3 += s2 * inv;
  }
  t2 = wave_sum(t2);
  t3 = wave_sum(t3);
  __syncthreads();   // red2 / red3 reused after newton_nu
  if ((threadIdx.x & 63) == 0) {
    red2[threadIdx.x >> 6] = t2;
    red3[threadIdx.x >> 6] = t3;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int k = 0; k < SEC_THREADS / 64; ++k) {
      a += red2[k];
      b += red3[k];
    }
    p2[c] = a;
    p3[c] = b;
  }
}

// The last Newton step: workgroup j takes it from the last pass's partials
// and stores nu_j to the block factors.
__global__ __launch_bounds__(SEC_THREADS) void k_sec_update(const double* __restrict__ p2,
                                                            const double* __restrict__ p3,
                                                            const int32_t* __restrict__ coff,
                                                            const double* __restrict__ eps,
                                                            const double* __restrict__ pnu,
                                                            double2* __restrict__ bfac) {
  __shared__ double red2[SEC_THREADS / 64], red3[SEC_THREADS / 64], s_nu;
  const int j = blockIdx.x;
  const double nu = newton_nu(p2, p3, coff[j], coff[j + 1], eps[j], pnu ? pnu[j] : 0.0, red2, red3, &s_nu);
  if (threadIdx.x == 0) bfac[j] = make_double2(nu, 0.0);
}

// The whole solve as one launch, with (a^2, U) of every point in registers and
// the tagged partials and bounded waits of k_alg2_persistent (two sums per
// block and step).  A block is done when a step leaves nu where it was: a
// relative step of 2^-50 puts r within that of eps (-g / g' >= (r / eps - 1)
// nu), and the steps left would only repeat its rounding.  So a solve costs
// the steps its blocks need, n_newton at most, and none costs a launch: at
// 512 x 256, 200003 points and 12 steps one launch of 24.5 us instead of 13 of
// 4.2 and the gaps between them; ten eager iterations 1291 -> 1065 us,
// and with one barrier a step 1008.
// A wait that gives up costs time, not the result: the workgroups run to the
// end and the last one out solves all blocks alone, from memory.  So other
// work on the device, and workgroups that are not resident at once, are no
// error.
struct SecArgs {
  int steps, G, d, spin_limit;
  int64_t M;
  const float2* v; const float2* ga; const float2* y; const double* U;
  const int32_t* voff; const int32_t* wgb0; const int32_t* gfirst; const int32_t* glast;
  const double* eps;
  double2* bfac;
  uint64_t* part;   // [2][G][PA_MAXB][2] tagged partials
  uint32_t* sync;   // [1] exits, [3] give-up flag, [4] solves by one workgroup
};

__device__ __forceinline__ double sec_a2(const SecArgs& a, int64_t i, double Ue) {
  const double2 we = dual_arg(a.v[i], Ue, a.ga[i]);
  const float2 ye = a.y[i];
  const double dx = we.x - double(ye.x), dy = we.y - double(ye.y);
  return Ue * Ue * (dx * dx + dy * dy);
}

// bfac[j].x = nu.  At device scope: after a give-up the last workgroup out
// stores once more what another one may have stored before its exit.
__device__ __forceinline__ void sec_store(const SecArgs& a, int j, double nu) {
  __hip_atomic_store(&a.bfac[j].x, nu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bool sec_done(double nu, double nu0) {
  return nu == nu0 || fabs(nu - nu0) <= 0x1p-50 * nu;
}

// Waits for the two tagged partials of a slot at once; false after a give-up.
__device__ bool sec_wait(uint64_t* slot, uint64_t tag, uint32_t* flag, int spin_limit, double& v2, double& v3) {
  int polls = 0;
  while (true) {
    const uint64_t b2 = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t b3 = __hip_atomic_load(slot + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (b2 != PA_EMPTY && b3 != PA_EMPTY && (b2 & PA_SIGN) == tag && (b3 & PA_SIGN) == tag) {
      v2 = __longlong_as_double(int64_t(b2 & ~PA_SIGN));
      v3 = __longlong_as_double(int64_t(b3 & ~PA_SIGN));
      return true;
    }
    if ((polls & 31) == 31 && __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) return false;
    if (++polls > spin_limit) {
      __hip_atomic_store(flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return false;
    }
#if PPD_PA_SLEEP > 0
    __builtin_amdgcn_s_sleep(PPD_PA_SLEEP);
#endif
  }
}

template <int PER>
__global__ __launch_bounds__(PA_THREADS) void k_sec_persistent(SecArgs a) {
  static_assert(PA_THREADS == 256, "partials are summed over exactly 4 waves");
  constexpr int WAVES = PA_THREADS / 64;
  __shared__ double red[2][WAVES][PA_MAXB][2];   // partials of the even and the odd steps
  __shared__ double s_nu[WAVES][PA_MAXB];        // every wave takes the Newton steps itself
  __shared__ int done[WAVES][PA_MAXB], left[2][WAVES], quit[2], last_out, gave_up;
  const int g = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & 63, wid = tid >> 6;
  const int64_t i0 = int64_t(g) * PER * PA_THREADS;
  const int64_t i1 = min(i0 + int64_t(PER) * PA_THREADS, a.M);
  const int b0 = a.wgb0[g];
  int nb = 1;
  while (nb < PA_MAXB && b0 + nb < a.d && a.voff[b0 + nb] < i1) ++nb;
  double a2[PER], U[PER];
  int sl[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int64_t i = i0 + int64_t(k) * PA_THREADS + tid;
    sl[k] = -1;
    a2[k] = 0.0;
    U[k] = 1.0;
    if (i < i1) {
      U[k] = a.U[i];
      a2[k] = sec_a2(a, i, U[k]);
      int b = 0;
      while (b + 1 < nb && i >= a.voff[b0 + b + 1]) ++b;
      sl[k] = b;
    }
  }
  if (lane < PA_MAXB) {
    s_nu[wid][lane] = 0.0;
    done[wid][lane] = lane >= nb;
  }
  if (tid < 2) quit[tid] = 0;
  if (lane == 0) left[1][wid] = 1;
  __syncthreads();
  // One barrier a step: behind it the waves know of each other's partials and
  // of the step before, whether a wave gave up and whether a block is left (in
  // two copies, as a wave may be a step ahead of another's reading).
  for (int s = 0; s < a.steps; ++s) {
    const int h = s & 1;
    // the workgroup's partials per block, summed in a fixed order
    for (int b = 0; b < nb; ++b) {
      if (done[wid][b]) continue;
      const double nu = s_nu[wid][b];
      double t2 = 0.0, t3 = 0.0;
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const double inv = 1.0 / (U[k] + nu);
        const double s2 = sl[k] == b ? a2[k] * inv * inv : 0.0;
        t2 += s2;
        t3 += s2 * inv;
      }
      t2 = wave_sum(t2);
      t3 = wave_sum(t3);
      if (lane == 0) {
        red[h][wid][b][0] = t2;
        red[h][wid][b][1] = t3;
      }
    }
    __syncthreads();
    if (quit[h ^ 1] || !(left[h ^ 1][0] | left[h ^ 1][1] | left[h ^ 1][2] | left[h ^ 1][3])) break;   // uniform
    uint64_t* part = a.part + size_t(h) * size_t(a.G) * (2 * PA_MAXB);
    const uint64_t tag = (s & 2) ? PA_SIGN : 0ull;
    if (wid == 0) {
      // as in k_alg2_persistent: this wave's earlier exchanges are
      // acknowledged before the slot of step s - 2 is overwritten
      __builtin_amdgcn_s_waitcnt(0);
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
    }
    if (tid < 2 * nb && !done[0][tid >> 1]) {
      const int b = tid >> 1, q = tid & 1;
      const double p = ((red[h][0][b][q] + red[h][1][b][q]) + red[h][2][b][q]) + red[h][3][b][q];
      uint64_t bits = uint64_t(__double_as_longlong(p)) & ~PA_SIGN;
      if (bits == PA_EMPTY) bits |= 1ull;   // a NaN partial must not read as an empty slot
      (void)__hip_atomic_exchange(&part[size_t(g) * (2 * PA_MAXB) + tid], bits | tag, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
    }
    // the same in every wave of every workgroup of a block
    int any = 0;
    for (int b = 0; b < nb; ++b) {
      if (done[wid][b]) continue;
      const int j = b0 + b;
      double t2 = 0.0, t3 = 0.0;
      int bad = 0;
      for (int gg = a.gfirst[j] + lane; gg <= a.glast[j] && !bad; gg += 64) {
        double v2, v3;
        if (sec_wait(&part[size_t(gg) * (2 * PA_MAXB) + 2 * (j - a.wgb0[gg])], tag, &a.sync[3], a.spin_limit, v2, v3)) {
          t2 += v2;
          t3 += v3;
        } else {
          bad = 1;
        }
      }
      t2 = wave_sum(t2);
      t3 = wave_sum(t3);
      if (bad) quit[h] = 1;
      const double nu0 = s_nu[wid][b], nu = newton_step(t2, t3, a.eps[j], nu0);
      const bool end = sec_done(nu, nu0);
      any |= !end;
      wave_sync();   // every lane has read the wave's nu
      if (lane == 0) {
        s_nu[wid][b] = nu;
        done[wid][b] = end;
      }
      wave_sync();
    }
    if (lane == 0) left[h][wid] = any;
  }
  __syncthreads();
  // stored by the first workgroup of each block (all others hold the same)
  if (tid < nb && a.gfirst[b0 + tid] == g && !(quit[0] | quit[1])) sec_store(a, b0 + tid, s_nu[0][tid]);
  // what each wave stored (partials, results, the flag) is acknowledged before
  // the exit is counted
  __builtin_amdgcn_s_waitcnt(0);
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __syncthreads();
  if (tid == 0) {
    const uint32_t out = __hip_atomic_fetch_add(&a.sync[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last_out = out == uint32_t(a.G) - 1u;
  }
  __syncthreads();
  if (!last_out) return;
  // the last workgroup out empties every slot for the next launch and clears
  // the exit count and the flag
  for (size_t e = tid; e < 4 * size_t(a.G) * PA_MAXB; e += PA_THREADS)
    __hip_atomic_store(&a.part[e], PA_EMPTY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (tid == 0) {
    __hip_atomic_store(&a.sync[1], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    gave_up = int(__hip_atomic_exchange(&a.sync[3], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    if (gave_up) (void)__hip_atomic_fetch_add(&a.sync[4], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!gave_up) return;
  for (int j = 0; j < a.d; ++j) {
    double nu = 0.0;
    for (int s = 0; s < a.steps; ++s) {
      double t2 = 0.0, t3 = 0.0;
      for (int64_t i = a.voff[j] + tid; i < a.voff[j + 1]; i += PA_THREADS) {
        const double Ue = a.U[i], inv = 1.0 / (Ue + nu), s2 = sec_a2(a, i, Ue) * inv * inv;
        t2 += s2;
        t3 += s2 * inv;
      }
      t2 = wave_sum(t2);
      t3 = wave_sum(t3);
      __syncthreads();
      if (lane == 0) {
        red[0][wid][0][0] = t2;
        red[0][wid][0][1] = t3;
      }
      __syncthreads();
      const double nu0 = nu;
      nu = newton_step(((red[0][0][0][0] + red[0][1][0][0]) + red[0][2][0][0]) + red[0][3][0][0],
                       ((red[0][0][0][1] + red[0][1][0][1]) + red[0][2][0][1]) + red[0][3][0][1], a.eps[j], nu0);
      if (sec_done(nu, nu0)) break;   // the same in every thread
    }
    if (tid == 0) sec_store(a, j, nu);
  }
}

// z = (U w + nu y) / (U + nu) with the block's nu (z = w when nu = 0).
__global__ void k_prox_apply(int64_t M, const int32_t* __restrict__ vblk, const double2* __restrict__ w,
                             const float2* __restrict__ y, const double* __restrict__ U,
                             const double2* __restrict__ bfac, double2* __restrict__ z) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < M; i += int64_t(gridDim.x) * blockDim.x) {
    const double nu = bfac[vblk[i]].x, Ue = U[i];
    const double2 we = w[i];
    const float2 ye = y[i];
    const double inv = 1.0 / (Ue + nu);
    z[i] = nu == 0.0 ? we   // inside the ellipsoid: the prox is w itself
                     : make_double2((Ue * we.x + nu * double(ye.x)) * inv, (Ue * we.y + nu * double(ye.y)) * inv);
  }
}

// ---- plain form: one block at a time, each step its own launch ---------
constexpr int PL_THREADS = 256;
constexpr int PL_MAX_BLOCKS = 512;

// w = U^-1 v + yhat, and partials of ||yhat - y||^2 (residual statistics)
__global__ void k_pl_w(int64_t b0, int64_t b1, const float2* __restrict__ v, const double* __restrict__ U,
                       const float2* __restrict__ yhat, const float2* __restrict__ y,
                       double2* __restrict__ w, double* __restrict__ part) {
  __shared__ double red[16];
  double rn = 0.0;
  for (int64_t i = b0 + blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < b1; i += int64_t(gridDim.x) * blockDim.x) {
    const float2 ve = v[i], g = yhat[i], ye = y[i];
    const double Ue = U[i];
    w[i] = dual_arg(ve, Ue, g);
    const double ex = double(g.x) - double(ye.x), ey = double(g.y) - double(ye.y);
    rn += ex * ex + ey * ey;
  }
  rn = block_sum(rn, red);
  if (threadIdx.x == 0) part[blockIdx.x] = rn;
}

// q = z - mu U (z - w) and partials of ||q - y||^2
__global__ void k_pl_q(int64_t b0, int64_t b1, const double2* __restrict__ w, const double2* __restrict__ z,
                       const double* __restrict__ U, const float2* __restrict__ y, double mu,
                       double2* __restrict__ q, double* __restrict__ part) {
  __shared__ double red[16];
  double qn = 0.0;
  for (int64_t i = b0 + blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < b1; i += int64_t(gridDim.x) * blockDim.x) {
    const double2 we = w[i], ze = z[i];
    const double mU = mu * U[i];
    const double qx = ze.x - mU * (ze.x - we.x), qy = ze.y - mU * (ze.y - we.y);
    q[i] = make_double2(qx, qy);
    const float2 ye = y[i];
    const double dx = qx - double(ye.x), dy = qy - double(ye.y);
    qn += dx * dx + dy * dy;
  }
  qn = block_sum(qn, red);
  if (threadIdx.x == 0) part[blockIdx.x] = qn;
}

// out[slot] = sum of n partials (one wave, fixed order)
__global__ void k_pl_reduce(const double* __restrict__ part, int n, double* __restrict__ out, int slot) {
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 64) s += part[i];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (threadIdx.x == 0) out[slot] = s;
}

// z = P_B(q) (Sec. 3.3, eq. proj-L2) with ||q - y||^2 in *norm2
__global__ void k_pl_proj(int64_t b0, int64_t b1, const double2* __restrict__ q, const float2* __restrict__ y,
                          const double* __restrict__ norm2, const double* __restrict__ eps, int j,
                          double2* __restrict__ z) {
  const double r = sqrt(*norm2), e = eps[j];
  const bool inside = r <= e;
  const double f = inside ? 1.0 : e / r;
  for (int64_t i = b0 + blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < b1; i += int64_t(gridDim.x) * blockDim.x) {
    const double2 qe = q[i];
    if (inside) {
      z[i] = qe;
    } else {
      const float2 ye = y[i];
      z[i] = make_double2(double(ye.x) + (qe.x - double(ye.x)) * f, double(ye.y) + (qe.y - double(ye.y)) * f);
    }
  }
}

// vbar = U (w - z); v <- v + lambda (vbar - v)
__global__ void k_pl_finish(int64_t b0, int64_t b1, const double2* __restrict__ w, const double2* __restrict__ z,
                            const double* __restrict__ U, double lambda, float2* __restrict__ v) {
  for (int64_t i = b0 + blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < b1; i += int64_t(gridDim.x) * blockDim.x) {
    const double2 we = w[i], ze = z[i];
    const double Ue = U[i];
    const float2 vo = v[i];
    const double vbx = Ue * (we.x - ze.x), vby = Ue * (we.y - ze.y);
    v[i] = make_float2(float(double(vo.x) + lambda * (vbx - double(vo.x))),
                       float(double(vo.y) + lambda * (vby - double(vo.y))));
  }
}

// ---- uniform-weighting preconditioner ----------------------------------
__device__ __forceinline__ int density_cell(float w, int n) {
  // floor((w + pi) n / (2 pi)), evaluated exactly in this order, clamped
  const double a = __dadd_rn(double(w), M_PI);
  const double b = __dmul_rn(a, double(n));
  const double c = __ddiv_rn(b, 2.0 * M_PI);
  int i = int(floor(c));
  return i < 0 ? 0 : (i > n - 1 ? n - 1 : i);
}

__global__ void k_hist(const float* __restrict__ wu, const float* __restrict__ wv, int64_t M, int nx, int ny,
                       int32_t* __restrict__ counts) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < M; i += int64_t(gridDim.x) * blockDim.x) {
    const int cu = density_cell(wu[i], nx), cv = density_cell(wv[i], ny);
    atomicAdd(&counts[cv * nx + cu], 1);
  }
}

__global__ void k_hist_min(const float* __restrict__ wu, const float* __restrict__ wv, int64_t M, int nx, int ny,
                           const int32_t* __restrict__ counts, int32_t* __restrict__ cmin) {
  int m = 0x7fffffff;
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < M; i += int64_t(gridDim.x) * blockDim.x) {
    const int cu = density_cell(wu[i], nx), cv = density_cell(wv[i], ny);
    m = min(m, counts[cv * nx + cu]);
  }
  for (int o = 32; o > 0; o >>= 1) m = min(m, __shfl_xor(m, o));
  if ((threadIdx.x & 63) == 0) atomicMin(cmin, m);
}

__global__ void k_hist_u(const float* __restrict__ wu, const float* __restrict__ wv, int64_t M, int nx, int ny,
                         const int32_t* __restrict__ counts, const int32_t* __restrict__ cmin,
                         double* __restrict__ U) {
  const double c0 = double(*cmin);
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < M; i += int64_t(gridDim.x) * blockDim.x) {
    const int cu = density_cell(wu[i], nx), cv = density_cell(wv[i], ny);
    U[i] = c0 / double(counts[cv * nx + cu]);
  }
}

__global__ void k_fill_i32(int32_t* __restrict__ a, int64_t n, int32_t v) {
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) a[i] = v;
}

int grid_blocks(int64_t n) { return int(std::min<int64_t>((n + PL_THREADS - 1) / PL_THREADS, PL_MAX_BLOCKS)); }

}  // namespace

int ball_factors(ppd_plan* p, const double* pin) {
  int slot;
  PPD_TRY(timer_begin(p, KK_MISC, &slot));
  hipLaunchKernelGGL(k_ball_factors, dim3(p->d), dim3(256), 0, p->stream, p->sec_coff, p->eps_d, pin, p->bfac);
  PPD_HIP(hipGetLastError());
  return timer_end(p, slot);
}

int ball_step(ppd_plan* p, const BallIn& in, double2* z, const double2* fac, const double* pin, double* pout) {
  if (pin && !fac && !p->own_sums) {   // blocks of too many chunks for every workgroup to add up
    PPD_TRY(ball_factors(p, pin));
    fac = p->bfac;
  }
  int slot;
  PPD_TRY(timer_begin(p, KK_SUBITER, &slot));
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(p->n_sec_chunks), dim3(256), 0, p->stream, in, p->sec_cstart, p->sec_cblock,
                       p->sec_coff, p->eps_d, fac, pin, z, pout);
  };
  if (!fac && !pin) launch(k_ball_step<false, true>);
  else if (pout) launch(k_ball_step<true, true>);
  else launch(k_ball_step<true, false>);
  PPD_HIP(hipGetLastError());
  return timer_end(p, slot);
}

using SecKernel = void (*)(SecArgs);
static SecKernel sec_kernel(int per) {
  return per == 2 ? k_sec_persistent<2> : per == 4 ? k_sec_persistent<4> : k_sec_persistent<PA_PER_MAX>;
}

// Workgroups of a persistent kernel that the device holds at once.
static int resident_groups(const void* kernel) {
  int dev = 0, cus = 0, blocks = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, kernel, PA_THREADS, 0) != hipSuccess) return 0;
  return cus * blocks;
}

int sec_persistent_capacity(int per) { return resident_groups(reinterpret_cast<const void*>(sec_kernel(per))); }

static int secular_persistent(ppd_plan* p, const float2* v, const float2* ga, const float2* y, const double* U,
                              int n_newton, int spin_limit) {
  const SecArgs a{n_newton, p->pa_groups, p->d, spin_limit > 0 ? spin_limit : PA_SPIN, p->M, v, ga, y, U,
                  p->voff_d, p->pa_wgb0, p->pa_gfirst, p->pa_glast, p->eps_d, p->bfac, p->pa_part, p->pa_sync};
  int slot;
  PPD_TRY(timer_begin(p, KK_SUBITER, &slot));
  hipLaunchKernelGGL(sec_kernel(p->pa_per), dim3(a.G), dim3(PA_THREADS), 0, p->stream, a);
  PPD_HIP(hipGetLastError());
  return timer_end(p, slot);
}

int secular_solve(ppd_plan* p, const double2* w, const float2* v, const float2* ga, const float2* y,
                  const double* U, int n_newton, bool persistent, int spin_limit) {
  if (persistent && p->sec_ok) return secular_persistent(p, v, ga, y, U, n_newton, spin_limit);
  // pass s writes its partials to buffer s & 1 and (s >= 1) its nu to
  // nu buffer s & 1
  const int nc = p->n_nw_chunks;
  double* part[2] = {p->sec_part, p->sec_part + 2 * nc};
  double* nub[2] = {p->sec_nu, p->sec_nu + p->d};
  for (int s = 0; s < n_newton; ++s) {
    double* p2 = part[s & 1];
    double* p3 = part[s & 1] + nc;
    const double* q2 = part[(s + 1) & 1];
    const double* q3 = part[(s + 1) & 1] + nc;
    const double* pnu = s >= 2 ? nub[(s + 1) & 1] : nullptr;
    int slot;
    PPD_TRY(timer_begin(p, KK_SUBITER, &slot));
    if (s == 0)
      hipLaunchKernelGGL(k_sec_chunk<true>, dim3(nc), dim3(SEC_THREADS), 0, p->stream, p->nw_cstart, p->nw_cblock,
                         p->nw_coff, p->eps_d, w, v, ga, y, U, p->qbuf, nullptr, nullptr, nullptr, nullptr, p2, p3);
    else
      hipLaunchKernelGGL(k_sec_chunk<false>, dim3(nc), dim3(SEC_THREADS), 0, p->stream, p->nw_cstart,
                         p->nw_cblock, p->nw_coff, p->eps_d, w, v, ga, y, U, p->qbuf, q2, q3, pnu, nub[s & 1], p2,
                         p3);
    PPD_HIP(hipGetLastError());
    PPD_TRY(timer_end(p, slot));
  }
  const int last = n_newton - 1;
  int slot;
  PPD_TRY(timer_begin(p, KK_MISC, &slot));
  hipLaunchKernelGGL(k_sec_update, dim3(p->d), dim3(SEC_THREADS), 0, p->stream, part[last & 1],
                     part[last & 1] + nc, p->nw_coff, p->eps_d, last >= 1 ? nub[last & 1] : nullptr, p->bfac);
  PPD_HIP(hipGetLastError());
  return timer_end(p, slot);
}

using PaKernel = void (*)(PaArgs);
static PaKernel pa_kernel(int per) {
  return per == 2 ? k_alg2_persistent<2> : per == 4 ? k_alg2_persistent<4> : k_alg2_persistent<PA_PER_MAX>;
}

int alg2_persistent_capacity(int per) { return resident_groups(reinterpret_cast<const void*>(pa_kernel(per))); }

int alg2_persistent(ppd_plan* p, const DualArgs& a, int spin_limit) {
  if (!p->pa_ok) return fail(PPD_EUNSUPPORTED, "persistent Algorithm 2 is not available for this plan");
  PaArgs pa;
  pa.steps = a.n_itr - 1;
  pa.G = p->pa_groups;
  pa.d = p->d;
  pa.spin_limit = spin_limit > 0 ? spin_limit : PA_SPIN;
  pa.report = spin_limit > 0;
  pa.M = p->M;
  pa.mu = a.mu;
  pa.v = a.v;
  pa.ga = p->gabuf;
  pa.y = a.y;
  pa.U = a.U;
  pa.z = a.z;
  pa.zout = p->qbuf;
  pa.active = a.active;
  pa.voff = p->voff_d;
  pa.wgb0 = p->pa_wgb0;
  pa.gfirst = p->pa_gfirst;
  pa.glast = p->pa_glast;
  pa.eps = p->eps_d;
  pa.bfac = p->bfac;
  pa.part = p->pa_part;
  pa.sync = p->pa_sync;
  int slot;
  PPD_TRY(timer_begin(p, KK_SUBITER, &slot));
  hipLaunchKernelGGL(pa_kernel(p->pa_per), dim3(pa.G), dim3(PA_THREADS), 0, p->stream, pa);
  PPD_HIP(hipGetLastError());
  return timer_end(p, slot);
}

int block_factors(ppd_plan* p, const double* part, const SaraJob* with) {
  int slot;
  PPD_TRY(timer_begin(p, KK_MISC, &slot));
  if (with)
    hipLaunchKernelGGL((with->W ? k_block_factors_dwt<true> : k_block_factors_dwt<false>), dim3(p->d + with->blocks()), dim3(BF_THREADS), 0, p->stream, part,
                       p->bseg_ids, p->bseg_off_d, p->eps_d, p->bfac, *with);
  else
    hipLaunchKernelGGL(k_block_factors, dim3(p->d), dim3(BF_THREADS), 0, p->stream, part, p->bseg_ids, p->bseg_off_d,
                       p->eps_d, p->bfac);
  PPD_HIP(hipGetLastError());
  return timer_end(p, slot);
}

// Unfused reference form of the data-dual update: per block, per sub-iteration,
// separate FP64 launches.  Expects Theta G F Z x~ in p->ybuf (plan order).
int plain_dual(ppd_plan* p, const DualArgs& a) {
  for (int j = 0; j < p->d; ++j) {
    const int64_t b0 = p->block_off[j], b1 = p->block_off[j + 1];
    const int G = grid_blocks(b1 - b0);
    int slot;
    PPD_TRY(timer_begin(p, KK_PLAIN_DUAL, &slot));
    hipLaunchKernelGGL(k_pl_w, dim3(G), dim3(PL_THREADS), 0, p->stream, b0, b1, a.v, a.U, p->ybuf, a.y,
                       p->wbuf, p->pl_part);
    hipLaunchKernelGGL(k_pl_reduce, dim3(1), dim3(64), 0, p->stream, p->pl_part, G, p->res_sq, j);
    for (int s = 0; s < a.n_itr; ++s) {
      hipLaunchKernelGGL(k_pl_q, dim3(G), dim3(PL_THREADS), 0, p->stream, b0, b1, p->wbuf, a.z, a.U, a.y,
                         a.mu, p->qbuf, p->pl_part);
      hipLaunchKernelGGL(k_pl_reduce, dim3(1), dim3(64), 0, p->stream, p->pl_part, G, p->pl_scalar, 0);
      hipLaunchKernelGGL(k_pl_proj, dim3(G), dim3(PL_THREADS), 0, p->stream, b0, b1, p->qbuf, a.y,
                         p->pl_scalar, p->eps_d, j, a.z);
    }
    hipLaunchKernelGGL(k_pl_finish, dim3(G), dim3(PL_THREADS), 0, p->stream, b0, b1, p->wbuf, a.z, a.U,
                       a.lambda, a.v);
    PPD_HIP(hipGetLastError());
    PPD_TRY(timer_end(p, slot));
  }
  return PPD_OK;
}

}  // namespace ppd

using namespace ppd;

extern "C" int ppd_ellipsoid_proj(ppd_plan* p, const double* w, const float* y, const double* U,
                                  const double* eps, int n_itr, double mu, double* zbar) {
  if (!p || !w || !y || !U || !eps || !zbar) return fail(PPD_EINVAL, "ppd_ellipsoid_proj: NULL argument");
  if (n_itr < 1) return fail(PPD_EINVAL, "ppd_ellipsoid_proj: n_itr must be >= 1");
  if (!(mu > 0.0) || !std::isfinite(mu)) return fail(PPD_EINVAL, "ppd_ellipsoid_proj: mu must be > 0");
  PPD_TRY(upload_eps(p, eps));
  const BallIn in{reinterpret_cast<const double2*>(w), nullptr, nullptr, reinterpret_cast<const float2*>(y), U, mu,
                  nullptr};
  double2* z2 = reinterpret_cast<double2*>(zbar);
  double* part[2] = {p->sec_part, p->sec_part + p->n_sec_chunks};
  PPD_TRY(ball_step(p, in, z2, nullptr, nullptr, part[0]));
  for (int s = 1; s < n_itr; ++s) PPD_TRY(ball_step(p, in, z2, nullptr, part[(s - 1) & 1], part[s & 1]));
  return ball_step(p, in, z2, nullptr, part[(n_itr - 1) & 1], nullptr);
}

extern "C" int ppd_prox_metric(ppd_plan* p, const double* w, const float* y, const double* U, const double* eps,
                               int n_newton, double* z, double* nu) {
  if (!p || !w || !y || !U || !eps || !z) return fail(PPD_EINVAL, "ppd_prox_metric: NULL argument");
  if (n_newton < 1 || n_newton > 64) return fail(PPD_EINVAL, "ppd_prox_metric: n_newton must be in [1, 64]");
  PPD_TRY(upload_eps(p, eps));
  const double2* w2 = reinterpret_cast<const double2*>(w);
  const float2* y2 = reinterpret_cast<const float2*>(y);
  // step by step: nothing here could turn the waits of the one launch off
  PPD_TRY(secular_solve(p, w2, nullptr, nullptr, y2, U, n_newton, false, 0));
  int slot;
  PPD_TRY(timer_begin(p, KK_MISC, &slot));
  hipLaunchKernelGGL(k_prox_apply, dim3(int(std::min<int64_t>((p->M + 255) / 256, 4096))), dim3(256), 0, p->stream,
                     p->M, p->vis_block, w2, y2, U, p->bfac, reinterpret_cast<double2*>(z));
  PPD_HIP(hipGetLastError());
  PPD_TRY(timer_end(p, slot));
  if (nu) {
    PPD_HIP(hipMemcpy2DAsync(nu, sizeof(double), p->bfac, sizeof(double2), sizeof(double), p->d,
                             hipMemcpyDeviceToDevice, p->stream));
  }
  return PPD_OK;
}

extern "C" int ppd_uniform_weights(ppd_plan* p, double* U) {
  if (!p || !U) return fail(PPD_EINVAL, "ppd_uniform_weights: NULL argument");
  int slot;
  PPD_TRY(timer_begin(p, KK_HIST, &slot));
  const int64_t N = int64_t(p->nx) * p->ny;
  const int gb = int(std::min<int64_t>((p->M + 255) / 256, 2048));
  hipLaunchKernelGGL(k_fill_i32, dim3(int(std::min<int64_t>((N + 255) / 256, 2048))), dim3(256), 0,
                     p->stream, p->icount, N, 0);
  hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, p->stream, p->imin, int64_t(1), 0x7fffffff);
  hipLaunchKernelGGL(k_hist, dim3(gb), dim3(256), 0, p->stream, p->wu, p->wv, p->M, p->nx, p->ny, p->icount);
  hipLaunchKernelGGL(k_hist_min, dim3(gb), dim3(256), 0, p->stream, p->wu, p->wv, p->M, p->nx, p->ny,
                     p->icount, p->imin);
  hipLaunchKernelGGL(k_hist_u, dim3(gb), dim3(256), 0, p->stream, p->wu, p->wv, p->M, p->nx, p->ny,
                     p->icount, p->imin, U);
  PPD_HIP(hipGetLastError());
  return timer_end(p, slot);
}
