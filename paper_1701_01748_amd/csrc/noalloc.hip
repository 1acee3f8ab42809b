// Algorithm 2 (Sec. 4.1) without any device allocation: the same
// forward-backward iterations as ppd_ellipsoid_proj, for callers that
// cannot allocate (graph capture, serving loops), with every intermediate
// in one file-scope device array instead of a plan's buffers.
//
// The visibilities of block j are the contiguous range
// [block_off[j], block_off[j+1]); each block is cut into chunks of
// consecutive points, one workgroup each: 512 points up to 2048 chunks, twice
// as many while there are more, at most 8192.  A step applies z <- P_B(q) and
// forms, per chunk, the partial sum of ||q - y_j||^2 of the next
// q = z - mu U (z - w); every workgroup of a block adds up the previous
// step's partials itself, in the same order, so a step is one launch (a block
// of more than NA_OWN_SUM chunks has its sum formed by a launch between).  All
// partial and factor slots are written before they are read in every call, so
// nothing has to start at zero.  Up to NA_ARG_BLOCKS blocks the block tables
// are kernel arguments: nothing is copied, and a captured call holds them.
//
// Bound by the launches' latency at the sizes of one observation: 307,780
// points in 7 blocks, 5 steps, took 98 us as 3 table copies and 11 launches of
// 41 workgroups, now 31 us as 6 launches of 603.
#include <algorithm>
#include <mutex>

#include "ppd_internal.h"

namespace ppd {
namespace {

constexpr int NA_CHUNK = 8192;        // most points per workgroup
constexpr int NA_MIN_CHUNK = 512;
constexpr int NA_FILL_CHUNKS = 2048;  // chunks that fill the chip
constexpr int NA_OWN_SUM = 4096;      // partials of a block that every workgroup adds up itself
constexpr int NA_ARG_BLOCKS = 64;
constexpr int NA_THREADS = 256;
constexpr int NA_MAX_BLOCKS = 4096;
constexpr int NA_MAX_CHUNKS = 65536;

// Layout of the array (byte offsets): eps [d] f64, block offsets [d+1] i64,
// chunk offsets [d+1] i32 (chunks of block j: [coff[j], coff[j+1])), block
// factors [d] (factor, inside) f64 pairs, two buffers of chunk partials
// [n_chunks] f64 (steps alternate).
constexpr size_t NA_OFF_EPS = 0;
constexpr size_t NA_OFF_BOFF = NA_OFF_EPS + 8 * NA_MAX_BLOCKS;
constexpr size_t NA_OFF_COFF = NA_OFF_BOFF + 8 * (NA_MAX_BLOCKS + 1);
constexpr size_t NA_OFF_FAC = (NA_OFF_COFF + 4 * (NA_MAX_BLOCKS + 1) + 255) / 256 * 256;
constexpr size_t NA_OFF_PART = NA_OFF_FAC + 16 * NA_MAX_BLOCKS;
constexpr size_t NA_BYTES = NA_OFF_PART + 2 * 8 * NA_MAX_CHUNKS;

// One copy per GPU, held until the process ends (about 1.2 MiB).  Host code
// never uses this name as an address: it takes the device address from
// hipGetSymbolAddress once per device (see scratch_for_device).
static __device__ __align__(256) unsigned char scratch[NA_BYTES];

// Block tables of a call: as a kernel argument, or in the array.
struct NaArgs {
  int64_t boff[NA_ARG_BLOCKS + 1];
  double eps[NA_ARG_BLOCKS];
  int32_t coff[NA_ARG_BLOCKS + 1];
};
struct NaNone {};

struct NaView {
  const double* eps;
  const int64_t* boff;
  const int32_t* coff;
  double2* fac;
  double* part;
};

__device__ __forceinline__ NaView na_view(unsigned char* base) {
  return {reinterpret_cast<const double*>(base + NA_OFF_EPS), reinterpret_cast<const int64_t*>(base + NA_OFF_BOFF),
          reinterpret_cast<const int32_t*>(base + NA_OFF_COFF), reinterpret_cast<double2*>(base + NA_OFF_FAC),
          reinterpret_cast<double*>(base + NA_OFF_PART)};
}
__device__ __forceinline__ NaView na_tables(const NaArgs& t, unsigned char* base) {
  NaView s = na_view(base);
  s.eps = t.eps;
  s.boff = t.boff;
  s.coff = t.coff;
  return s;
}
__device__ __forceinline__ NaView na_tables(const NaNone&, unsigned char* base) { return na_view(base); }

// Sum over the workgroup in a fixed order, in every thread.
__device__ __forceinline__ double na_block_sum(double v, double* red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int k = 0; k < NA_THREADS / 64; ++k) s += red[k];
  return s;
}

// P_B factor from the block's squared norm: (eps / r, 0) if r > eps, else
// (1, 1) (Sec. 3.3, eq. proj-L2).
__device__ __forceinline__ double2 na_factor(double r2, double e) {
  const double r = sqrt(r2);
  return r > e ? make_double2(e / r, 0.0) : make_double2(1.0, 1.0);
}

// mode 0: partials of ||q - y||^2 from z; mode 1: z <- P_B(q), then partials
// of the next q; mode 2: z <- P_B(q) only.  The factors are those of the
// partials in buffer `from`, or with own = 0 the ones stored.
template <typename Tab>
__global__ __launch_bounds__(NA_THREADS) void k_na_step(int mode, int own, int from, int chunk, int d, Tab tab,
                                                        const double2* __restrict__ w,
                                                        const float2* __restrict__ y, const double* __restrict__ U,
                                                        double2* __restrict__ z, double mu,
                                                        unsigned char* __restrict__ base) {
  __shared__ double red[2 * (NA_THREADS / 64)];
  const NaView s = na_tables(tab, base);
  const int c = blockIdx.x;
  int lo = 0, hi = d;   // the block of chunk c: the last j with coff[j] <= c
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (s.coff[mid] <= c) lo = mid;
    else hi = mid;
  }
  const int j = lo;
  const int64_t i0 = s.boff[j] + int64_t(c - s.coff[j]) * chunk;
  const int64_t i1 = min(i0 + chunk, s.boff[j + 1]);
  double2 bf = make_double2(1.0, 1.0);
  if (mode != 0) {
    if (own) {
      const double* pin = s.part + size_t(from) * NA_MAX_CHUNKS;
      double t = 0.0;
      for (int k = s.coff[j] + int(threadIdx.x); k < s.coff[j + 1]; k += NA_THREADS) t += pin[k];
      bf = na_factor(na_block_sum(t, red), s.eps[j]);
    } else {
      bf = s.fac[j];
    }
  }
  double acc = 0.0;
#pragma unroll 2
  for (int64_t i = i0 + threadIdx.x; i < i1; i += NA_THREADS) {
    const double Ue = U[i], mU = mu * Ue;
    const double2 we = w[i];
    const float2 ye = y[i];
    double2 ze = z[i];
    if (mode != 0) {
      const double qx = ze.x - mU * (ze.x - we.x), qy = ze.y - mU * (ze.y - we.y);
      ze.x = bf.y != 0.0 ? qx : double(ye.x) + (qx - double(ye.x)) * bf.x;
      ze.y = bf.y != 0.0 ? qy : double(ye.y) + (qy - double(ye.y)) * bf.x;
      z[i] = ze;
    }
    if (mode != 2) {
      const double dx = (ze.x - mU * (ze.x - we.x)) - double(ye.x);
      const double dy = (ze.y - mU * (ze.y - we.y)) - double(ye.y);
      acc += dx * dx + dy * dy;
    }
  }
  if (mode != 2) {
    acc = na_block_sum(acc, red + NA_THREADS / 64);
    if (threadIdx.x == 0) s.part[size_t(mode == 0 ? 0 : 1 - from) * NA_MAX_CHUNKS + c] = acc;
  }
}

// Block j's factor from its chunk partials in buffer `from`, stored.
template <typename Tab>
__global__ __launch_bounds__(NA_THREADS) void k_na_factors(int from, Tab tab, unsigned char* __restrict__ base) {
  __shared__ double red[NA_THREADS / 64];
  const NaView s = na_tables(tab, base);
  const int j = blockIdx.x;
  double acc = 0.0;
  for (int c = s.coff[j] + int(threadIdx.x); c < s.coff[j + 1]; c += NA_THREADS)
    acc += s.part[size_t(from) * NA_MAX_CHUNKS + c];
  acc = na_block_sum(acc, red);
  if (threadIdx.x == 0) s.fac[j] = na_factor(acc, s.eps[j]);
}

struct NaCall {
  int d, n_itr, chunk, nchunks, own;
  const double2* w; const float2* y; const double* U; double2* z;
  double mu;
  unsigned char* base;
  hipStream_t stream;
};

template <typename Tab>
int na_run(const NaCall& a, const Tab& tab) {
  for (int k = 0; k <= a.n_itr; ++k) {
    const int mode = k == 0 ? 0 : k < a.n_itr ? 1 : 2, from = (k + 1) & 1;
    if (k > 0 && !a.own)
      hipLaunchKernelGGL(k_na_factors<Tab>, dim3(a.d), dim3(NA_THREADS), 0, a.stream, from, tab, a.base);
    hipLaunchKernelGGL(k_na_step<Tab>, dim3(a.nchunks), dim3(NA_THREADS), 0, a.stream, mode, a.own, from, a.chunk, a.d,
                       tab, a.w, a.y, a.U, a.z, a.mu, a.base);
  }
  PPD_HIP(hipGetLastError());
  return PPD_OK;
}

constexpr int NA_MAX_DEVICES = 64;
std::mutex g_na_mutex;
unsigned char* g_na_ptr[NA_MAX_DEVICES] = {};

// The device address of `scratch` on the current device, looked up once per
// device with that device current.
int scratch_for_device(unsigned char** out) {
  int dev = 0;
  PPD_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= NA_MAX_DEVICES) return fail(PPD_EUNSUPPORTED, "device index beyond the supported count");
  std::lock_guard<std::mutex> lock(g_na_mutex);
  if (!g_na_ptr[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(PPD_EDEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    g_na_ptr[dev] = static_cast<unsigned char*>(ptr);
  }
  *out = g_na_ptr[dev];
  return PPD_OK;
}

}  // namespace
}  // namespace ppd

using namespace ppd;

extern "C" int ppd_ellipsoid_proj_noalloc(const double* w, const float* y, const double* U, int32_t d,
                                          const int64_t* block_off, const double* eps, int n_itr, double mu,
                                          double* zbar, void* stream) {
  if (!w || !y || !U || !block_off || !eps || !zbar)
    return fail(PPD_EINVAL, "ppd_ellipsoid_proj_noalloc: NULL argument");
  if (d < 1 || d > NA_MAX_BLOCKS)
    return fail(PPD_EINVAL, "ppd_ellipsoid_proj_noalloc: d must be in [1, " + std::to_string(NA_MAX_BLOCKS) + "]");
  if (n_itr < 1) return fail(PPD_EINVAL, "ppd_ellipsoid_proj_noalloc: n_itr must be >= 1");
  if (!(mu > 0.0) || !std::isfinite(mu)) return fail(PPD_EINVAL, "ppd_ellipsoid_proj_noalloc: mu must be > 0");
  if (block_off[0] != 0) return fail(PPD_EINVAL, "ppd_ellipsoid_proj_noalloc: block_off[0] must be 0");
  int32_t coff[NA_MAX_BLOCKS + 1];
  coff[0] = 0;
  for (int j = 0; j < d; ++j) {
    const int64_t mj = block_off[j + 1] - block_off[j];
    if (mj < 1) return fail(PPD_EINVAL, "ppd_ellipsoid_proj_noalloc: block_off must be strictly increasing");
    if (block_off[j + 1] >= (int64_t(1) << 40))
      return fail(PPD_EINVAL, "ppd_ellipsoid_proj_noalloc: too many visibilities");
    if (!(eps[j] > 0.0) || !std::isfinite(eps[j]))
      return fail(PPD_EINVAL, "ppd_ellipsoid_proj_noalloc: eps must be finite and > 0");
    const int64_t nc = coff[j] + (mj + NA_CHUNK - 1) / NA_CHUNK;
    if (nc > NA_MAX_CHUNKS)
      return fail(PPD_EINVAL, "ppd_ellipsoid_proj_noalloc: more than " + std::to_string(NA_MAX_CHUNKS) +
                                  " chunks of " + std::to_string(NA_CHUNK) + " points (about " +
                                  std::to_string(int64_t(NA_MAX_CHUNKS) * NA_CHUNK) + " visibilities)");
    coff[j + 1] = int32_t(nc);
  }
  NaCall c{};
  c.d = d;
  c.n_itr = n_itr;
  c.chunk = NA_CHUNK;
  for (int len = NA_MIN_CHUNK; len < NA_CHUNK; len *= 2) {   // the shortest chunks that do not overfill the chip
    int64_t n = 0;
    for (int j = 0; j < d; ++j) n += (block_off[j + 1] - block_off[j] + len - 1) / len;
    if (n <= std::max(NA_FILL_CHUNKS, d)) {
      c.chunk = len;
      break;
    }
  }
  c.own = 1;
  for (int j = 0; j < d; ++j) {
    coff[j + 1] = coff[j] + int32_t((block_off[j + 1] - block_off[j] + c.chunk - 1) / c.chunk);
    if (coff[j + 1] - coff[j] > NA_OWN_SUM) c.own = 0;
  }
  c.nchunks = coff[d];
  PPD_TRY(scratch_for_device(&c.base));
  c.w = reinterpret_cast<const double2*>(w);
  c.y = reinterpret_cast<const float2*>(y);
  c.U = U;
  c.z = reinterpret_cast<double2*>(zbar);
  c.mu = mu;
  c.stream = static_cast<hipStream_t>(stream);
  if (d <= NA_ARG_BLOCKS) {
    NaArgs t{};
    std::copy(eps, eps + d, t.eps);
    std::copy(block_off, block_off + d + 1, t.boff);
    std::copy(coff, coff + d + 1, t.coff);
    return na_run(c, t);
  }
  // the block tables into the array (pageable host sources are staged by the
  // runtime before these calls return)
  PPD_HIP(hipMemcpyAsync(c.base + NA_OFF_EPS, eps, sizeof(double) * d, hipMemcpyHostToDevice, c.stream));
  PPD_HIP(hipMemcpyAsync(c.base + NA_OFF_BOFF, block_off, sizeof(int64_t) * (d + 1), hipMemcpyHostToDevice, c.stream));
  PPD_HIP(hipMemcpyAsync(c.base + NA_OFF_COFF, coff, sizeof(int32_t) * (d + 1), hipMemcpyHostToDevice, c.stream));
  return na_run(c, NaNone{});
}
