// Internal declarations of libppd (gfx950).  Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/ppd.h"

namespace ppd {

// ---- errors -------------------------------------------------------------
void set_error(const std::string& msg);
int fail(int status, const std::string& msg);

#define PPD_HIP(expr)                                                           \
  do {                                                                          \
    hipError_t e_ = (expr);                                                     \
    if (e_ != hipSuccess)                                                       \
      return ::ppd::fail(PPD_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

#define PPD_TRY(expr)                 \
  do {                                \
    int s_ = (expr);                  \
    if (s_ != PPD_OK) return s_;      \
  } while (0)

// ---- constants ----------------------------------------------------------
constexpr int KB_TAPS = 8;        // kernel width per axis
constexpr int KB_DEG = 9;         // polynomial degree per tap
constexpr int KB_NC = KB_DEG + 1; // coefficients per tap
constexpr int N_BASES = 9;        // Dirac + db1..db8
constexpr int FILT_STRIDE = 16;   // max Daubechies taps (db8)
// Points per workgroup of the passes over plan-order chunks of one block
// (Algorithm 2 steps, the differentiable dual update): fewer
// points where the chip would be left empty, and few enough chunks for every
// workgroup to add up its block's partials itself.
inline int64_t sec_chunk(int64_t M) { return M <= (int64_t(1) << 20) ? 512 : M <= (int64_t(1) << 22) ? 1024 : 2048; }
// The same for the launches of a Newton step each, which read 16 bytes a point
// instead of 40 to 72 and two sums of every chunk, so that with few blocks the
// reading of the partials weighs more.  A 12-step solve at 512, 1024 and 2048
// points, us: 250000 points in one block 61, 54, 58; 500000 79, 64, 65; a million
// 121, 88, 80, in 16 blocks 86, 78, 75; 4 million 773, 336, 236.
inline int64_t newton_chunk(int64_t M) { return M <= (int64_t(1) << 19) ? 1024 : 2048; }
// Chunks of a block up to which the workgroups of a step do that (each reads all the
// block's partials: 32 KB, 16 a thread); beyond it a launch of one workgroup
// per block forms the block's sum.
constexpr int OWN_SUM_CHUNKS = 4096;
constexpr int MAX_ITEM_SEGS = 64; // per-block segments of one work item (one wave scans them)
constexpr int MAX_XCD = 8;
constexpr int PA_THREADS = 256;   // persistent Algorithm 2: threads per workgroup
// Points per thread held in registers: 12 (2 waves per SIMD: 512 workgroups on
// the device) leaves few workgroups to wait for at each step and still fits the
// co-residency limit at 1.3M points.  Fewer points are spread over more
// compute units: a step's own arithmetic is then short against the exchange
// (four middle steps at 65536 points: 28.3 us at 12, 18.2 at 4, 16.2 at 2).
// But then the launch takes a larger share of the device (2048 workgroups at 2
// points per thread, 1280 at 4), so the shorter chunks end where PA_BESIDE such
// launches still fit beside each other.
constexpr int PA_PER_MAX = 12;
inline int pa_points(int64_t M) { return M <= (1 << 17) ? 2 : M <= 320 * 1024 ? 4 : PA_PER_MAX; }
constexpr int PA_CHUNK_MAX = PA_THREADS * PA_PER_MAX;
constexpr int PA_MAXB = 4;        // data blocks one workgroup's points may span
// Launches whose workgroups wait for each other that must fit the device beside
// each other: as many as a process's hardware queues run at once (HIP's default).
constexpr int PA_BESIDE = 4;
constexpr int PA_SYNC_WORDS = 32;   // [1] exit count, [2] give-up to report, [3] give-up flag, [4] solves by one workgroup
// Polls of one wait of a persistent launch before it gives up and the last
// workgroup out does the work alone: 2 ms at 0.25 us a poll, where a step takes 4
// us and the work of one workgroup, for Newton steps at 200003 points, 0.9 to 1.4 ms.
constexpr int PA_SPIN = 1 << 13;
// tagged partial slots of the persistent launch (see k_alg2_persistent)
constexpr uint64_t PA_SIGN = 0x8000000000000000ull;
constexpr uint64_t PA_EMPTY = 0x7ff8000000000000ull;   // quiet NaN: no partial yet
#ifndef PPD_FOLD_HEAVY
#define PPD_FOLD_HEAVY 16
#endif
constexpr int FOLD_HEAVY = PPD_FOLD_HEAVY;   // item regions above which a tile's fold takes a whole workgroup
// Where a tile has more items than fold_group_from, every FOLD_GROUP regions of
// the tiles with more than that are added up in a launch before the fold.  Phi^H
// without and with it, us: 8 x 8 tiles with up to 94 to 117 items (four waves
// share a tile there) 26 and 25, 22 and 20, 31 and 34, 53 and 53, with 246 and 297
// 27 and 19, 39 and 25; larger ones with 25 to 30 items 34 and 34, 37 and 38, 93
// and 92, with 72 and 78 49 and 37, 56 and 42.
constexpr int FOLD_GROUP = 16;
inline int fold_group_from(int T) { return T == 8 ? 128 : 32; }
// Item count up to which two waves share each item in the 8 x 8 kernels: with
// fewer waves than the chip holds (4096 at 4 per SIMD), the length of one
// wave's chain is the kernel's time.  Gridding 10.8 -> 5.4 us at 64^2, 4096
// points, 8.6 -> 7.4 at 256^2, 65536; 15.6 -> 16.6 at 512^2, 250k, where the
// waves suffice.
constexpr int SHARE_ITEMS = 4096;
// Item count up to which SARA's launches ride in the data path's (each launch
// then has the registers and LDS of the larger part).  Per replayed iteration,
// on two streams and in pairs: 50 and 31 us at 64^2 (125 items), 51 and 40 at
// 128^2 (1043), 51 and 48.5 at 256^2 (1777), 57 and 72 at 256^2 (3118); eager,
// where the host sets the pace of two streams, 59-74 and 36, 59-74 and 43,
// 60-74 and 49.5, 63-78 and 75.
constexpr int PAIR_ITEMS = 2048;
// The same for replayed iterations with middle Algorithm 2 steps or the exact
// prox, in which the second stream has SARA run beside those: five steps 54 and
// 50 us at 128^2 (471 items), 55.5 and 59 at 128^2 (1043), 58.5 and 68 at 256^2
// (1777); exact 59 and 56 at 64^2 (140), 61 and 63 at 128^2 (502).
constexpr int PAIR_ITEMS_MIDDLE = 480;
// Block count up to which they do: a block is a workgroup of 1024 threads in the
// launch of the block factors, and beside an analysis level's registers and LDS
// few of those are resident.  Per replayed iteration in pairs and on two
// streams, in 1024 and in 4096 blocks sorted by radius: 65536 points at 256^2 81
// and 56 us, 119 and 77 (the factors alone, of one block a point, 509 and 266);
// 20000 at 128^2 51 and 52, 76 and 67; 4096 at 64^2 50 and 53, 73 and 67.
constexpr int PAIR_BLOCKS = 1024;
// Largest 2 ny of the launches that a SARA level rides in (its kernels exist
// for the lengths up to there).
constexpr int PAIR_MAX_KY = 1024;
// Captured-iteration graphs per plan: one iteration without statistics
// partials, one with them and the periodic reduction, one with the partials
// only, and a captured run (a statistics period, or GRAPH_RUN iterations
// without partials).
constexpr int GRAPH_SLOTS = 4;
#ifndef PPD_GRAPH_RUN
#define PPD_GRAPH_RUN 8
#endif
constexpr int GRAPH_RUN = PPD_GRAPH_RUN;
// The spectrum of the (real) image is Hermitian, so the grids hold the columns
// c = -GRID_PAD .. Kx/2 + GRID_PAD - 1 only, at padded index c + GRID_PAD: the
// columns 0 .. Kx/2 and, beyond either end, the mirror images that taps reach.
// A visibility whose first tap lies left of -GRID_PAD is taken at its mirror
// frequency, conjugated (see mirrored).  8 columns of padding leave the points
// around the v axis, of either sign, unmirrored in one tile column.
constexpr int GRID_PAD = 8;
// Columns per block of the grids and of the row-pass buffers: a block holds
// all rows of FFT_CB columns, row by row, so a column pass on a block, and the
// region of an 8 x 8 tile, are runs of consecutive addresses.
constexpr int FFT_CB = 4;
__host__ __device__ __forceinline__ size_t grid_index(int p, int row, int Ky) {
  return (size_t(p / FFT_CB) * Ky + row) * FFT_CB + p % FFT_CB;
}
__host__ __device__ __forceinline__ size_t half_index(int c, int row, int ny) { return grid_index(c, row, ny); }
// Whether a visibility at u grid coordinate tu (K omega_u / 2 pi) is gridded
// at its mirror frequency: its first tap floor(tu) - 3 is left of -GRID_PAD.
__host__ __device__ __forceinline__ bool mirrored(double tu) { return tu < 3.0 - GRID_PAD; }

// Elements per thread of a row and of a column transform of length L, and
// columns per workgroup (more where that is less than a wave).  Short
// transforms leave the chip nearly empty (64 to 512 sequences), so they take
// few elements per thread, which shortens every wave's chain of dependent work:
// rows with the primal update, L = 1024: 12.6 / 9.0 / 8.0 us at 16 / 8 / 4
// elements; columns 6.7 us at any of these, 5.4 us with 2 instead of 4 columns
// per workgroup (twice the workgroups).  From L = 2048 on the chip is full and
// fewer, larger stages win: columns at L = 4096 (2048^2), in SQ busy cycles,
// 1.76M / 2.33M forward at 16 elements and 4 columns / 8 and 2, rows 2.93M /
// 2.74M at 16 / 8 elements.
template <int L>
struct FftShape {
  static constexpr int ROW_E = L <= 1024 ? 4 : 8;
  static constexpr int COL_E = L <= 1024 ? 4 : L == 2048 ? 8 : 16;
  static constexpr int COL_C = L <= 2048 ? 2 : 4;
};
// Two exchange buffers where a workgroup's LDS then still leaves room for a
// second workgroup on the compute unit (160 KB).
constexpr int FFT_TWO_LDS = 80 * 1024;
struct FftTwiddles {
  std::vector<float2> row, col;   // in the order the threads of a transform read them
};

// Launch order of the work items over the XCDs: the items, in spatial
// order, are cut into 8 contiguous bands of near-equal work (64-point
// batches plus one per item for its region), XCD k taking the items
// [off[k], off[k+1]).  Workgroup ids go round-robin over the XCDs, so
// workgroup b runs item off[b mod 8] + b / 8 of band b mod 8, if that band
// has it.
struct XcdSplit {
  int32_t off[MAX_XCD + 1];
  int32_t launch;   // workgroups to launch: 8 x the longest band
};

// A segment: plan-order visibilities [start, start+count) of one data
// block whose first tap lies in one grid tile.
struct Seg {
  int32_t start, count, block, item;
};
// A work item (one workgroup): the segments [seg0, seg1) of tile (tx, ty),
// `total` visibilities, at most chunk_max.  Items are ordered tile by tile in
// row-major tile order.  The first segment is repeated here: most items have
// no other (one radial block per tile), and then need no segment table.
struct Item {
  int32_t tx, ty, seg0, seg1;
  int32_t start, block, total, pad_;
};

// Kernel kinds for the optional per-launch event timer.
enum KernelKind {
  KK_FFT_ROWS_FWD, KK_FFT_COLS_FWD, KK_DEGRID, KK_GRID, KK_FFT_COLS_INV, KK_FFT_ROWS_INV,
  KK_FOLD, KK_PERMUTE, KK_SUBITER, KK_DWT, KK_IDWT, KK_STATS, KK_PLAIN_DUAL, KK_HIST,
  KK_NORM, KK_MISC, KK_COUNT
};
const char* kernel_kind_name(int k);

}  // namespace ppd

struct ppd_plan {
  // geometry
  int nx = 0, ny = 0, Kx = 0, Ky = 0;
  int PW = 0;                              // grid columns held: Kx/2 + 2 GRID_PAD
  int64_t M = 0;
  int d = 0, levels = 3, T = 32, chunk_max = 1024;
  int tiles_x = 0, tiles_y = 0;
  double beta = 0.0;
  double su_scale = 0.0, sv_scale = 0.0;   // K / (2 pi) per axis
  bool has_theta = false;
  hipStream_t stream = nullptr;
  int device = 0;
  // second stream of an iteration (the SARA dual step runs there, forked
  // from and joined back to `stream` through the two events)
  hipStream_t aux = nullptr;
  double2* bfac = nullptr;                 // [d] (factor, inside) of the last block_factors call
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;

  // host copies
  std::vector<int64_t> block_off;          // [d+1]
  std::vector<int32_t> perm_host;          // plan -> user
  std::vector<ppd::Item> items_host;       // launch order
  std::vector<ppd::Seg> segs_host;
  std::vector<int32_t> bseg_off;           // [d+1] into bseg_ids
  int n_items = 0, n_segs = 0;
  ppd::XcdSplit split1{};
  int n_tiles = 0;

  // device: coverage and plan tables
  float* wu = nullptr;
  float* wv = nullptr;
  float* theta = nullptr;
  int32_t* perm = nullptr;
  ppd::Item* items = nullptr;
  ppd::Seg* segs = nullptr;
  int32_t* tile_item_off = nullptr;        // [n_tiles+1] items of each tile
  int32_t* fold_wg = nullptr;              // [n_fold_wg][4] tiles per 4-wave fold workgroup
  int n_fold_wg = 0;                       // multiple of MAX_XCD
  int32_t* fold_groups = nullptr;          // [n_fold_groups][2] first item and items of each group
  int n_fold_groups = 0;                   // 0: no tile has so many items
  int32_t* bseg_ids = nullptr;             // segment ids grouped by block
  int32_t* bseg_off_d = nullptr;           // [d+1]
  float2* gscratch = nullptr;              // [n_items][(T+7)^2] gridding partials
  int32_t* vis_block = nullptr;            // plan index -> block (plain form)
  float* kbc = nullptr;                    // [8][10] tap polynomials
  float* dpx = nullptr;                    // [nx] 1/phi_hat(n_c / Kx)
  float* dpy = nullptr;                    // [ny] 1/phi_hat(n_r / Ky)
  float2* twx = nullptr;                   // row transform's twiddles (fft_twiddles(Kx).row)
  float2* twy = nullptr;                   // column transform's (fft_twiddles(Ky).col)
  float* filt = nullptr;                   // [8][2][16] lo / hi Daubechies filters

  // device: work buffers
  float2* grid_f = nullptr;                // forward spectrum, Ky x PW (grid_index)
  float2* grid_a = nullptr;                // adjoint accumulation, Ky x PW
  float2* half = nullptr;                  // ny x Kx/2 row-pass intermediate (half_index)
  float2* half_f = nullptr;                // ny x Kx/2 forward row pass of x~ (iterations)
  float2* ybuf = nullptr;                  // [M] complex64 scratch
  double2* wbuf = nullptr;                 // [M] complex128 w (plain form)
  float2* gabuf = nullptr;                 // [M] complex64 Theta G a (fused form; w is rebuilt from it)
  double2* qbuf = nullptr;                 // [M] complex128 (plain form; (a^2, U) of the Newton passes)
  // Algorithm 2 steps and the differentiable dual update: chunks of consecutive
  // plan-order visibilities inside one block
  int n_sec_chunks = 0;
  bool own_sums = true;                    // no block has more than OWN_SUM_CHUNKS chunks
  int32_t* sec_cstart = nullptr;           // [n_sec_chunks + 1] first visibility of each chunk
  int32_t* sec_cblock = nullptr;           // [n_sec_chunks] block of each chunk
  int32_t* sec_coff = nullptr;             // [d + 1] chunks of block j: [sec_coff[j], sec_coff[j+1])
  double* sec_part = nullptr;              // [2][2][n_sec_chunks] partials: two sums, two passes
  // the same for the Newton passes, whose chunks are as long or longer
  int n_nw_chunks = 0;
  int32_t* nw_cstart = nullptr;
  int32_t* nw_cblock = nullptr;
  int32_t* nw_coff = nullptr;
  double* sec_nu = nullptr;                // [2][d] nu of the last two Newton passes
  double4* du_blk = nullptr;               // [d] block terms of the differentiable dual update
  // persistent Algorithm 2 middle steps (one launch, state in registers):
  // workgroup g holds the pa_per PA_THREADS plan-order points from there on
  int pa_per = 0;                          // points per thread
  int pa_groups = 0;                       // workgroups of the persistent launch
  bool pa_ok = false;                      // every workgroup co-resident and within PA_MAXB blocks
  bool sec_ok = false;                     // the same for the exact prox's persistent Newton steps
  int32_t* voff_d = nullptr;               // [d+1] block offsets (plan order)
  int32_t* pa_wgb0 = nullptr;              // [pa_groups] first block of each workgroup
  int32_t* pa_gfirst = nullptr;            // [d] first workgroup of each block
  int32_t* pa_glast = nullptr;             // [d] last workgroup of each block
  uint64_t* pa_part = nullptr;             // [2][pa_groups][PA_MAXB][2] tagged per-workgroup block partials
  uint32_t* pa_sync = nullptr;             // [PA_SYNC_WORDS] exit count, give-up flags, solves by one workgroup
  bool last_paired = false;                // forms of the last ppd_iterate call (ppd_plan_get_forms)
  bool last_one_launch = false;
  double* part = nullptr;                  // [n_segs] block-norm partials
  double* rpart = nullptr;                 // [n_segs] residual partials (per item in the fidelity)
  double* eps_d = nullptr;                 // [d]
  std::vector<double> eps_cache;
  double* ppart = nullptr;                 // [ny][4] primal statistics partials
  double* stats_d = nullptr;               // [8 + d]
  int32_t* hist_cursor = nullptr;          // [1] next statistics history row of a graph replay
  double* rj_d = nullptr;                  // [d] block residuals of the last statistics reduction
  double* host_stats = nullptr;            // pinned host [8 + d + 1]: a call's statistics and give-up flag
  double* host_stats_dev = nullptr;        // its device-side address
  float* sara_ll = nullptr;                // LL temporaries, analysis
  float* sara_rec = nullptr;               // reconstruction temporaries
  float* ut = nullptr;                     // [ny][nx] Psi u
  float* img_tmp = nullptr;                // [ny][nx]
  float* vec_tmp = nullptr;                // [ny][nx] power iteration
  double* pl_part = nullptr;               // [1024] plain-form / image partials
  double* res_sq = nullptr;                // [d] plain-form residual norms^2
  double* pl_scalar = nullptr;             // [4]
  int32_t* icount = nullptr;               // [ny][nx] sampling-density counts
  int32_t* imin = nullptr;                 // [1]
  size_t sara_ll_floats = 0;
  size_t device_bytes = 0;
  std::vector<void*> allocations;          // hipMalloc'd buffers (plans without a workspace)
  // caller-owned workspace the buffers are carved from (256-byte aligned
  // offsets), or a sizing pass that only adds up the bytes
  char* ws = nullptr;
  size_t ws_bytes = 0, ws_used = 0;
  bool ws_measure = false;

  // graph replay of one iteration: slot 0 without the statistics partials,
  // slot 1 with them and the periodic reduction, slot 2 with them only
  hipGraphExec_t graph_exec[ppd::GRAPH_SLOTS] = {};
  hipGraph_t graph[ppd::GRAPH_SLOTS] = {};
  std::string graph_key[ppd::GRAPH_SLOTS];

  // optional per-launch timing
  bool timing = false;
  std::vector<hipEvent_t> ev_pool;
  std::vector<std::pair<int, int>> ev_pending;   // (kind, event pair index)
  int64_t t_counts[ppd::KK_COUNT] = {};
  double t_ms[ppd::KK_COUNT] = {};
};

namespace ppd {

// launch bracketing for the per-kernel timer
int timer_begin(ppd_plan* p, int kind, int* slot);
int timer_end(ppd_plan* p, int slot);

struct SaraGeom {
  int nx, ny, L;
  size_t N;
  size_t off[8];   // per-level temporaries: off[l] for level l (1 <= l < L)
};
// One SARA launch of an iteration (sara_jobs), to ride in a launch of the data
// path (`with` below; NULL: nothing rides).
enum SaraKind { SARA_DWT, SARA_IDWT2, SARA_IDWT, SARA_FINAL };
struct SaraJob {
  int kind;
  const float* in; float* tmp; float* out;
  const float* filt; const float* W;
  SaraGeom g;
  int l;
  float alpha, lambda;
  const uint8_t* active;
  int vec, gx, gy, gz;
  __host__ __device__ int blocks() const { return gx * gy * gz; }
};

// ---- component launchers (each returns a PPD_* status) -------------------
int fft_forward(ppd_plan* p, const float* x);                  // x -> grid_f (via half)
int fft_rows_forward(ppd_plan* p, const float* x, float2* dst);  // x -> dst (row-pass buffer)
// src (row-pass buffer) -> grid_f; with: a SARA analysis level
int fft_cols_forward(ppd_plan* p, const float2* src, const SaraJob* with = nullptr);
int fft_adjoint(ppd_plan* p, float* x, bool add = false);      // grid_a -> x, or added to x (plain)
int fft_cols_inverse(ppd_plan* p);                             // grid_a -> half
struct PrimalArgs {
  float* x; float* xt; const float* ut; const float* x_true;
  double tau, eta, zeta, lambda;
  double* part;                    // [ny][4] statistics partials, or NULL to skip them
};
// half -> primal update and the forward row pass of the new x~ into next
// (row-pass buffer)
int fft_rows_inverse_primal(ppd_plan* p, const PrimalArgs& a, float2* next);
int fold_grid(ppd_plan* p, const SaraJob* with = nullptr);     // gscratch -> grid_a; with: a synthesis level

// grid_f -> out, in plan order, or with uperm (plan -> caller) in the caller's
int degrid_plain(ppd_plan* p, float2* out, const int32_t* uperm = nullptr);
// grid_f -> Theta G a - y (plan order), squared norms per item in rpart
int degrid_residual(ppd_plan* p, const float2* y, float2* out);
struct DualArgs {
  const float2* y; const double* U; float2* v; double2* z;
  double mu, lambda;
  int n_itr;
  const uint8_t* active;   // DEVICE [d] block mask of this iteration, NULL = all
  const double2* zin = nullptr;   // gridding: the iterate before the last projection, NULL = z
  double* rpart = nullptr; // DEVICE [n_segs] residual partials for the statistics, NULL = skip them
};
// grid_f -> gabuf; part_out NULL: no Algorithm 2 partials; with: a SARA analysis level
int degrid_dual(ppd_plan* p, const DualArgs& a, double* part_out, const SaraJob* with = nullptr);
// v -> grid_a; v in plan order, or with uperm in the caller's
int grid_plain(ppd_plan* p, const float2* v, const int32_t* uperm = nullptr);
int grid_dual(ppd_plan* p, const DualArgs& a, const double* part_in);  // dual finish + grid
// the same with the block factors already in bfac
int grid_dual_factored(ppd_plan* p, const DualArgs& a);
// the same, or with the exact prox, and a synthesis launch (a level or the two
// coarsest) beside the gridding, one (a level or the last) beside the fold
int grid_dual_paired(ppd_plan* p, const DualArgs& a, int exact, const SaraJob* with, const SaraJob* with_fold);

int plain_dual(ppd_plan* p, const DualArgs& a);               // per-block unfused dual update
// z <- P_B(q) for every block and, if pout, chunk partials of the next
// ||q - y_j||^2; the factors of P_B come from fac, else from the chunk
// partials pin.  Without either: the partials of the present z only.  w, or
// v and ga (w = U^-1 v + ga); active: DEVICE [d] mask, NULL = all.
struct BallIn {
  const double2* w; const float2* v; const float2* ga; const float2* y; const double* U;
  double mu;
  const uint8_t* active;
};
int ball_step(ppd_plan* p, const BallIn& in, double2* z, const double2* fac, const double* pin, double* pout);
int ball_factors(ppd_plan* p, const double* pin);   // bfac from chunk partials
// Per-block projection factors of P_B from per-segment partials of
// ||q - y||^2: bfac[j] = (min(1, eps_j / r_j), r_j <= eps_j), r_j the block norm.
// with: a SARA analysis level.
int block_factors(ppd_plan* p, const double* part, const SaraJob* with = nullptr);
// The n_itr - 1 middle Algorithm 2 steps of the fused form in one persistent
// launch (needs p->pa_ok and the first step's factors in bfac; leaves the
// last step's factors in bfac and the iterate in qbuf).  spin_limit bounds each
// wait (0: PA_SPIN); a given one that runs out is reported.
int alg2_persistent(ppd_plan* p, const DualArgs& a, int spin_limit);
// Maximum co-resident workgroups of the persistent launch at `per` points per
// thread on the current device (0 if it cannot be determined).
int alg2_persistent_capacity(int per);
int sec_persistent_capacity(int per);
// n_newton Newton steps of the exact prox per block; nu_j in bfac[j].x.
// The prox argument is w if non-NULL, else U^-1 v + ga (see dual_arg).
// persistent (w NULL): as one launch where the plan's points fit a quarter of the device.
int secular_solve(ppd_plan* p, const double2* w, const float2* v, const float2* ga, const float2* y,
                  const double* U, int n_newton, bool persistent, int spin_limit);
int grid_dual_exact(ppd_plan* p, const DualArgs& a);   // dual finish with the exact prox + grid
int permute(ppd_plan* p, int direction, const void* in, void* out, int elem_bytes);

// The SARA launches of one iteration: analysis levels with the dual update of
// u from x, then the synthesis levels, the last one into out.  For plans where
// sara_pairs: at most SARA_PAIR_LEVELS levels and low analysis tiles.
constexpr int SARA_PAIR_LEVELS = 4;
struct SaraJobs {
  SaraJob dwt[SARA_PAIR_LEVELS], synth[3];
  int n_dwt, n_synth;
};
bool sara_pairs(const ppd_plan* p);
SaraJobs sara_jobs(ppd_plan* p, const float* x, float* u, float alpha, float lambda, const float* W,
                   const uint8_t* active, float* out);
int sara_launch(ppd_plan* p, const SaraJob& j);   // a launch of its own
int sara_analysis(ppd_plan* p, const float* x, float* coef, const float* W);
int sara_dual(ppd_plan* p, const float* x, float* u, float alpha, float lambda, const float* W,
              const uint8_t* active = nullptr);   // active: DEVICE [9] basis mask, NULL = all
int sara_synthesis(ppd_plan* p, const float* u, float* out, const float* W);

// out: [8 + d], or with a cursor row *cursor of rows of `stride` doubles (advanced)
int stats_finalize(ppd_plan* p, int has_truth, int use_res_sq, double* out, int32_t* cursor, int stride);
int upload_eps(ppd_plan* p, const double* eps_host);

// host-side setup helpers
void kb_tap_polynomials(double beta, float* coef /* [8][KB_NC] */);
double kb_ft(double xi, double beta);
void daubechies(int p, double* h);
FftTwiddles fft_twiddles(int L);

}  // namespace ppd

namespace ppd {

// Runs the plan's launches on another stream for the lifetime of the object.
struct OnStream {
  ppd_plan* p;
  hipStream_t saved;
  OnStream(ppd_plan* pl, hipStream_t s) : p(pl), saved(pl->stream) { p->stream = s; }
  ~OnStream() { p->stream = saved; }
};

}  // namespace ppd

// ---- device helpers --------------------------------------------------------
namespace ppd {

// The 8 tap weights at fractional offset s in [0, 1), x = 2s - 1.  The
// kernel is even, so tap 7-m at x equals tap m at -x: with the even and odd
// parts of tap m's polynomial, P(+-x) = E(x^2) +- x O(x^2), four polynomial
// pairs give all eight weights (half the multiply-adds of eight Horner
// evaluations).  c holds the coefficients of taps 0..3 (of 8) in powers of x.
__host__ __device__ inline void kb_weights(float s, const float* __restrict__ c, float* w) {
  const float x = 2.0f * s - 1.0f;
  const float y = x * x;
#pragma unroll
  for (int m = 0; m < KB_TAPS / 2; ++m) {
    const float* cm = c + m * KB_NC;
    float e = cm[KB_DEG - 1], o = cm[KB_DEG];   // KB_DEG is odd
#pragma unroll
    for (int k = KB_DEG - 3; k >= 0; k -= 2) {
      e = fmaf(e, y, cm[k]);
      o = fmaf(o, y, cm[k + 1]);
    }
    const float xo = x * o;
    w[m] = e + xo;
    w[KB_TAPS - 1 - m] = e - xo;
  }
}
static_assert(KB_DEG % 2 == 1, "even / odd split assumes an odd degree");

// argument of the data-dual update of Algorithm 3, w = U^-1 v + Theta G a, in FP64; the fused form
// stores Theta G a (complex64) and rebuilds w where it is needed, bitwise
// the same each time.
__device__ __forceinline__ double2 dual_arg(float2 v, double U, float2 ga) {
  const double r = 1.0 / U;   // one division per visibility, shared by both parts
  return make_double2(double(v.x) * r + double(ga.x), double(v.y) * r + double(ga.y));
}

// Segment table of a work item in LDS: the offsets of its segments in the
// item's flattened visibility range (pre[n] = total), their first visibility
// in plan order and their data block.
struct ItemTab {
  int pre[MAX_ITEM_SEGS + 1];
  int start[MAX_ITEM_SEGS];
  int block[MAX_ITEM_SEGS];
};

// Wave 0 loads the item's segments (one per lane) and scans their counts;
// the caller synchronises before use.
__device__ inline void load_item_tab(const Item& it, const Seg* __restrict__ segs, ItemTab& tab) {
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    int cnt = 0;
    if (lane < it.seg1 - it.seg0) {
      const Seg sg = segs[it.seg0 + lane];
      cnt = sg.count;
      tab.start[lane] = sg.start;
      tab.block[lane] = sg.block;
    }
    int inc = cnt;
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(inc, o);
      if (lane >= o) inc += t;
    }
    tab.pre[lane + 1] = inc;
    if (lane == 0) tab.pre[0] = 0;
  }
}

// Segment of flattened index li, searching forward from segment s.
__device__ __forceinline__ int seg_of(int li, int s, const int* pre) {
  while (li >= pre[s + 1]) ++s;
  return s;
}

// Value of the lane that a data-parallel permutation within 16 lanes names.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, int(b), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, int(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane(int(b), lane), hi = __builtin_amdgcn_readlane(int(b >> 32), lane);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}

// Sum over the 64 lanes of a wave in a fixed order, the same in every lane:
// within 16 lanes by permuted operands (quads, half rows, rows), then the four
// rows.  No LDS: a shuffle butterfly takes 12 LDS permutes one after another.
// All 64 lanes must be active.
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_move<0xB1>(v);    // quad_perm 1 0 3 2
  v += dpp_move<0x4E>(v);    // quad_perm 2 3 0 1
  v += dpp_move<0x141>(v);   // row_half_mirror
  v += dpp_move<0x140>(v);   // row_mirror
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// The item a workgroup takes in a work-balanced XCD split, or -1 when its
// XCD's band has none left for it.
__device__ __forceinline__ int xcd_item(int bid, const XcdSplit& s) {
  const int k = bid % MAX_XCD;
  const int u = s.off[k] + bid / MAX_XCD;
  return u < s.off[k + 1] ? u : -1;
}

// XCD-aware remap: consecutive workgroup ids go round-robin over the XCDs;
// give each XCD a contiguous range of the (spatially ordered) work list so
// its L2 holds one band of the grid.
__device__ inline int xcd_remap(int bid, int nlaunch) {
  const int per = nlaunch / MAX_XCD;     // nlaunch is a multiple of MAX_XCD
  return (bid % MAX_XCD) * per + bid / MAX_XCD;
}

}  // namespace ppd
