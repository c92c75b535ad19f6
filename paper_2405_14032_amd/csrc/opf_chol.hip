// Static-pivot sparse Cholesky of the condensed matrix (Sec. III-B): device
// kernels and the opf_chol_* entry points.
//
// Numeric scheme (multifrontal, the plan from opf_chol_symbolic.cpp):
//   * the factor of every interior front s of every period lives in one
//     column-major (p+u) x p block (p pivots, u update rows); its update
//     matrix (u x u, lower part) lives in a workspace arena until the
//     parent has collected it;
//   * K's entries are written straight into the factor blocks; each front
//     then pulls its children's update matrices (extend-add, no atomics: a
//     work item owns a set of the parent's columns), is factored in place
//     (small fronts in registers by one wavefront, large ones by blocked panel
//     + trailing-update kernels), batched over the periods of a chunk;
//   * the pg front of period t (G pivots) collects the period's tree roots
//     and its chain neighbour's update: a chain over t, eliminated from both
//     ends at once (fronts t < m carry update rows pg_{t+1}, fronts t > m
//     update rows pg_{t-1}, front m closes it; m = (T - 1) / 2), one front of
//     each side per launch; over long horizons by cyclic reduction instead
//     (every other front at once, see k_cyc_add), with few generators by one
//     launch (k_chain_wave).
// Solves run the same tree forward (update vectors pulled by the parent)
// and backward (gathers of the ancestors' solution), batched over periods.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/opf.h"
#include "opf_api_internal.h"
#include "opf_chol_host.h"

namespace opf {
namespace {

constexpr int kSmall = 64;   // largest front of one wavefront, a row per lane
constexpr int kNB = 64;      // panel width of the blocked fronts
constexpr int kTile = 64;    // trailing-update tile
constexpr int kChainCols = 128;  // columns summed together in the chain's L21 z (a multiple of kNB)
constexpr int kStep = 1024;      // columns per trailing update of a blocked front
constexpr int kWide = 256;       // columns whose panels update each other within their launches
constexpr int kTreeT = 512;      // threads of k_fwd_tree, k_bwd_tree: eight fronts at a time
constexpr int kTreeFronts = 16;  // levels of at most this many fronts share their launch (two per wavefront)
constexpr int kFewTiles = 256;   // updates of fewer 64 x 64 tiles take 32 x 32 ones (one block per CU)
// The pg chain by cyclic reduction (see k_cyc_add) from kCycT periods, up to
// fronts of kCycG: factor + solve, from both ends against by reduction, 54
// generators x 64 periods 2.05 / 0.92 ms, 400 x 64 21.4 / 14.8, 400 x 168 53 /
// 34, 1000 x 168 110 / 70, 1400 x 168 173 / 138, 1600 x 168 198 / 172, but 2000 x
// 168 602 / 644: the work it adds outgrows the steps it saves.  The line on the
// horizon is not one of speed (400 x 24 takes 9.2 / 7.3 ms, 54 x 24 1.10 / 0.74):
// an interior-point iterate shows a changed elimination order at 1e-8, and
// short horizons keep theirs bit for bit.  The memory it takes beyond the chain's (G^2 per period
// for the pg fronts, 2 G^2 for a level's update blocks, which the instances of
// a batch share) is held to kCycBytes over all instances together.
constexpr int kCycT = 64, kCycG = 1536;
constexpr int64_t kCycBytes = 16LL << 30;
// The pg chain by two wavefronts (see k_chain_wave, k_chain_wave_solve) over
// horizons of fewer than kCycT periods, up to this many generators in the
// factorization and in the solves.  Factorization, launched front by front
// against one launch: 5 generators x 4 periods (14 buses) 140 / 72 us, 7 x 63
// (57 buses) 763 / 313, 16 x 24 (60 buses) 511 / 395, 17 x 24 574 / 623 (a front
// of more than 32 rows spills).  Solve: 68 / 48 us, 405 / 145, 213 / 110, 32 x 48
// (90 buses) 391 / 224, 48 x 24 283 / 210, 54 x 24 (118 buses) 327 / 298, 64 x 24
// 301 / 290.
constexpr int kWaveG = 16, kWaveSolveG = 64;
constexpr int kBwdCols = 32;     // earlier columns updated per block of a backward launch, at least

// Device view of one instance's plan.
struct CDev {
  const int32_t *node_p, *node_u, *rel, *kids, *rows;
  const int64_t *node_loff, *node_uoff, *node_woff, *row_ptr;
  // extend-add: per node its rows by position in its parent's front (inv, -1:
  // none); per column of a large front (col_off) or of the pg front (from
  // col_root) the children with an entry there in their order, con[col[q]] ..
  // con[col[q + 1] - 1]: where the child's column starts in the workspace and
  // its inverse map in inv
  const int32_t* inv;
  const int64_t* col_off;
  const int32_t* col;
  const longlong2* con;
  // per child, in kid_ptr's order: where its update matrix and its inverse map
  // start, its rows, where its update vector starts
  const longlong4* kid;
  int64_t col_root;
  int64_t lsize, usize, wsize;
  int32_t n_p, n_int, G;
  const int32_t* stop;  // the static-pivot count when the factor stops at the first one, else NULL
};

// One front as the blocked kernels see it: p pivots, u update rows and where
// its parts start in a period's storage: factor block ((p+u) x p, leading
// dimension ld), diagonal blocks (see diag_size), update block (u x u), update
// vector of the solves, row list; its first elimination position and its children (CDev::kid).
struct FrontRec {
  int64_t L, D, U, W, R;
  int32_t p, u, ld, f, k0, k1;
};

// Front z of a batch: rec's, or the one given by value where rec is NULL (no
// load before the first address), in scalar registers either way.
__device__ __forceinline__ FrontRec pick_front(const FrontRec* __restrict__ rec, const FrontRec& one, int z) {
  const FrontRec g = rec ? rec[z] : one;
  constexpr int N = sizeof(FrontRec) / 4;
  int32_t w[N];
  __builtin_memcpy(w, &g, sizeof(g));
#pragma unroll
  for (int k = 0; k < N; ++k) w[k] = __builtin_amdgcn_readfirstlane(w[k]);
  FrontRec f;
  __builtin_memcpy(&f, w, sizeof(f));
  return f;
}

// A batch of fronts for one launch (front blockIdx.z of rec, in falling order
// of p: the ones that still have columns come first) over several periods
// (blockIdx.y): the first period's storage and the strides from one to the
// next.
struct Fronts {
  const FrontRec* rec;  // NULL: the one front below
  FrontRec one;
  double *L, *D, *U;
  int64_t sL, sD, sU;
  const int32_t* stop;  // as CDev::stop
  int32_t fresh;        // the update blocks hold nothing yet: the first trailing update stores into them
};

// The factored 64 x 64 diagonal blocks of a blocked front live apart from
// its factor block, one after the other, the last one kb x kb (leading
// dimension kb), the triangle mirrored: the forward solve wants its rows side
// by side, the backward solve its columns.  Every block of a panel launch
// reads the unfactored block from the front while one of them stores the
// factored one.
__host__ __device__ __forceinline__ int64_t diag_size(int p) {
  const int64_t np = (p + kNB - 1) / kNB, kb = p - (np - 1) * kNB;
  return (np - 1) * kNB * kNB + kb * kb;
}

// Whether the factorization stops at its first static pivot and one has
// been counted: the count read once per block by its first thread and
// shared, so every thread of the block takes the same branch.  A count
// raised by a concurrent kernel may be seen one launch late; the factor is
// then only discarded later.
__device__ __forceinline__ bool stopped(const int32_t* stop) {
  if (!stop) return false;
  __shared__ int32_t seen;
  if (threadIdx.x == 0) seen = *reinterpret_cast<const volatile int32_t*>(stop);
  __syncthreads();
  return seen > 0;
}

// The start of a factorization: factor blocks, pg fronts and (where given) the
// count of static pivots cleared.
__global__ void k_clear(double* __restrict__ p, int64_t n, double* __restrict__ q, int64_t m,
                        int32_t* __restrict__ npert) {
  const int64_t at = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
  if (at == 0 && npert) *npert = 0;
  for (int64_t i = at; i < n; i += step) p[i] = 0.0;
  for (int64_t i = at; i < m; i += step) q[i] = 0.0;
}

// K's template slots of periods t0 .. t0+nt-1 into the factor blocks (or the
// pg front's pivot block).  Every destination receives one entry.
__global__ void k_scatter(const double* __restrict__ kv, int64_t k_off, int64_t nnzk_p, int32_t G, int32_t t0,
                          int32_t nslots, const int64_t* __restrict__ dst, const int32_t* __restrict__ kpos0,
                          const int32_t* __restrict__ kpos1, double* __restrict__ Lf, int64_t lsize,
                          double* __restrict__ Cf, int64_t csize) {
  const int t = t0 + (int)blockIdx.y;
  const int64_t kp = k_off + (int64_t)t * nnzk_p + (t >= 1 ? (int64_t)(t - 1) * G : 0);
  for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < nslots; q += gridDim.x * blockDim.x) {
    const double v = kv[kp + (t == 0 ? kpos0[q] : kpos1[q])];
    const int64_t d = dst[q];
    if (d >= 0) Lf[(int64_t)t * lsize + d] = v;
    else Cf[(int64_t)t * csize + (-1 - d)] = v;
  }
}

// The ramp pairs (pg_t,g , pg_{t-1},g), t in [t0, t0 + gridDim.y), t >= 1:
// entries of the coupling block of the one of the two pg fronts that is
// eliminated first.  Two-ended chain (m >= 0): row G + g of front t-1 when t <=
// m (the left side), of front t otherwise (the right side).  Cyclic reduction
// (m < 0): the even one of the two, its right neighbour's rows at G, its left
// neighbour's at 2 G.
__global__ void k_scatter_ramp(const double* __restrict__ kv, int64_t k_off, int64_t nnzk_p, int32_t G, int32_t t0,
                               int32_t m, const int32_t* __restrict__ ramp_pos, double* __restrict__ Cf,
                               int64_t csize, int32_t cld) {
  const int t = t0 + (int)blockIdx.y;
  const int64_t kp = k_off + (int64_t)t * nnzk_p + (int64_t)(t - 1) * G;
  const int f = m >= 0 ? (t <= m ? t - 1 : t) : (t & ~1);
  const int row = m < 0 && f == t ? 2 * G : G;
  for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < G; g += gridDim.x * blockDim.x)
    Cf[(int64_t)f * csize + (int64_t)g * cld + row + g] = kv[kp + ramp_pos[g]];
}

// One column of a front by extend-add, by one wavefront: rows [j, n) of dst
// (pivot columns: on top of what is there) plus the entries of the children
// that have this column, child after child.  Every entry is written once.
__device__ __forceinline__ void extend_column(const CDev& D, const double* __restrict__ Ut, int32_t q0, int32_t q1,
                                              int j, int n, bool pivot, double* __restrict__ dst) {
  constexpr int UN = 4;  // rows per lane in flight
  const int lane = (int)threadIdx.x & 63;
  for (int i0 = j + lane; i0 - lane < n; i0 += 64 * UN) {
    double v[UN];
#pragma unroll
    for (int k = 0; k < UN; ++k) v[k] = pivot && i0 + 64 * k < n ? dst[i0 + 64 * k] : 0.0;
    for (int32_t q = q0; q < q1; ++q) {
      const longlong2 e = D.con[q];
      const int32_t* inv = D.inv + e.y;
      const double* Uc = Ut + e.x;
      int ic[UN];
      double w[UN];
#pragma unroll
      for (int k = 0; k < UN; ++k) ic[k] = i0 + 64 * k < n ? inv[i0 + 64 * k] : -1;
#pragma unroll
      for (int k = 0; k < UN; ++k) w[k] = ic[k] >= 0 ? Uc[ic[k]] : 0.0;
#pragma unroll
      for (int k = 0; k < UN; ++k) v[k] = ic[k] >= 0 ? v[k] + w[k] : v[k];
    }
#pragma unroll
    for (int k = 0; k < UN; ++k)
      if (i0 + 64 * k < n) dst[i0 + 64 * k] = v[k];
  }
}

// Columns per extend-add item of a front of n rows: the longest columns a
// wavefront or two, so that a few fronts still fill the chip.
__host__ __device__ __forceinline__ int extend_cols(int n) { return n > 256 ? 8 : 32; }

// Extend-add for the large fronts of one level: work item (s, c0) owns columns
// [c0, c0 + extend_cols) of front s, one wavefront a column.  Gathered by the
// front's entries through the children's inverse maps: each entry is read and
// written once, where clearing the update part and adding child by child into
// scattered entries took twice as long (2000 buses x 24 periods 1.93 -> 0.95 ms
// per factorization, 10000 x 168 about 112 -> 60, then the rate of memory).
__global__ void __launch_bounds__(256) k_extend(CDev D, const int32_t* __restrict__ items, int64_t item0, int32_t t0,
                                                double* __restrict__ Lf, double* __restrict__ Ar) {
  if (stopped(D.stop)) return;
  const int tt = (int)blockIdx.y;
  const int s = items[2 * (item0 + blockIdx.x)], c0 = items[2 * (item0 + blockIdx.x) + 1];
  const int p = D.node_p[s], u = D.node_u[s], ld = p + u;
  const int c1 = min(c0 + extend_cols(ld), ld);
  double* L = Lf + (int64_t)(t0 + tt) * D.lsize + D.node_loff[s];
  double* Ut = Ar + (int64_t)tt * D.usize;
  double* U = Ut + D.node_uoff[s];
  const int32_t* col = D.col + D.col_off[s];
  for (int j = c0 + (int)(threadIdx.x >> 6); j < c1; j += 4) {
    const int32_t q0 = col[j], q1 = col[j + 1];
    if (j < p && q0 == q1) continue;
    extend_column(D, Ut, q0, q1, j, ld, j < p, j < p ? L + (int64_t)j * ld : U + (int64_t)(j - p) * u - p);
  }
}

// The period's tree roots into its pg front (leading dimension ld, pivot block
// only), four columns per block.
__global__ void __launch_bounds__(256) k_extend_root(CDev D, int32_t t0, double* __restrict__ Cf, int64_t csize,
                                                     int64_t ld, const double* __restrict__ Ar) {
  if (stopped(D.stop)) return;
  const int tt = (int)blockIdx.y, j = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  if (j >= D.G) return;
  const int32_t* col = D.col + D.col_root;
  if (col[j] < col[j + 1])
    extend_column(D, Ar + (int64_t)tt * D.usize, col[j], col[j + 1], j, D.G, true,
                  Cf + (int64_t)(t0 + tt) * csize + (int64_t)j * ld);
}

// Broadcast of lane l's value to the whole wavefront (l uniform).
__device__ __forceinline__ double lane_bcast(double v, int l) {
  const int2 w = __builtin_bit_cast(int2, v);
  int2 r;
  r.x = __builtin_amdgcn_readlane(w.x, l);
  r.y = __builtin_amdgcn_readlane(w.y, l);
  return __builtin_bit_cast(double, r);
}

// sqrt(d) and the reciprocal of that square root, both rounded as sqrt() and
// the division round them: one hardware estimate refined by two coupled
// (Goldschmidt) steps and a last correction each, where the two functions one
// after the other are a dependent chain about three times as long -- and a
// front's pivots are one serial chain.  d outside [2^-500, 2^500] is scaled
// by a power of four first; neither zero nor infinite (see odd_pivot).
__device__ __forceinline__ void sqrt_recip(double d, double& s, double& r) {
  const bool lo = d < 0x1p-500, hi = d > 0x1p500;
  const double x = d * (lo ? 0x1p400 : (hi ? 0x1p-400 : 1.0));
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  double e = fma(-h, g, 0.5);
  g = fma(g, e, g);
  h = fma(h, e, h);
  e = fma(-h, g, 0.5);
  g = fma(g, e, g);
  h = fma(h, e, h);
  g = fma(fma(-g, g, x), h, g);
  h = h + h;
  h = fma(fma(-g, h, 1.0), h, h);
  g *= lo ? 0x1p-200 : (hi ? 0x1p200 : 1.0);
  h *= lo ? 0x1p200 : (hi ? 0x1p-200 : 1.0);
  s = g;
  r = h;
}

// The static pivot rule as the elimination uses it: the threshold, the square
// root of the replacement and its reciprocal.
struct PivotRule {
  double tol, s_repl, r_repl;
};

// Square root and reciprocal of a pivot that is static, infinite, NaN, zero
// (under a threshold below 0) or far from 1 in size: rare, kept out of the pivot
// chain.  An infinite pivot keeps inf and 0, a zero one 0 and inf.
__device__ __forceinline__ void odd_pivot(double d, const PivotRule& R, bool count, double& s, double& r, int& low) {
  const bool bad = !(d > R.tol), end = __builtin_amdgcn_class(d, 0x260);  // +-0 or infinity
  const double r_end = d > 0.0 ? 0.0 : copysign(INFINITY, d);
  const double s_not = bad ? R.s_repl : d, r_not = bad ? R.r_repl : r_end;
  sqrt_recip(d, s, r);
  asm("" : "+v"(s), "+v"(r));  // selects, not a branch around the above
  s = bad || end ? s_not : s;
  r = bad || end ? r_not : r;
  low += bad && count;
}

// Whether a pivot takes that way: not above the threshold, or outside about
// [2^-500, 2^500] (a negative one, a NaN or an infinity lies outside too, by
// its leading word as an unsigned number).
__device__ __forceinline__ bool is_odd(double d, double tol) {
  const uint32_t hi = (uint32_t)(__builtin_bit_cast(uint64_t, d) >> 32);
  return hi - 0x20c00000u > 0x5f200000u - 0x20c00000u || !(d > tol);
}

// One step of an elimination held a row per lane, a[0] the column eliminated
// (l its factored entries, lane k its pivot's row): the columns behind it take
// their update and move one to the left.  The new a[0] comes first, and its
// pivot's square root and reciprocal (s, r), the serial chain of the whole
// elimination, run between the updates of the others, an eighth of them after
// each of its dependent instructions; the empty asm statements hold that order.
// (One after the other: 37.5 us for a launch of fronts of 48 rows, now 32.6; 13.2
// and 11.0 for up to 32 rows.)
template <int FM>
__device__ __forceinline__ void next_column(double (&a)[FM], double l, int k, bool count, const PivotRule& R,
                                            double& s, double& r, int& low) {
  a[0] = fma(-l, lane_bcast(l, (k + 1) & 63), a[1]);
  const double d = lane_bcast(a[0], (k + 1) & 63);
  auto fill = [&](auto eighth) {
    constexpr int q = decltype(eighth)::value, j0 = 2 + (FM - 2) * q / 8, j1 = 2 + (FM - 2) * (q + 1) / 8;
#pragma unroll
    for (int j = j0; j < j1; ++j) {
      a[j - 1] = fma(-l, lane_bcast(l, (k + j) & 63), a[j]);
      asm volatile("" : "+v"(a[j - 1]));
    }
  };
  double y = __builtin_amdgcn_rsq(d);
  asm volatile("" : "+v"(y));
  fill(std::integral_constant<int, 0>());
  double g = d * y, h = 0.5 * y;
  asm volatile("" : "+v"(g), "+v"(h));
  fill(std::integral_constant<int, 1>());
  double e = fma(-h, g, 0.5);
  asm volatile("" : "+v"(e));
  fill(std::integral_constant<int, 2>());
  g = fma(g, e, g);
  h = fma(h, e, h);
  asm volatile("" : "+v"(g), "+v"(h));
  fill(std::integral_constant<int, 3>());
  e = fma(-h, g, 0.5);
  asm volatile("" : "+v"(e));
  fill(std::integral_constant<int, 4>());
  g = fma(g, e, g);
  h = fma(h, e, h);
  asm volatile("" : "+v"(g), "+v"(h));
  fill(std::integral_constant<int, 5>());
  e = fma(-g, g, d);
  asm volatile("" : "+v"(e));
  fill(std::integral_constant<int, 6>());
  g = fma(e, h, g);
  h = h + h;
  asm volatile("" : "+v"(g), "+v"(h));
  fill(std::integral_constant<int, 7>());
  a[FM - 1] = 0.0;
  e = fma(-g, h, 1.0);
  s = g;
  r = fma(e, h, h);
  if (is_odd(d, R.tol)) odd_pivot(d, R, count, s, r, low);
}

// A small front (p + u = f <= FM <= 64) by one wavefront: lane i owns row i in
// registers (entries above the diagonal are scratch that no valid entry ever
// reads, so the updates run unmasked).  The children's update matrices are
// gathered on the way in (no launch and no pass over memory of their own),
// child after child.  The front moves one column left at every step, a[0]
// always the column to eliminate, so that the steps are a loop of one body:
// unrolled over the columns they spilled some 400 scalar registers.
template <int FM>
__device__ __forceinline__ void small_front(const CDev& D, const FrontRec& F, double* __restrict__ L,
                                            double* __restrict__ Ut, const PivotRule& R, int& low) {
  const int p = F.p, u = F.u, f = p + u, i = (int)threadIdx.x & 63;
  double a[FM];
#pragma unroll
  for (int j = 0; j < FM; ++j) a[j] = j < p && i >= j && i < f ? L[j * f + i] : 0.0;
  // the next child's map is on its way while one is added
  const int q0 = F.k0, q1 = F.k1;
  const int at = min(i, f - 1);
  int icn = q0 < q1 ? D.inv[D.kid[q0].y + at] : -1;
  for (int q = q0; q < q1; ++q) {
    const longlong4 kd = D.kid[q];
    const int uc = (int)kd.z, ic = i < f ? icn : -1;
    const double* Uc = Ut + kd.x;
    if (q + 1 < q1) icn = D.inv[D.kid[q + 1].y + at];
    // 8 columns' loads in flight (an entry the child does not have reads its
    // first one)
#pragma unroll
    for (int j0 = 0; j0 < FM; j0 += 8) {
      double w[8];
      bool ok[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int jc = __builtin_amdgcn_readlane(ic, j0 + j);
        ok[j] = jc >= 0 && ic >= jc;
        w[j] = Uc[ok[j] ? jc * uc + ic : 0];
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) a[j0 + j] = ok[j] ? a[j0 + j] + w[j] : a[j0 + j];
    }
  }
  double s, r;
  odd_pivot(lane_bcast(a[0], 0), R, p > 0, s, r, low);
  for (int k = 0; k < p; ++k) {
    const double l = i == k ? s : a[0] * r;
    if (i >= k && i < f) L[k * f + i] = l;
    next_column(a, l, k, k + 1 < p, R, s, r, low);
  }
  double* U = Ut + F.U;
#pragma unroll
  for (int j = 0; j < FM; ++j)
    if (j < u && i >= p + j && i < f) U[j * u + (i - p)] = a[j];
}

template <bool BIG>
__device__ __forceinline__ void small_any(const CDev& D, const FrontRec& F, double* __restrict__ L,
                                          double* __restrict__ Ut, const PivotRule& R, int& low) {
  const int f = F.p + F.u;
  if (BIG) {
    if (f <= 48) small_front<48>(D, F, L, Ut, R, low);
    else small_front<64>(D, F, L, Ut, R, low);
  } else {
    if (f <= 16) small_front<16>(D, F, L, Ut, R, low);
    else if (f <= 24) small_front<24>(D, F, L, Ut, R, low);
    else small_front<32>(D, F, L, Ut, R, low);
  }
}

// The small fronts of one level, one wavefront per (front, period); those of
// more than 32 rows in launches of their own (BIG), which need twice the
// registers.
template <bool BIG>
__global__ void __launch_bounds__(64) k_factor_small(CDev D, const FrontRec* __restrict__ rec, int32_t t0,
                                                     double* __restrict__ Lf, double* __restrict__ Ar, double tol,
                                                     double repl, int32_t* __restrict__ npert) {
  if (stopped(D.stop)) return;
  const int tt = (int)blockIdx.y;
  const FrontRec F = rec[blockIdx.x];
  PivotRule R;
  R.tol = tol;
  sqrt_recip(repl, R.s_repl, R.r_repl);
  int low = 0;
  small_any<BIG>(D, F, Lf + (int64_t)(t0 + tt) * D.lsize + F.L, Ar + (int64_t)tt * D.usize, R, low);
  if (low && threadIdx.x == 0) atomicAdd(npert, low);
}

// Right-looking elimination of 16 columns, one row per lane, lanes 0-15 the
// diagonal rows; low counts the static pivots among the first n columns.
// Column k updates column k + 1 first; then that column's pivot is taken
// (a hardware estimate refined step by step, some 15 dependent operations)
// with the updates of the columns further right in between, some after each
// step: one wavefront issues an instruction every 4 cycles at best, so the
// chain's waits are where the updates belong, and every instruction counts.
// (Its steps: one coupled refinement, two corrections of the root and one of
// the reciprocal, where sqrt_recip and next_column refine twice and correct
// each once.  Either way both round as sqrt() and the division.)
// The empty asm statements hold that order; left to itself the compiler
// collects a column's updates in front of its pivot, one dependent chain, and
// spills the broadcast entries.
__device__ __forceinline__ void eliminate16(double (&a)[16], int lane, int n, const PivotRule& R, int& low) {
  double s, r;
  odd_pivot(lane_bcast(a[0], 0), R, 0 < n, s, r, low);
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    a[k] = lane == k ? s : a[k] * r;
    if (k + 1 == 16) break;
    a[k + 1] = fma(-a[k], lane_bcast(a[k], k + 1), a[k + 1]);
    const double d = lane_bcast(a[k + 1], k + 1);
    int j = k + 2, left = 8;
    auto fill = [&]() {
      const int c = (16 - j + left - 1) / left;
      --left;
#pragma unroll
      for (int q = 0; q < c; ++q, ++j) {
        a[j] = fma(-a[k], lane_bcast(a[k], j), a[j]);
        asm volatile("" : "+v"(a[j]));
      }
    };
    double y = __builtin_amdgcn_rsq(d);
    asm volatile("" : "+v"(y));
    fill();
    double g = d * y, h = 0.5 * y;
    asm volatile("" : "+v"(g), "+v"(h));
    fill();
    double e = fma(-h, g, 0.5);
    asm volatile("" : "+v"(e));
    fill();
    g = fma(g, e, g);
    h = fma(h, e, h);
    asm volatile("" : "+v"(g), "+v"(h));
    fill();
    e = fma(-g, g, d);
    asm volatile("" : "+v"(e));
    fill();
    g = fma(e, h, g);
    asm volatile("" : "+v"(g));
    fill();
    e = fma(-g, g, d);
    asm volatile("" : "+v"(e));
    fill();
    g = fma(e, h, g);
    h = h + h;
    asm volatile("" : "+v"(g), "+v"(h));
    fill();
    e = fma(-g, h, 1.0);
    s = g;
    r = fma(e, h, h);
    if (is_odd(d, R.tol)) odd_pivot(d, R, k + 1 < n, s, r, low);
  }
}

typedef double dbl4 __attribute__((ext_vector_type(4)));

// Blocked front, one panel of kb <= 64 columns [k0, k0+kb): its update by the
// columns [kbeg, k0) before it, its diagonal block's factorization and the
// solve of the kTR rows of each block against it, in one launch.  Grid (row
// blocks below the panel of the largest front, at least one; periods; fronts).
//
// What bounds it is latency: a front's panels follow one another, 64 serial
// pivots each.  So every block repeats the diagonal block's work (64 rows
// beside its own kTR) instead of waiting for another launch, the pivot chain
// runs in registers, one row per lane, 16 columns at a time: lanes 0-15 of
// every wavefront hold the 16 diagonal rows, lanes 16-63 another 48 of the
// rows below, so the pivot and column entries are broadcast within the
// wavefront and the rows' solve costs no steps of its own; the columns to the
// right take their 16-column update from the matrix cores.  8 wavefronts: the update by the columns
// before needs two per SIMD to fill the matrix cores.
// (Before: one wavefront per diagonal block, 19 us, one launch for the rows,
// 31 us, and one matrix-core update launch per 64 columns, 16 us at least.)
constexpr int kTR = 64;
constexpr int kPT = 512;  // threads
__global__ void __launch_bounds__(kPT) k_panel(Fronts F, int32_t kbeg, int32_t k0, double tol, double repl,
                                               int32_t* __restrict__ npert) {
  constexpr int NG = (kNB + kTR) / 16;      // 16-row groups, one per wavefront: 4 of the diagonal block, then the block's own rows
  constexpr int S = kNB + kTR + 16;         // column stride: the 4 columns an operand load touches fall on distinct banks
  constexpr int NWV = kPT / 64;
  static_assert(NG == NWV && kTR == 64, "one row group per wavefront, one own row per lane");
  __shared__ double P[kNB * S];
  const FrontRec f = pick_front(F.rec, F.one, blockIdx.z);
  const int rows = f.p + f.u, kb = min(kNB, f.p - k0);
  const int r0 = k0 + kb + (int)blockIdx.x * kTR;
  if (blockIdx.x > 0 && r0 >= rows) return;
  if (stopped(F.stop)) return;
  double* __restrict__ L = F.L + (int64_t)blockIdx.y * F.sL + f.L;
  const int64_t ld = f.ld;
  const int tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  // rows and columns past the front are clamped onto its last ones: what is
  // computed for them is never stored
  const int last = rows - 1;
  const int row = min(wv < 4 ? k0 + wv * 16 + lr : r0 + (wv - 4) * 16 + lr, last);
  dbl4 x[4];
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) x[c][e] = L[(int64_t)min(k0 + c * 16 + lk + 4 * e, f.p - 1) * ld + row];
  // the columns before, 64 at a time through LDS, the next 64 loaded while the
  // matrix cores work on these; in the blocks of the recursive elimination
  // order (the 128 first ones, then 64: k0 - kbeg is 0, 64, 128 or 192), each
  // block's product summed by itself and then subtracted; formed transposed
  // (see k_update)
  if (k0 > kbeg) {
    // thread: row tid % 128 of the 64 + 64 rows, columns tid / 128 + 4 i
    const int sr = tid & 127, sc = tid >> 7;
    const double* ps = L + (int64_t)(kbeg + sc) * ld + min(sr < kNB ? k0 + sr : r0 + sr - kNB, last);
    double v[16];
    auto fetch = [&]() {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        v[i] = *ps;
        ps += 4 * ld;
      }
    };
    dbl4 acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = (dbl4){0.0, 0.0, 0.0, 0.0};
    auto mul = [&](auto nc) {
#pragma unroll
      for (int k4 = 0; k4 < 16; ++k4) {
        const double* col = P + (4 * k4 + lk) * S + lr;
        const double bw = col[wv * 16];
#pragma unroll
        for (int c = 0; c < nc(); ++c) acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(col[c * 16], bw, acc[c], 0, 0, 0);
      }
    };
    fetch();
    for (int k = kbeg; k < k0; k += 64) {
#pragma unroll
      for (int i = 0; i < 16; ++i) P[(sc + 4 * i) * S + sr] = v[i];
      __syncthreads();
      if (k + 64 < k0) fetch();
      // the diagonal block's groups above its diagonal are not needed
      if (wv == 0) mul(std::integral_constant<int, 1>());
      else if (wv == 1) mul(std::integral_constant<int, 2>());
      else if (wv == 2) mul(std::integral_constant<int, 3>());
      else mul(std::integral_constant<int, 4>());
      __syncthreads();
      if (k + 64 == k0 || k + 64 - kbeg == 128) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          x[c] -= acc[c];
          acc[c] = (dbl4){0.0, 0.0, 0.0, 0.0};
        }
      }
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) P[(c * 16 + lk + 4 * e) * S + wv * 16 + lr] = x[c][e];
  __syncthreads();
  PivotRule rule;
  rule.tol = tol;
  sqrt_recip(repl, rule.s_repl, rule.r_repl);
  int bad = 0;  // static pivots
  const int nb = (kb + 15) / 16;
  constexpr int CW = (kNB + kTR - 16 + 47) / 48;  // wavefronts that hold rows in the column phase
  for (int jb = 0; jb < nb; ++jb) {
    // one 16 x 16 tile of the columns to the right, on or below the diagonal:
    // column group c, row group g, its update by the 16 columns of block b
    auto tile = [&](int b, int c, int g) {
      dbl4 y;
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = -P[(c * 16 + lk + 4 * e) * S + g * 16 + lr];
#pragma unroll
      for (int k4 = 0; k4 < 4; ++k4) {
        const double* col = P + (b * 16 + 4 * k4 + lk) * S;
        y = __builtin_amdgcn_mfma_f64_16x16x4f64(col[c * 16 + lr], col[g * 16 + lr], y, 0, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) P[(c * 16 + lk + 4 * e) * S + g * 16 + lr] = -y[e];
    };
    // the column phase: this lane's row of the tile is a diagonal row, or one
    // of the rows below
    double a[16];
    const int t = lane < 16 ? jb * 16 + lane : (jb + 1) * 16 + wv * 48 + lane - 16;
    if (wv < CW) {
      const bool in = t < kNB + kTR;
#pragma unroll
      for (int j = 0; j < 16; ++j) a[j] = in ? P[(jb * 16 + j) * S + t] : 0.0;
      // columns past kb are carried along, and used by nothing
      eliminate16(a, lane, kb - jb * 16, rule, bad);
      if (in && lane >= 16) {
#pragma unroll
        for (int j = 0; j < 16; ++j) P[(jb * 16 + j) * S + t] = a[j];
      }
    } else if (jb > 0) {
      // meanwhile the other wavefronts give the columns right of this block
      // their update by the block before
      int q = wv - CW;
      for (int c = jb + 1; c < nb; ++c)
        for (int g = c; g < NG; ++g, q = q == 0 ? NWV - CW - 1 : q - 1)
          if (q == 0) tile(jb - 1, c, g);
    }
    __syncthreads();
    // the 16 diagonal rows are the same in every wavefront, and a slower one
    // may only now have read the unfactored ones
    if (wv == 0 && lane < 16) {
#pragma unroll
      for (int j = 0; j < 16; ++j) P[(jb * 16 + j) * S + t] = a[j];
    }
    if (jb + 1 < nb && jb + 1 + wv < NG) tile(jb, jb + 1, jb + 1 + wv);
    __syncthreads();
  }
  // the rows' solution to the front, the diagonal block once
#pragma unroll 4
  for (int c = wv; c < kb; c += NWV)
    if (r0 + lane < rows) L[(int64_t)(k0 + c) * ld + r0 + lane] = P[c * S + kNB + lane];
  if (blockIdx.x == 0) {
    double* Dq = F.D + (int64_t)blockIdx.y * F.sD + f.D + (int64_t)k0 * kNB;
#pragma unroll 4
    for (int c = wv; c < kb; c += NWV)
      if (lane >= c && lane < kb) {
        const double v = P[c * S + lane];
        Dq[c * kb + lane] = v;
        Dq[lane * kb + c] = v;
      }
  }
  if (bad && tid == 0 && blockIdx.x == 0) atomicAdd(npert, bad);
}

// Trailing update after a panel of kb = min(w, p - k0) columns from k0 on, r0
// = k0 + kb: C -= P P^T on the lower part of the rows from r0 on x the columns
// from r0 on -- inner: the next w pivot columns only, else all of them.
// Columns < p live in the factor block, the others in the update block.  Grid
// (tiles of the largest front; periods; fronts).
//
// FP64 matrix cores: v_mfma_f64_16x16x4, lane l supplies A(l%16, l/16) and
// B(l/16, l%16) and holds D(l/16 + 4r, l%16), r < 4.  The product is formed
// transposed (rows of the tile along the lanes) so that each lane group writes
// 16 consecutive rows of a column of the column-major front; every entry is
// one ascending chain over the panel's columns, whatever the tile.
//
// What bounds a large launch is keeping the matrix cores issued: a block in its
// first loads or its last read-modify-write has to leave others running.  64 x
// 64 tiles of 4 wavefronts (32 x 32 each, 63 VGPRs) with 8 panel columns per
// LDS round (20 KB for both buffers) leave 7 blocks on a CU (its LDS holds no
// more; the launch bounds only keep the registers to 6 or more): 58 TFLOP/s at
// 4323 columns x 1024 panel columns x 8 periods, 47 at 4114 x 204 x 8, 55 at
// 2976 x 1024 x 2; 128 x 128 tiles of 4 wavefronts (2 blocks on a CU) reached
// 51, 33 and 37, of 8 wavefronts 60, 45 and 43, and twice the time on launches
// of few tiles.  Tiles are taken in column groups of kGroup, row by row, and
// each XCD gets a contiguous run of (period, tile) items, so that the tiles
// running side by side share panel slices in its L2.
// What bounds a launch that leaves CUs without a block is the latency of one
// block: 32 x 32 tiles, a quarter of the matrix-core chain, and 64 columns per
// round, so that few round trips to memory follow one another (see
// launch_update).
constexpr int kGroup = 8;
template <int TM, int KC>
__global__ void __launch_bounds__(256, TM == 64 ? 6 : 1)
k_update(Fronts F, int32_t k0, int32_t w, int32_t inner) {
  constexpr int S = TM + 16;         // column stride: an operand load's 4 columns fall on distinct banks
  constexpr int CS = 256 / TM;       // columns a load of the block covers
  constexpr int NLD = KC / CS;       // loads per thread and side
  constexpr int W = TM / 2, N = W / 16;  // a wavefront's quarter, in rows and 16-row groups
  // two LDS buffers: the next round is loaded into registers while the
  // matrix cores work on the current one
  __shared__ double Pi[2][KC * S], Pj[2][KC * S];
  const FrontRec f = pick_front(F.rec, F.one, blockIdx.z);
  const int rows = f.p + f.u, kb = min(w, f.p - k0), r0 = k0 + kb, cend = inner ? min(r0 + w, f.p) : rows;
  if (cend <= r0) return;
  const int R = (rows - r0 + TM - 1) / TM, Cn = (cend - r0 + TM - 1) / TM;
  // blocks are dealt round-robin to the 8 XCDs in launch order
  const int ntl = (int)gridDim.x, total = ntl * (int)gridDim.y;
  int item = (int)(blockIdx.y * gridDim.x + blockIdx.x);
  const int q8 = total >> 3;
  if (item < (q8 << 3)) item = (item & 7) * q8 + (item >> 3);
  const int per = item / ntl;
  int x = item % ntl, ti = 0, tj = 0;
  if (x >= Cn * R - Cn * (Cn - 1) / 2) return;
  if (stopped(F.stop)) return;
  for (int g = 0;; g += kGroup) {
    // column group [g, g + gw): a triangle of gw rows, then full rows
    const int gw = min(kGroup, Cn - g), tri = gw * (gw + 1) / 2, cnt = tri + (R - g - gw) * gw;
    if (x >= cnt) {
      x -= cnt;
      continue;
    }
    if (x < tri) {
      int i = 0;
      while (x > i) x -= ++i;
      ti = g + i;
      tj = g + x;
    } else {
      ti = g + gw + (x - tri) / gw;
      tj = g + (x - tri) % gw;
    }
    break;
  }
  double* L = F.L + (int64_t)per * F.sL + f.L;
  double* U = F.U + (int64_t)per * F.sU + f.U;
  const int64_t ld = f.ld;
  const int i0 = r0 + ti * TM, j0 = r0 + tj * TM;
  const int tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int wr = wv & 1, wc = wv >> 1;  // the wavefront's quarter
  // a quarter wholly above the diagonal or right of the region contributes nothing
  const bool skip = i0 + wr * W + W - 1 < j0 + wc * W || j0 + wc * W >= cend;
  dbl4 acc[N][N];
#pragma unroll
  for (int c = 0; c < N; ++c)
#pragma unroll
    for (int r = 0; r < N; ++r) acc[c][r] = (dbl4){0.0, 0.0, 0.0, 0.0};
  const int lr = lane & 15, lk = lane >> 4;
  // this thread's row of both slices (rows past the front are clamped onto
  // its last one: what is computed for them is never stored)
  const int rr = tid % TM, lc = tid / TM;
  const double* pi = L + (int64_t)(k0 + lc) * ld + min(i0 + rr, rows - 1);
  const double* pj = L + (int64_t)(k0 + lc) * ld + min(j0 + rr, rows - 1);
  const int64_t step = CS * ld;
  double ri[NLD], rj[NLD];
  auto fetch = [&](int l0) {
    if (l0 + KC <= kb) {
#pragma unroll
      for (int q = 0; q < NLD; ++q) {
        ri[q] = pi[q * step];
        rj[q] = pj[q * step];
      }
    } else {
#pragma unroll
      for (int q = 0; q < NLD; ++q) {
        const bool in = l0 + lc + CS * q < kb;
        ri[q] = in ? pi[q * step] : 0.0;
        rj[q] = in ? pj[q * step] : 0.0;
      }
    }
    pi += KC * ld;
    pj += KC * ld;
  };
  auto park = [&](int buf) {
#pragma unroll
    for (int q = 0; q < NLD; ++q) {
      Pi[buf][(lc + CS * q) * S + rr] = ri[q];
      Pj[buf][(lc + CS * q) * S + rr] = rj[q];
    }
  };
  fetch(0);
  park(0);
  __syncthreads();
  int buf = 0;
  for (int l0 = 0; l0 < kb; l0 += KC) {
    const bool more = l0 + KC < kb;
    if (more) fetch(l0 + KC);
    if (!skip) {
#pragma unroll 4
      for (int k4 = 0; k4 < KC; k4 += 4) {
        double aj[N], bi[N];
#pragma unroll
        for (int q = 0; q < N; ++q) {
          aj[q] = Pj[buf][(k4 + lk) * S + wc * W + q * 16 + lr];
          bi[q] = Pi[buf][(k4 + lk) * S + wr * W + q * 16 + lr];
        }
#pragma unroll
        for (int c = 0; c < N; ++c)
#pragma unroll
          for (int r = 0; r < N; ++r) acc[c][r] = __builtin_amdgcn_mfma_f64_16x16x4f64(aj[c], bi[r], acc[c][r], 0, 0, 0);
      }
    }
    if (more) park(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
  if (skip) return;
  const bool fresh = F.fresh && k0 == 0;
#pragma unroll
  for (int c = 0; c < N; ++c)
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const int i = i0 + wr * W + r * 16 + lr;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = j0 + wc * W + c * 16 + lk + 4 * e;
        if (i >= rows || j >= cend || i < j) continue;
        if (j < f.p) {
          L[(int64_t)j * ld + i] -= acc[c][r][e];
        } else {
          double* q = U + (int64_t)(j - f.p) * f.u + (i - f.p);
          *q = (fresh ? 0.0 : *q) - acc[c][r][e];
        }
      }
    }
}

// G x G lower update blocks of the pg fronts before them into the pivot blocks
// of fronts: entry blockIdx.y of both sides.
__global__ void k_add_chain(const double* __restrict__ Us, int64_t sU, int32_t G, double* __restrict__ C, int64_t sC) {
  const double* U = Us + (int64_t)blockIdx.y * sU;
  double* c = C + (int64_t)blockIdx.y * sC;
  const int64_t n = (int64_t)G * G;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = e / G, i = e % G;
    if (i >= j) c[j * 2 * G + i] += U[e];
  }
}

// ---- the pg chain of few generators
//
// The pg chain of G <= FM / 2 generators by one block: one wavefront eliminates
// the left fronts, one the right ones, front by front in step, a front's row
// per lane as in small_front, its update block handed to the next front
// through LDS; then the first one eliminates front m.  Launched front by front
// such a chain spends three launches of 3 to 12 us on an elimination of G
// dependent pivots, about 0.5 us each (6 generators x 24 periods: 44 us in all).  Arithmetic as in k_panel, k_update and
// k_add_chain.  sC: from one front to the next; the ramp rows' part of the
// factor stays in place, the diagonal blocks go to Dc (mirrored).
template <int FM>
__global__ void __launch_bounds__(128) k_chain_wave(int32_t G, int32_t T, double* __restrict__ Cf, int64_t sC,
                                                    double* __restrict__ Dc, int64_t sD,
                                                    const int32_t* __restrict__ stop, double tol, double repl,
                                                    int32_t* __restrict__ npert) {
  constexpr int H = FM / 2;
  __shared__ double U[2][H * H];
  __shared__ int32_t bad[2][2];
  if (stopped(stop)) return;
  const int i = (int)threadIdx.x & 63, side = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int m = (T - 1) / 2, ld = 2 * G;
  PivotRule R;
  R.tol = tol;
  sqrt_recip(repl, R.s_repl, R.r_repl);
  int low = 0;
  double a[FM], nx[H];
  // the pivot columns of a front of n rows
  auto load = [&](int t, int n) {
    const double* C = Cf + (int64_t)t * sC;
#pragma unroll
    for (int j = 0; j < H; ++j) nx[j] = j < G && i >= j && i < n ? C[j * ld + i] : 0.0;
  };
  // plus what the front before on side q leaves
  auto take = [&](int q) {
#pragma unroll
    for (int j = 0; j < H; ++j)
      if (j < G && i >= j && i < G) a[j] += U[q][j * H + i];
  };
  auto begin = [&]() {
#pragma unroll
    for (int j = 0; j < FM; ++j) a[j] = j < H ? nx[j] : 0.0;
  };
  auto eliminate = [&](int t, int n) {
    double *C = Cf + (int64_t)t * sC, *D = Dc + (int64_t)t * sD;
    double s, r;
    odd_pivot(lane_bcast(a[0], 0), R, true, s, r, low);
    for (int k = 0; k < G; ++k) {
      const double l = i == k ? s : a[0] * r;
      if (i >= G && i < n) C[k * ld + i] = l;
      if (i >= k && i < G) {
        D[k * G + i] = l;
        D[i * G + k] = l;
      }
      next_column(a, l, k, k + 1 < G, R, s, r, low);
    }
  };
  const int steps = T - 1 - m;  // the right side's fronts, as many as the left's or one more
  if (side == 1 ? steps > 0 : m > 0) load(side ? T - 1 : 0, 2 * G);
  for (int s = 0; s < steps; ++s) {
    const bool on = side || s < m;
    if (on) {
      begin();
      if (s > 0) take(side);
      if (s + 1 < (side ? steps : m)) load(side ? T - 2 - s : s + 1, 2 * G);
      eliminate(side ? T - 1 - s : s, 2 * G);
#pragma unroll
      for (int j = 0; j < H; ++j)
        if (j < G && i >= G + j && i < 2 * G) U[side][j * H + i - G] = a[j];
    }
    if (i == 0) bad[s & 1][side] = low;
    __syncthreads();
    if (stop && bad[s & 1][0] + bad[s & 1][1] > 0) {
      if (i == 0 && low) atomicAdd(npert, low);
      return;
    }
  }
  if (side == 0) {
    load(m, G);
    begin();
    if (m > 0) take(0);
    if (steps > 0) take(1);
    eliminate(m, G);
  }
  if (i == 0 && low) atomicAdd(npert, low);
}

// ---- cyclic reduction of the pg chain
//
// At level k (h = 2^k) the fronts h - 1 + j h, j < n = T / h, are left; the
// even ones, c = (n + 1) / 2 of them, are eliminated together, front j = 2 i
// with its right (j + 1) and left (j - 1) neighbours' pg variables as update
// rows, in this order (a missing neighbour's rows are zero; a level of one
// front has no left rows).  Its update block links the two.  T = 168 periods
// take 8 levels where the two-ended chain takes 84 steps, at 19/3 G^3 instead
// of 7/3 G^3 flops (a multiply-add two) for most fronts.

// Front i's updates (2G x 2G blocks Ub, ub rows) into the pivot blocks of the
// fronts that stay: front s = 2 i + 1 takes its left neighbour's (i, its right
// rows) and its right one's (i + 1, its left rows; i + 1 < c).  Grid (elements;
// fronts that stay).
__global__ void k_cyc_add(const double* __restrict__ Ub, int32_t ub, int32_t c, int32_t G, double* __restrict__ C0,
                          int64_t sC, int64_t ld, const int32_t* __restrict__ stop) {
  if (stopped(stop)) return;
  const int i = (int)blockIdx.y;
  const double* Ul = Ub + (int64_t)i * ub * ub;
  const double* Ur = i + 1 < c ? Ul + (int64_t)ub * ub + (int64_t)G * ub + G : nullptr;
  double* C = C0 + (int64_t)i * sC;
  const int64_t n = (int64_t)G * G;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t q = e / G, r = e % G;
    if (r < q) continue;
    double v = C[q * ld + r] + Ul[q * ub + r];
    if (Ur) v += Ur[q * ub + r];
    C[q * ld + r] = v;
  }
}

// The coupling of the neighbours that stay, s and s + 1 (s = i, counted among
// the ones that stay): the (left, right) block of front i + 1's update, into
// the one of the two that goes first at the next level -- the even one: s
// itself, its right rows (transposed), or s + 1, its left rows.  32 x 32 tiles.
// Grid (tile column, tile row, pairs).
__global__ void __launch_bounds__(256) k_cyc_link(const double* __restrict__ Ub, int32_t ub, int32_t G,
                                                  double* __restrict__ C0, int64_t sC, int64_t ld,
                                                  const int32_t* __restrict__ stop) {
  __shared__ double tile[32][33];
  if (stopped(stop)) return;
  const int s = (int)blockIdx.z;
  const double* X = Ub + (int64_t)(s + 1) * ub * ub + G;  // row a (left), column b (right) at X[b * ub + a]
  const int a0 = (int)blockIdx.x * 32, b0 = (int)blockIdx.y * 32, x = (int)threadIdx.x & 31, y = (int)threadIdx.x >> 5;
  if (s & 1) {
    double* C = C0 + (int64_t)(s + 1) * sC + 2 * G;
    for (int j = y; j < 32; j += 8)
      if (a0 + x < G && b0 + j < G) C[(int64_t)(b0 + j) * ld + a0 + x] = X[(int64_t)(b0 + j) * ub + a0 + x];
    return;
  }
  for (int j = y; j < 32; j += 8) tile[j][x] = (a0 + x < G && b0 + j < G) ? X[(int64_t)(b0 + j) * ub + a0 + x] : 0.0;
  __syncthreads();
  double* C = C0 + (int64_t)s * sC + G;
  for (int j = y; j < 32; j += 8)
    if (b0 + x < G && a0 + j < G) C[(int64_t)(a0 + j) * ld + b0 + x] = tile[x][j];
}

// ------------------------------------------------------------------ solves
// y -= u, then -= w (either may be NULL).
__global__ void k_sub(double* __restrict__ y, const double* __restrict__ u, const double* __restrict__ w, int32_t n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    double v = y[i];
    if (u) v -= u[i];
    if (w) v -= w[i];
    y[i] = v;
  }
}

__global__ void k_gather(const double* __restrict__ b, int32_t n_p, int32_t T, const int32_t* __restrict__ perm,
                         double* __restrict__ Y) {
  const int64_t n = (int64_t)n_p * T;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t t = e / n_p, k = e % n_p;
    Y[e] = b[t * n_p + perm[k]];
  }
}

__global__ void k_scatter_out(const double* __restrict__ Y, int32_t n_p, int32_t T,
                              const int32_t* __restrict__ perm, double* __restrict__ x) {
  const int64_t n = (int64_t)n_p * T;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t t = e / n_p, k = e % n_p;
    x[t * n_p + perm[k]] = Y[e];
  }
}

// Forward, a small front by one wavefront, lane i its row i: v = b(pivots) -
// the children's pivot-row updates, their other rows summed into this front's
// update vector (gathered through the inverse maps, child after child), then
// L11 z = v and w += L21 z, 8 columns of L in flight.  W holds, per front, what
// its subtree subtracts from the right-hand side at the front's update rows.
__device__ __forceinline__ void fwd_small(const CDev& D, const FrontRec& F, const double* __restrict__ Lt,
                                          double* __restrict__ Yt, double* __restrict__ Wt, int i) {
  const int p = F.p, f = p + F.u, fs = F.f, at = min(i, f - 1);
  const double* L = Lt + F.L;
  const double d = L[(i < p ? i : 0) * f + (i < p ? i : 0)];
  double v = i < p ? Yt[fs + i] : 0.0;
  const int q0 = F.k0, q1 = F.k1;
  int icn = q0 < q1 ? D.inv[D.kid[q0].y + at] : -1;
  for (int q = q0; q < q1; ++q) {
    const int ic = i < f ? icn : -1;
    const double w = Wt[D.kid[q].w + max(ic, 0)];
    if (q + 1 < q1) icn = D.inv[D.kid[q + 1].y + at];
    v = ic >= 0 ? (i < p ? v - w : v + w) : v;
  }
  for (int k0 = 0; k0 < p; k0 += 8) {
    double t[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) t[j] = L[min(k0 + j, p - 1) * f + at];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = k0 + j;
      if (k >= p) break;
      const double x = lane_bcast(v / d, k);
      const double z = x * t[j];
      v = i == k ? x : (i > k ? (i < p ? v - z : v + z) : v);
    }
  }
  if (i < p) Yt[fs + i] = v;
  else if (i < f) Wt[F.W + i - p] = v;
}

// The small fronts of one level, a wavefront each (k_fwd_small); and
// consecutive levels of at most kTreeFronts fronts, all small, in one launch,
// a block per period, the levels separated by barriers (k_fwd_tree; ptr: the
// levels' starts in rec).  Four such levels of a 57-bus network are 13.7 us
// against 4 x 7 (backward 12.3 against 4 x 6): what a launch waits for is the
// latency of its one chain, and a barrier costs less than a launch.  With more
// fronts than two per wavefront a level's launch has the chip to spread over.
// The factorization's levels stay apart: held together they took 78 us against
// 4 x 15, every front size's code in one kernel spilling its scalars.
__global__ void __launch_bounds__(64) k_fwd_small(CDev D, const FrontRec* __restrict__ rec,
                                                  const double* __restrict__ Lf, double* __restrict__ Y,
                                                  double* __restrict__ W) {
  const int t = (int)blockIdx.y;
  const FrontRec F = rec[blockIdx.x];
  fwd_small(D, F, Lf + (int64_t)t * D.lsize, Y + (int64_t)t * D.n_p, W + (int64_t)t * D.wsize,
            (int)threadIdx.x);
}
__global__ void __launch_bounds__(kTreeT) k_fwd_tree(CDev D, const FrontRec* __restrict__ rec,
                                                     const int64_t* __restrict__ ptr, int32_t h0, int32_t h1,
                                                     const double* __restrict__ Lf, double* __restrict__ Y,
                                                     double* __restrict__ W) {
  const int t = (int)blockIdx.x, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  for (int h = h0; h < h1; ++h) {
    for (int q = (int)ptr[h] + wv; q < (int)ptr[h + 1]; q += kTreeT / 64) {
      const FrontRec F = rec[q];
      fwd_small(D, F, Lf + (int64_t)t * D.lsize, Y + (int64_t)t * D.n_p, W + (int64_t)t * D.wsize,
                (int)threadIdx.x & 63);
    }
    __syncthreads();
  }
}

// Forward, large fronts of one level, step 1: pull the children's update
// vectors (pivot rows subtracted from Y in place, other rows summed into this
// front's W).  Grid (periods; 1; fronts).
__global__ void __launch_bounds__(256) k_fwd_pull(CDev D, const FrontRec* __restrict__ rec, double* __restrict__ Y,
                                                  double* __restrict__ W) {
  const FrontRec f = rec[blockIdx.z];
  const int t = (int)blockIdx.x;
  double* Ys = Y + (int64_t)t * D.n_p + f.f;
  double* Wt = W + (int64_t)t * D.wsize;
  double* Ws = Wt + f.W;
  for (int a = (int)threadIdx.x; a < f.u; a += (int)blockDim.x) Ws[a] = 0.0;
  __syncthreads();
  for (int q = f.k0; q < f.k1; ++q) {
    const int c = D.kids[q];
    const int uc = D.node_u[c];
    const int32_t* rel = D.rel + D.row_ptr[c];
    const double* Wc = Wt + D.node_woff[c];
    for (int a = (int)threadIdx.x; a < uc; a += (int)blockDim.x) {
      const int r = rel[a];
      if (r < f.p) Ys[r] -= Wc[a];
      else Ws[r - f.p] += Wc[a];
    }
    __syncthreads();
  }
}

// The period's tree roots' update vectors into its pg right-hand side.
__global__ void __launch_bounds__(256) k_fwd_root_pull(CDev D, const int32_t* __restrict__ roots, int32_t nroots,
                                                       double* __restrict__ Y, const double* __restrict__ W) {
  const int t = (int)blockIdx.x;
  double* Yp = Y + (int64_t)t * D.n_p + D.n_int;
  const double* Wt = W + (int64_t)t * D.wsize;
  for (int k = 0; k < nroots; ++k) {
    const int c = roots[k];
    const int uc = D.node_u[c];
    const int32_t* rel = D.rel + D.row_ptr[c];
    const double* Wc = Wt + D.node_woff[c];
    for (int a = (int)threadIdx.x; a < uc; a += (int)blockDim.x) Yp[rel[a]] -= Wc[a];
    __syncthreads();
  }
}

// A batch of fronts as the blocked solve kernels see it (front blockIdx.z of
// rec, batch entry blockIdx.y: a period, or a pg front of the chain): factor
// and diagonal blocks, right-hand side / solution y, forward solution z,
// update vector w and its running sums v, each with its stride.
struct Tri {
  const FrontRec* rec;  // NULL: the one front below
  FrontRec one;
  const double *L, *D;
  double *y, *z, *w, *v;
  int64_t sL, sD, sy, sw, sv;
};

// The 64 x 64 triangle of a panel (or a smaller front's N x N one, N a multiple
// of 16), solved by one wavefront: lane i holds row i
// of the symmetric diagonal block in registers (forward: its entries left of
// the diagonal, backward those right of it, which are column i below the
// diagonal; 0 elsewhere, or finite past kb, where the steps multiply by 0: never
// the diagonal, which may be infinite), its entry v of the right-hand side and
// its pivot's reciprocal.  Step k: every lane's product v r, of which lane k's is entry k
// of the solution, broadcast, and one update -- four instructions, and 64 of
// these steps are what a solve launch waits for.  Lanes past kb hold zeros.
// Every step runs in every lane, with a zero where there is no entry, so an
// entry that is infinite or NaN makes all lanes NaN, the last one broadcast too:
// then the steps run once more, from memory, each in the lanes it belongs to.
template <int N = 64>
struct Triangle {
  double t[N], r;
};
template <bool FWD, int N>
__device__ __forceinline__ void load_triangle(Triangle<N>& T, const double* __restrict__ D, int kb, int lane) {
  const int at = min(lane, kb - 1);
#pragma unroll
  for (int k = 0; k < N; ++k) T.t[k] = D[min(k, kb - 1) * kb + at];
  const double d = D[at * kb + at];
  // (backward, the last row has no entries; past kb it would meet its diagonal)
  int ln = FWD ? (lane < kb ? lane : 0) : (lane < kb - 1 ? lane : 64);
  // the masks below are taken when they are needed (kept over a front's
  // panels they would fill the scalar registers four times over)
  asm volatile("" : "+v"(ln));
#pragma unroll
  for (int k = 0; k < N; ++k) T.t[k] = (FWD ? k < ln : k > ln) ? T.t[k] : 0.0;
  T.r = lane < kb ? 1.0 / d : 0.0;
}
template <bool FWD, int N>
__device__ __forceinline__ double solve_triangle(const Triangle<N>& T, const double* __restrict__ D, int kb, int lane,
                                                 double y) {
  double v = y, x = 0.0;
#pragma unroll
  for (int q = 0; q < N / 16; ++q) {
    const int b = FWD ? q : N / 16 - 1 - q;
    if (b * 16 >= kb) continue;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int k = b * 16 + (FWD ? j : 15 - j);
      x = lane_bcast(v * T.r, k);
      v = fma(-T.t[k], x, v);
    }
  }
  const uint32_t hi = (uint32_t)(__builtin_bit_cast(uint64_t, x) >> 32) & 0x7ff00000u;
  if (__builtin_expect(hi == 0x7ff00000u, 0)) {
    v = y;
#pragma unroll 1
    for (int q = 0; q < kb; ++q) {
      const int k = FWD ? q : kb - 1 - q;
      x = lane_bcast(v * T.r, k);
      if (lane < kb && (FWD ? k < lane : k > lane)) v = fma(-D[k * kb + lane], x, v);
    }
  }
  return v * T.r;
}

// Sum over a wavefront, the same in every lane: the butterfly over lane
// distances 32, 16, 8, 4, 2, 1.  The first two swap halves and rows of 16
// lanes; after them every row holds the same values, and the lanes of a row
// repeat with the next distance's period, so a rotation within the row pairs
// the same values as an exchange would.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const int2 w = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_update_dpp(0, w.x, CTRL, 0xf, 0xf, false),
                                              __builtin_amdgcn_update_dpp(0, w.y, CTRL, 0xf, 0xf, false)));
}
template <int N>
__device__ __forceinline__ void wave_sum(double (&v)[N]) {
  auto words = [](double x) { return __builtin_bit_cast(uint2, x); };
  auto both = [](uint32_t x, uint32_t y) { return __builtin_bit_cast(double, make_uint2(x, y)); };
#pragma unroll
  for (int n = 0; n < N; ++n) {
    const uint2 w = words(v[n]);
    const auto x = __builtin_amdgcn_permlane32_swap(w.x, w.x, false, false);
    const auto y = __builtin_amdgcn_permlane32_swap(w.y, w.y, false, false);
    v[n] = both(x[0], y[0]) + both(x[1], y[1]);
  }
#pragma unroll
  for (int n = 0; n < N; ++n) {
    const uint2 w = words(v[n]);
    const auto x = __builtin_amdgcn_permlane16_swap(w.x, w.x, false, false);
    const auto y = __builtin_amdgcn_permlane16_swap(w.y, w.y, false, false);
    v[n] = both(x[0], y[0]) + both(x[1], y[1]);
  }
#pragma unroll
  for (int n = 0; n < N; ++n) v[n] += dpp_move<0x128>(v[n]);  // row_ror:8
#pragma unroll
  for (int n = 0; n < N; ++n) v[n] += dpp_move<0x124>(v[n]);  // row_ror:4
#pragma unroll
  for (int n = 0; n < N; ++n) v[n] += dpp_move<0x122>(v[n]);  // row_ror:2
#pragma unroll
  for (int n = 0; n < N; ++n) v[n] += dpp_move<0x121>(v[n]);  // row_ror:1
}

// Forward, kSolve columns from k0 on of each front per launch, grid (row blocks
// below them of the largest front, at least one; batch; fronts).  The launches
// of a front follow one another, so a launch goes as far as one block can
// alone: the columns' 64-column panels one after the other, each one's triangle
// by one of two wavefronts in turn (solve_triangle; the other loads the next), while
// the others load their rows of the panel -- the rows of the later panels,
// which every block repeats, and the block's own ROWS.  (A launch per panel
// took 8 us, most of it the way to the first loads and back; four panels of two
// 800-row fronts in one take 20.)  Block 0 stores the solution in z.  Each row takes a panel's products
// as one sum: pivot rows subtract it from y, update rows carry one running sum
// over the panels in v.  Of y the launch's own columns are only read and z is
// only written, so the blocks of one launch never touch an entry another block
// writes.
// chunk 0 (interior fronts): the sum over all columns goes onto w at the last
// panel.  chunk > 0 (the pg chain, a multiple of 64): the sums over chunk
// columns are added up in w one after the other, from 0; at the last panel w
// is also subtracted from next, the right-hand side of the chain neighbour
// (stride sn), by the batch entries whose bit in pass is set.
constexpr int kSolve = 256;           // columns per launch
constexpr int kInner = kSolve - kNB;  // of which rows of later panels
template <int ROWS>
__global__ void __launch_bounds__(kInner + ROWS + 128) k_fwd_panel(Tri A, int32_t k0, int32_t chunk,
                                                                   double* __restrict__ next, int64_t sn,
                                                                   int32_t pass) {
  __shared__ double xs[kNB], ys[kSolve];
  const FrontRec f = pick_front(A.rec, A.one, blockIdx.z);
  const int rows = f.p + f.u, kend = min(k0 + kSolve, f.p);
  const int tid = (int)threadIdx.x;
  const int own = kend + (int)blockIdx.x * ROWS;  // first own row
  if (blockIdx.x > 0 && own >= rows) return;
  const double* L = A.L + (int64_t)blockIdx.y * A.sL + f.L;
  const double* D = A.D + (int64_t)blockIdx.y * A.sD + f.D;
  double* y = A.y + (int64_t)blockIdx.y * A.sy + f.f;
  double* z = A.z + (int64_t)blockIdx.y * A.sy + f.f;
  if (tid >= kInner + ROWS) {
    const int lane = tid & 63, odd = (tid - kInner - ROWS) >> 6;
    Triangle<> T;
    auto load = [&](int k) {
      if (k < kend) load_triangle<true>(T, D + (int64_t)k * kNB, min(kNB, kend - k), lane);
    };
    double v = lane < kend - k0 ? y[k0 + lane] : 0.0;
    load(k0 + odd * kNB);
    for (int k = k0, q = 0; k < kend; k += kNB, ++q) {
      const int kb = min(kNB, kend - k);
      const bool mine = (q & 1) == odd;
      if (mine) {
        const double x = solve_triangle<true>(T, D + (int64_t)k * kNB, kb, lane, v);
        xs[lane] = x;
        if (blockIdx.x == 0 && lane < kb) z[k + lane] = x;
      }
      __syncthreads();
      if (mine) load(k + 2 * kNB);
      __syncthreads();
      v = k + kNB + lane < kend ? ys[k + kNB - k0 + lane] : 0.0;
    }
    return;
  }
  const bool inner = tid < kInner;
  const int i = inner ? k0 + kNB + tid : own + tid - kInner;
  const bool row = i < (inner ? kend : rows);
  const int j = i - f.p;  // update row
  const bool up = row && j >= 0;
  // the row's entries of the panel, 16 at a time; rows of no use read row k0's
  const int64_t ld = f.ld;
  const double* Li = L + (row ? i : k0);
  double rv[64];
  auto load = [&](int k, int q) {
    const double* at = Li + (int64_t)(k + q * 16) * ld;
    if (k + q * 16 + 16 <= kend) {
#pragma unroll
      for (int l = 0; l < 16; ++l, at += ld) rv[q * 16 + l] = *at;
    } else {
#pragma unroll
      for (int l = 0; l < 16; ++l, at += ld) rv[q * 16 + l] = k + q * 16 + l < kend ? *at : 0.0;
    }
  };
#pragma unroll
  for (int q = 0; q < 4; ++q) load(k0, q);
  // pivot rows: the right-hand side; update rows: the running sum, w and next
  double* w = A.w + (int64_t)blockIdx.y * A.sw + f.W + j;
  double* v = A.v + (int64_t)blockIdx.y * A.sv + f.W + j;
  double yi = row && !up ? y[i] : 0.0;
  double sum = up && (chunk ? k0 % chunk != 0 : k0 != 0) ? *v : 0.0;
  double wi = up && (chunk ? k0 >= chunk : true) ? *w : 0.0;
  for (int k = k0; k < kend; k += kNB) {
    const int kb = min(kNB, kend - k);
    __syncthreads();  // the panel's solution
    // (an inner wavefront holds one panel's rows: none of them is below k then)
    if (inner && (tid & ~63) + k0 < k) {
      __syncthreads();
      continue;
    }
    double acc = up && !(chunk && k % chunk == 0) ? sum : 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (q * 16 < kb) {
#pragma unroll
        for (int l = q * 16; l < q * 16 + 16; ++l) acc += rv[l] * xs[l];
      }
      if (k + kNB < kend && !(inner && (tid & ~63) + k0 < k + kNB)) load(k + kNB, q);
    }
    if (up) {
      sum = acc;
      if (chunk && (k + kb == f.p || (k + kb) % chunk == 0)) wi += sum;
    } else {
      yi -= acc;
      if (inner) ys[i - k0] = yi;
    }
    __syncthreads();
  }
  if (!row || inner) return;
  if (!up) {
    y[i] = yi;
  } else if (!chunk) {
    if (kend == f.p) *w = wi + sum;
    else *v = sum;
  } else {
    *w = wi;
    *v = sum;
    if (kend == f.p && blockIdx.y < 2 && (pass >> blockIdx.y & 1)) next[(int64_t)blockIdx.y * sn + j] -= wi;
  }
}

// Backward, z[j] -= sum_i L21[i, j] x_u[i] for the pivot columns, one
// wavefront per column; x_u gathered through the front's row list (interior:
// rows, x the period's solution) or contiguous (rows NULL).  Grid (column
// blocks of 4; batch; fronts).
__global__ void __launch_bounds__(256) k_bwd_gemv(Tri A, const int32_t* __restrict__ rows,
                                                  const double* __restrict__ x, int64_t sx) {
  const FrontRec f = pick_front(A.rec, A.one, blockIdx.z);
  const int j = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  const int lane = (int)(threadIdx.x & 63);
  if (j >= f.p) return;
  const double* col = A.L + (int64_t)blockIdx.y * A.sL + f.L + (int64_t)j * f.ld + f.p;
  const double* xs = x + (int64_t)blockIdx.y * sx;
  const int32_t* rr = rows ? rows + f.R : nullptr;
  double acc = 0.0;
#pragma unroll 4
  for (int a = lane; a < f.u; a += 64) acc += col[a] * xs[rr ? rr[a] : a];
  double sum[1] = {acc};
  wave_sum(sum);
  if (lane == 0) A.z[(int64_t)blockIdx.y * A.sy + f.f + j] -= sum[0];
}

// Cyclic reduction, forward: what the level's c fronts subtract from the
// right-hand sides of the fronts that stay (front i: its left neighbour's
// right rows, then its right one's left rows).  Grid (rows; fronts that stay).
__global__ void k_cyc_pull(const double* __restrict__ W, int64_t sw, int32_t c, int32_t G, double* __restrict__ Y,
                           int64_t sy) {
  const int i = (int)blockIdx.y;
  const double* w = W + (int64_t)i * sw;
  double* y = Y + (int64_t)i * sy;
  for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < G; g += gridDim.x * blockDim.x) {
    double v = y[g] - w[g];
    if (i + 1 < c) v -= w[sw + G + g];
    y[g] = v;
  }
}

// Cyclic reduction, backward: z[j] -= sum L21[., j] x over the solutions of the
// right (x + sh) and left (x - sh) neighbours of the fronts (x: the first
// front's own), one wavefront per column.  n as above.  Grid (column blocks of
// 4; fronts).
__global__ void __launch_bounds__(256) k_cyc_gemv(Tri A, int32_t n, const double* __restrict__ x, int64_t sh) {
  const FrontRec f = A.one;
  const int i = (int)blockIdx.y, lane = (int)(threadIdx.x & 63);
  const int j = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  if (j >= f.p) return;
  const double* col = A.L + (int64_t)i * A.sL + (int64_t)j * f.ld + f.p;
  const double* xs = x + (int64_t)i * A.sy;
  double acc = 0.0;
  if (2 * i + 1 < n) {
#pragma unroll 4
    for (int a = lane; a < f.p; a += 64) acc += col[a] * xs[sh + a];
  }
  if (i > 0) {
#pragma unroll 4
    for (int a = lane; a < f.p; a += 64) acc += col[f.p + a] * xs[a - sh];
  }
  double sum[1] = {acc};
  wave_sum(sum);
  if (lane == 0) A.z[(int64_t)i * A.sy + j] -= sum[0];
}

// Backward triangle L11^T x = z, kSolve columns of each front per launch, from
// the last (the q-th kSolve columns counted from the front's last panel), as
// the forward launch: the 64-column panels one after the other, each one's
// triangle by one of the last two wavefronts in turn from z (the launch's own
// columns are only read), the others subtract the panel's contribution from the columns of the
// launch's earlier panels, which every block repeats (held in LDS), and from
// the block's own columns of z before them: a column per wavefront, lanes over
// the panel's rows, 4 columns' loads in flight.  Block 0 stores x in y.  Grid
// (blocks of cols columns; batch; fronts).
constexpr int kBwdT = 512 + 128;
__global__ void __launch_bounds__(kBwdT) k_bwd_panel(Tri A, int32_t q, int32_t cols) {
  __shared__ double xs[kNB], zs[kSolve];
  const FrontRec f = pick_front(A.rec, A.one, blockIdx.z);
  // the launch's columns [k0, kend), whole panels from the front's last one
  const int np = (f.p + kNB - 1) / kNB, pe = np - q * (kSolve / kNB), pb = max(0, pe - kSolve / kNB);
  if (pe <= 0) return;
  const int k0 = pb * kNB, kend = min(pe * kNB, f.p);
  const int jb = (int)blockIdx.x * cols, je = min(jb + cols, k0);
  if (blockIdx.x > 0 && jb >= k0) return;
  const double* L = A.L + (int64_t)blockIdx.y * A.sL + f.L;
  const double* D = A.D + (int64_t)blockIdx.y * A.sD + f.D;
  double* y = A.y + (int64_t)blockIdx.y * A.sy + f.f;
  double* z = A.z + (int64_t)blockIdx.y * A.sy + f.f;
  const int tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int e = tid; e < kend - k0; e += kBwdT) zs[e] = z[k0 + e];
  __syncthreads();
  constexpr int NW = kBwdT / 64 - 2, UN = 4;
  if (wv >= NW) {
    const int odd = wv - NW;
    Triangle<> T;
    auto load = [&](int k) {
      if (k >= k0) load_triangle<false>(T, D + (int64_t)k * kNB, min(kNB, f.p - k), lane);
    };
    load((pe - 1 - odd) * kNB);
    for (int k = (pe - 1) * kNB, c = 0; k >= k0; k -= kNB, ++c) {
      const int kb = min(kNB, f.p - k);
      const bool mine = (c & 1) == odd;
      if (mine) {
        const double x = solve_triangle<false>(T, D + (int64_t)k * kNB, kb, lane,
                                               lane < kb ? zs[k - k0 + lane] : 0.0);
        xs[lane] = x;
        if (blockIdx.x == 0 && lane < kb) y[k + lane] = x;
      }
      __syncthreads();
      if (mine) load(k - 2 * kNB);
      __syncthreads();
    }
    return;
  }
  for (int k = (pe - 1) * kNB; k >= k0; k -= kNB) {
    const int kb = min(kNB, f.p - k);
    // columns: the launch's earlier ones, then the block's own
    const int ni = k - k0, n = ni + max(0, je - jb);
    bool waited = false;
    for (int c0 = wv; c0 < n || !waited; c0 += NW * UN) {
      double cv[UN];
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const int c = c0 + u * NW, j = c < ni ? k0 + c : jb + c - ni;
        cv[u] = c < n && lane < kb ? L[(int64_t)j * f.ld + k + lane] : 0.0;
      }
      if (!waited) {
        __syncthreads();  // the panel's solution
        waited = true;
      }
      const double xk = xs[lane];
#pragma unroll
      for (int u = 0; u < UN; ++u) cv[u] = lane < kb ? cv[u] * xk : 0.0;
      wave_sum(cv);
      // lane u keeps column u's
      const double acc = lane == 0 ? cv[0] : lane == 1 ? cv[1] : lane == 2 ? cv[2] : cv[3];
      const int c = c0 + lane * NW;
      if (lane < UN && c < n) {
        if (c < ni) zs[c] -= acc;
        else z[jb + c - ni] -= acc;
      }
    }
    __syncthreads();
  }
}

// Both solves along a chain factored by k_chain_wave, in one block of two
// wavefronts: the left and the right fronts' forward solves, front m's two, the
// backward solves outwards, the next front's factor loaded meanwhile.  Y, Z:
// the pg right-hand side / solution and forward solution of period 0, sy from
// one period to the next.  Sums as in k_fwd_panel, k_sub, k_bwd_gemv (whose
// butterfly over the lanes is a tree over a column's entries here) and
// k_bwd_panel.
template <int N>
__global__ void __launch_bounds__(128) k_chain_wave_solve(int32_t G, int32_t T, const double* __restrict__ Cf,
                                                          int64_t sC, const double* __restrict__ Dc, int64_t sD,
                                                          double* __restrict__ Y, double* __restrict__ Z, int64_t sy) {
  constexpr bool kAhead = N <= 32;  // two fronts of more do not fit the registers
  __shared__ double sh[2][64], xm[64];
  const int i = (int)threadIdx.x & 63, side = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int m = (T - 1) / 2, ld = 2 * G, g = min(i, G - 1);
  const int n = side ? T - 1 - m : m;  // the side's fronts
  auto front = [&](int s) { return side ? T - 1 - s : s; };
  struct Front {
    Triangle<N> T;
    double l[N], y;
  } A, B;
  // forward: lane i its ramp row's entries; backward: its column's
  auto load = [&](Front& F, int s, auto fwd) {
    const int t = front(s);
    const double *C = Cf + (int64_t)t * sC + G, *v = (fwd() ? Y : Z) + (int64_t)t * sy;
    load_triangle<fwd()>(F.T, Dc + (int64_t)t * sD, G, i);
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const double e = fwd() ? C[min(k, G - 1) * ld + g] : C[g * ld + min(k, G - 1)];
      F.l[k] = k < G ? e : 0.0;
    }
    F.y = i < G ? v[i] : 0.0;
  };
  constexpr std::true_type fwd;
  constexpr std::false_type bwd;
  double sum = 0.0;
  if (kAhead && n > 0) load(A, 0, fwd);
  for (int s = 0; s < n; ++s) {
    if (!kAhead) load(A, s, fwd);
    else if (s + 1 < n) load(B, s + 1, fwd);
    const double z = solve_triangle<true>(A.T, Dc + (int64_t)front(s) * sD, G, i,
                                          s > 0 && i < G ? A.y - sum : A.y);
    if (i < G) Z[(int64_t)front(s) * sy + i] = z;
    sum = 0.0;
#pragma unroll
    for (int k = 0; k < N; ++k) sum += A.l[k] * lane_bcast(z, k);
    if (kAhead) A = B;
  }
  if (kAhead && n > 0) load(B, n - 1, bwd);
  sh[side][i] = sum;
  __syncthreads();
  if (side == 0) {
    double v = i < G ? Y[(int64_t)m * sy + i] : 0.0;
    if (m > 0 && i < G) v -= sh[0][i];
    if (T > 1 && i < G) v -= sh[1][i];
    Triangle<N> M;
    load_triangle<true>(M, Dc + (int64_t)m * sD, G, i);
    v = solve_triangle<true>(M, Dc + (int64_t)m * sD, G, i, v);
    load_triangle<false>(M, Dc + (int64_t)m * sD, G, i);
    v = solve_triangle<false>(M, Dc + (int64_t)m * sD, G, i, v);
    if (i < G) Y[(int64_t)m * sy + i] = v;
    xm[i] = v;
  }
  __syncthreads();
  double x = xm[i];
  for (int s = n - 1; s >= 0; --s) {
    if (kAhead) A = B;
    if (!kAhead) load(A, s, bwd);
    else if (s > 0) load(B, s - 1, bwd);
    double w[N];
#pragma unroll
    for (int k = 0; k < N; ++k) w[k] = A.l[k] * lane_bcast(x, k);
#pragma unroll
    for (int d = N > 32 ? 32 : N / 2; d > 0; d /= 2)
#pragma unroll
      for (int k = 0; k < d && k + d < N; ++k) w[k] += w[k + d];
    x = solve_triangle<false>(A.T, Dc + (int64_t)front(s) * sD, G, i, i < G ? A.y - w[0] : 0.0);
    if (i < G) Y[(int64_t)front(s) * sy + i] = x;
  }
}

// Backward, a small front by one wavefront, lane i its pivot column i: gather x
// at the update rows, v = y - L21^T x_u, then L11^T x = v, 8 rows of L in
// flight.
__device__ __forceinline__ void bwd_small(const CDev& D, const FrontRec& F, const double* __restrict__ Lt,
                                          double* __restrict__ Yt, int i) {
  const int p = F.p, u = F.u, f = p + u, fs = F.f;
  const int at = min(i, p - 1);
  const double* col = Lt + F.L + at * f;
  const double d = col[at];
  const double xu = i < u ? Yt[D.rows[F.R + i]] : 0.0;
  double v = i < p ? Yt[fs + i] : 0.0;
  for (int a0 = 0; a0 < u; a0 += 8) {
    double t[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) t[j] = col[min(p + a0 + j, f - 1)];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (a0 + j >= u) break;
      v -= t[j] * lane_bcast(xu, a0 + j);
    }
  }
  for (int k0 = p - 1; k0 >= 0; k0 -= 8) {
    double t[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) t[j] = col[max(k0 - j, 0)];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = k0 - j;
      if (k < 0) break;
      const double x = lane_bcast(v / d, k);
      const double w = v - t[j] * x;
      v = i == k ? x : (i < k ? w : v);
    }
  }
  if (i < p) Yt[fs + i] = v;
}
__global__ void __launch_bounds__(64) k_bwd_small(CDev D, const FrontRec* __restrict__ rec,
                                                  const double* __restrict__ Lf, double* __restrict__ Y) {
  const int t = (int)blockIdx.y;
  const FrontRec F = rec[blockIdx.x];
  bwd_small(D, F, Lf + (int64_t)t * D.lsize, Y + (int64_t)t * D.n_p, (int)threadIdx.x);
}
__global__ void __launch_bounds__(kTreeT) k_bwd_tree(CDev D, const FrontRec* __restrict__ rec,
                                                     const int64_t* __restrict__ ptr, int32_t h0, int32_t h1,
                                                     const double* __restrict__ Lf, double* __restrict__ Y) {
  const int t = (int)blockIdx.x, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  for (int h = h1 - 1; h >= h0; --h) {
    for (int q = (int)ptr[h] + wv; q < (int)ptr[h + 1]; q += kTreeT / 64) {
      const FrontRec F = rec[q];
      bwd_small(D, F, Lf + (int64_t)t * D.lsize, Y + (int64_t)t * D.n_p, (int)threadIdx.x & 63);
    }
    __syncthreads();
  }
}

int grid_for(int64_t n, int block) {
  const int64_t g = (n + block - 1) / block;
  return (int)std::max<int64_t>(1, std::min<int64_t>(g, 65535));
}

}  // namespace
}  // namespace opf

using namespace opf;

// ------------------------------------------------------------------ object
namespace {

struct CholInst {
  CholPlan plan;
  const InstHost* I = nullptr;
  CDev dev{};
  int32_t *d_node_p = nullptr, *d_node_u = nullptr, *d_rel = nullptr, *d_kids = nullptr,
          *d_rows = nullptr, *d_perm = nullptr, *d_items = nullptr, *d_roots = nullptr,
          *d_kpos0 = nullptr, *d_kpos1 = nullptr, *d_ramp = nullptr, *d_inv = nullptr, *d_col = nullptr;
  int64_t *d_coloff = nullptr, *d_smallptr = nullptr;
  std::vector<int32_t> run_end;  // per level: the end of the run of small levels it starts or continues, else itself
  longlong2* d_con = nullptr;
  longlong4* d_kid = nullptr;
  std::vector<int64_t> lvl_item, lvl_big;  // per level: extend-add items; the first small front of more than 32 rows
  int64_t *d_loff = nullptr, *d_uoff = nullptr, *d_woff = nullptr, *d_rowptr = nullptr, *d_slot = nullptr;
  double *Lf = nullptr, *Cf = nullptr, *Df = nullptr, *Dc = nullptr, *Ar = nullptr, *W = nullptr, *V = nullptr, *Wc = nullptr, *Y = nullptr, *Z = nullptr;
  double* Gp = nullptr;  // running sums of the chain's L21 z (a step's fronts)
  std::vector<FrontRec> rec;  // the large fronts, by level
  FrontRec crec[3];           // the pg fronts: with no, G and 2 G update rows
  bool cyclic = false;        // pg fronts by cyclic reduction, else from both ends:
  bool wave = false, wave_solve = false;  // by two wavefronts
  int32_t cld = 0;            // their leading dimension: 2 G or 3 G
  double* Uc = nullptr;       // cyclic reduction: a level's update blocks (in Ar, or opf_chol::Uc)
  FrontRec *d_rec = nullptr, *d_srec = nullptr;  // large fronts; small ones, by level
  int64_t csize = 0, wsize = 0, dsize = 0, dcsize = 0;
  int32_t chunk = 1;
};

}  // namespace

struct opf_chol {
  opf_model* model = nullptr;
  int device = -1;
  std::vector<CholInst> inst;
  double* Us = nullptr;  // two G x G update blocks of the pg chain, one per end (largest G)
  double* Uc = nullptr;  // cyclic reduction's update blocks, where an instance's Ar does not hold them (largest level)
  // the pg chain runs on a stream of its own, chunk by chunk, behind the
  // interior fronts of the next chunk (events order the two)
  hipStream_t cs = nullptr;
  std::vector<hipEvent_t> evs;
  // the solve recorded once into a HIP graph per (b, x) pair and replayed
  // on the model's stream (its launch sequence is fixed for the object)
  hipStream_t gs = nullptr;
  hipGraphExec_t gexec = nullptr;
  const double* gb = nullptr;
  double* gx = nullptr;
  bool use_graph = true;
  bool stop_on_pivot = false;  // skip the rest of a factorization after its first static pivot
  std::vector<void*> allocs;
  void* work = nullptr;  // chol_workspace
  double flops = 0.0, flops_int = 0.0;
  int64_t factor_entries = 0, arena_entries = 0;
};

const opf_model* opf::chol_model(const opf_chol* F) { return F ? F->model : nullptr; }

int opf::chol_workspace(opf_chol* F, size_t bytes, void** out) {
  if (!F->work && hipMalloc(&F->work, bytes) != hipSuccess) {
    F->work = nullptr;
    return api_fail(OPF_ENOMEM, "device allocation of " + std::to_string(bytes) + " bytes failed");
  }
  *out = F->work;
  return OPF_OK;
}

namespace {

// bytes of update-matrix workspace per instance: 25 periods of the
// 10000-bus grid (measured per factorization with the chain eliminated from
// both ends and the chunks cut from both ends in turn: 12 periods 0.858 s,
// 25 0.793 s, 38 0.832 s, 51 0.862 s, 76 0.838 s, before the symmetric cut)
constexpr int64_t kArenaBudget = 16LL << 30;

// Workspace budget: OPF_CHOL_ARENA_BYTES (bytes, > 0) overrides the default.
int64_t arena_budget() {
  const char* e = std::getenv("OPF_CHOL_ARENA_BYTES");
  if (e && *e) {
    const long long v = std::atoll(e);
    if (v > 0) return (int64_t)v;
  }
  return kArenaBudget;
}

// Budget of cyclic reduction's additional memory: OPF_CHOL_CYCLIC_BYTES (bytes,
// 0: the chain from both ends at every size) overrides the default.
int64_t cyclic_budget() {
  const char* e = std::getenv("OPF_CHOL_CYCLIC_BYTES");
  if (e && *e) {
    const long long v = std::atoll(e);
    if (v >= 0) return (int64_t)v;
  }
  return kCycBytes;
}

// Update blocks of cyclic reduction, in doubles: the first level has the most.
int64_t cyclic_blocks(const CholPlan& P) { return (P.T + 1) / 2 * 4LL * P.G * P.G; }

// Flops of cyclic reduction (p^3 / 3 + p^2 u + p u^2 a front, counted as the
// plan counts the chain's), level by level.
double cyclic_flops(const CholPlan& P) {
  const double G = P.G;
  double f = 0.0;
  for (int64_t h = 1; h <= P.T; h *= 2) {
    const int64_t n = P.T / h, c = (n + 1) / 2;
    f += (double)c * G * G * G * (c > 1 ? 19.0 : (n > 1 ? 7.0 : 1.0)) / 3.0;
  }
  return f;
}

template <class T>
int upload(opf_chol* F, const std::vector<T>& h, T** d) {
  const size_t bytes = std::max<size_t>(1, h.size()) * sizeof(T);
  if (hipMalloc((void**)d, bytes) != hipSuccess) return api_fail(OPF_ENOMEM, "chol: device allocation failed");
  F->allocs.push_back(*d);
  if (!h.empty() && hipMemcpy(*d, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice) != hipSuccess)
    return api_fail(OPF_EHIP, "chol: upload failed");
  return OPF_OK;
}

int dalloc(opf_chol* F, int64_t n, double** d) {
  if (hipMalloc((void**)d, (size_t)std::max<int64_t>(1, n) * sizeof(double)) != hipSuccess)
    return api_fail(OPF_ENOMEM, "chol: device allocation of " + std::to_string(n * 8) + " bytes failed");
  F->allocs.push_back(*d);
  return OPF_OK;
}

void release(opf_chol* F) {
  for (void* p : F->allocs) (void)hipFree(p);
  F->allocs.clear();
  F->Us = F->Uc = nullptr;
  if (F->work) (void)hipFree(F->work);
  F->work = nullptr;
}

#define CHK(x)                      \
  do {                              \
    int rc_ = (x);                  \
    if (rc_ != OPF_OK) return rc_;  \
  } while (0)

#define LAUNCH_OK(what)                                                                       \
  do {                                                                                        \
    hipError_t e_ = hipGetLastError();                                                        \
    if (e_ != hipSuccess) return api_fail(OPF_EHIP, std::string(what) + ": " + hipGetErrorString(e_)); \
  } while (0)

// The extend-add's tables (see CDev and k_extend) and the small fronts' lists.
int setup_extend(opf_chol* F, CholInst& C, const std::vector<int64_t>& woff) {
  const CholPlan& P = C.plan;
  auto order = [&](int32_t s) { return P.node_p[s] + P.node_u[s]; };
  std::vector<int32_t> inv, col, items, small;
  std::vector<int64_t> inv_off(P.nnodes, 0), col_off(P.nnodes, 0);
  std::vector<longlong2> con;
  auto invert = [&](int32_t c, int32_t n) {
    inv_off[c] = (int64_t)inv.size();
    inv.resize(inv.size() + n, -1);
    const int32_t* rel = P.rel.data() + P.row_ptr[c];
    for (int32_t b = 0; b < P.node_u[c]; ++b) inv[inv_off[c] + rel[b]] = b;
  };
  // the columns of a front of n rows and the children that have them
  auto columns = [&](int32_t n, const int32_t* k0, const int32_t* k1) {
    const int64_t at = (int64_t)col.size();
    std::vector<int32_t> cnt(n + 1, 0);
    for (const int32_t* c = k0; c < k1; ++c)
      for (int32_t b = 0; b < P.node_u[*c]; ++b) ++cnt[P.rel[P.row_ptr[*c] + b] + 1];
    for (int32_t j = 0; j < n; ++j) cnt[j + 1] += cnt[j];
    const int32_t base = (int32_t)con.size();
    for (int32_t j = 0; j <= n; ++j) col.push_back(base + cnt[j]);
    con.resize(con.size() + cnt[n]);
    for (const int32_t* c = k0; c < k1; ++c)
      for (int32_t b = 0; b < P.node_u[*c]; ++b)
        con[base + cnt[P.rel[P.row_ptr[*c] + b]]++] =
            make_longlong2(P.node_uoff[*c] + (int64_t)b * P.node_u[*c], inv_off[*c]);
    return at;
  };
  C.lvl_item.assign(P.nlevels + 1, 0);
  C.lvl_big.assign(P.nlevels, 0);
  for (int32_t s = 0; s < P.nnodes; ++s) {
    const int32_t *k0 = P.kids.data() + P.kid_ptr[s], *k1 = P.kids.data() + P.kid_ptr[s + 1];
    for (const int32_t* c = k0; c < k1; ++c) invert(*c, order(s));
    if (order(s) > kSmall) col_off[s] = columns(order(s), k0, k1);
  }
  for (int32_t c : P.roots) invert(c, P.G);
  std::vector<longlong4> kid;
  for (int32_t c : P.kids) kid.push_back(make_longlong4(P.node_uoff[c], inv_off[c], P.node_u[c], woff[c]));
  C.dev.col_root = columns(P.G, P.roots.data(), P.roots.data() + P.roots.size());
  for (int32_t h = 0; h < P.nlevels; ++h) {
    for (int64_t q = P.lvl_large_ptr[h]; q < P.lvl_large_ptr[h + 1]; ++q) {
      const int32_t s = P.lvl_large[q], n = order(s);
      for (int32_t c0 = 0; c0 < n; c0 += extend_cols(n)) {
        items.push_back(s);
        items.push_back(c0);
      }
    }
    C.lvl_item[h + 1] = (int64_t)items.size() / 2;
    for (int big = 0; big < 2; ++big) {
      if (big) C.lvl_big[h] = (int64_t)small.size();
      for (int64_t q = P.lvl_small_ptr[h]; q < P.lvl_small_ptr[h + 1]; ++q)
        if ((order(P.lvl_small[q]) > 32) == (big == 1)) small.push_back(P.lvl_small[q]);
    }
  }
  // levels with at most kTreeFronts fronts, all small, in runs of two or more
  C.run_end.resize(P.nlevels);
  for (int32_t h = P.nlevels - 1; h >= 0; --h) {
    const bool fit = P.lvl_large_ptr[h] == P.lvl_large_ptr[h + 1] &&
                     P.lvl_small_ptr[h + 1] - P.lvl_small_ptr[h] <= kTreeFronts;
    C.run_end[h] = !fit ? h : (h + 1 < P.nlevels && C.run_end[h + 1] > h + 1 ? C.run_end[h + 1] : h + 1);
  }
  CHK(upload(F, P.lvl_small_ptr, &C.d_smallptr));
  CHK(upload(F, items, &C.d_items));
  std::vector<FrontRec> srec;
  for (int32_t s : small)
    srec.push_back({P.node_loff[s], 0, P.node_uoff[s], woff[s], P.row_ptr[s], P.node_p[s], P.node_u[s], order(s),
                    P.node_f[s], (int32_t)P.kid_ptr[s], (int32_t)P.kid_ptr[s + 1]});
  CHK(upload(F, srec, &C.d_srec));
  CHK(upload(F, inv, &C.d_inv));
  CHK(upload(F, col, &C.d_col));
  CHK(upload(F, col_off, &C.d_coloff));
  CHK(upload(F, con, &C.d_con));
  CHK(upload(F, kid, &C.d_kid));
  C.dev.inv = C.d_inv;
  C.dev.col = C.d_col;
  C.dev.col_off = C.d_coloff;
  C.dev.con = C.d_con;
  C.dev.kid = C.d_kid;
  return OPF_OK;
}

int setup_device(opf_chol* F, CholInst& C) {
  const CholPlan& P = C.plan;
  std::vector<int64_t> woff(P.nnodes, 0);  // per-front offsets of the forward update vectors
  int64_t w = 0;
  for (int32_t s = 0; s < P.nnodes; ++s) {
    woff[s] = w;
    w += P.node_u[s];
  }
  C.wsize = std::max<int64_t>(w, 1);
  // the large fronts, level by level, those with more pivots first
  for (int32_t h = 0; h < P.nlevels; ++h) {
    std::vector<int32_t> v(P.lvl_large.begin() + P.lvl_large_ptr[h], P.lvl_large.begin() + P.lvl_large_ptr[h + 1]);
    std::stable_sort(v.begin(), v.end(), [&](int32_t x, int32_t y) { return P.node_p[x] > P.node_p[y]; });
    for (int32_t s : v) {
      C.rec.push_back({P.node_loff[s], C.dsize, P.node_uoff[s], woff[s], P.row_ptr[s], P.node_p[s], P.node_u[s],
                       P.node_p[s] + P.node_u[s], P.node_f[s], (int32_t)P.kid_ptr[s], (int32_t)P.kid_ptr[s + 1]});
      C.dsize += diag_size(P.node_p[s]);
    }
  }
  C.dcsize = diag_size(P.G);
  C.wave = P.T < kCycT && P.G >= 1 && P.G <= kWaveG;
  C.wave_solve = P.T < kCycT && P.G >= 1 && P.G <= kWaveSolveG;
  C.cld = (C.cyclic ? 3 : 2) * P.G;
  for (int k = 0; k < 3; ++k) C.crec[k] = {0, 0, 0, 0, 0, P.G, k * P.G, C.cld, 0, 0, 0};
  CHK(upload(F, C.rec, &C.d_rec));
  CHK(upload(F, P.node_p, &C.d_node_p));
  CHK(upload(F, P.node_u, &C.d_node_u));
  CHK(upload(F, P.rel, &C.d_rel));
  CHK(upload(F, P.kids, &C.d_kids));
  CHK(upload(F, P.rows, &C.d_rows));
  CHK(upload(F, P.perm, &C.d_perm));
  CHK(setup_extend(F, C, woff));
  CHK(upload(F, P.roots, &C.d_roots));
  CHK(upload(F, P.kpos0, &C.d_kpos0));
  CHK(upload(F, P.kpos1, &C.d_kpos1));
  CHK(upload(F, P.ramp_pos, &C.d_ramp));
  CHK(upload(F, P.node_loff, &C.d_loff));
  CHK(upload(F, P.node_uoff, &C.d_uoff));
  CHK(upload(F, woff, &C.d_woff));
  CHK(upload(F, P.row_ptr, &C.d_rowptr));
  const int64_t T = P.T, G = P.G;
  // the plan numbers a pg front's entries with leading dimension 2 G
  std::vector<int64_t> slot = P.slot_dst;
  for (int64_t& d : slot)
    if (d < 0) d = -1 - ((-1 - d) / (2 * G) * C.cld + (-1 - d) % (2 * G));
  CHK(upload(F, slot, &C.d_slot));
  C.csize = C.cld * G;
  C.chunk = (int32_t)std::max<int64_t>(1, std::min<int64_t>(T, arena_budget() / (P.usize * 8)));
  CHK(dalloc(F, P.lsize * T, &C.Lf));
  CHK(dalloc(F, C.csize * T, &C.Cf));
  CHK(dalloc(F, C.dsize * T, &C.Df));
  CHK(dalloc(F, C.dcsize * T, &C.Dc));
  CHK(dalloc(F, P.usize * C.chunk, &C.Ar));
  CHK(dalloc(F, C.wsize * T, &C.W));
  CHK(dalloc(F, (C.cyclic ? 2 : 1) * G * T, &C.Wc));
  CHK(dalloc(F, (int64_t)P.n_p * T, &C.Y));
  CHK(dalloc(F, (int64_t)P.n_p * T, &C.Z));
  CHK(dalloc(F, C.cyclic ? (T + 1) / 2 * 2 * G : 2 * G, &C.Gp));
  CHK(dalloc(F, C.wsize * T, &C.V));
  CDev& D = C.dev;
  D.node_p = C.d_node_p;
  D.node_u = C.d_node_u;
  D.rel = C.d_rel;
  D.kids = C.d_kids;
  D.rows = C.d_rows;
  D.node_loff = C.d_loff;
  D.node_uoff = C.d_uoff;
  D.node_woff = C.d_woff;
  D.row_ptr = C.d_rowptr;
  D.lsize = P.lsize;
  D.usize = P.usize;
  D.wsize = C.wsize;
  D.n_p = P.n_p;
  D.n_int = P.n_int;
  D.G = P.G;
  return OPF_OK;
}

// The instances' forms, device tables and storage; cyc: what cyclic reduction
// may add to the chain's memory, all instances together.
int setup_instances(opf_chol* F, int64_t cyc) {
  int64_t fronts = 0, blocks = 0, uc = 0, maxG = 0;
  bool any = false;
  for (auto& C : F->inst) {
    const CholPlan& P = C.plan;
    const int64_t f = fronts + (int64_t)P.G * P.G * P.T, b = std::max(blocks, cyclic_blocks(P));
    C.cyclic = P.T >= kCycT && P.G <= kCycG && 8 * (f + b) <= cyc;
    if (C.cyclic) {
      fronts = f;
      blocks = b;
      any = true;
    }
    maxG = std::max<int64_t>(maxG, P.G);
  }
  F->arena_entries = F->factor_entries = 0;
  F->flops = F->flops_int;
  for (auto& C : F->inst) {
    CHK(setup_device(F, C));
    const int64_t ar = C.plan.usize * C.chunk;
    F->arena_entries += ar;
    F->factor_entries += (C.plan.lsize + C.csize + C.dsize + C.dcsize) * C.plan.T;
    F->flops += C.cyclic ? cyclic_flops(C.plan) : C.plan.flops_chain;
    // the interior fronts' workspace is free when the reduction starts, and
    // the instances are factored one after another
    if (C.cyclic && cyclic_blocks(C.plan) <= ar) C.Uc = C.Ar;
    else if (C.cyclic) uc = std::max(uc, cyclic_blocks(C.plan));
  }
  if (uc > 0) CHK(dalloc(F, uc, &F->Uc));
  F->arena_entries += uc;
  for (auto& C : F->inst)
    if (C.cyclic && !C.Uc) C.Uc = F->Uc;
  CHK(dalloc(F, 2 * maxG * maxG, &F->Us));
  const char* inj = std::getenv("OPF_TEST_FAIL_ALLOC");
  if (any && inj && std::strcmp(inj, "cyclic") == 0)
    return api_fail(OPF_ENOMEM, "allocation failure injected by OPF_TEST_FAIL_ALLOC");
  return OPF_OK;
}

// A batch of fronts as the host launches it: the records on both sides and
// the number of periods.
struct Batch {
  Fronts F;
  const FrontRec* rec;
  int n, nt;
  // the fronts with pivots from position k on
  int active(int k) const {
    int a = 0;
    while (a < n && rec[a].p > k) ++a;
    return a;
  }
};

// Small tiles where 64 x 64 ones would leave CUs without a block: at 256
// panel columns, 144 columns and 544 rows of two fronts 9.6 us against 20.
int launch_update(const Batch& B, int k0, int w, bool inner, hipStream_t st) {
  const int n = B.active(inner ? k0 + w : k0);
  int64_t most[2] = {0, 0}, sum = 0;  // tiles of the largest front, by tile size; 64 x 64 tiles of all
  for (int i = 0; i < n; ++i) {
    const FrontRec& f = B.rec[i];
    const int rows = f.p + f.u, r0 = k0 + std::min(w, f.p - k0), cend = inner ? std::min(r0 + w, f.p) : rows;
    if (cend <= r0) continue;
    for (int s = 0; s < 2; ++s) {
      const int64_t tm = s ? 32 : kTile, R = (rows - r0 + tm - 1) / tm, Cn = (cend - r0 + tm - 1) / tm;
      const int64_t t = Cn * R - Cn * (Cn - 1) / 2;
      most[s] = std::max(most[s], t);
      if (!s) sum += t;
    }
  }
  if (sum == 0) return OPF_OK;
  if (most[1] > 0x7fffffff) return api_fail(OPF_EINVAL, "chol: front too large");
  if (sum * B.nt < kFewTiles)
    hipLaunchKernelGGL((k_update<32, 64>), dim3((unsigned)most[1], B.nt, n), dim3(256), 0, st, B.F, k0, w, (int)inner);
  else
    hipLaunchKernelGGL((k_update<kTile, 8>), dim3((unsigned)most[0], B.nt, n), dim3(256), 0, st, B.F, k0, w, (int)inner);
  LAUNCH_OK("chol update");
  return OPF_OK;
}

// Columns [k, k+w) of a batch of fronts, w a power of two >= kWide: up to
// kWide columns by panels that each take their update from the block's columns
// before them; wider blocks recursively: the first half, the first half's
// update of the second half's columns, the second half.  The trailing columns
// are left to the caller.
int factor_cols(const Batch& B, int k, int w, double tol, double repl, int32_t* npert, hipStream_t st) {
  if (w == kWide) {
    for (int k0 = k; k0 < k + kWide; k0 += kNB) {
      const int n = B.active(k0);
      if (n == 0) break;
      int g = 1;
      for (int i = 0; i < n; ++i) {
        const FrontRec& f = B.rec[i];
        g = std::max(g, (f.p + f.u - k0 - std::min(kNB, f.p - k0) + kTR - 1) / kTR);
      }
      hipLaunchKernelGGL(k_panel, dim3(g, B.nt, n), dim3(kPT), 0, st, B.F, k, k0, tol, repl, npert);
      LAUNCH_OK("chol panel");
    }
    return OPF_OK;
  }
  const int h = w / 2;
  CHK(factor_cols(B, k, h, tol, repl, npert, st));
  if (B.active(k + h) > 0) {
    CHK(launch_update(B, k, h, true, st));
    CHK(factor_cols(B, k + h, h, tol, repl, npert, st));
  }
  return OPF_OK;
}

// A batch of fronts: kStep-column steps, each factored recursively, then one
// trailing update with the kStep-wide panel.
int factor_fronts(const Batch& B, double tol, double repl, int32_t* npert, hipStream_t st) {
  for (int k0 = 0; B.active(k0) > 0; k0 += kStep) {
    CHK(factor_cols(B, k0, kStep, tol, repl, npert, st));
    CHK(launch_update(B, k0, kStep, false, st));
  }
  return OPF_OK;
}

// The pg chain by cyclic reduction, after the interior fronts.
int factor_cyclic(CholInst& C, double tol, double repl, int32_t* npert, hipStream_t st) {
  const int T = C.plan.T, G = C.plan.G;
  for (int h = 1; h <= T; h *= 2) {
    const int n = T / h, c = (n + 1) / 2, u = c > 1 ? 2 : (n > 1 ? 1 : 0), ub = u * G;
    const int64_t s2 = 2 * (int64_t)h;  // from one eliminated front to the next
    Batch B;
    B.F = {nullptr, C.crec[u], C.Cf + (h - 1) * C.csize, C.Dc + (h - 1) * C.dcsize, C.Uc, s2 * C.csize, s2 * C.dcsize,
           (int64_t)ub * ub, C.dev.stop, 1};
    B.rec = C.crec + u;
    B.n = 1;
    B.nt = c;
    CHK(factor_fronts(B, tol, repl, npert, st));
    const int m = n - c;  // fronts that stay: 2 h - 1, 4 h - 1, ...
    if (m == 0) break;
    double* C0 = C.Cf + (s2 - 1) * C.csize;
    hipLaunchKernelGGL(k_cyc_add, dim3(std::min(grid_for((int64_t)G * G, 256), 2048), m), dim3(256), 0, st, C.Uc, ub, c,
                       G, C0, s2 * C.csize, (int64_t)C.cld, C.dev.stop);
    if (m > 1)
      hipLaunchKernelGGL(k_cyc_link, dim3((G + 31) / 32, (G + 31) / 32, m - 1), dim3(256), 0, st, C.Uc, ub, G, C0,
                         s2 * C.csize, (int64_t)C.cld, C.dev.stop);
    LAUNCH_OK("chol cyclic update");
  }
  return OPF_OK;
}

int factor_inst(opf_chol* F, CholInst& C, bool first, const double* kv, double tol, double repl, int32_t* npert,
                hipStream_t st) {
  const CholPlan& P = C.plan;
  const InstHost& I = *C.I;
  const int T = P.T, G = P.G;
  hipLaunchKernelGGL(k_clear, dim3(grid_for(std::max(P.lsize, C.csize) * T, 256)), dim3(256), 0, st, C.Lf, P.lsize * T,
                     C.Cf, C.csize * T, first ? npert : (int32_t*)nullptr);
  LAUNCH_OK("chol clear");
  // every ramp pair up front: they land in the pg front of the period
  // before, which the chain stream may be factoring while a later chunk's
  // interior runs
  if (T > 1) {
    hipLaunchKernelGGL(k_scatter_ramp, dim3(grid_for(G, 256), T - 1), dim3(256), 0, st, kv, I.k_off, I.nnzk_p, G, 1,
                       C.cyclic ? -1 : (T - 1) / 2, C.d_ramp, C.Cf, C.csize, C.cld);
    LAUNCH_OK("chol ramp scatter");
  }
  const int nslots = (int)P.slot_dst.size();
  // The pg chain from both ends: left fronts kl = 0 .. m-1, right fronts
  // kr = T-1 .. m+1, a left and a right front per step while both sides
  // have one ready, then front m.  The interior chunks are cut from both
  // ends of the horizon in turn (C.chunk periods each, the rest in the
  // middle last), so both sides of the chain become ready together and the
  // steps left after the last chunk are about half of that chunk.
  const int m = (T - 1) / 2;
  std::vector<std::pair<int, int>> chunks;  // (first period, periods)
  {
    int a = 0, b = T;
    bool left = true;
    while (b - a > C.chunk) {
      if (left) {
        chunks.push_back({a, C.chunk});
        a += C.chunk;
      } else {
        chunks.push_back({b - C.chunk, C.chunk});
        b -= C.chunk;
      }
      left = !left;
    }
    if (b > a) chunks.push_back({a, b - a});
  }
  const int nchunk = (int)chunks.size();
  if (!C.cyclic && !C.wave && nchunk + 1 > (int)F->evs.size()) return api_fail(OPF_EINVAL, "chol: more period chunks than events");
  std::vector<char> ready(T, 0);
  int kl = 0, kr = T - 1;
  double* UsL = F->Us;
  double* UsR = F->Us + (int64_t)G * G;
  const int64_t gg = (int64_t)G * G;
  // front t's incoming chain update (from t-1 on the left, t+1 on the
  // right) into its pivot block
  auto add_in = [&](int t, const double* Ub, int n = 1, int t2 = 0) -> int {
    hipLaunchKernelGGL(k_add_chain, dim3(grid_for(gg, 256), n), dim3(256), 0, F->cs, Ub, gg, G,
                       C.Cf + (int64_t)t * C.csize, n > 1 ? (t2 - t) * C.csize : 0);
    LAUNCH_OK("chol chain add");
    return OPF_OK;
  };
  // nt = 2: fronts kl and kr in one batch (period stride kr - kl)
  auto chain_front = [&](int t, int nt, int t2, int u, double* Ub) -> int {
    Batch B;
    B.F = {nullptr, C.crec[u ? 1 : 0], C.Cf + (int64_t)t * C.csize, C.Dc + (int64_t)t * C.dcsize, Ub,
           (int64_t)(t2 - t) * C.csize, (int64_t)(t2 - t) * C.dcsize, gg, C.dev.stop, 1};
    B.rec = C.crec + (u ? 1 : 0);
    B.n = 1;
    B.nt = nt;
    return factor_fronts(B, tol, repl, npert, F->cs);
  };
  auto chain_steps = [&](bool all) -> int {
    for (;;) {
      const bool l = kl < m && ready[kl], r = kr > m && ready[kr];
      if (l && r) {
        if (kl >= 1 && kr <= T - 2) {
          CHK(add_in(kl, UsL, 2, kr));
        } else {
          if (kl >= 1) CHK(add_in(kl, UsL));
          if (kr <= T - 2) CHK(add_in(kr, UsR));
        }
        CHK(chain_front(kl, 2, kr, G, UsL));
        ++kl;
        --kr;
      } else if (l && (kr <= m || all)) {
        if (kl >= 1) CHK(add_in(kl, UsL));
        CHK(chain_front(kl, 1, kl, G, UsL));
        ++kl;
      } else if (r && (kl >= m || all)) {
        if (kr <= T - 2) CHK(add_in(kr, UsR));
        CHK(chain_front(kr, 1, kr, G, UsR));
        --kr;
      } else {
        break;
      }
    }
    return OPF_OK;
  };
  for (int chunk_id = 0; chunk_id < nchunk; ++chunk_id) {
    const int t0 = chunks[chunk_id].first;
    const int nt = chunks[chunk_id].second;
    hipLaunchKernelGGL(k_scatter, dim3(grid_for(nslots, 256), nt), dim3(256), 0, st, kv, I.k_off, I.nnzk_p, G, t0,
                       nslots, C.d_slot, C.d_kpos0, C.d_kpos1, C.Lf, P.lsize, C.Cf, C.csize);
    LAUNCH_OK("chol scatter");
    for (int h = 0; h < P.nlevels; ++h) {
      const int64_t i0 = C.lvl_item[h], i1 = C.lvl_item[h + 1];
      if (i1 > i0) {
        hipLaunchKernelGGL(k_extend, dim3((unsigned)(i1 - i0), nt), dim3(256), 0, st, C.dev, C.d_items, i0, t0, C.Lf,
                           C.Ar);
        LAUNCH_OK("chol extend-add");
      }
      const int64_t s0 = P.lvl_small_ptr[h], s1 = P.lvl_small_ptr[h + 1], sb = C.lvl_big[h];
      if (sb > s0)
        hipLaunchKernelGGL(k_factor_small<false>, dim3((unsigned)(sb - s0), nt), dim3(64), 0, st, C.dev, C.d_srec + s0,
                           t0, C.Lf, C.Ar, tol, repl, npert);
      if (s1 > sb)
        hipLaunchKernelGGL(k_factor_small<true>, dim3((unsigned)(s1 - sb), nt), dim3(64), 0, st, C.dev, C.d_srec + sb,
                           t0, C.Lf, C.Ar, tol, repl, npert);
      LAUNCH_OK("chol small fronts");
      const int64_t q0 = P.lvl_large_ptr[h], q1 = P.lvl_large_ptr[h + 1];
      if (q1 > q0) {
        Batch B;
        B.F = {C.d_rec + q0, FrontRec(), C.Lf + (int64_t)t0 * P.lsize, C.Df + (int64_t)t0 * C.dsize, C.Ar, P.lsize, C.dsize, P.usize,
               C.dev.stop, 0};
        B.rec = C.rec.data() + q0;
        B.n = (int)(q1 - q0);
        B.nt = nt;
        CHK(factor_fronts(B, tol, repl, npert, st));
      }
    }
    hipLaunchKernelGGL(k_extend_root, dim3((G + 3) / 4, nt), dim3(256), 0, st, C.dev, t0, C.Cf, C.csize,
                       (int64_t)C.cld, C.Ar);
    LAUNCH_OK("chol pg front assembly");
    if (C.cyclic || C.wave) continue;
    // the chain steps this chunk makes ready, on the chain stream
    if (hipEventRecord(F->evs[chunk_id], st) != hipSuccess || hipStreamWaitEvent(F->cs, F->evs[chunk_id], 0) != hipSuccess)
      return api_fail(OPF_EHIP, "chol: chain stream ordering");
    for (int t = t0; t < t0 + nt; ++t) ready[t] = 1;
    CHK(chain_steps(chunk_id + 1 == nchunk));
  }
  if (C.cyclic) return factor_cyclic(C, tol, repl, npert, st);
  if (C.wave) {
    auto go = [&](auto k) {
      hipLaunchKernelGGL(k, dim3(1), dim3(128), 0, st, (int32_t)G, (int32_t)T, C.Cf, C.csize, C.Dc, C.dcsize, C.dev.stop,
                         tol, repl, npert);
    };
    if (G <= 8) go(k_chain_wave<16>);
    else go(k_chain_wave<32>);
    LAUNCH_OK("chol chain by wavefronts");
    return OPF_OK;
  }
  // front m: both sides' last updates, no update rows
  if (m >= 1) CHK(add_in(m, UsL));
  if (m + 1 <= T - 1) CHK(add_in(m, UsR));
  CHK(chain_front(m, 1, m, 0, UsL));
  // the model's stream waits for the chain
  hipEvent_t done = F->evs.back();
  if (hipEventRecord(done, F->cs) != hipSuccess || hipStreamWaitEvent(st, done, 0) != hipSuccess)
    return api_fail(OPF_EHIP, "chol: chain stream join");
  return OPF_OK;
}

// Forward / backward triangle of a batch of fronts (nb batch entries, in
// falling order of p), see k_fwd_panel / k_bwd_panel: y is the
// right-hand side in, z the forward solution; the backward pass reads z and
// leaves x in y.
int fwd_tri(const Tri& A, const FrontRec* rec, int n, int nb, int chunk, double* next, int64_t sn, int pass,
            hipStream_t st) {
  for (int k0 = 0; n > 0; k0 += kSolve) {
    int below = 1;
    for (int i = 0; i < n; ++i) below = std::max(below, rec[i].p + rec[i].u - std::min(k0 + kSolve, rec[i].p));
    // 64 rows per block while those blocks fit the chip at once (one CU loads
    // no more than about 64 bytes a cycle), else 192, as every block repeats
    // the launch's triangles
    if ((int64_t)(below + 63) / 64 * nb * n <= 512)
      hipLaunchKernelGGL(k_fwd_panel<64>, dim3((below + 63) / 64, nb, n), dim3(kInner + 64 + 128), 0, st, A, k0, chunk,
                         next, sn, pass);
    else
      hipLaunchKernelGGL(k_fwd_panel<192>, dim3((below + 191) / 192, nb, n), dim3(kInner + 192 + 128), 0, st, A, k0,
                         chunk, next, sn, pass);
    while (n > 0 && rec[n - 1].p <= k0 + kSolve) --n;
  }
  LAUNCH_OK("chol forward panel");
  return OPF_OK;
}

int bwd_tri(const Tri& A, const FrontRec* rec, int n, int nb, hipStream_t st) {
  constexpr int per = kSolve / kNB;
  for (int q = 0; n > 0; ++q) {
    const int k0 = std::max(0, (rec[0].p + kNB - 1) / kNB - (q + 1) * per) * kNB;  // columns before the launch's
    // as few columns per block as leave it no more of them than the chip takes
    // at once: each block repeats the launch's triangles
    int cols = kBwdCols;
    while (cols < 1024 && (int64_t)(k0 + cols - 1) / cols * nb * n > 512) cols *= 2;
    hipLaunchKernelGGL(k_bwd_panel, dim3(std::max(1, (k0 + cols - 1) / cols), nb, n), dim3(kBwdT), 0, st, A, q, cols);
    while (n > 0 && (rec[n - 1].p + kNB - 1) / kNB <= (q + 1) * per) --n;
  }
  LAUNCH_OK("chol backward panel");
  return OPF_OK;
}

// The pg chain's two solves by cyclic reduction: the levels forward, then back.
int solve_cyclic(CholInst& C, hipStream_t st) {
  const int T = C.plan.T, G = C.plan.G;
  const int64_t np = C.plan.n_p, o = C.plan.n_int;
  auto level = [&](int h, int u) {
    const int64_t s2 = 2 * (int64_t)h, t = h - 1;
    return Tri{nullptr, C.crec[u], C.Cf + t * C.csize, C.Dc + t * C.dcsize, C.Y + t * np + o, C.Z + t * np + o,
               C.Wc + t * 2 * G, C.Gp, s2 * C.csize, s2 * C.dcsize, s2 * np, s2 * 2 * G, 2 * (int64_t)G};
  };
  constexpr int kAll = 1 << 30;  // one sum over all columns
  int top = 1;
  for (int h = 1; h <= T; h *= 2) {
    const int n = T / h, c = (n + 1) / 2, u = c > 1 ? 2 : (n > 1 ? 1 : 0);
    top = h;
    const Tri A = level(h, u);
    CHK(fwd_tri(A, C.crec + u, 1, c, kAll, nullptr, 0, 0, st));
    if (n == c) break;
    hipLaunchKernelGGL(k_cyc_pull, dim3((G + 255) / 256, n - c), dim3(256), 0, st, (const double*)A.w, A.sw, c, G,
                       C.Y + (2 * (int64_t)h - 1) * np + o, A.sy);
    LAUNCH_OK("chol forward cyclic");
  }
  for (int h = top; h >= 1; h /= 2) {
    const int n = T / h, c = (n + 1) / 2, u = c > 1 ? 2 : (n > 1 ? 1 : 0);
    const Tri A = level(h, u);
    if (u) {
      hipLaunchKernelGGL(k_cyc_gemv, dim3((G + 3) / 4, c), dim3(256), 0, st, A, n, (const double*)A.y, h * np);
      LAUNCH_OK("chol backward cyclic");
    }
    CHK(bwd_tri(A, C.crec + u, 1, c, st));
  }
  return OPF_OK;
}

int solve_inst(CholInst& C, const double* b, double* x, hipStream_t st) {
  const CholPlan& P = C.plan;
  const InstHost& I = *C.I;
  const int T = P.T, G = P.G;
  const int64_t np = P.n_p;
  hipLaunchKernelGGL(k_gather, dim3(grid_for(np * T, 256)), dim3(256), 0, st, b + I.x_off, P.n_p, T, C.d_perm, C.Y);
  LAUNCH_OK("chol gather");
  auto tree = [&](int64_t q0) {
    return Tri{C.d_rec + q0, FrontRec(), C.Lf, C.Df, C.Y, C.Z, C.W, C.V, P.lsize, C.dsize, np, C.wsize, C.wsize};
  };
  // forward through the interior trees, all periods at once (small fronts
  // leave their forward solution in Y, large ones in Z)
  for (int h = 0; h < P.nlevels; ++h) {
    if (C.run_end[h] > h + 1) {
      hipLaunchKernelGGL(k_fwd_tree, dim3(T), dim3(kTreeT), 0, st, C.dev, C.d_srec, C.d_smallptr, h, C.run_end[h], C.Lf,
                         C.Y, C.W);
      LAUNCH_OK("chol forward small levels");
      h = C.run_end[h] - 1;
      continue;
    }
    const int64_t s0 = P.lvl_small_ptr[h], s1 = P.lvl_small_ptr[h + 1];
    if (s1 > s0) {
      hipLaunchKernelGGL(k_fwd_small, dim3((unsigned)(s1 - s0), T), dim3(64), 0, st, C.dev, C.d_srec + s0, C.Lf,
                         C.Y, C.W);
      LAUNCH_OK("chol forward small");
    }
    const int64_t q0 = P.lvl_large_ptr[h];
    const int nl = (int)(P.lvl_large_ptr[h + 1] - q0);
    if (nl > 0) {
      hipLaunchKernelGGL(k_fwd_pull, dim3(T, 1, nl), dim3(256), 0, st, C.dev, C.d_rec + q0, C.Y, C.W);
      CHK(fwd_tri(tree(q0), C.rec.data() + q0, nl, T, 0, nullptr, 0, 0, st));
    }
  }
  hipLaunchKernelGGL(k_fwd_root_pull, dim3(T), dim3(256), 0, st, C.dev, C.d_roots, (int32_t)P.roots.size(), C.Y,
                     (const double*)C.W);
  LAUNCH_OK("chol forward roots");
  // forward along the pg chain, from both ends as it was factored: left
  // fronts ascending, right fronts descending, a left and a right front per
  // step while both sides have one, then front m
  const int m = (T - 1) / 2;
  auto off = [&](int t) { return (int64_t)t * np + P.n_int; };
  // fronts t and, when nb = 2, t2 as one batch
  auto chain = [&](int t, int nb, int t2) {
    const int64_t d = nb > 1 ? t2 - t : 0;
    return Tri{nullptr, C.crec[t == m ? 0 : 1], C.Cf + (int64_t)t * C.csize, C.Dc + (int64_t)t * C.dcsize, C.Y + off(t),
               C.Z + off(t), C.Wc + (int64_t)t * G, C.Gp, d * C.csize, d * C.dcsize, d * np, d * G, G};
  };
  if (C.cyclic) {
    CHK(solve_cyclic(C, st));
  } else if (C.wave_solve) {
    auto go = [&](auto k) {
      hipLaunchKernelGGL(k, dim3(1), dim3(128), 0, st, (int32_t)G, (int32_t)T, (const double*)C.Cf, C.csize,
                         (const double*)C.Dc, C.dcsize, C.Y + P.n_int, C.Z + P.n_int, np);
    };
    if (G <= 16) go(k_chain_wave_solve<16>);
    else if (G <= 32) go(k_chain_wave_solve<32>);
    else if (G <= 48) go(k_chain_wave_solve<48>);
    else go(k_chain_wave_solve<64>);
    LAUNCH_OK("chol chain solve by wavefronts");
  } else {
    int kl = 0, kr = T - 1;
    while (kl < m || kr > m) {
      const bool l = kl < m, r = kr > m;
      const int t = l ? kl : kr, nb = l && r ? 2 : 1;
      // each side's last panel passes its update on, except to front m, which
      // collects its two neighbours' (Wc), left then right
      const int nl = kl + 1, nr = kr - 1;
      int pass = 0;
      if (l && nl != m) pass |= 1;
      if (r && nr != m) pass |= nb > 1 ? 2 : 1;
      CHK(fwd_tri(chain(t, nb, kr), C.crec + 1, 1, nb, kChainCols, C.Y + off(l ? nl : nr),
                  nb > 1 ? (int64_t)(nr - nl) * np : 0, pass, st));
      if (l) ++kl;
      if (r) --kr;
    }
    if (T > 1) {
      hipLaunchKernelGGL(k_sub, dim3((G + 255) / 256), dim3(256), 0, st, C.Y + off(m),
                         (const double*)(m >= 1 ? C.Wc + (int64_t)(m - 1) * G : nullptr),
                         (const double*)(m + 1 < T ? C.Wc + (int64_t)(m + 1) * G : nullptr), G);
      LAUNCH_OK("chol forward chain");
    }
    CHK(fwd_tri(chain(m, 1, m), C.crec, 1, 1, kChainCols, nullptr, 0, 0, st));
  }
  // backward along the pg chain: front m, then outwards (each front reads
  // its chain neighbour's solution, held in Y)
  if (!C.cyclic && !C.wave_solve) {
    CHK(bwd_tri(chain(m, 1, m), C.crec, 1, 1, st));
    int kl = m - 1, kr = m + 1;
    while (kl >= 0 || kr <= T - 1) {
      const bool l = kl >= 0, r = kr <= T - 1;
      const int t = l ? kl : kr, nb = l && r ? 2 : 1;
      const Tri A = chain(t, nb, kr);
      hipLaunchKernelGGL(k_bwd_gemv, dim3((G + 3) / 4, nb, 1), dim3(256), 0, st, A, (const int32_t*)nullptr,
                         (const double*)(C.Y + off(l ? kl + 1 : kr - 1)), nb > 1 ? (int64_t)(kr - kl - 2) * np : 0);
      LAUNCH_OK("chol backward chain");
      CHK(bwd_tri(A, C.crec + 1, 1, nb, st));
      if (l) --kl;
      if (r) ++kr;
    }
  }
  // backward through the interior trees, top down
  for (int h = P.nlevels - 1; h >= 0; --h) {
    // a run of small levels, from its first one on
    int h0 = h;
    while (h0 > 0 && C.run_end[h] == h + 1 && C.run_end[h0 - 1] == h + 1) --h0;
    if (h0 < h) {
      hipLaunchKernelGGL(k_bwd_tree, dim3(T), dim3(kTreeT), 0, st, C.dev, C.d_srec, C.d_smallptr, h0, h + 1, C.Lf, C.Y);
      LAUNCH_OK("chol backward small levels");
      h = h0;
      continue;
    }
    const int64_t q0 = P.lvl_large_ptr[h];
    const int nl = (int)(P.lvl_large_ptr[h + 1] - q0);
    if (nl > 0) {
      const Tri A = tree(q0);
      hipLaunchKernelGGL(k_bwd_gemv, dim3((C.rec[q0].p + 3) / 4, T, nl), dim3(256), 0, st, A,
                         (const int32_t*)C.d_rows, (const double*)C.Y, np);
      LAUNCH_OK("chol backward large");
      CHK(bwd_tri(A, C.rec.data() + q0, nl, T, st));
    }
    const int64_t s0 = P.lvl_small_ptr[h], s1 = P.lvl_small_ptr[h + 1];
    if (s1 > s0) {
      hipLaunchKernelGGL(k_bwd_small, dim3((unsigned)(s1 - s0), T), dim3(64), 0, st, C.dev, C.d_srec + s0, C.Lf,
                         C.Y);
      LAUNCH_OK("chol backward small");
    }
  }
  hipLaunchKernelGGL(k_scatter_out, dim3(grid_for(np * T, 256)), dim3(256), 0, st, (const double*)C.Y, P.n_p, T,
                     C.d_perm, x + I.x_off);
  LAUNCH_OK("chol scatter");
  return OPF_OK;
}

}  // namespace

// ============================================================== C ABI
extern "C" {

int opf_chol_analyze(opf_model* model, opf_chol** out) {
  if (!out) return api_fail(OPF_EINVAL, "out is NULL");
  *out = nullptr;
  if (!model) return api_fail(OPF_EINVAL, "model is NULL");
  opf_chol* F = nullptr;
  try {
    F = new opf_chol();
    F->model = model;
    F->device = model_device(model);
    const auto& insts = model_insts(model);
    F->inst.resize(insts.size());
    CholOptions opt;
    for (size_t k = 0; k < insts.size(); ++k) {
      CholInst& C = F->inst[k];
      C.I = &insts[k];
      std::string err;
      const int rc = chol_plan_build(insts[k], opt, C.plan, err);
      if (rc != OPF_OK) {
        delete F;
        return api_fail(rc, "instance " + std::to_string(k) + ": " + err);
      }
      const CholPlan& P = C.plan;
      F->flops += P.flops_period * P.T + P.flops_chain;
      F->flops_int += P.flops_period * P.T;
      F->factor_entries += P.lsize * P.T + 2LL * P.G * P.G * P.T;
    }
    if (F->device >= 0) {
      if (hipSetDevice(F->device) != hipSuccess) {
        delete F;
        return api_fail(OPF_EHIP, "chol: hipSetDevice failed");
      }
      int rc = setup_instances(F, cyclic_budget());
      // what the chain from both ends leaves room for is not refused
      if (rc == OPF_ENOMEM && std::any_of(F->inst.begin(), F->inst.end(), [](const CholInst& C) { return C.cyclic; })) {
        release(F);
        (void)hipGetLastError();  // the failed allocation's
        for (auto& C : F->inst) {
          CholInst fresh;
          fresh.plan = std::move(C.plan);
          fresh.I = C.I;
          C = std::move(fresh);
        }
        rc = setup_instances(F, 0);
      }
      if (rc != OPF_OK) {
        release(F);
        delete F;
        return rc;
      }
      // default priority, no implicit ordering with the null stream
      int nev = 1;
      for (auto& C : F->inst) nev = std::max(nev, (C.plan.T + C.chunk - 1) / C.chunk + 1);
      bool ok = hipStreamCreateWithFlags(&F->cs, hipStreamNonBlocking) == hipSuccess &&
                hipStreamCreateWithFlags(&F->gs, hipStreamNonBlocking) == hipSuccess;
      for (int k = 0; ok && k < nev; ++k) {
        hipEvent_t e = nullptr;
        ok = hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess;
        if (ok) F->evs.push_back(e);
      }
      if (!ok) {
        opf_chol_destroy(F);
        return api_fail(OPF_EHIP, "chol: stream or event creation failed");
      }
    } else {
      for (auto& C : F->inst) {
        C.chunk = (int32_t)std::max<int64_t>(1, std::min<int64_t>(C.plan.T, arena_budget() / (C.plan.usize * 8)));
        F->arena_entries += C.plan.usize * C.chunk;
      }
    }
  } catch (const std::bad_alloc&) {
    if (F) {
      release(F);
      delete F;
    }
    return api_fail(OPF_ENOMEM, "chol: host allocation failed");
  }
  *out = F;
  return OPF_OK;
}

void opf_chol_destroy(opf_chol* chol) {
  if (!chol) return;
  if (chol->device >= 0) (void)hipSetDevice(chol->device);
  if (chol->cs) (void)hipStreamSynchronize(chol->cs);
  if (chol->device >= 0) (void)hipDeviceSynchronize();
  if (chol->gexec) (void)hipGraphExecDestroy(chol->gexec);
  for (hipEvent_t e : chol->evs) (void)hipEventDestroy(e);
  if (chol->cs) (void)hipStreamDestroy(chol->cs);
  if (chol->gs) (void)hipStreamDestroy(chol->gs);
  release(chol);
  delete chol;
}

int opf_chol_get_info(const opf_chol* F, opf_chol_info* info) {
  if (!F || !info) return api_fail(OPF_EINVAL, "chol or info is NULL");
  std::memset(info, 0, sizeof(*info));
  info->factor_entries = F->factor_entries;
  info->arena_entries = F->arena_entries;
  info->flops = F->flops;
  info->flops_interior = F->flops_int;
  info->chunk = F->inst.empty() ? 0 : 0x7fffffff;
  for (const auto& C : F->inst) {
    info->nodes += C.plan.nnodes;
    info->levels = std::max(info->levels, C.plan.nlevels);
    info->chunk = std::min(info->chunk, C.chunk);
    info->large_nodes += (int32_t)C.plan.lvl_large.size();
  }
  return OPF_OK;
}

int opf_chol_tree_size(const opf_chol* F, int32_t inst, int32_t* nodes, int64_t* rows) {
  if (!F || !nodes || !rows) return api_fail(OPF_EINVAL, "NULL argument");
  if (inst < 0 || inst >= (int32_t)F->inst.size()) return api_fail(OPF_EINVAL, "instance out of range");
  *nodes = F->inst[inst].plan.nnodes;
  *rows = (int64_t)F->inst[inst].plan.rows.size();
  return OPF_OK;
}

int opf_chol_tree(const opf_chol* F, int32_t inst, int32_t* perm, int32_t* first, int32_t* npiv, int32_t* parent,
                  int64_t* rowptr, int32_t* rows) {
  if (!F || !perm || !first || !npiv || !parent || !rowptr || !rows) return api_fail(OPF_EINVAL, "NULL argument");
  if (inst < 0 || inst >= (int32_t)F->inst.size()) return api_fail(OPF_EINVAL, "instance out of range");
  const CholPlan& P = F->inst[inst].plan;
  std::copy(P.perm.begin(), P.perm.end(), perm);
  std::copy(P.node_f.begin(), P.node_f.end(), first);
  std::copy(P.node_p.begin(), P.node_p.end(), npiv);
  std::copy(P.node_parent.begin(), P.node_parent.end(), parent);
  std::copy(P.row_ptr.begin(), P.row_ptr.end(), rowptr);
  std::copy(P.rows.begin(), P.rows.end(), rows);
  return OPF_OK;
}

int opf_chol_factor(opf_chol* F, const double* kvals, double pivot_tol, double pivot_repl, int32_t* npert) {
  if (!F || !kvals || !npert) return api_fail(OPF_EINVAL, "chol, kvals or npert is NULL");
  if (F->device < 0) return api_fail(OPF_ENODEV, "model is host-only");
  if (!(pivot_repl > 0.0) || !std::isfinite(pivot_repl)) return api_fail(OPF_EINVAL, "pivot_repl must be > 0");
  if (std::isnan(pivot_tol)) return api_fail(OPF_EINVAL, "pivot_tol is NaN");
  if (hipSetDevice(F->device) != hipSuccess) return api_fail(OPF_EHIP, "hipSetDevice failed");
  hipStream_t st = model_stream(F->model);
  for (auto& C : F->inst) {
    C.dev.stop = F->stop_on_pivot ? npert : nullptr;
    CHK(factor_inst(F, C, &C == F->inst.data(), kvals, pivot_tol, pivot_repl, npert, st));
  }
  return OPF_OK;
}

int opf_chol_solve(opf_chol* F, const double* b, double* x) {
  if (!F || !b || !x) return api_fail(OPF_EINVAL, "chol, b or x is NULL");
  if (F->device < 0) return api_fail(OPF_ENODEV, "model is host-only");
  if (hipSetDevice(F->device) != hipSuccess) return api_fail(OPF_EHIP, "hipSetDevice failed");
  hipStream_t st = model_stream(F->model);
  if (!F->use_graph) {
    for (auto& C : F->inst) CHK(solve_inst(C, b, x, st));
    return OPF_OK;
  }
  if (!F->gexec || F->gb != b || F->gx != x) {
    if (F->gexec) {
      (void)hipStreamSynchronize(st);
      (void)hipGraphExecDestroy(F->gexec);
      F->gexec = nullptr;
    }
    if (hipStreamBeginCapture(F->gs, hipStreamCaptureModeThreadLocal) != hipSuccess)
      return api_fail(OPF_EHIP, "chol: solve capture");
    int rc = OPF_OK;
    for (auto& C : F->inst)
      if (rc == OPF_OK) rc = solve_inst(C, b, x, F->gs);
    hipGraph_t g = nullptr;
    const hipError_t e = hipStreamEndCapture(F->gs, &g);
    if (rc != OPF_OK) {
      if (g) (void)hipGraphDestroy(g);
      return rc;
    }
    if (e != hipSuccess || !g) return api_fail(OPF_EHIP, "chol: solve capture end");
    const hipError_t ei = hipGraphInstantiate(&F->gexec, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (ei != hipSuccess) {
      F->gexec = nullptr;
      return api_fail(OPF_EHIP, std::string("chol: solve graph: ") + hipGetErrorString(ei));
    }
    F->gb = b;
    F->gx = x;
  }
  if (hipGraphLaunch(F->gexec, st) != hipSuccess) return api_fail(OPF_EHIP, "chol: solve graph launch");
  return OPF_OK;
}

int opf_chol_set_stop_on_pivot(opf_chol* F, int enable) {
  if (!F) return api_fail(OPF_EINVAL, "chol is NULL");
  F->stop_on_pivot = enable != 0;
  return OPF_OK;
}

int opf_chol_stop_on_pivot(const opf_chol* F) { return F && F->stop_on_pivot ? 1 : 0; }

int opf_chol_set_graph(opf_chol* F, int enable) {
  if (!F) return api_fail(OPF_EINVAL, "chol is NULL");
  F->use_graph = enable != 0;
  return OPF_OK;
}

}  // extern "C"
