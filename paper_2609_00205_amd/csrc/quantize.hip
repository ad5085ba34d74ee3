// ROI tolerance maps and the reciprocal quantizer (Sec. IV-C, IV-D).
//
// Block-wise tolerance assignment: a level-1 block takes the minimum voxel
// tolerance over its closed node range (a partly covered block is strict;
// padded nodes count as the node they copy).  Conservative propagation
// (Eq. 2): a block of local level s+1 takes the minimum over the level-s
// blocks that share a node with it.  Global levels use tau_global, the
// minimum over the last local level.
//
// Budget (the L-infinity bound of Sec. II-B): level s gets the share w_s of
// every tolerance (proportional to its coefficient count, equal among the
// global levels, floored at 1/(64 T) and renormalised; see level_weights);
// a detail of level s on a node with tolerance tau gets bin width
// Delta = tau * kappa_s, kappa_s = 2 (1 - eta) w_s / A_s, where A_s is the
// level's L-infinity gain; the coarsest values get kappa = 2 (1 - eta) w_c.
// q = rint(c * (1/Delta)) in FP64 (the per-block reciprocal quantizer of
// Sec. IV-D), c_hat = q * Delta.  A node inside several blocks of its level
// uses the smallest Delta (largest reciprocal) of those blocks; because
// rounding is monotone this equals computing Delta from the smallest tau.

#include <algorithm>
#include <cmath>

#include <cstring>

#include "internal.h"

namespace bm {
namespace {

constexpr int NT = 256;

inline unsigned grid_for(int64_t tot) {
  int64_t g = (tot + NT - 1) / NT;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return unsigned(g);
}

// tolerances are positive doubles: their bit patterns order like the values
__device__ inline void atomic_min_pos(double* p, double v) {
  atomicMin(reinterpret_cast<unsigned long long*>(p), static_cast<unsigned long long>(__double_as_longlong(v)));
}

__global__ void k_fill(double* p, int64_t n, double v) {
  for (int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x; i < n; i += int64_t(gridDim.x) * NT) p[i] = v;
}

struct BoxArgs {
  const double* boxes;   // nbox x 7
  int nbox;
  double background;
  int64_t n[3];          // logical dims
  int64_t nb[3];
  int64_t w;             // block width in nodes (b-1); 0 when L == 0 (one block)
  double* out;
};

// Up to kArgBoxes boxes come with the launch, longer lists from device memory
// (a copy from staging that the call has to wait for: map, quantization and
// reconstruction of 129^3 under new boxes 102 -> 81 us).
constexpr int kArgBoxes = 32;
struct BoxList {
  double r[kArgBoxes * 7];
};

template <bool ARG>
__global__ void k_tol_boxes(BoxArgs a, BoxList l) {
  const int64_t nbt = a.nb[0] * a.nb[1] * a.nb[2];
  for (int64_t k = int64_t(blockIdx.x) * NT + threadIdx.x; k < nbt; k += int64_t(gridDim.x) * NT) {
    const int64_t bx = k % a.nb[2], t = k / a.nb[2], by = t % a.nb[1], bz = t / a.nb[1];
    const int64_t bi[3] = {bz, by, bx};
    int64_t lo[3], hi[3];
    for (int d = 0; d < 3; ++d) {
      if (a.w == 0) {
        lo[d] = 0;
        hi[d] = a.n[d] - 1;
      } else {
        lo[d] = i64min(bi[d] * a.w, a.n[d] - 1);
        hi[d] = i64min((bi[d] + 1) * a.w, a.n[d] - 1);
      }
    }
    double v = a.background;
    for (int j = 0; j < a.nbox; ++j) {
      const double* r = (ARG ? l.r : a.boxes) + 7 * j;
      bool hit = true;
      for (int d = 0; d < 3; ++d) {
        const int64_t b0 = int64_t(r[d]), b1 = int64_t(r[d + 3]);
        hit = hit && b0 < b1 && b0 <= hi[d] && b1 > lo[d];
      }
      if (hit && r[6] < v) v = r[6];
    }
    a.out[k] = v;
  }
}

struct VoxArgs {
  const double* vt;
  int64_t n[3];
  int64_t nb[3];
  int64_t w;
  double* out;
};

// one workgroup per block: min over the block's closed node range
__global__ __launch_bounds__(NT) void k_tol_voxels(VoxArgs a) {
  __shared__ double red[NT];
  const int64_t k = blockIdx.x;
  const int64_t bx = k % a.nb[2], t = k / a.nb[2], by = t % a.nb[1], bz = t / a.nb[1];
  const int64_t bi[3] = {bz, by, bx};
  int64_t lo[3], ext[3];
  for (int d = 0; d < 3; ++d) {
    lo[d] = i64min(bi[d] * a.w, a.n[d] - 1);
    ext[d] = i64min((bi[d] + 1) * a.w, a.n[d] - 1) - lo[d] + 1;
  }
  double v = INFINITY;
  const int64_t cnt = ext[0] * ext[1] * ext[2];
  for (int64_t i = threadIdx.x; i < cnt; i += NT) {
    const int64_t x = i % ext[2], r = i / ext[2], y = r % ext[1], z = r / ext[1];
    const double tv = a.vt[((lo[0] + z) * a.n[1] + lo[1] + y) * a.n[2] + lo[2] + x];
    v = tv < v ? tv : v;
  }
  red[threadIdx.x] = v;
  __syncthreads();
  for (int s = NT / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] = fmin(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) a.out[k] = red[0];
}

// min over everything (L == 0): grid-stride + atomic min into out[0] (pre-filled with +inf)
__global__ __launch_bounds__(NT) void k_min_all(const double* v, int64_t n, double* out) {
  __shared__ double red[NT];
  double m = INFINITY;
  for (int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x; i < n; i += int64_t(gridDim.x) * NT) m = fmin(m, v[i]);
  red[threadIdx.x] = m;
  __syncthreads();
  for (int s = NT / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] = fmin(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) atomic_min_pos(out, red[0]);
}



struct QArgs {
  uint32_t tot;               // padded node count (< 2^32)
  Unflat32 uf;                // flat index -> (z, y, x) of the padded grid
  int L, M;
  int D[3];                   // levels each axis coarsens
  int lw;                     // log2(b - 1), b of the first block level
  int nested;                 // nested block schedule: every level's blocks span b - 1 padded cells
  // 27-class Delta and 1/Delta tables per block: slot s-1 for the details of
  // local level s; slot kCoarseSlot for the coarsest values when M == 0
  // (level-L blocks)
  const double* cdel[9];
  const double* cinv[9];
  uint32_t nb[9][3];
  const double* q;            // scalar Delta / inverse per level (index s-1), coarsest at L+M
  int64_t* counters;          // [0] outliers, [1] max |q|, [2] out of range
  const double* pdel;         // optional per-node Delta (padded grid); 1/Delta is its IEEE reciprocal
};

__device__ inline int ctz32(uint32_t v) { return v == 0 ? 32 : __builtin_ctz(v); }

// level of a node: 1..L+M for a detail of that level, L+M+1 for a coarsest value
__device__ inline int node_level(const QArgs& a, uint32_t g0, uint32_t g1, uint32_t g2) {
  int lev = a.L + a.M + 1;
  const uint32_t g[3] = {g0, g1, g2};
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int t = ctz32(g[d]);
    if (t < a.D[d] && t + 1 < lev) lev = t + 1;
  }
  return lev;
}

constexpr int kCoarseSlot = 8;

// Delta and 1/Delta of a node whose tolerance comes from the blocks of local
// level s (grid coordinates q = g >> (s-1)), from table slot `slot`.  Block i
// spans nodes [i w, (i+1) w]: a node on a shared face lies in two blocks per
// axis, and the block's class table holds the smallest Delta (largest
// 1/Delta) of the up to eight: one load per node instead of a walk over them
// (k_qoi_final at 384 x 384 x 256 FP32: 0.227 -> 0.166 ms, with the share no
// longer read there).  In the nested schedule the blocks of every level span the same
// padded-grid regions, so the padded coordinates g index them directly.
__device__ inline void block_delta(const QArgs& a, int s, int slot, uint32_t g0, uint32_t g1, uint32_t g2,
                                   double& del, double& inv) {
  const int sh = a.nested ? 0 : s - 1;
  const uint32_t q[3] = {g0 >> sh, g1 >> sh, g2 >> sh};
  const uint32_t wm = (1u << a.lw) - 1;
  uint32_t f[3], cls = 0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    f[d] = q[d] >> a.lw;
    uint32_t c = 1;                       // inside a block
    if ((q[d] & wm) == 0) {
      const bool far = f[d] >= a.nb[slot][d];
      f[d] = far ? a.nb[slot][d] - 1 : f[d];
      c = far ? 2 : 0;                    // the far end of the grid, or the face block f starts on
    }
    cls = cls * 3 + c;
  }
  const uint32_t k = ((f[0] * a.nb[slot][1] + f[1]) * a.nb[slot][2] + f[2]) * 27u + cls;
  del = a.cdel[slot][k];
  inv = a.cinv[slot][k];
}

__device__ inline void node_delta(const QArgs& a, uint32_t z, uint32_t y, uint32_t x, double& del, double& inv) {
  const int lev = node_level(a, z, y, x);
  if (lev <= a.L) {
    block_delta(a, lev, lev - 1, z, y, x, del, inv);
  } else if (lev == a.L + a.M + 1 && a.M == 0) {
    block_delta(a, a.L, kCoarseSlot, z, y, x, del, inv);
  } else {
    del = a.q[2 * (lev - 1)];
    inv = a.q[2 * (lev - 1) + 1];
  }
}

// Each thread handles QU nodes of a tile of NT*QU consecutive nodes per
// iteration, so the independent loads of those nodes overlap.
constexpr int QU = 4;
constexpr int kMaxQGroups = 8192;

inline unsigned qgroups(uint32_t tot) {
  const int64_t tiles = (int64_t(tot) + NT * QU - 1) / (NT * QU);
  return unsigned(tiles < kMaxQGroups ? (tiles > 0 ? tiles : 1) : kMaxQGroups);
}

// Per-workgroup statistics go to partials[3 * group]: outliers, max |q|,
// out-of-range flag; k_reduce_stats folds them into counters[0..2].
template <typename T>
__global__ __launch_bounds__(NT) void k_quantize(QArgs a, const T* c, int32_t* codes, int64_t* partials) {
  int64_t nout = 0, mx = 0, bad = 0;
  const uint32_t ntiles = (a.tot + NT * QU - 1) / (NT * QU);
  for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const uint32_t base = tile * (NT * QU) + threadIdx.x;
    double cv[QU], inv[QU];
#pragma unroll
    for (int k = 0; k < QU; ++k) {
      const uint32_t i = base + k * NT;
      cv[k] = 0.0;
      inv[k] = 0.0;
      if (i < a.tot) {
        uint32_t z, y, x;
        a.uf(i, z, y, x);
        double del;
        if (a.pdel) {
          inv[k] = 1.0 / a.pdel[i];
        } else {
          node_delta(a, z, y, x, del, inv[k]);
        }
        cv[k] = double(c[i]);
      }
    }
#pragma unroll
    for (int k = 0; k < QU; ++k) {
      const uint32_t i = base + k * NT;
      if (i >= a.tot) continue;
      const double v = rint(mul_rn(cv[k], inv[k]));
      int32_t qv;
      if (!(fabs(v) <= 2147483647.0)) {
        bad |= int64_t(code_flag(double(cv[k])));
        qv = 0;
      } else {
        qv = int32_t(v);
      }
      codes[i] = qv;
      const int64_t aq = qv < 0 ? -int64_t(qv) : int64_t(qv);
      nout += aq >= 32768;
      mx = aq > mx ? aq : mx;
    }
  }
  __shared__ int64_t red[3][NT / 64];
  for (int off = 32; off > 0; off >>= 1) {
    nout += __shfl_down(nout, off, 64);
    const int64_t o = __shfl_down(mx, off, 64);
    mx = o > mx ? o : mx;
    bad |= __shfl_down(bad, off, 64);
  }
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    red[0][wv] = nout;
    red[1][wv] = mx;
    red[2][wv] = bad;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t s0 = 0, s1 = 0, s2 = 0;
    for (int k = 0; k < NT / 64; ++k) {
      s0 += red[0][k];
      s1 = red[1][k] > s1 ? red[1][k] : s1;
      s2 |= red[2][k];
    }
    partials[3 * blockIdx.x] = s0;
    partials[3 * blockIdx.x + 1] = s1;
    partials[3 * blockIdx.x + 2] = s2;
  }
}

__global__ __launch_bounds__(NT) void k_reduce_stats(const int64_t* partials, int n, int64_t* counters) {
  __shared__ int64_t r[3][NT];
  int64_t s0 = 0, s1 = 0, s2 = 0;
  for (int k = threadIdx.x; k < n; k += NT) {
    s0 += partials[3 * k];
    s1 = partials[3 * k + 1] > s1 ? partials[3 * k + 1] : s1;
    s2 |= partials[3 * k + 2];
  }
  r[0][threadIdx.x] = s0;
  r[1][threadIdx.x] = s1;
  r[2][threadIdx.x] = s2;
  __syncthreads();
  for (int s = NT / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      r[0][threadIdx.x] += r[0][threadIdx.x + s];
      r[1][threadIdx.x] = r[1][threadIdx.x + s] > r[1][threadIdx.x] ? r[1][threadIdx.x + s] : r[1][threadIdx.x];
      r[2][threadIdx.x] |= r[2][threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    counters[0] = r[0][0];
    counters[1] = r[1][0];
    counters[2] = r[2][0];
  }
}

template <typename T>
__global__ __launch_bounds__(NT) void k_dequantize(QArgs a, const int32_t* codes, T* c) {
  const uint32_t ntiles = (a.tot + NT * QU - 1) / (NT * QU);
  for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const uint32_t base = tile * (NT * QU) + threadIdx.x;
    double q[QU], del[QU];
#pragma unroll
    for (int k = 0; k < QU; ++k) {
      const uint32_t i = base + k * NT;
      q[k] = 0.0;
      del[k] = 0.0;
      if (i < a.tot) {
        uint32_t z, y, x;
        a.uf(i, z, y, x);
        double inv;
        if (a.pdel)
          del[k] = a.pdel[i];
        else
          node_delta(a, z, y, x, del[k], inv);
        q[k] = double(codes[i]);
      }
    }
#pragma unroll
    for (int k = 0; k < QU; ++k) {
      const uint32_t i = base + k * NT;
      if (i < a.tot) c[i] = T(mul_rn(q[k], del[k]));
    }
  }
}

int64_t prod3(const int64_t n[3]) { return n[0] * n[1] * n[2]; }

}  // namespace

// Adjoint-guided widths for a linear quantity of interest Q = <g, x>: with
// s = R^T g, quantization moves Q by at most sum |s_i| Delta_i / 2.  Each
// coefficient's share |s_i| Delta_i / 2 is one level lambda, except where the
// node's L-inf width cap_i is smaller: share = min(a_i, lambda) with
// a_i = |s_i| cap_i / 2, and lambda the root of f(lambda) =
// sum_i min(a_i, lambda) = (1 - eta) tol_q.  f is concave and piecewise
// linear; a pass evaluates it at kQoiK candidates and keeps the bracket
// f(lo) <= target < f(hi).
//
// HBM reads bound a pass, so a pass drops the shares that no later pass
// needs one by one: a share <= lo adds itself to every later sum, one >= hi
// adds the candidate.  Each wavefront compacts the others, in order, over the
// chunks it has read already (in place, no atomics, the same result on every
// run), so only the first pass goes over all nodes.  The next candidates lie
// between the bounds that concavity gives (chords from outside the bracket
// below, the bracket's own chord above), which closes in quadratically where
// an even split of the bracket gains a factor 16; the steps run on the device,
// so passes follow each other without a host round trip.  384 x 384 x 256
// FP32: shares 0.309 -> 0.184 ms (152 MB read, the shares above lo written),
// search 1.88 ms (15 passes over 306 MB and their folds) -> 0.17 ms.
// Sums are reduced per workgroup in a fixed order, then by one workgroup
// (deterministic).
constexpr int kQoiK = 15;           // candidate levels per pass
constexpr int kQoiGroups = 1024;    // workgroups of a pass
constexpr int kQoiPasses = 10;      // passes launched before the host looks whether the search has ended
constexpr int kQoiU = 4;            // chunks in flight per wavefront

// the search's state in the plan's statistics scratch
struct QoiState {
  double target, lo, hi, flo, fhi;  // f at lo and hi (NaN while unknown)
  double c[kQoiK];                  // the next pass's candidates, ascending
  double lambda;
  int done, passes;
};
struct QoiScratch {
  QoiState st;
  double sum[kQoiGroups], max[kQoiGroups];            // of all shares, per workgroup
  double f[kQoiGroups * kQoiK];                       // candidates' sums over the kept shares
  double low[kQoiGroups], high[kQoiGroups];           // dropped: sum of the low ones, count of the high ones
  int kept[kQoiGroups * (NT / 64)];                   // kept shares per wavefront
};
static_assert(sizeof(QoiScratch) <= 3 * 8192 * sizeof(double), "QoI scratch exceeds the statistics scratch");

__device__ inline double block_sum(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int w = NT / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

__device__ inline double block_max(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int w = NT / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

// The 64-share chunks of wavefront w (of W) in the share array: chunk k at
// (k W + w) 64.  Keeps v (where `keep`) at position `at` of the wavefront's
// compacted list and advances it; a list never overtakes the chunks read.
__device__ inline void qoi_keep(double* share, uint32_t W, uint32_t w, int lane, bool keep, double v, uint32_t& at) {
  const unsigned long long m = __ballot(keep);
  if (keep) {
    const uint32_t p = at + __popcll(m & ((1ull << lane) - 1));
    share[(uint64_t(p >> 6) * W + w) * 64 + (p & 63)] = v;
  }
  at += __popcll(m);
}

// a_i = |s_i| cap_i / 2 of every node: their sum and max, f at the first
// candidates, and the ones above lo kept in share.
template <typename T>
__global__ __launch_bounds__(NT) void k_qoi_shares(QArgs a, const T* s, double* share, QoiScratch* q) {
  __shared__ double red[NT];
  const int lane = threadIdx.x & 63;
  const uint32_t W = gridDim.x * (NT / 64), w = blockIdx.x * (NT / 64) + (threadIdx.x >> 6);
  const uint32_t nchunk = uint32_t((uint64_t(a.tot) + 63) / 64);
  const double lo = q->st.lo;
  double c[kQoiK], acc[kQoiK];
#pragma unroll
  for (int j = 0; j < kQoiK; ++j) {
    c[j] = q->st.c[j];
    acc[j] = 0.0;
  }
  double sum = 0.0, mx = 0.0, low = 0.0;
  uint32_t at = 0;
  for (uint32_t k0 = w; k0 < nchunk; k0 += kQoiU * W) {
    double v[kQoiU];
#pragma unroll
    for (int u = 0; u < kQoiU; ++u) {
      const uint64_t i = (uint64_t(k0) + uint64_t(u) * W) * 64 + lane;
      v[u] = 0.0;
      if (i < a.tot) {
        uint32_t z, y, x;
        a.uf(uint32_t(i), z, y, x);
        double del, inv;
        node_delta(a, z, y, x, del, inv);
        v[u] = fabs(double(s[i])) * del * 0.5;
      }
    }
#pragma unroll
    for (int u = 0; u < kQoiU; ++u) {
      sum += v[u];
      mx = fmax(mx, v[u]);
      const bool keep = !(v[u] <= lo);
      if (!keep) low += v[u];
      qoi_keep(share, W, w, lane, keep, v[u], at);
      if (keep) {
#pragma unroll
        for (int j = 0; j < kQoiK; ++j) acc[j] += fmin(v[u], c[j]);
      }
    }
  }
  if (lane == 0) q->kept[w] = int(at);
  sum = block_sum(sum, red);
  mx = block_max(mx, red);
  low = block_sum(low, red);
  if (threadIdx.x == 0) {
    q->sum[blockIdx.x] = sum;
    q->max[blockIdx.x] = mx;
    q->low[blockIdx.x] = low;
    q->high[blockIdx.x] = 0.0;
  }
  for (int j = 0; j < kQoiK; ++j) {
    const double r = block_sum(acc[j], red);
    if (threadIdx.x == 0) q->f[blockIdx.x * kQoiK + j] = r;
  }
}

// one later pass over the kept shares (same grid as k_qoi_shares)
__global__ __launch_bounds__(NT) void k_qoi_eval(double* share, QoiScratch* q) {
  __shared__ double red[NT];
  if (q->st.done) return;
  const int lane = threadIdx.x & 63;
  const uint32_t W = gridDim.x * (NT / 64), w = blockIdx.x * (NT / 64) + (threadIdx.x >> 6);
  const double lo = q->st.lo, hi = q->st.hi;
  double c[kQoiK], acc[kQoiK];
#pragma unroll
  for (int j = 0; j < kQoiK; ++j) {
    c[j] = q->st.c[j];
    acc[j] = 0.0;
  }
  const uint32_t n = uint32_t(q->kept[w]);
  double low = 0.0, high = 0.0;
  uint32_t at = 0;
  for (uint32_t p0 = 0; p0 < n; p0 += 64 * kQoiU) {
    double v[kQoiU];
    bool in[kQoiU];
#pragma unroll
    for (int u = 0; u < kQoiU; ++u) {
      const uint32_t p = p0 + 64 * u + lane;
      in[u] = p < n;
      v[u] = in[u] ? share[(uint64_t(p >> 6) * W + w) * 64 + lane] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kQoiU; ++u) {
      const bool dl = v[u] <= lo, dh = v[u] >= hi;
      const bool keep = in[u] && !dl && !dh;
      if (in[u] && dl) low += v[u];
      if (in[u] && dh) high += 1.0;
      qoi_keep(share, W, w, lane, keep, v[u], at);
      if (keep) {
#pragma unroll
        for (int j = 0; j < kQoiK; ++j) acc[j] += fmin(v[u], c[j]);
      }
    }
  }
  if (lane == 0) q->kept[w] = int(at);
  low = block_sum(low, red);
  high = block_sum(high, red);
  if (threadIdx.x == 0) {
    q->low[blockIdx.x] += low;
    q->high[blockIdx.x] += high;
  }
  for (int j = 0; j < kQoiK; ++j) {
    const double r = block_sum(acc[j], red);
    if (threadIdx.x == 0) q->f[blockIdx.x * kQoiK + j] = r;
  }
}

// The search starts at lo = target / n (f(lo) <= n lo) with candidates a
// factor 4 apart; the largest share, hi, is known after the first pass.
__global__ void k_qoi_begin(QoiScratch* q, double target, double n, unsigned long long* count) {
  if (threadIdx.x != 0) return;
  *count = 0;
  QoiState& t = q->st;
  t.target = target;
  t.lo = target / n;
  t.hi = INFINITY;
  t.flo = t.fhi = NAN;
  t.lambda = 0.0;
  t.done = t.passes = 0;
  double c = t.lo;
  for (int j = 0; j < kQoiK; ++j) t.c[j] = c *= 4.0;
}

__device__ inline double from_bits(long long b) { return __longlong_as_double(b); }

// The new bracket [lo, hi] from the candidates' sums f, and the next
// candidates (or the end: no double strictly inside, lambda = lo).
__device__ inline void qoi_narrow(QoiState& t, const double* f) {
  double lo = t.lo, hi = t.hi, flo = t.flo, fhi = t.fhi;
  // the points around the bracket's ends, outside it (NaN: none)
  double plo = NAN, pflo = NAN, phi = NAN, pfhi = NAN;
  for (int j = 0; j < kQoiK; ++j) {       // the largest candidate with f <= target
    const double c = t.c[j];
    if (c > t.lo && c < t.hi && f[j] <= t.target && c > lo) {
      plo = lo;
      pflo = flo;
      lo = c;
      flo = f[j];
    }
  }
  for (int j = kQoiK - 1; j >= 0; --j) {  // the smallest with f > target
    const double c = t.c[j];
    if (c > t.lo && c < t.hi && !(f[j] <= t.target) && c < hi) {
      phi = hi;
      pfhi = fhi;
      hi = c;
      fhi = f[j];
    }
  }
  t.passes += 1;
  if (lo >= hi) {                         // sums not monotone at rounding level
    t.lambda = lo;
    t.done = 1;
    return;
  }
  t.lo = lo;
  t.hi = hi;
  t.flo = flo;
  t.fhi = fhi;
  const long long blo = __double_as_longlong(lo), bhi = __double_as_longlong(hi);   // positive: ordered like the values
  if (bhi - blo <= 1 || t.passes >= 80) {
    t.lambda = lo;
    t.done = 1;
    return;
  }
  // where the root can lie
  double L = lo, U = hi;
  const double slope = (fhi - flo) / (hi - lo);
  if (slope > 0 && isfinite(slope)) {
    // sums carry a few roundings of the target, candidates one of their own
    const double slack = 2e-15 * t.target / slope + 4e-16 * lo;
    U = fmin(U, lo + (t.target - flo) / slope + slack);
    const double sl = (flo - pflo) / (lo - plo), sh = (pfhi - fhi) / (phi - hi);
    if (sl > 0 && isfinite(sl)) L = fmax(L, lo + (t.target - flo) / sl - slack);
    if (sh > 0 && isfinite(sh)) L = fmax(L, hi - (fhi - t.target) / sh - slack);
  }
  if (!(L >= lo && L < U && U <= hi)) {
    L = lo;
    U = hi;
  }
  const long long bL = __double_as_longlong(L), bU = __double_as_longlong(U);
  if (bU - bL <= kQoiK - 3) {             // every double there, and one on either side
    for (int j = 0; j < kQoiK; ++j) t.c[j] = from_bits(bL - 1 + j);
  } else if (L == lo && U == hi) {        // nothing known: geometric steps, then even ones
    for (int j = 0; j < kQoiK; ++j) {
      const double u = double(j + 1) / double(kQoiK + 1);
      t.c[j] = hi > 2.0 * lo ? lo * pow(hi / lo, u) : lo + (hi - lo) * u;
    }
  } else {                                // even steps over [L, U], and one point on either side of it
    t.c[0] = lo + 0.5 * (L - lo);
    for (int j = 0; j < kQoiK - 2; ++j) t.c[j + 1] = L + (U - L) * (double(j) / double(kQoiK - 3));
    t.c[kQoiK - 1] = U + 0.5 * (hi - U);
  }
}

// Folds a pass's sums (wavefront j: candidate j) and takes the next step of
// the search; after the first pass also the sum and the largest share.
__global__ __launch_bounds__(1024) void k_qoi_step(QoiScratch* q, int ng, int first) {
  __shared__ double f[16], red[4][16];
  if (!first && q->st.done) return;
  const int lane = threadIdx.x & 63, j = threadIdx.x >> 6;
  // sums over the workgroups, 16 wavefronts each a 16th of them
  double v[4] = {0.0, 0.0, 0.0, 0.0};     // low, high, sum, max
  for (int g = threadIdx.x; g < ng; g += 1024) {
    v[0] += q->low[g];
    v[1] += q->high[g];
    if (first) {
      v[2] += q->sum[g];
      v[3] = fmax(v[3], q->max[g]);
    }
  }
  double s = 0.0;
  if (j < kQoiK)
    for (int g = lane; g < ng; g += 64) s += q->f[g * kQoiK + j];
  for (int off = 32; off > 0; off >>= 1) {
    s += __shfl_down(s, off, 64);
#pragma unroll
    for (int k = 0; k < 3; ++k) v[k] += __shfl_down(v[k], off, 64);
    v[3] = fmax(v[3], __shfl_down(v[3], off, 64));
  }
  if (lane == 0) {
    f[j] = s;
#pragma unroll
    for (int k = 0; k < 4; ++k) red[k][j] = v[k];
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  double low = 0.0, high = 0.0, sum = 0.0, mx = 0.0;
  for (int k = 0; k < 16; ++k) {
    low += red[0][k];
    high += red[1][k];
    sum += red[2][k];
    mx = fmax(mx, red[3][k]);
  }
  QoiState& t = q->st;
  if (first) {
    t.hi = mx;
    if (!(sum > t.target)) {              // every cap fits: no width is set by the quantity
      t.lambda = INFINITY;
      t.done = 1;
      return;
    }
    if (isinf(mx) || !(mx > t.lo)) {      // (no bracket to search)
      t.lambda = t.lo;
      t.done = 1;
      return;
    }
    t.fhi = sum;
  }
  for (int k = 0; k < kQoiK; ++k) f[k] = f[k] + low + high * t.c[k];
  qoi_narrow(t, f);
}

// Delta_i = 2 lambda / |s_i| where a_i > lambda (the quantity sets the
// width), else the node's L-inf width; counts the former.  Nothing is
// written while the search has not ended.
template <typename T>
__global__ __launch_bounds__(NT) void k_qoi_final(QArgs a, const T* s, const QoiScratch* q, double* delta,
                                                  unsigned long long* count) {
  __shared__ double red[NT];
  if (!q->st.done) return;
  const double lambda = q->st.lambda;
  double c = 0.0;
  const uint32_t ntiles = (a.tot + NT * QU - 1) / (NT * QU);
  for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const uint32_t base = tile * (NT * QU) + threadIdx.x;
    double sv[QU], del[QU];
#pragma unroll
    for (int k = 0; k < QU; ++k) {
      const uint32_t i = base + k * NT;
      sv[k] = del[k] = 0.0;
      if (i < a.tot) {
        uint32_t z, y, x;
        a.uf(i, z, y, x);
        double inv;
        node_delta(a, z, y, x, del[k], inv);
        sv[k] = fabs(double(s[i]));
      }
    }
#pragma unroll
    for (int k = 0; k < QU; ++k) {
      const uint32_t i = base + k * NT;
      if (i >= a.tot) continue;
      const bool set = sv[k] * del[k] * 0.5 > lambda;
      delta[i] = set ? 2.0 * lambda / sv[k] : del[k];
      if (set) c += 1.0;
    }
  }
  c = block_sum(c, red);
  if (threadIdx.x == 0 && c > 0.0) atomicAdd(count, (unsigned long long)c);
}

QPrep qprep_layout(bm_plan_s& p, const double* block_tol) {
  const std::vector<double> w = level_weights(p);
  const double eta = p.cfg.eta;
  if (p.L > 8) fail(BM_EUNSUPPORTED, "more than 8 local levels");
  QPrep a{};
  a.flag = p.ws.counters + 2;
  const int64_t tot = p.ws.tol_off[p.L + 1];
  double* tg = p.ws.tolbuf + tot;         // tau_global
  const int64_t nlastb = p.L > 0 ? prod3(p.lv[p.L - 1].nb) : 0;
  double* cls = tg + 8;                   // 27-class tables: level s at 54 tol_off[s], coarsest at 54 tot
  for (int s = 1; s <= p.L; ++s) {
    const int64_t nbs = prod3(p.lv[s - 1].nb);
    const int64_t off = p.ws.tol_off[s];
    QTab& t = a.lv[s - 1];
    t.tau = s == 1 ? block_tol : p.ws.tolbuf + off;
    t.kap = (2.0 * (1.0 - eta)) * w[s - 1] / p.lv[s - 1].gain;
    t.cdel = cls + 54 * off;
    t.cinv = cls + 54 * off + 27 * nbs;
    for (int d = 0; d < 3; ++d) t.nb[d] = p.lv[s - 1].nb[d];
  }
  if (p.L > 0 && p.M == 0) {
    // coarsest values (no gain), over the level-L blocks
    QTab& t = a.lv[kCoarseSlotHost];
    t.tau = a.lv[p.L - 1].tau;
    t.kap = (2.0 * (1.0 - eta)) * w[p.nlev];
    t.cdel = cls + 54 * tot;
    t.cinv = cls + 54 * tot + 27 * nlastb;
    for (int d = 0; d < 3; ++d) t.nb[d] = p.lv[p.L - 1].nb[d];
  }
  a.q = p.ws.qparam;
  return a;
}

// One plan's tables are built by the many-field kernels with one field: one
// launch per propagation step, one per table level, one for tau_global and
// the scalar Deltas (which also clears the overflow flag).  The field record
// is stored only when it changes.
namespace {
__global__ void k_clear_flag(int64_t* flag) {
  if (threadIdx.x == 0) *flag = 0;
}
}  // namespace

// The preparation's record reaches the device as a launch's argument, in
// stream order, with no copy to wait for: a new plan's first call.
struct PrepImage {
  uint64_t w[kPrepBytes / 8];
};

__global__ __launch_bounds__(512) void k_prep_store(PrepImage im, uint64_t* dst) {
  static_assert(kPrepBytes % 8 == 0 && kPrepBytes / 8 <= 512, "a lane per word");
  if (threadIdx.x < kPrepBytes / 8) dst[threadIdx.x] = im.w[threadIdx.x];
}

static bool capturing(hipStream_t st) {
  hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
  BM_HIP(hipStreamIsCapturing(st, &c));
  return c != hipStreamCaptureStatusNone;
}

QPrep quant_prepare(bm_plan_s& p, const double* block_tol, hipStream_t st, bool clear_flag, bool tables) {
  const QPrep a = qprep_layout(p, block_tol);
  if (block_tol && block_tol == p.ws.kept_tol) {   // the kept tables are this map's
    if (clear_flag) {
      hipLaunchKernelGGL(k_clear_flag, dim3(1), dim3(64), 0, st, a.flag);
      BM_HIP(hipGetLastError());
    }
    return a;
  }
  p.ws.kept_tol = nullptr;   // the tables built here replace the kept ones
  // the record holds everything but the map, which comes with each launch: a
  // new map costs no upload
  const PrepField f = prep_field(p, nullptr, a);
  static_assert(sizeof(PrepField) <= kPrepFirst, "field record too large");
  int64_t cnt_prop[9] = {}, cnt_tab[9] = {};
  if (p.L > 1 && prod3(p.lv[1].nb) > kPropOneGroup)
    for (int s = 1; s < 9; ++s) cnt_prop[s] = p.L > s ? prod3(p.lv[s].nb) : 0;
  auto wants = [&](int s) { return tables || p.lv[s - 1].b == 33; };
  for (int s = 1; s < 9; ++s) cnt_tab[s] = p.L >= s && wants(s) ? 27 * prod3(p.lv[s - 1].nb) : 0;
  cnt_tab[0] = (p.L > 0 && p.M == 0 && wants(p.L)) ? 27 * prod3(p.lv[p.L - 1].nb) : 0;
  const uint8_t* fb = reinterpret_cast<const uint8_t*>(&f);
  if (!p.ws.prep_set || p.ws.prep_key.size() != sizeof(f) || std::memcmp(p.ws.prep_key.data(), fb, sizeof(f)) != 0) {
    PrepImage im{};
    std::memcpy(im.w, fb, sizeof(f));
    int64_t* first = reinterpret_cast<int64_t*>(im.w) + kPrepFirst / sizeof(int64_t);
    for (int s = 0; s < 9; ++s) {
      first[2 * s + 1] = s >= 1 && p.L > s ? prod3(p.lv[s].nb) : 0;
      first[18 + 2 * s + 1] = s == 0 ? (p.L > 0 && p.M == 0 ? 27 * prod3(p.lv[p.L - 1].nb) : 0)
                                     : (p.L >= s ? 27 * prod3(p.lv[s - 1].nb) : 0);
    }
    if (capturing(st)) {   // (a captured copy would leave the record unset: the wait refuses it)
      BM_HIP(hipMemcpyAsync(p.ws.prep_dev, im.w, sizeof(im), hipMemcpyHostToDevice, st));
      BM_HIP(hipStreamSynchronize(st));
    } else {
      hipLaunchKernelGGL(k_prep_store, dim3(1), dim3(512), 0, st, im, static_cast<uint64_t*>(p.ws.prep_dev));
      BM_HIP(hipGetLastError());
    }
    if (!p.ws.prep_set) p.dev_bytes += kPrepBytes;
    p.ws.prep_set = true;
    p.ws.prep_key.assign(fb, fb + sizeof(f));
  }
  PrepStages g;
  const int64_t* first = reinterpret_cast<const int64_t*>(static_cast<uint8_t*>(p.ws.prep_dev) + kPrepFirst);
  for (int s = 0; s < 9; ++s) {
    g.prop_first[s] = first + 2 * s;
    g.prop_n[s] = cnt_prop[s];
    g.tab_first[s] = first + 18 + 2 * s;
    g.tab_n[s] = cnt_tab[s];
  }
  g.fields = clear_flag || p.L != 1 || p.M > 0;
  launch_prep_batch(g, static_cast<const PrepField*>(p.ws.prep_dev), 1, block_tol, clear_flag, st);
  return a;
}

void quant_keep(bm_plan_s& p, const double* block_tol, hipStream_t st) {
  p.ws.kept_tol = nullptr;
  if (!block_tol) return;
  quant_prepare(p, block_tol, st);
  p.ws.kept_tol = block_tol;
}

// ---- many fields per launch -------------------------------------------------

namespace {

// taus of local level s (1-based); map: the level-1 map of a record without one
__device__ inline const double* taus(const PrepField& P, int s, const double* map) {
  return s == 1 && map ? map : P.tau[s - 1];
}

// Eq. 2: block i of level s+1 takes the smallest tau of the level-s blocks
// that share a node with it.  It spans blocks 2Z, 2Z+1 of level s and touches
// 2Z-1, 2Z+2 (nested: it is block Z itself, touching Z-1, Z+1); the 4^3 box
// is read with clamped coordinates (a repeated block changes no minimum), so
// that its loads overlap instead of following each other.
__device__ inline double propagate_task(const PrepField& P, int s, const double* tau, uint32_t i) {
  const uint32_t n0 = uint32_t(P.nb[s - 1][0]), n1 = uint32_t(P.nb[s - 1][1]), n2 = uint32_t(P.nb[s - 1][2]);
  const uint32_t m1 = uint32_t(P.nb[s][1]), m2 = uint32_t(P.nb[s][2]);
  const uint32_t t = i / m2, X = i - t * m2, Z = t / m1, Y = t - Z * m1;
  const uint32_t f = P.nested ? 1u : 2u;
  uint32_t z[4], y[4], x[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int o = (k < int(f) + 2 ? k : int(f) + 1) - 1;
    auto at = [&](uint32_t c, uint32_t n) {
      const int v = int(c * f) + o;
      return uint32_t(v < 0 ? 0 : v >= int(n) ? int(n) - 1 : v);
    };
    z[k] = at(Z, n0);
    y[k] = at(Y, n1);
    x[k] = at(X, n2);
  }
  double v = INFINITY;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    double r[16];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int c = 0; c < 4; ++c) r[4 * b + c] = tau[(z[a] * n1 + y[b]) * n2 + x[c]];
#pragma unroll
    for (int k = 0; k < 16; ++k) v = fmin(v, r[k]);
  }
  return v;
}

// one step for every field that has level s+1
__global__ void k_batch_propagate(const PrepField* F, const int64_t* first, int nf, int64_t ntot, int s,
                                  const double* map) {
  for (int64_t k = int64_t(blockIdx.x) * NT + threadIdx.x; k < ntot; k += int64_t(gridDim.x) * NT) {
    const int f = task_field(first, nf, k);
    const PrepField& P = F[f];
    const int64_t i = k - first[f];
    const_cast<double*>(P.tau[s])[i] = propagate_task(P, s, taus(P, s, map), uint32_t(i));
  }
}

// The 27-class Delta and 1/Delta tables of local level s (s = 0: the
// coarsest values of a field with M == 0) straight from the taus: rounding
// of tau * kappa is monotone, so the smallest Delta over a set of blocks is
// the smallest tau times kappa, and its reciprocal is the largest 1/Delta.
// Task = (block, class), consecutive tasks write consecutive entries.  Along an axis, class 0
// (first face) takes the block and the one before, 1 the block alone, 2
// (last face) the block and the one after.  32-bit index arithmetic (a
// level has fewer than 2^32 / 27 blocks).
// one task of k_batch_tables: task i of field P
__device__ inline void table_task(const PrepField& P, int s, uint32_t i, const double* map) {
  const int li = s > 0 ? s - 1 : P.L - 1;
  const QTab& T = s > 0 ? P.tab[li] : P.tab[kCoarseSlotHost];
  const double kap = s > 0 ? P.kap[li] : P.kapc;
  const double* tau = taus(P, li + 1, map);
  const uint32_t blk = i / 27u;
  const int c = int(i - blk * 27u);
  const int cls[3] = {c / 9, (c / 3) % 3, c % 3};
  const uint32_t n0 = uint32_t(P.nb[li][0]), n1 = uint32_t(P.nb[li][1]), n2 = uint32_t(P.nb[li][2]);
  const uint32_t t = blk / n2;
  const uint32_t b[3] = {t / n1, t - (t / n1) * n1, blk - t * n2};
  const uint32_t nb[3] = {n0, n1, n2};
  uint32_t lo[3], hi[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    lo[d] = (cls[d] == 0 && b[d] > 0) ? b[d] - 1 : b[d];
    hi[d] = (cls[d] == 2 && b[d] + 1 < nb[d]) ? b[d] + 1 : b[d];
  }
  // each axis spans at most two blocks: the eight corners of the box
  // (repeated where lo == hi) are loaded together, then reduced
  double tv[8];
#pragma unroll
  for (int j = 0; j < 8; ++j)
    tv[j] = tau[(((j & 4) ? hi[0] : lo[0]) * n1 + ((j & 2) ? hi[1] : lo[1])) * n2 + ((j & 1) ? hi[2] : lo[2])];
  const double m = fmin(fmin(fmin(tv[0], tv[1]), fmin(tv[2], tv[3])), fmin(fmin(tv[4], tv[5]), fmin(tv[6], tv[7])));
  const double d = m * kap, iv = 1.0 / d;
  const_cast<double*>(T.cdel)[i] = d;
  const_cast<double*>(T.cinv)[i] = iv;
}

__global__ void k_batch_tables(const PrepField* F, const int64_t* first, int nf, int64_t ntot, int s,
                               const double* map) {
  if (nf == 1) {
    // one field: its record is the same for every lane (scalar loads)
    for (int64_t k = int64_t(blockIdx.x) * NT + threadIdx.x; k < ntot; k += int64_t(gridDim.x) * NT)
      table_task(F[0], s, uint32_t(k - first[0]), map);
    return;
  }
  for (int64_t k = int64_t(blockIdx.x) * NT + threadIdx.x; k < ntot; k += int64_t(gridDim.x) * NT) {
    const int f = task_field(first, nf, k);
    table_task(F[f], s, uint32_t(k - first[f]), map);
  }
}

// One workgroup per field: the propagation (prop: unless launches of many
// workgroups did it), tau_global (minimum over the last block level, or the
// single map value when there is none) and the scalar Deltas where a global
// level or the coarsest values use them, and the overflow flag cleared.
constexpr int kScalarNT = 1024;

__global__ __launch_bounds__(kScalarNT) void k_batch_prep(const PrepField* F, const double* map, int prop, int clear) {
  __shared__ double red[kScalarNT / 64];
  const PrepField& P = F[blockIdx.x];
  const int tid = threadIdx.x;
  if (clear && tid == 0) *P.flag = 0;
  if (prop) {
    for (int s = 1; s < P.L; ++s) {
      const uint32_t n = uint32_t(P.nb[s][0] * P.nb[s][1] * P.nb[s][2]);
      const double* tau = taus(P, s, map);
      double* out = const_cast<double*>(P.tau[s]);
      for (uint32_t i = tid; i < n; i += kScalarNT) out[i] = propagate_task(P, s, tau, i);
      __syncthreads();   // the next level reads what this workgroup wrote
    }
  }
  if (P.L > 0 && P.M == 0) return;
  double m = INFINITY;
  if (P.L > 0) {
    const int64_t* nb = P.nb[P.L - 1];
    const int64_t n = nb[0] * nb[1] * nb[2];
    const double* tau = taus(P, P.L, map);
    // eight independent loads in flight per lane
    double mm[8] = {INFINITY, INFINITY, INFINITY, INFINITY, INFINITY, INFINITY, INFINITY, INFINITY};
    int64_t i = tid;
    for (; i + 7 * kScalarNT < n; i += 8 * kScalarNT)
#pragma unroll
      for (int u = 0; u < 8; ++u) mm[u] = fmin(mm[u], tau[i + u * kScalarNT]);
    for (; i < n; i += kScalarNT) mm[0] = fmin(mm[0], tau[i]);
#pragma unroll
    for (int u = 0; u < 8; ++u) m = fmin(m, mm[u]);
  } else if (tid == 0) {
    m = taus(P, 1, map)[0];
  }
  for (int off = 32; off > 0; off >>= 1) m = fmin(m, __shfl_down(m, off, 64));
  if ((tid & 63) == 0) red[tid >> 6] = m;
  __syncthreads();
  m = red[0];
#pragma unroll
  for (int k = 1; k < kScalarNT / 64; ++k) m = fmin(m, red[k]);
  if (tid == 0) *P.tg = m;
  if (tid <= P.nlev) {
    const double d = m * P.kq[tid];
    P.q[2 * tid] = d;
    P.q[2 * tid + 1] = 1.0 / d;
  }
}

}  // namespace

PrepField prep_field(bm_plan_s& p, const double* block_tol, const QPrep& q) {
  PrepField f{};
  const double eta = p.cfg.eta;
  const std::vector<double> w = level_weights(p);
  f.L = p.L;
  f.M = p.M;
  f.nlev = p.nlev;
  f.nested = p.cfg.nested;
  if (p.nlev + 1 > 26) fail(BM_EUNSUPPORTED, "too many levels");
  for (int s = 1; s <= p.L; ++s) {
    f.tau[s - 1] = s == 1 ? block_tol : p.ws.tolbuf + p.ws.tol_off[s];
    for (int d = 0; d < 3; ++d) f.nb[s - 1][d] = p.lv[s - 1].nb[d];
    f.kap[s - 1] = q.lv[s - 1].kap;
    f.tab[s - 1] = q.lv[s - 1];
    f.tab[s - 1].tau = nullptr;
  }
  if (p.L == 0) f.tau[0] = block_tol;
  f.kapc = (2.0 * (1.0 - eta)) * w[p.nlev];
  f.tab[kCoarseSlotHost] = q.lv[kCoarseSlotHost];
  f.tab[kCoarseSlotHost].tau = nullptr;   // (the record holds no map pointer of its own)
  f.tg = p.ws.tolbuf + p.ws.tol_off[p.L + 1];
  f.q = p.ws.qparam;
  for (int s = 1; s <= p.nlev; ++s) f.kq[s - 1] = (2.0 * (1.0 - eta)) * w[s - 1] / p.lv[s - 1].gain;
  f.kq[p.nlev] = (2.0 * (1.0 - eta)) * w[p.nlev];
  f.flag = q.flag;
  return f;
}

void launch_prep_batch(const PrepStages& g, const PrepField* F, int nf, const double* map, bool clear_flag,
                       hipStream_t st) {
  for (int s = 1; s < 9; ++s)
    if (g.prop_n[s] > 0)
      hipLaunchKernelGGL(k_batch_propagate, dim3(grid_for(g.prop_n[s])), dim3(NT), 0, st, F, g.prop_first[s], nf,
                         g.prop_n[s], s, map);
  if (g.fields)
    hipLaunchKernelGGL(k_batch_prep, dim3(unsigned(nf)), dim3(kScalarNT), 0, st, F, map, g.prop_n[1] > 0 ? 0 : 1,
                       clear_flag ? 1 : 0);
  for (int s = 0; s < 9; ++s)
    if (g.tab_n[s] > 0)
      hipLaunchKernelGGL(k_batch_tables, dim3(grid_for(g.tab_n[s])), dim3(NT), 0, st, F, g.tab_first[s], nf,
                         g.tab_n[s], s, map);
  BM_HIP(hipGetLastError());
}

namespace {

QArgs prepare(bm_plan_s& p, const double* block_tol, hipStream_t st, bool tables = true, bool clear_flag = true) {
  const QPrep qp = tables ? quant_prepare(p, block_tol, st, clear_flag) : qprep_layout(p, block_tol);
  QArgs a{};
  const int64_t npad = prod3(p.pdims);
  if (npad >= (int64_t(1) << 32)) fail(BM_EUNSUPPORTED, "quantizer: padded grid of 2^32 nodes or more");
  a.tot = uint32_t(npad);
  a.uf = Unflat32(p.pdims[1], p.pdims[2]);
  for (int d = 0; d < 3; ++d) {
    int D = 0;
    for (auto& L : p.lv) D += L.coarsen[d] ? 1 : 0;
    a.D[d] = D;
  }
  a.L = p.L;
  a.M = p.M;
  a.lw = 0;
  if (p.L > 0)
    while ((1 << a.lw) < p.cfg.block - 1) ++a.lw;
  a.nested = p.cfg.nested;
  a.counters = p.ws.counters;
  for (int k = 0; k < 9; ++k) {
    a.cdel[k] = qp.lv[k].cdel;
    a.cinv[k] = qp.lv[k].cinv;
    for (int d = 0; d < 3; ++d) a.nb[k][d] = uint32_t(qp.lv[k].nb[d]);
  }
  a.q = qp.q;
  return a;
}

}  // namespace

void tolmap_from_boxes(bm_plan_s& p, const double* boxes, int nbox, double background, double* block_tol,
                       hipStream_t st) {
  if (nbox < 0 || (nbox > 0 && !boxes)) fail(BM_EINVAL, "bad box list");
  if (!(background > 0) || !std::isfinite(background)) fail(BM_ENONFINITE, "background tolerance must be positive and finite");
  for (int j = 0; j < nbox; ++j)
    if (!(boxes[7 * j + 6] > 0) || !std::isfinite(boxes[7 * j + 6])) fail(BM_ENONFINITE, "box tolerance must be positive and finite");
  if (nbox > kMaxBoxes) fail(BM_EINVAL, "at most 4096 boxes");
  BoxArgs a{nullptr, nbox, background, {p.dims[0], p.dims[1], p.dims[2]}, {p.nb1[0], p.nb1[1], p.nb1[2]},
            p.L > 0 ? p.cfg.block - 1 : 0, block_tol};
  const dim3 g(grid_for(prod3(p.nb1)));
  if (nbox <= kArgBoxes && (nbox == 0 || !capturing(st))) {
    BoxList l{};
    std::copy(boxes, boxes + 7 * nbox, l.r);
    hipLaunchKernelGGL(k_tol_boxes<true>, g, dim3(NT), 0, st, a, l);
    BM_HIP(hipGetLastError());
    return;
  }
  // the caller's list goes through pinned staging; the call then waits for
  // the copy so the staging buffer can be reused
  if (!p.ws.boxhost)
    BM_HIP(hipHostMalloc(&p.ws.boxhost, size_t(kMaxBoxes) * 7 * sizeof(double), hipHostMallocDefault));
  std::copy(boxes, boxes + 7 * nbox, p.ws.boxhost);
  BM_HIP(hipMemcpyAsync(p.ws.boxbuf, p.ws.boxhost, size_t(nbox) * 7 * sizeof(double), hipMemcpyHostToDevice, st));
  a.boxes = p.ws.boxbuf;
  hipLaunchKernelGGL(k_tol_boxes<false>, g, dim3(NT), 0, st, a, BoxList{});
  BM_HIP(hipGetLastError());
  BM_HIP(hipStreamSynchronize(st));
}

void tolmap_from_voxels(bm_plan_s& p, const double* voxel_tol, double* block_tol, hipStream_t st) {
  if (p.L > 0) {
    VoxArgs a{voxel_tol, {p.dims[0], p.dims[1], p.dims[2]}, {p.nb1[0], p.nb1[1], p.nb1[2]}, p.cfg.block - 1, block_tol};
    hipLaunchKernelGGL(k_tol_voxels, dim3(unsigned(prod3(p.nb1))), dim3(NT), 0, st, a);
  } else {
    hipLaunchKernelGGL(k_fill, dim3(1), dim3(NT), 0, st, block_tol, int64_t(1), double(INFINITY));
    hipLaunchKernelGGL(k_min_all, dim3(grid_for(prod3(p.dims))), dim3(NT), 0, st, voxel_tol, prod3(p.dims), block_tol);
  }
  BM_HIP(hipGetLastError());
}

void quantize(bm_plan_s& p, const void* coeff, const double* block_tol, int32_t* codes, bm_qstats* stats,
              hipStream_t st) {
  const int64_t tot = prod3(p.pdims);
  {
    TimedScope ts(p, 2 * p.nlev, st);
    QArgs a = prepare(p, block_tol, st);
    const unsigned g = qgroups(a.tot);
    int64_t* partials = p.ws.counters + 16;
    if (p.cfg.dtype == BM_F32)
      hipLaunchKernelGGL(k_quantize<float>, dim3(g), dim3(NT), 0, st, a, static_cast<const float*>(coeff), codes,
                         partials);
    else
      hipLaunchKernelGGL(k_quantize<double>, dim3(g), dim3(NT), 0, st, a, static_cast<const double*>(coeff), codes,
                         partials);
    hipLaunchKernelGGL(k_reduce_stats, dim3(1), dim3(NT), 0, st, partials, int(g), p.ws.counters);
    BM_HIP(hipGetLastError());
  }
  if (stats) {
    int64_t h[4];
    BM_HIP(hipMemcpyAsync(h, p.ws.counters, sizeof(h), hipMemcpyDeviceToHost, st));
    BM_HIP(hipStreamSynchronize(st));
    stats->n_codes = tot;
    stats->n_outliers = h[0];
    stats->max_abs_code = h[1];
    check_code_flag(h[2], "tolerance too small for the data");
  }
}

void dequantize(bm_plan_s& p, const int32_t* codes, const double* block_tol, void* coeff, hipStream_t st) {
  TimedScope ts(p, 2 * p.nlev + 1, st);
  QArgs a = prepare(p, block_tol, st, true, false);
  const int64_t tot = prod3(p.pdims);
  (void)tot;
  const unsigned g = qgroups(a.tot);
  if (p.cfg.dtype == BM_F32)
    hipLaunchKernelGGL(k_dequantize<float>, dim3(g), dim3(NT), 0, st, a, codes, static_cast<float*>(coeff));
  else
    hipLaunchKernelGGL(k_dequantize<double>, dim3(g), dim3(NT), 0, st, a, codes, static_cast<double*>(coeff));
  BM_HIP(hipGetLastError());
}

int64_t qoi_deltas(bm_plan_s& p, const void* g, double tol_q, const double* block_tol, double* delta,
                   hipStream_t st) {
  if (!(tol_q > 0) || !std::isfinite(tol_q)) fail(BM_ENONFINITE, "tol_q must be positive and finite");
  const size_t npad = size_t(prod3(p.pdims));
  if (!p.ws.coeff) plan_alloc(p, &p.ws.coeff, npad * p.esize);
  // sensitivities s = R^T g of the quantity to the coefficients
  recompose_adjoint(p, g, p.ws.coeff, st);
  QArgs a = prepare(p, block_tol, st);
  const bool f32 = p.cfg.dtype == BM_F32;
  auto* q = reinterpret_cast<QoiScratch*>(p.ws.counters + 16);
  auto* cnt = reinterpret_cast<unsigned long long*>(p.ws.counters + 3);
  const unsigned gs = std::min<unsigned>(grid_for(int64_t(a.tot)), unsigned(kQoiGroups));
  hipLaunchKernelGGL(k_qoi_begin, dim3(1), dim3(64), 0, st, q, (1.0 - p.cfg.eta) * tol_q, double(a.tot), cnt);
  // (the kept shares wait in delta until the last pass)
  if (f32)
    hipLaunchKernelGGL(k_qoi_shares<float>, dim3(gs), dim3(NT), 0, st, a, static_cast<const float*>(p.ws.coeff),
                       delta, q);
  else
    hipLaunchKernelGGL(k_qoi_shares<double>, dim3(gs), dim3(NT), 0, st, a, static_cast<const double*>(p.ws.coeff),
                       delta, q);
  hipLaunchKernelGGL(k_qoi_step, dim3(1), dim3(1024), 0, st, q, int(gs), 1);
  BM_HIP(hipGetLastError());
  const unsigned gq = qgroups(a.tot);
  for (;;) {   // (a search that has not ended after its passes leaves delta to more of them)
    for (int pass = 0; pass < kQoiPasses; ++pass) {
      hipLaunchKernelGGL(k_qoi_eval, dim3(gs), dim3(NT), 0, st, delta, q);
      hipLaunchKernelGGL(k_qoi_step, dim3(1), dim3(1024), 0, st, q, int(gs), 0);
    }
    if (f32)
      hipLaunchKernelGGL(k_qoi_final<float>, dim3(gq), dim3(NT), 0, st, a, static_cast<const float*>(p.ws.coeff), q,
                         delta, cnt);
    else
      hipLaunchKernelGGL(k_qoi_final<double>, dim3(gq), dim3(NT), 0, st, a, static_cast<const double*>(p.ws.coeff), q,
                         delta, cnt);
    BM_HIP(hipGetLastError());
    unsigned long long nset = 0;
    int done = 0;
    BM_HIP(hipMemcpyAsync(&nset, cnt, sizeof(nset), hipMemcpyDeviceToHost, st));
    BM_HIP(hipMemcpyAsync(&done, &q->st.done, sizeof(done), hipMemcpyDeviceToHost, st));
    BM_HIP(hipStreamSynchronize(st));
    if (done) return int64_t(nset);
  }
}

void quantize_delta(bm_plan_s& p, const void* coeff, const double* delta, int32_t* codes, bm_qstats* stats,
                    hipStream_t st) {
  QArgs a = prepare(p, nullptr, st, false);
  a.pdel = delta;
  const unsigned g = qgroups(a.tot);
  int64_t* partials = p.ws.counters + 16;
  if (p.cfg.dtype == BM_F32)
    hipLaunchKernelGGL(k_quantize<float>, dim3(g), dim3(NT), 0, st, a, static_cast<const float*>(coeff), codes, partials);
  else
    hipLaunchKernelGGL(k_quantize<double>, dim3(g), dim3(NT), 0, st, a, static_cast<const double*>(coeff), codes,
                       partials);
  BM_HIP(hipGetLastError());
  if (stats) {
    hipLaunchKernelGGL(k_reduce_stats, dim3(1), dim3(NT), 0, st, partials, int(g), p.ws.counters);
    BM_HIP(hipGetLastError());
    int64_t h[4];
    BM_HIP(hipMemcpyAsync(h, p.ws.counters, sizeof(h), hipMemcpyDeviceToHost, st));
    BM_HIP(hipStreamSynchronize(st));
    stats->n_codes = int64_t(a.tot);
    stats->n_outliers = h[0];
    stats->max_abs_code = h[1];
    check_code_flag(h[2], "Delta too small for the data");
  }
}

void dequantize_delta(bm_plan_s& p, const int32_t* codes, const double* delta, void* coeff, hipStream_t st) {
  QArgs a = prepare(p, nullptr, st, false);
  a.pdel = delta;
  const unsigned g = qgroups(a.tot);
  if (p.cfg.dtype == BM_F32)
    hipLaunchKernelGGL(k_dequantize<float>, dim3(g), dim3(NT), 0, st, a, codes, static_cast<float*>(coeff));
  else
    hipLaunchKernelGGL(k_dequantize<double>, dim3(g), dim3(NT), 0, st, a, codes, static_cast<double*>(coeff));
  BM_HIP(hipGetLastError());
}

}  // namespace bm
