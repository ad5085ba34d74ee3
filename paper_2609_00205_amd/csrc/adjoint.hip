// Transposes of the multilevel transform: D^T (decompose) and R^T
// (recompose), level by level in the reverse order of the forward map.  They
// give gradients through the transform and the coefficient sensitivities of
// a quantity of interest.
//
// One decomposition level (Sec. II-B) on a grid F with coarse nodes C maps u
// to  w = (I - P3 S) u on the fine-only nodes and  c = S u + K3 w on C,
// with S the selection of C, P3 the multilinear interpolation and
// K3 = (Mc^{-1} P^T M) per axis.  Its transpose takes (g on F\C, cbar on C) to
//   fine-only nodes:  v = g + K3^T cbar        (K^T = M P Mc^{-1} per axis)
//   coarse nodes:     cbar - P3^T v0           (v0 = v with zeros on C).
// One recomposition level u = P3 (c - K3 w) + w has the transpose
//   coarse nodes:     r = P3^T g,
//   fine-only nodes:  g - K3^T r.
// K^T along one axis is a solve with Mc followed by the transposed rows of
// P^T M (a spread from m to n nodes); P3^T is a gather over the 3^3
// neighbourhood of each coarse node with weights 1, 1/2, 1/4, 1/8.
//
// Block levels (Sec. IV-A, face-fixed): every block applies the transpose of
// its own level to the values of the nodes it owns and adds the result into
// every node it covers, shared faces included.  The order in which the up to
// eight contributions of a shared node are summed is fixed: by the parity
// class of the contributing block, even before odd, z slowest.  The blocks of
// a slab (a few layers along z, of a strip along y and x where a layer is too
// large) leave their contributions, b^3 values each, in a scratch array; a
// second launch sums them node by node in that order.  HBM traffic is what
// bounds a level, and a slab's scratch is kept small enough to stay in the
// 256 MB Infinity Cache between its two launches.
// (As 8 launches, one per parity class, that added into the grid in place,
// every line was fetched and written several times: 384 x 384 x 256 FP32
// 0.324 ms, now 0.18 ms.)  The transpose of the clamp padding adds the
// gradient of every padded node into the node it copied.

#include <algorithm>

#include "adjoint_slab.h"
#include "block.h"
#include "internal.h"
#include "line_solve.h"

namespace bm {
namespace {

constexpr int NT = 256;

inline unsigned grid_for(int64_t tot) {
  int64_t g = (tot + NT - 1) / NT;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return unsigned(g);
}

// --------------------------------------------------------------- block levels

// K_D^T on one line of a face-fixed block: s = Mc_I^{-1} y on the MI interior
// coarse nodes (3 Mc_I = tridiag(1, 4, 1)), then the transposed interior rows
// of P^T M ({1/12, 1/2, 5/6, 1/2, 1/12} around node 2J+2) spread s over the B
// nodes of the line.  SPLIT: the last term of a coarse node's sum is a product
// rounded on its own (else contracted): the z spread of a recomposition's
// transpose, whose bits set the widths of a quantity of interest and with
// them its codes, has that rounding.
template <typename T>
__device__ inline T add_product(T acc, T a, T b) {
#pragma clang fp contract(off)
  return acc + a * b;
}

template <typename T, int B, bool SPLIT = false>
__device__ inline void solve_spread(const T (&yv)[Geo<B>::MI], T (&out)[B]) {
  constexpr int MI = Geo<B>::MI;
  constexpr Pivots<MI> P{};
  T d[MI], s[MI];
#pragma unroll
  for (int J = 0; J < MI; ++J) d[J] = J == 0 ? T(3) * yv[0] * T(P.v[0]) : (T(3) * yv[J] - d[J - 1]) * T(P.v[J]);
  s[MI - 1] = d[MI - 1];
#pragma unroll
  for (int J = MI - 2; J >= 0; --J) s[J] = d[J] - T(P.v[J]) * s[J + 1];
  const T C0 = T(5.0 / 6.0), C1 = T(0.5), C2 = T(1.0 / 12.0);
#pragma unroll
  for (int i = 0; i < B; ++i) out[i] = T(0);
#pragma unroll
  for (int J = 0; J < MI; ++J) {
    const int c = 2 * J + 2;
    if (SPLIT)
      out[c - 2] = add_product(out[c - 2], C2, s[J]);
    else
      out[c - 2] += C2 * s[J];
    out[c - 1] += C1 * s[J];
    out[c] += C0 * s[J];
    out[c + 1] += C1 * s[J];
    out[c + 2] += C2 * s[J];
  }
}

// Transposed passes x, y (LDS lines) and z (registers) of K_D^T:
// Z[J][I][K] -> T2[J][I][x] -> T1[J][y][x] -> t[z] of column tb.
template <typename T, int B>
__device__ inline void kd_transpose_xy(const T* Z, T* T2, T* T1, int tb, bool act) {
  constexpr int MI = Geo<B>::MI, BB = Geo<B>::BB;
  if (act && tb < MI * MI) {
    T l[MI], o[B];
#pragma unroll
    for (int K = 0; K < MI; ++K) l[K] = Z[tb * MI + K];
    solve_spread<T, B>(l, o);
#pragma unroll
    for (int x = 0; x < B; ++x) T2[tb * B + x] = o[x];
  }
  __syncthreads();
  if (act && tb < MI * B) {
    const int J = tb / B, x = tb - (tb / B) * B;
    T l[MI], o[B];
#pragma unroll
    for (int I = 0; I < MI; ++I) l[I] = T2[(J * MI + I) * B + x];
    solve_spread<T, B>(l, o);
#pragma unroll
    for (int y = 0; y < B; ++y) T1[J * BB + y * B + x] = o[y];
  }
  __syncthreads();
}

// z part of P3^T at the even planes of one column: R[j] = v[2j] + (v[2j-1] + v[2j+1]) / 2
// (skip: with v[2j] taken as zero)
template <typename T, int B>
__device__ inline void restrict_z(const T (&v)[B], T* R, int tb, bool skip) {
  constexpr int MC = Geo<B>::MC, BB = Geo<B>::BB;
#pragma unroll
  for (int j = 0; j < MC; ++j) {
    T r = skip ? T(0) : v[2 * j];
    if (j > 0 && j < MC - 1)
      r += T(0.5) * (v[2 * j - 1] + v[2 * j + 1]);
    else if (j > 0)
      r += T(0.5) * v[2 * j - 1];
    else
      r += T(0.5) * v[2 * j + 1];
    R[j * BB + tb] = r;
  }
}

// y and x parts of P3^T at the coarse nodes of an even column (y, x)
template <typename T, int B>
__device__ inline T gather_yx(const T* R, int j, int y, int x) {
  constexpr int BB = Geo<B>::BB;
  const T* pl = R + j * BB;
  T acc = pl[y * B + x];
  T side = T(0), corner = T(0);
  if (y > 0) side += pl[(y - 1) * B + x];
  if (y < B - 1) side += pl[(y + 1) * B + x];
  if (x > 0) side += pl[y * B + x - 1];
  if (x < B - 1) side += pl[y * B + x + 1];
  if (y > 0 && x > 0) corner += pl[(y - 1) * B + x - 1];
  if (y > 0 && x < B - 1) corner += pl[(y - 1) * B + x + 1];
  if (y < B - 1 && x > 0) corner += pl[(y + 1) * B + x - 1];
  if (y < B - 1 && x < B - 1) corner += pl[(y + 1) * B + x + 1];
  return acc + T(0.5) * side + T(0.25) * corner;
}

// One slab of a level's blocks, from block o on, s per axis, and its scratch:
// block (bz, by, bx) leaves its B^3 contributions in slot (bz mod ring, by,
// bx) of rows of s[2] and layers of s[1] rows: the kernels' pointer to the
// scratch lies where block (., 0, 0) would be.
struct Slab {
  int64_t nb[3];          // blocks per axis of the level
  int64_t o[3], s[3];     // first block of the slab, blocks per axis
  int64_t nblocks;
  int64_t nwg, per;
  uint32_t ring;
  FastDiv fs2, fs1, fring;
  __device__ inline int64_t slot(int64_t bz, int64_t by, int64_t bx) const {
    const uint32_t r = uint32_t(bz) - fring.div(uint32_t(bz)) * ring;
    return (int64_t(r) * s[1] + by) * s[2] + bx;
  }
  // block k of the slab
  __device__ inline void block(int64_t k, int64_t& bz, int64_t& by, int64_t& bx) const {
    block_coords(uint32_t(k), fs2, fs1, s, bz, by, bx);
    bz += o[0];
    by += o[1];
    bx += o[2];
  }
};

template <typename T>
struct BlockTArgs {
  // decomposition: gradient of the coefficients, this level's view, and of
  // the coarse grid G^s (compact, dims cn)
  const T* gc;
  int64_t cs[3];
  const T* gcur;
  int64_t cn[3];
  // recomposition: gradient of G^{s-1} (dense, dims in; zero at or beyond lim)
  const T* gin;
  int64_t in[3], lim[3];
  T* part;                // contributions [slot][B][B][B]
  Slab sl;
};

// The element `lane` past a base that all lanes of a workgroup share: the
// base stays in scalar registers and every access of a column takes the same
// lane offset, where a pointer per lane and plane costs two vector registers
// each.  64 bits: from 2^25 doubles or 2^26 floats a row on, the byte offset
// of a block's last row does not fit in 32 (which take the same registers and
// time).
template <typename T>
__device__ inline T* lane_at(T* base, uint64_t lane) {
  return reinterpret_cast<T*>(reinterpret_cast<uintptr_t>(base) + lane * sizeof(T));
}

// A workgroup's block for this lane (several 9^3 blocks share a workgroup).
template <int B>
struct BlockLane {
  static constexpr int NB = Geo<B>::NB1, BB = B * B, NT = (NB * BB + 63) / 64 * 64;
  int bl, tb, y, x;
  bool act, ecol;
  int64_t bz, by, bx;
  __device__ inline BlockLane(const Slab& sl, int64_t g) {
    const int tid = threadIdx.x;
    bl = NB == 1 ? 0 : tid / BB;          // (one block: its coordinates are scalars)
    tb = tid - bl * BB;
    act = NB == 1 ? tid < BB : bl < NB && g * NB + bl < sl.nblocks;
    const int64_t blk = NB == 1 || act ? g * NB + bl : 0;
    sl.block(blk, bz, by, bx);
    if (NB > 1 && bl >= NB) bl = 0;
    y = tb / B;
    x = tb - (tb / B) * B;
    ecol = ((y | x) & 1) == 0;
  }
};

template <typename T, int B>
__global__ __launch_bounds__(BlockLane<B>::NT) void k_local_decompose_T(BlockTArgs<T> a) {
  using G = Geo<B, sizeof(T)>;
  constexpr int BB = G::BB, MC = G::MC, MI = G::MI;
  __shared__ T lds[BlockLane<B>::NB * G::ADJ_LDS];
  const int64_t g = xcd_group(blockIdx.x, a.sl.per);
  if (g >= a.sl.nwg) return;
  const BlockLane<B> k(a.sl, g);
  const int tb = k.tb, y = k.y, x = k.x;
  const bool act = k.act, ecol = k.ecol;
  T* T1 = lds + k.bl * G::ADJ_LDS;                   // [MI][B][B]
  T* T2 = T1 + MI * BB;                              // [MI][MI][B]
  T* Z = T2 + MI * MI * B;                           // [MI][MI][MI]
  T* R = T1;                                         // [MC][B][B], once T1 and T2 are dead
  const int64_t oz = k.bz * (B - 1), oy = k.by * (B - 1), ox = k.bx * (B - 1);
  // the gradient on the nodes this block owns (zero elsewhere)
  T v[B];
  if (act) {
    const bool own_yx = (y < B - 1 || k.by == a.sl.nb[1] - 1) && (x < B - 1 || k.bx == a.sl.nb[2] - 1);
    const bool lastz = k.bz == a.sl.nb[0] - 1;
    const int64_t cpl = a.cn[1] * a.cn[2];
    const T* col = a.gc + oz * a.cs[0] + oy * a.cs[1] + ox * a.cs[2];
    const T* ccol = a.gcur + (oz >> 1) * cpl + (oy >> 1) * a.cn[2] + (ox >> 1);
    const uint64_t l = y * a.cs[1] + x * a.cs[2];
    const uint64_t cl = (y >> 1) * a.cn[2] + (x >> 1);
#pragma unroll
    for (int z = 0; z < B; ++z) {
      T w = T(0);
      if (own_yx && (z < B - 1 || lastz))
        w = (ecol && !(z & 1)) ? *lane_at(ccol + (z >> 1) * cpl, cl) : *lane_at(col + z * a.cs[0], l);
      v[z] = w;
    }
    if (ecol && y >= 2 && y <= B - 3 && x >= 2 && x <= B - 3) {
      const int I = (y - 2) >> 1, K = (x - 2) >> 1;
#pragma unroll
      for (int J = 0; J < MI; ++J) Z[(J * MI + I) * MI + K] = v[2 * J + 2];
    }
  }
  __syncthreads();
  kd_transpose_xy<T, B>(Z, T2, T1, tb, act);
  if (act) {
    T l[MI], t[B];
#pragma unroll
    for (int J = 0; J < MI; ++J) l[J] = T1[J * BB + tb];
    solve_spread<T, B>(l, t);
    // v = g + t on the fine nodes; the coarse ones keep cbar, which P3^T
    // leaves out
#pragma unroll
    for (int z = 0; z < B; ++z)
      if (!(ecol && !(z & 1))) v[z] = v[z] + t[z];
    // R aliases T1 (this column only, read above) and the dead T2 / Z
    restrict_z<T, B>(v, R, tb, ecol);
  }
  __syncthreads();
  if (act) {
    if (ecol) {
#pragma unroll
      for (int j = 0; j < MC; ++j) v[2 * j] = v[2 * j] - gather_yx<T, B>(R, j, y, x);
    }
    T* dst = a.part + a.sl.slot(k.bz, k.by, k.bx) * (B * BB);
#pragma unroll
    for (int z = 0; z < B; ++z) *lane_at(dst + z * BB, uint32_t(tb)) = v[z];
  }
}

template <typename T, int B>
__global__ __launch_bounds__(BlockLane<B>::NT) void k_local_recompose_T(BlockTArgs<T> a) {
  using G = Geo<B, sizeof(T)>;
  constexpr int BB = G::BB, MC = G::MC, MI = G::MI;
  __shared__ T lds[BlockLane<B>::NB * G::ADJ_LDS];
  const int64_t g = xcd_group(blockIdx.x, a.sl.per);
  if (g >= a.sl.nwg) return;
  const BlockLane<B> k(a.sl, g);
  const int tb = k.tb, y = k.y, x = k.x;
  const bool act = k.act, ecol = k.ecol;
  T* T1 = lds + k.bl * G::ADJ_LDS;
  T* T2 = T1 + MI * BB;
  T* Z = T2 + MI * MI * B;
  T* R = T1;
  const int64_t oz = k.bz * (B - 1), oy = k.by * (B - 1), ox = k.bx * (B - 1);
  T gv[B];
  if (act) {
    const bool own_yx = (y < B - 1 || k.by == a.sl.nb[1] - 1) && (x < B - 1 || k.bx == a.sl.nb[2] - 1) &&
                        oy + y < a.lim[1] && ox + x < a.lim[2];
    const bool lastz = k.bz == a.sl.nb[0] - 1;
    const int64_t pl = a.in[1] * a.in[2];
    const T* col = a.gin + oz * pl + oy * a.in[2] + ox;
    const uint64_t l = y * a.in[2] + x;
#pragma unroll
    for (int z = 0; z < B; ++z)
      gv[z] = (own_yx && (z < B - 1 || lastz) && oz + z < a.lim[0]) ? *lane_at(col + z * pl, l) : T(0);
    restrict_z<T, B>(gv, R, tb, false);
  }
  __syncthreads();
  T rc[MC];
  if (act && ecol) {
#pragma unroll
    for (int j = 0; j < MC; ++j) rc[j] = gather_yx<T, B>(R, j, y, x);
  }
  __syncthreads();
  if (act && ecol && y >= 2 && y <= B - 3 && x >= 2 && x <= B - 3) {
    const int I = (y - 2) >> 1, K = (x - 2) >> 1;
#pragma unroll
    for (int J = 0; J < MI; ++J) Z[(J * MI + I) * MI + K] = rc[J + 1];
  }
  __syncthreads();
  kd_transpose_xy<T, B>(Z, T2, T1, tb, act);
  if (act) {
    T l[MI], t[B];
#pragma unroll
    for (int J = 0; J < MI; ++J) l[J] = T1[J * BB + tb];
    solve_spread<T, B, true>(l, t);
    T* dst = a.part + a.sl.slot(k.bz, k.by, k.bx) * (B * BB);
#pragma unroll
    for (int z = 0; z < B; ++z)
      *lane_at(dst + z * BB, uint32_t(tb)) = (ecol && !(z & 1)) ? rc[z >> 1] : gv[z] - t[z];
  }
}

// Where a node's summed gradient goes.  REC (coefficients of a recomposition
// level): coarse nodes (every coordinate even) into the compact coarse grid
// b, the others into the level view a.  Otherwise (gradient of G^{s-1}):
// nodes below lim on every axis into a, the others into b (the padded grid,
// at the padded strides; null: dropped).
template <typename T>
struct NodeOut {
  T* a;
  int64_t as[3];
  T* b;
  int64_t bs[3];
  int64_t lim[3];
};

template <typename T>
struct SumArgs {
  const T* part;
  Slab sl;
  NodeOut<T> out;
  // first node of the slab's own; y0 in groups of kSumR rows: that y is a
  // multiple of kSumR there settles at compile time which rows can lie on a
  // face (0.254 against 0.236 ms for 384 x 384 x 256 FP32)
  uint32_t z0, y0, x0;
  uint32_t n1, n2;        // rows and columns end here
  uint32_t ntask;         // wavefront tasks: kSumR rows of one plane, 64 nodes of each
  Unflat32 uf;            // task -> (plane, group of rows, 64 nodes)
};

// the blocks along one axis that cover node c, even block first: block and
// local coordinate; returns how many
template <int B>
__device__ inline int cover(uint32_t c, int64_t nb, int (&blk)[2], int (&loc)[2]) {
  const uint32_t f = c / (B - 1);
  const int l = int(c - f * (B - 1));
  blk[0] = int(f);
  loc[0] = l;
  blk[1] = loc[1] = 0;
  if (l != 0 || f == 0) return 1;
  if (f == uint32_t(nb)) {
    blk[0] = int(f) - 1;
    loc[0] = B - 1;
    return 1;
  }
  const bool odd = f & 1;                // block f is odd: block f-1 comes first
  blk[0] = int(f) - odd;
  loc[0] = odd ? B - 1 : 0;
  blk[1] = int(f) - !odd;
  loc[1] = odd ? 0 : B - 1;
  return 2;
}

// A wavefront sums 64 nodes of kSumR neighbouring rows: what depends on z and
// y (the blocks of a row, its place in the output) is scalar, what depends on
// x is formed once for all rows, and the first contributions of all rows are
// fetched before any other.  One lane per node with all of that per node was
// bound by its index arithmetic: the 15 M nodes of a slab of 113 x 513 x 513
// 53 us, 37 to 41 us this way.
constexpr int kSumR = 4;

template <typename T, int B, bool REC>
__global__ __launch_bounds__(NT) void k_block_sum(SumArgs<T> a) {
  constexpr int64_t B3 = int64_t(B) * B * B;
  const uint32_t nwg = (a.ntask + NT / 64 - 1) / (NT / 64);
  const uint32_t g = uint32_t(xcd_group(blockIdx.x, (nwg + 7) / 8));
  const uint32_t w = __builtin_amdgcn_readfirstlane(g * (NT / 64) + (threadIdx.x >> 6));
  if (w >= a.ntask) return;
  uint32_t z, yg, seg;
  a.uf(w, z, yg, seg);
  z += a.z0;
  const uint32_t x = a.x0 + seg * 64 + (threadIdx.x & 63);
  const bool in = x < a.n2;
  int bx[2], lx[2], by[2], ly[2], bz[2], lz[2];
  const bool two = cover<B>(in ? x : a.x0, a.sl.nb[2], bx, lx) > 1;
  const int64_t o0 = bx[0] * B3 + lx[0], o1 = bx[1] * B3 + lx[1];
  const int nz = cover<B>(z, a.sl.nb[0], bz, lz);
  // a row of a block row's contributions at node (0, iz-th z, iy-th y)
  auto row = [&](int iz, int iy) {
    return a.part + a.sl.slot(bz[iz], by[iy], 0) * B3 + (lz[iz] * B + ly[iy]) * B;
  };
  const uint32_t y0 = (a.y0 + yg) * kSumR;
  T acc[kSumR], v1[kSumR];
#pragma unroll
  for (int r = 0; r < kSumR; ++r) {
    acc[r] = v1[r] = T(0);
    if (y0 + r >= a.n1) continue;
    cover<B>(y0 + r, a.sl.nb[1], by, ly);
    const T* p = row(0, 0);
    if (in) acc[r] = p[o0];
    if (in && two) v1[r] = p[o1];
  }
#pragma unroll
  for (int r = 0; r < kSumR; ++r) {
    const uint32_t y = y0 + r;
    if (y >= a.n1) continue;
    const int ny = cover<B>(y, a.sl.nb[1], by, ly);
    if (two) acc[r] += v1[r];
    auto add = [&](int iz, int iy) {
      const T* p = row(iz, iy);
      if (in) {
        acc[r] += p[o0];
        if (two) acc[r] += p[o1];
      }
    };
    if (ny > 1) add(0, 1);
    if (nz > 1) {
      add(1, 0);
      if (ny > 1) add(1, 1);
    }
    if (!in) continue;
    const NodeOut<T>& o = a.out;
    if (REC) {
      if (((z | y) & 1) == 0 && (x & 1) == 0)
        o.b[(z >> 1) * o.bs[0] + (y >> 1) * o.bs[1] + (x >> 1)] = acc[r];
      else
        o.a[z * o.as[0] + y * o.as[1] + x * o.as[2]] = acc[r];
    } else if (z < o.lim[0] && y < o.lim[1] && x < o.lim[2]) {
      o.a[z * o.as[0] + y * o.as[1] + x] = acc[r];
    } else if (o.b) {
      o.b[z * o.bs[0] + y * o.bs[1] + x] = acc[r];
    }
  }
}

// Runs a level slab by slab (slab_cut): blocks(slab) launches what leaves the
// contributions of the slab's blocks in the plan's scratch (kept; sized for
// the largest level on first use), then the slab's own nodes are summed.
template <typename T, int B, bool REC, typename F>
void run_slabs(bm_plan_s& p, int s, const NodeOut<T>& out, int per_wg, hipStream_t st, F blocks) {
  const Level& L = p.lv[s - 1];
  if (!p.ws.contrib) {
    size_t need = 0;
    for (const Level& l : p.lv)
      if (l.local)
        need = std::max(need, size_t(slab_cut(l.nb, l.b, p.esize).blocks()) * l.b * l.b * l.b * p.esize);
    plan_alloc_late(p, &p.ws.contrib, need);
  }
  const SlabCut c = slab_cut(L.nb, B, p.esize);
  // nodes of blocks [lo, hi): up to the next one's first, the far face with the last
  auto first = [](int64_t lo) { return uint32_t(lo * (B - 1)); };
  auto end = [&](int a, int64_t hi) { return hi == L.nb[a] ? L.n[a] : hi * (B - 1); };
  for (int64_t ky = 0; ky * c.cut[0] < L.nb[1]; ++ky)
    for (int64_t kx = 0; kx * c.cut[1] < L.nb[2]; ++kx) {
      const BlockRange y = strip(L.nb[1], c.cut[0], ky), x = strip(L.nb[2], c.cut[1], kx);
      for (int64_t k0 = 0; k0 < L.nb[0]; k0 += c.layers) {
        const int64_t k1 = std::min(L.nb[0], k0 + c.layers);
        Slab sl{};
        for (int k = 0; k < 3; ++k) sl.nb[k] = L.nb[k];
        sl.o[0] = k0;
        sl.o[1] = y.run;
        sl.o[2] = x.run;
        sl.s[0] = k1 - k0;
        sl.s[1] = y.hi - y.run;
        sl.s[2] = x.hi - x.run;
        sl.nblocks = sl.s[0] * sl.s[1] * sl.s[2];
        sl.nwg = (sl.nblocks + per_wg - 1) / per_wg;
        sl.per = (sl.nwg + 7) / 8;
        sl.ring = uint32_t(c.ring);
        sl.fring = FastDiv(uint32_t(c.ring));
        sl.fs2 = FastDiv(uint32_t(sl.s[2]));
        sl.fs1 = FastDiv(uint32_t(sl.s[1]));
        T* const part = reinterpret_cast<T*>(reinterpret_cast<intptr_t>(p.ws.contrib) -
                                             (sl.o[1] * sl.s[2] + sl.o[2]) * int64_t(B) * B * B * int64_t(sizeof(T)));
        blocks(sl, part);
        BM_HIP(hipGetLastError());
        const int64_t z1 = end(0, k1), n1 = end(1, y.hi), n2 = end(2, x.hi);
        static_assert((B - 1) % kSumR == 0, "a strip's rows start a group");
        SumArgs<T> a{part, sl, out, first(k0), first(y.lo) / kSumR, first(x.lo), uint32_t(n1), uint32_t(n2), 0, {}};
        const int64_t ngy = (n1 + kSumR - 1) / kSumR - a.y0, nseg = (n2 - a.x0 + 63) / 64;
        a.ntask = uint32_t((z1 - a.z0) * ngy * nseg);   // (of a scratch full of blocks: below 2^32)
        a.uf = Unflat32(ngy, nseg);
        const unsigned nwg = (a.ntask + NT / 64 - 1) / (NT / 64);
        hipLaunchKernelGGL((k_block_sum<T, B, REC>), dim3((nwg + 7) / 8 * 8), dim3(NT), 0, st, a);
        BM_HIP(hipGetLastError());
      }
    }
}

// the outputs of a recomposition level's transpose
template <typename T>
NodeOut<T> rec_out(bm_plan_s& p, int s, void* gcoeff) {
  const Level& L = p.lv[s - 1];
  const View3 cv = level_view(p, s, gcoeff);
  NodeOut<T> o{};
  o.a = static_cast<T*>(cv.ptr);
  o.b = static_cast<T*>(p.ws.grid[s]);
  for (int k = 0; k < 3; ++k) o.as[k] = cv.s[k];
  o.bs[0] = L.m[1] * L.m[2];
  o.bs[1] = L.m[2];
  o.bs[2] = 1;
  return o;
}

template <typename T, int B>
void launch_local_dec_T(bm_plan_s& p, int s, const void* gcoeff, const NodeOut<T>& out, hipStream_t st) {
  const Level& L = p.lv[s - 1];
  BlockTArgs<T> a{};
  const View3 cv = level_view(p, s, const_cast<void*>(gcoeff));
  a.gc = static_cast<const T*>(cv.ptr);
  a.gcur = static_cast<const T*>(p.ws.grid[s]);
  for (int k = 0; k < 3; ++k) {
    a.cs[k] = cv.s[k];
    a.cn[k] = L.m[k];
  }
  run_slabs<T, B, false>(p, s, out, BlockLane<B>::NB, st, [&](const Slab& sl, T* part) {
    a.sl = sl;
    a.part = part;
    hipLaunchKernelGGL((k_local_decompose_T<T, B>), dim3(unsigned(8 * sl.per)), dim3(BlockLane<B>::NT), 0, st, a);
  });
}

template <typename T, int B>
void launch_local_rec_T(bm_plan_s& p, int s, const void* gin, const int64_t in[3], const int64_t lim[3],
                        void* gcoeff, hipStream_t st) {
  BlockTArgs<T> a{};
  a.gin = static_cast<const T*>(gin);
  for (int k = 0; k < 3; ++k) {
    a.in[k] = in[k];
    a.lim[k] = lim[k];
  }
  run_slabs<T, B, true>(p, s, rec_out<T>(p, s, gcoeff), BlockLane<B>::NB, st, [&](const Slab& sl, T* part) {
    a.sl = sl;
    a.part = part;
    hipLaunchKernelGGL((k_local_recompose_T<T, B>), dim3(unsigned(8 * sl.per)), dim3(BlockLane<B>::NT), 0, st, a);
  });
}

// ------------------------------------------------------- 33^3 block levels
// Transposes of the 33^3 block level, split like the forward kernels: a
// block is cut along x into halves, here overlapping by two columns (x in
// [0, 17] and [15, 32]) so that the transposed interpolation at the coarse
// columns next to the cut (16 and 18) has both neighbours; the first half
// stores x <= 16, the second x >= 17.  The transposed correction runs as an
// x spread per block into a scratch array (the plan's line-pass buffer),
// then the y and z spreads per half.  Halves of a block store disjoint nodes.
namespace w33 {
constexpr int B = 33, MC = 17, MI = 15, HW = 18, NCOL = B * HW, NT = 640, T2B = MI * MI * B, ZB = MI * MI * MI;
__device__ inline int x0(int h) { return h ? 15 : 0; }
__device__ inline bool stores(int h, int x) { return h ? x >= 17 : x <= 16; }
}  // namespace w33

template <typename T>
struct W33Args {
  const T* gc;            // decompose: gradient of the coefficients (level view)
  int64_t cs[3];
  const T* gcur;          // decompose: gradient of the coarse grid G^s (compact, dims cn)
  int64_t cn[3];
  const T* gin;           // recompose: gradient of G^{s-1} (dense, dims in, zero at or beyond lim)
  int64_t in[3], lim[3];
  T* zs;                  // recompose: interior coarse gradients per block [ZB]
  T* t2;                  // x-spread result per block [MI][MI][B]
  int64_t nb[3];
  T* part;                // contributions [slot][B][B][B]
  Slab sl;
};

// z part of P3^T at the even planes of a column of 33 values
template <typename T>
__device__ inline T restrict_z33(const T (&v)[w33::B], int j) {
  using namespace w33;
  T r = v[2 * j];
  if (j > 0 && j < MC - 1)
    r += T(0.5) * (v[2 * j - 1] + v[2 * j + 1]);
  else if (j > 0)
    r += T(0.5) * v[2 * j - 1];
  else
    r += T(0.5) * v[2 * j + 1];
  return r;
}

// y and x parts of P3^T at coarse node (j, y, x) from R[MC][B][HW] of half h
template <typename T>
__device__ inline T gather33(const T* R, int j, int y, int xl, int x) {
  using namespace w33;
  const T* pl = R + j * B * HW;
  auto at = [&](int yy, int dx) { return pl[yy * HW + xl + dx]; };
  T acc = at(y, 0);
  T side = T(0), corner = T(0);
  if (y > 0) side += at(y - 1, 0);
  if (y < B - 1) side += at(y + 1, 0);
  if (x > 0) side += at(y, -1);
  if (x < B - 1) side += at(y, 1);
  if (y > 0 && x > 0) corner += at(y - 1, -1);
  if (y > 0 && x < B - 1) corner += at(y - 1, 1);
  if (y < B - 1 && x > 0) corner += at(y + 1, -1);
  if (y < B - 1 && x < B - 1) corner += at(y + 1, 1);
  return acc + T(0.5) * side + T(0.25) * corner;
}

// x spread of the transposed correction, one workgroup per block: Z[MI]^3
// (from the coarse grid's interior nodes, or from zs) -> t2[MI][MI][B]
template <typename T>
__global__ __launch_bounds__(256) void k_w33_spread_x(W33Args<T> a, int from_zs) {
  using namespace w33;
  __shared__ T Z[ZB];
  int64_t bz, by, bx;                    // zs: the slab's blocks
  if (from_zs) {
    a.sl.block(blockIdx.x, bz, by, bx);
  } else {
    bx = blockIdx.x % a.nb[2];
    const int64_t t = blockIdx.x / a.nb[2];
    by = t % a.nb[1];
    bz = t / a.nb[1];
  }
  const int64_t blk = (bz * a.nb[1] + by) * a.nb[2] + bx;
  const int64_t c0 = bz * (MC - 1), c1 = by * (MC - 1), c2 = bx * (MC - 1), cpl = a.cn[1] * a.cn[2];
  for (int i = threadIdx.x; i < ZB; i += 256) {
    const int J = i / (MI * MI), r = i - J * MI * MI, I = r / MI, K = r - I * MI;
    Z[i] = from_zs ? a.zs[blk * ZB + i] : a.gcur[(c0 + J + 1) * cpl + (c1 + I + 1) * a.cn[2] + (c2 + K + 1)];
  }
  __syncthreads();
  if (threadIdx.x < MI * MI) {
    T l[MI], o[B];
#pragma unroll
    for (int K = 0; K < MI; ++K) l[K] = Z[threadIdx.x * MI + K];
    solve_spread<T, B>(l, o);
    T* dst = a.t2 + blk * T2B + threadIdx.x * B;
#pragma unroll
    for (int x = 0; x < B; ++x) dst[x] = o[x];
  }
}

// y spread of one half's columns: t2 -> T1[MI][B][HW]
template <typename T>
__device__ inline void w33_spread_y(const W33Args<T>& a, int64_t blk, int h, T* T1) {
  using namespace w33;
  const int tid = threadIdx.x;
  if (tid < MI * HW) {
    const int J = tid / HW, c = tid - (tid / HW) * HW;
    T l[MI], o[B];
    const T* src = a.t2 + blk * T2B + J * MI * B + x0(h) + c;
#pragma unroll
    for (int I = 0; I < MI; ++I) l[I] = src[I * B];
    solve_spread<T, B>(l, o);
#pragma unroll
    for (int y = 0; y < B; ++y) T1[(J * B + y) * HW + c] = o[y];
  }
}

// Transpose of a decomposition level, per half: v = g + K^T cbar on the
// fine nodes, then cbar - P3^T v on the coarse nodes.
template <typename T>
__global__ __launch_bounds__(w33::NT) void k_w33_dec_T(W33Args<T> a) {
  using namespace w33;
  __shared__ T lds[MC * B * HW];       // T1 [MI][B][HW], then R [MC][B][HW]
  const int64_t g = xcd_group(blockIdx.x, a.sl.per);
  if (g >= a.sl.nwg) return;
  const int h = int(g & 1);
  int64_t bz, by, bx;
  a.sl.block(g >> 1, bz, by, bx);
  const int64_t blk = (bz * a.nb[1] + by) * a.nb[2] + bx;
  w33_spread_y(a, blk, h, lds);
  __syncthreads();
  const int tid = threadIdx.x;
  const bool act = tid < NCOL;
  const int y = act ? tid / HW : 0, xl = act ? tid - (tid / HW) * HW : 0, x = x0(h) + xl;
  const bool ecol = ((y | x) & 1) == 0;
  const int64_t oz = bz * (B - 1), gy = by * (B - 1) + y, gx = bx * (B - 1) + x;
  T gv[B], v[B];
  if (act) {
    const bool own_yx = (y < B - 1 || by == a.nb[1] - 1) && (x < B - 1 || bx == a.nb[2] - 1);
    const bool lastz = bz == a.nb[0] - 1;
    const T* col = a.gc + gy * a.cs[1] + gx * a.cs[2];
    const T* ccol = a.gcur + (gy >> 1) * a.cn[2] + (gx >> 1);
    const int64_t cpl = a.cn[1] * a.cn[2];
#pragma unroll
    for (int z = 0; z < B; ++z) {
      T w = T(0);
      if (own_yx && (z < B - 1 || lastz))
        w = (ecol && !(z & 1)) ? ccol[((oz >> 1) + (z >> 1)) * cpl] : col[(oz + z) * a.cs[0]];
      gv[z] = w;
    }
    T l[MI], t[B];
#pragma unroll
    for (int J = 0; J < MI; ++J) l[J] = lds[(J * B + y) * HW + xl];
    solve_spread<T, B>(l, t);
#pragma unroll
    for (int z = 0; z < B; ++z) v[z] = (ecol && !(z & 1)) ? T(0) : gv[z] + t[z];
  }
  __syncthreads();                     // T1 is dead: R takes its place
  if (act) {
#pragma unroll
    for (int j = 0; j < MC; ++j) lds[(j * B + y) * HW + xl] = restrict_z33<T>(v, j);
  }
  __syncthreads();
  if (act && stores(h, x)) {
    if (ecol) {
#pragma unroll
      for (int j = 0; j < MC; ++j) v[2 * j] = gv[2 * j] - gather33<T>(lds, j, y, xl, x);
    }
    T* dst = a.part + a.sl.slot(bz, by, bx) * (B * B * B) + y * B + x;
#pragma unroll
    for (int z = 0; z < B; ++z) dst[z * B * B] = v[z];
  }
}

// gradient of G^{s-1} on the nodes a block owns (zero elsewhere), one column
template <typename T>
__device__ inline void w33_owned_column(const W33Args<T>& a, int64_t bz, int64_t by, int64_t bx, int y, int x,
                                        T (&gv)[w33::B]) {
  using namespace w33;
  const int64_t oz = bz * (B - 1), gy = by * (B - 1) + y, gx = bx * (B - 1) + x;
  const bool own_yx = (y < B - 1 || by == a.nb[1] - 1) && (x < B - 1 || bx == a.nb[2] - 1) && gy < a.lim[1] &&
                      gx < a.lim[2];
  const bool lastz = bz == a.nb[0] - 1;
  const T* col = a.gin + gy * a.in[2] + gx;
  const int64_t pl = a.in[1] * a.in[2];
#pragma unroll
  for (int z = 0; z < B; ++z)
    gv[z] = (own_yx && (z < B - 1 || lastz) && oz + z < a.lim[0]) ? col[(oz + z) * pl] : T(0);
}

// Transpose of a recomposition level, first part per half: r = P3^T g at
// the coarse nodes, part of the block's contributions; the interior ones
// also go to zs for the transposed correction.
template <typename T>
__global__ __launch_bounds__(w33::NT) void k_w33_rec_T_coarse(W33Args<T> a) {
  using namespace w33;
  __shared__ T R[MC * B * HW];
  const int64_t g = xcd_group(blockIdx.x, a.sl.per);
  if (g >= a.sl.nwg) return;
  const int h = int(g & 1);
  int64_t bz, by, bx;
  a.sl.block(g >> 1, bz, by, bx);
  const int64_t blk = (bz * a.nb[1] + by) * a.nb[2] + bx;
  const int tid = threadIdx.x;
  const bool act = tid < NCOL;
  const int y = act ? tid / HW : 0, xl = act ? tid - (tid / HW) * HW : 0, x = x0(h) + xl;
  const bool ecol = ((y | x) & 1) == 0;
  if (act) {
    T gv[B];
    w33_owned_column(a, bz, by, bx, y, x, gv);
#pragma unroll
    for (int j = 0; j < MC; ++j) R[(j * B + y) * HW + xl] = restrict_z33<T>(gv, j);
  }
  __syncthreads();
  if (act && ecol && stores(h, x)) {
    T* dst = a.part + a.sl.slot(bz, by, bx) * (B * B * B) + y * B + x;
    const bool icol = y >= 2 && y <= B - 3 && x >= 2 && x <= B - 3;
#pragma unroll
    for (int j = 0; j < MC; ++j) {
      const T rc = gather33<T>(R, j, y, xl, x);
      dst[2 * j * B * B] = rc;
      if (icol && j >= 1 && j <= MC - 2) a.zs[blk * ZB + ((j - 1) * MI + ((y - 2) >> 1)) * MI + ((x - 2) >> 1)] = rc;
    }
  }
}

// Transpose of a recomposition level, last part per half: g - K^T r on the
// fine nodes, added into the coefficients' gradient.
template <typename T>
__global__ __launch_bounds__(w33::NT) void k_w33_rec_T_fine(W33Args<T> a) {
  using namespace w33;
  __shared__ T T1[MI * B * HW];
  const int64_t g = xcd_group(blockIdx.x, a.sl.per);
  if (g >= a.sl.nwg) return;
  const int h = int(g & 1);
  int64_t bz, by, bx;
  a.sl.block(g >> 1, bz, by, bx);
  const int64_t blk = (bz * a.nb[1] + by) * a.nb[2] + bx;
  w33_spread_y(a, blk, h, T1);
  __syncthreads();
  const int tid = threadIdx.x;
  const bool act = tid < NCOL;
  const int y = act ? tid / HW : 0, xl = act ? tid - (tid / HW) * HW : 0, x = x0(h) + xl;
  if (!(act && stores(h, x))) return;
  const bool ecol = ((y | x) & 1) == 0;
  T gv[B], l[MI], t[B];
  w33_owned_column(a, bz, by, bx, y, x, gv);
#pragma unroll
  for (int J = 0; J < MI; ++J) l[J] = T1[(J * B + y) * HW + xl];
  solve_spread<T, B>(l, t);
  T* dst = a.part + a.sl.slot(bz, by, bx) * (B * B * B) + y * B + x;
#pragma unroll
  for (int z = 0; z < B; ++z)
    if (!(ecol && !(z & 1))) dst[z * B * B] = gv[z] - t[z];   // coarse nodes: the coarse part above
}

template <typename T>
W33Args<T> w33_args(const bm_plan_s& p, int s) {
  const Level& L = p.lv[s - 1];
  W33Args<T> a{};
  for (int k = 0; k < 3; ++k) {
    a.cn[k] = L.m[k];
    a.nb[k] = L.nb[k];
  }
  const int64_t nblocks = L.nb[0] * L.nb[1] * L.nb[2];
  if (size_t(nblocks) * w33::T2B > p.ws.t_elems) fail(BM_EINVAL, "plan workspace too small for 33^3 blocks");
  a.t2 = static_cast<T*>(p.ws.t1);
  a.zs = static_cast<T*>(p.ws.t2);
  return a;
}

// The slab in workgroups of half a block each.  The two halves of a block
// read 3 of 33 columns twice and share the cache lines between them, so they
// run on one XCD like its neighbours (dealt round-robin, 256 x 1024 x 1024
// FP32 took 2.38 ms against 2.06 for the decomposition's transpose, 2.76
// against 2.49 for the recomposition's).
Slab halves(Slab sl) {
  sl.nwg = 2 * sl.nblocks;
  sl.per = (sl.nwg + 7) / 8;
  return sl;
}

template <typename T>
void launch_w33_dec_T(bm_plan_s& p, int s, const void* gcoeff, const NodeOut<T>& out, hipStream_t st) {
  const Level& L = p.lv[s - 1];
  W33Args<T> a = w33_args<T>(p, s);
  const View3 cv = level_view(p, s, const_cast<void*>(gcoeff));
  a.gc = static_cast<const T*>(cv.ptr);
  a.gcur = static_cast<const T*>(p.ws.grid[s]);
  for (int k = 0; k < 3; ++k) a.cs[k] = cv.s[k];
  hipLaunchKernelGGL(k_w33_spread_x<T>, dim3(unsigned(L.nb[0] * L.nb[1] * L.nb[2])), dim3(256), 0, st, a, 0);
  BM_HIP(hipGetLastError());
  run_slabs<T, w33::B, false>(p, s, out, 1, st, [&](const Slab& sl, T* part) {
    a.sl = halves(sl);
    a.part = part;
    hipLaunchKernelGGL(k_w33_dec_T<T>, dim3(unsigned(8 * a.sl.per)), dim3(w33::NT), 0, st, a);
  });
}

template <typename T>
void launch_w33_rec_T(bm_plan_s& p, int s, const void* gin, const int64_t in[3], const int64_t lim[3],
                      void* gcoeff, hipStream_t st) {
  W33Args<T> a = w33_args<T>(p, s);
  a.gin = static_cast<const T*>(gin);
  for (int k = 0; k < 3; ++k) {
    a.in[k] = in[k];
    a.lim[k] = lim[k];
  }
  run_slabs<T, w33::B, true>(p, s, rec_out<T>(p, s, gcoeff), 1, st, [&](const Slab& sl, T* part) {
    a.sl = halves(sl);
    a.part = part;
    hipLaunchKernelGGL(k_w33_rec_T_coarse<T>, dim3(unsigned(8 * a.sl.per)), dim3(w33::NT), 0, st, a);
    hipLaunchKernelGGL(k_w33_spread_x<T>, dim3(unsigned(sl.nblocks)), dim3(256), 0, st, a, 1);
    hipLaunchKernelGGL(k_w33_rec_T_fine<T>, dim3(unsigned(8 * a.sl.per)), dim3(w33::NT), 0, st, a);
  });
}

template <typename T>
void local_dec_T(bm_plan_s& p, int s, const void* gcoeff, const NodeOut<T>& out, hipStream_t st) {
  if (p.lv[s - 1].b == 33)
    launch_w33_dec_T<T>(p, s, gcoeff, out, st);
  else if (p.lv[s - 1].b == 9)
    launch_local_dec_T<T, 9>(p, s, gcoeff, out, st);
  else
    launch_local_dec_T<T, 17>(p, s, gcoeff, out, st);
}

template <typename T>
void local_rec_T(bm_plan_s& p, int s, const void* gin, const int64_t in[3], const int64_t lim[3], void* gcoeff,
                 hipStream_t st) {
  if (p.lv[s - 1].b == 33)
    launch_w33_rec_T<T>(p, s, gin, in, lim, gcoeff, st);
  else if (p.lv[s - 1].b == 9)
    launch_local_rec_T<T, 9>(p, s, gin, in, lim, gcoeff, st);
  else
    launch_local_rec_T<T, 17>(p, s, gin, in, lim, gcoeff, st);
}

// --------------------------------------------------------------- global levels

// K^T along one axis: lines of m coarse values in, lines of nl values out.
template <typename T>
struct PassTArgs {
  const T* in;
  int64_t is[3];          // input strides (dims: n with m along axis)
  int axis;
  T* out;
  int64_t os[3];          // output strides (dims n)
  const T* base;          // optional: out = base + sgn * result
  int64_t bs[3];
  T sgn;
  int mask;               // write zero at the level's coarse nodes
  int cm[3];
  const double* inv;      // reciprocal Thomas pivots of 3 Mc (natural ends), length m
  int64_t nl, m;
  int W, lw;              // lines per tile (a power of two) and its log2
  int64_t nq, ntq;        // extent of the fastest other axis, tiles along it
  int pa, qa;             // the two other axes (q fastest)
};

template <typename T, int Q>
__global__ __launch_bounds__(NT) void k_line_pass_T(PassTArgs<T> a) {
  extern __shared__ unsigned char smem[];
  T* tin = reinterpret_cast<T*>(smem);               // [m][W+1]
  const int WP = a.W + 1;
  T* piv = tin + int(a.m) * WP;                      // [m] reciprocal pivots
  const uint32_t tile = blockIdx.x;
  const uint32_t p = tile / uint32_t(a.ntq);
  const int64_t q0 = int64_t(tile - p * uint32_t(a.ntq)) * a.W;
  const int wv = int(i64min(a.W, a.nq - q0));
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int m = int(a.m), nl = int(a.nl);
  const int64_t ibase = int64_t(p) * a.is[a.pa] + q0 * a.is[a.qa];
  for (int J = tid; J < m; J += NT) piv[J] = T(a.inv[J]);
  auto load = [&](int J, int w) { tin[J * WP + w] = a.in[ibase + w * a.is[a.qa] + J * a.is[a.axis]]; };
  if (a.axis == 2) {
    for (int w = wave; w < wv; w += NT / 64)
      for (int J = lane; J < m; J += 64) load(J, w);
  } else {
    const int w = tid & (a.W - 1);
    if (w < wv)
      for (int J = tid >> a.lw; J < m; J += NT >> a.lw) load(J, w);
  }
  __syncthreads();
  // in place: each lane reads, and later overwrites, only its own rows
  solve_lines<T, NT, Q>(m, piv, wv, tid, [&](int w, int J) { return T(3) * tin[J * WP + w]; },
                     [&](int w, int J, T x) { tin[J * WP + w] = x; });
  __syncthreads();
  const bool pe = !(a.cm[a.pa] && (p & 1));
  const int cmA = a.cm[a.axis], cmQ = a.cm[a.qa];
  auto store = [&](int i, int w) {
    // transposed rows of P^T M: row J has 5/6 (5/12 at the two ends) at
    // node 2J, 1/2 at 2J +- 1 and 1/12 at 2J +- 2
    const T* col = tin + w;
    const int h = i >> 1;
    T v;
    if (i & 1) {
      v = T(0.5) * (col[h * WP] + col[(h + 1) * WP]);
    } else {
      v = ((h == 0 || h == m - 1) ? T(5.0 / 12.0) : T(5.0 / 6.0)) * col[h * WP];
      T e = T(0);
      if (h > 0) e += col[(h - 1) * WP];
      if (h + 1 < m) e += col[(h + 1) * WP];
      v += T(1.0 / 12.0) * e;
    }
    int64_t c[3];
    c[a.axis] = i;
    c[a.pa] = p;
    c[a.qa] = q0 + w;
    if (a.mask && pe && !(cmA && (i & 1)) && !(cmQ && ((q0 + w) & 1))) v = T(0);
    else if (a.base) v = a.base[c[0] * a.bs[0] + c[1] * a.bs[1] + c[2] * a.bs[2]] + a.sgn * v;
    a.out[c[0] * a.os[0] + c[1] * a.os[1] + c[2] * a.os[2]] = v;
  };
  if (a.axis == 2) {
    for (int w = wave; w < wv; w += NT / 64)
      for (int i = lane; i < nl; i += 64) store(i, w);
  } else {
    const int w = tid & (a.W - 1);
    if (w < wv)
      for (int i = tid >> a.lw; i < nl; i += NT >> a.lw) store(i, w);
  }
}

template <typename T>
void launch_pass_T(const bm_plan_s& p, int s, int axis, const View3& in, const View3& out, const View3* base,
                   T sgn, bool mask, hipStream_t st) {
  const Level& L = p.lv[s - 1];
  PassTArgs<T> a{};
  a.in = static_cast<const T*>(in.ptr);
  a.out = static_cast<T*>(out.ptr);
  a.base = base ? static_cast<const T*>(base->ptr) : nullptr;
  for (int k = 0; k < 3; ++k) {
    a.is[k] = in.s[k];
    a.os[k] = out.s[k];
    a.bs[k] = base ? base->s[k] : 0;
    a.cm[k] = L.coarsen[k] ? 1 : 0;
  }
  a.sgn = sgn;
  a.mask = mask;
  a.axis = axis;
  a.nl = out.n[axis];
  a.m = in.n[axis];
  if (a.nl < 3 || a.m != (a.nl + 1) / 2 || a.m > 64 * kLineQ) fail(BM_EUNSUPPORTED, "line length not supported");
  a.inv = L.d_inv[axis];
  a.pa = axis == 0 ? 1 : 0;
  a.qa = axis == 2 ? 1 : 2;
  a.nq = out.n[a.qa];
  const int64_t np = out.n[a.pa];
  a.W = tile_width(a.m + 1, sizeof(T), np, a.nq);
  a.lw = 0;
  while ((1 << a.lw) < a.W) ++a.lw;
  a.ntq = (a.nq + a.W - 1) / a.W;
  const int64_t tiles = np * a.ntq;
  if (tiles >= (int64_t(1) << 31)) fail(BM_EUNSUPPORTED, "too many lines");
  const size_t shm = (size_t(a.m) * (a.W + 1) + size_t(a.m)) * sizeof(T);
  switch (row_q_for(a.m)) {
    case 3: hipLaunchKernelGGL((k_line_pass_T<T, 3>), dim3(unsigned(tiles)), dim3(NT), shm, st, a); break;
    case 5: hipLaunchKernelGGL((k_line_pass_T<T, 5>), dim3(unsigned(tiles)), dim3(NT), shm, st, a); break;
    case 9: hipLaunchKernelGGL((k_line_pass_T<T, 9>), dim3(unsigned(tiles)), dim3(NT), shm, st, a); break;
    case 11: hipLaunchKernelGGL((k_line_pass_T<T, 11>), dim3(unsigned(tiles)), dim3(NT), shm, st, a); break;
    case kRowQ: hipLaunchKernelGGL((k_line_pass_T<T, kRowQ>), dim3(unsigned(tiles)), dim3(NT), shm, st, a); break;
    default: hipLaunchKernelGGL((k_line_pass_T<T, 0>), dim3(unsigned(tiles)), dim3(NT), shm, st, a); break;
  }
  BM_HIP(hipGetLastError());
}

// P3^T at the coarse nodes (dims m) of a dense fine grid (dims n): the
// weighted sum over the 3^3 neighbourhood (an axis that does not coarsen
// contributes the node's own plane only).  self = 0 leaves out the node
// itself; with cbar the result is cbar - sum.  Written through a strided
// view; in place is safe when self = 0, since only coarse nodes are written
// and only fine-only nodes are read.
template <typename T>
struct RestrArgs {
  const T* src;
  int64_t n[3];
  int cm[3];
  int self;
  const T* cbar;          // optional, compact dims m
  T* out;
  int64_t os[3];
  int64_t m[3];
  Unflat32 uf;            // over dims m
};

template <typename T>
__global__ __launch_bounds__(NT) void k_restrict_T(RestrArgs<T> a) {
  const int64_t tot = a.m[0] * a.m[1] * a.m[2];
  for (int64_t i = int64_t(blockIdx.x) * NT + threadIdx.x; i < tot; i += int64_t(gridDim.x) * NT) {
    uint32_t uz, uy, ux;
    a.uf(uint32_t(i), uz, uy, ux);
    const int64_t cz = uz, cy = uy, cx = ux;
    const int64_t fz = a.cm[0] ? 2 * cz : cz, fy = a.cm[1] ? 2 * cy : cy, fx = a.cm[2] ? 2 * cx : cx;
    // all (up to 27) neighbours are fetched before the sum, which takes them
    // in the order z, y, x (weights are powers of two: exact products; an
    // absent neighbour adds +0, which changes nothing)
    T v[27];
#pragma unroll
    for (int t = 0; t < 27; ++t) {
      const int dz = t / 9 - 1, dy = (t / 3) % 3 - 1, dx = t % 3 - 1;
      const int64_t zz = fz + dz, yy = fy + dy, xx = fx + dx;
      const bool in = (dz == 0 || (a.cm[0] && zz >= 0 && zz < a.n[0])) &&
                      (dy == 0 || (a.cm[1] && yy >= 0 && yy < a.n[1])) &&
                      (dx == 0 || (a.cm[2] && xx >= 0 && xx < a.n[2])) && (t != 13 || a.self);
      v[t] = in ? a.src[(zz * a.n[1] + yy) * a.n[2] + xx] : T(0);
    }
    const T cb = a.cbar ? a.cbar[i] : T(0);
    T acc = T(0);
#pragma unroll
    for (int t = 0; t < 27; ++t) {
      const int d = (t / 9 != 1) + ((t / 3) % 3 != 1) + (t % 3 != 1);
      acc += T(d == 0 ? 1.0 : d == 1 ? 0.5 : d == 2 ? 0.25 : 0.125) * v[t];
    }
    a.out[cz * a.os[0] + cy * a.os[1] + cx * a.os[2]] = a.cbar ? cb - acc : acc;
  }
}

template <typename T>
void launch_restrict_T(const Level& L, const void* src, bool self, const void* cbar, const View3& out,
                       hipStream_t st) {
  RestrArgs<T> a{};
  a.src = static_cast<const T*>(src);
  a.self = self;
  a.cbar = static_cast<const T*>(cbar);
  a.out = static_cast<T*>(out.ptr);
  for (int k = 0; k < 3; ++k) {
    a.n[k] = L.n[k];
    a.cm[k] = L.coarsen[k] ? 1 : 0;
    a.os[k] = out.s[k];
    a.m[k] = L.m[k];
  }
  if (a.m[0] * a.m[1] * a.m[2] >= (int64_t(1) << 32)) fail(BM_EUNSUPPORTED, "coarse grid too large");
  a.uf = Unflat32(a.m[1], a.m[2]);
  hipLaunchKernelGGL(k_restrict_T<T>, dim3(grid_for(a.m[0] * a.m[1] * a.m[2])), dim3(NT), 0, st, a);
  BM_HIP(hipGetLastError());
}

// K3^T applied to the compact coarse grid G^s in the plan's grid buffer, one
// axis at a time (z, y, x, over the axes that coarsen); the last pass writes
// out (dims n) as base + sgn * result, or masked.
template <typename T>
void apply_K3_T(bm_plan_s& p, int s, const View3& out, const View3* base, T sgn, bool mask, hipStream_t st) {
  const Level& L = p.lv[s - 1];
  int axes[3], na = 0;
  for (int a : {0, 1, 2})
    if (L.coarsen[a]) axes[na++] = a;
  void* tmp[2] = {p.ws.t1, p.ws.t2};
  View3 cur = dense_view(p.ws.grid[s], L.m);
  for (int k = 0; k < na; ++k) {
    const int ax = axes[k];
    int64_t on[3] = {cur.n[0], cur.n[1], cur.n[2]};
    on[ax] = L.n[ax];
    if (k == na - 1) {
      launch_pass_T<T>(p, s, ax, cur, out, base, sgn, mask, st);
    } else {
      const View3 dst = dense_view(tmp[k & 1], on);
      launch_pass_T<T>(p, s, ax, cur, dst, nullptr, T(1), false, st);
      cur = dst;
    }
  }
}

// global decomposition level transposed: grid[s] holds cbar; out (dense, dims
// n) receives the gradient of G^{s-1}
template <typename T>
void global_dec_T(bm_plan_s& p, int s, const void* gcoeff, void* out, hipStream_t st) {
  const Level& L = p.lv[s - 1];
  const View3 ov = dense_view(out, L.n);
  const View3 gv = level_view(p, s, const_cast<void*>(gcoeff));
  apply_K3_T<T>(p, s, ov, &gv, T(1), true, st);
  View3 cview = ov;
  for (int k = 0; k < 3; ++k) {
    cview.n[k] = L.m[k];
    cview.s[k] = L.coarsen[k] ? 2 * ov.s[k] : ov.s[k];
  }
  launch_restrict_T<T>(L, out, false, p.ws.grid[s], cview, st);
}

// global recomposition level transposed: gin (dense, dims n) is the gradient
// of G^{s-1}; grid[s] receives r = P3^T gin, the coefficient view gin - K3^T r
template <typename T>
void global_rec_T(bm_plan_s& p, int s, const void* gin, void* gcoeff, hipStream_t st) {
  const Level& L = p.lv[s - 1];
  launch_restrict_T<T>(L, gin, true, nullptr, dense_view(p.ws.grid[s], L.m), st);
  const View3 base = dense_view(const_cast<void*>(gin), L.n);
  apply_K3_T<T>(p, s, level_view(p, s, gcoeff), &base, T(-1), false, st);
}

// Transpose of the clamp padding at the end nodes of the padded axes: gx =
// sum of the padded gradient over the padded nodes that copied the node.
// One lane per node on a face (its terms along one axis), one wavefront per
// node on an edge or the corner (up to the product of three axes' terms: as
// one lane's loop the corner of 100 x 500 x 500 took 0.32 ms by itself).
constexpr int kUT = 8;    // loads in flight per lane

template <typename T>
struct UnpadArgs {
  const T* gp;
  int64_t p[3];           // padded dims
  T* gx;
  int64_t n[3];           // logical dims
  int64_t e[3];           // logical dims without the end node of a padded axis
  Unflat32 uf[3];         // face tasks of axis k -> the other two coordinates
  uint64_t tf[3];         // face tasks per axis
  uint64_t te[3];         // edge tasks (the axis the edge runs along); then one corner
  uint64_t ngf;           // workgroups of the face tasks
};

template <typename T>
__global__ __launch_bounds__(NT) void k_unpad_ends(UnpadArgs<T> a) {
  const int64_t ps[3] = {a.p[1] * a.p[2], a.p[2], 1}, ns[3] = {a.n[1] * a.n[2], a.n[2], 1};
  if (blockIdx.x < a.ngf) {
    uint64_t i = uint64_t(blockIdx.x) * NT + threadIdx.x;
    for (int k = 0; k < 3; ++k) {
      if (i >= a.tf[k]) {
        i -= a.tf[k];
        continue;
      }
      const int u = k == 0 ? 1 : 0, v = k == 2 ? 1 : 2;
      uint32_t z, cu, cv;
      a.uf[k](uint32_t(i), z, cu, cv);
      const T* src = a.gp + int64_t(cu) * ps[u] + int64_t(cv) * ps[v] + (a.n[k] - 1) * ps[k];
      const int64_t cnt = a.p[k] - a.n[k] + 1;
      T acc = T(0);
      int64_t j = 0;
      for (; j < cnt; j += kUT) {
        T t[kUT];
#pragma unroll
        for (int q = 0; q < kUT; ++q) t[q] = j + q < cnt ? src[(j + q) * ps[k]] : T(0);
#pragma unroll
        for (int q = 0; q < kUT; ++q) acc += t[q];
      }
      a.gx[int64_t(cu) * ns[u] + int64_t(cv) * ns[v] + (a.n[k] - 1) * ns[k]] = acc;
      return;
    }
    return;
  }
  uint64_t i = (uint64_t(blockIdx.x) - a.ngf) * (NT / 64) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  int64_t c[3] = {a.n[0] - 1, a.n[1] - 1, a.n[2] - 1};
  int64_t cnt[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) cnt[k] = a.p[k] - a.n[k] + 1;
  bool found = false;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (found) continue;
    if (i < a.te[k]) {
      c[k] = int64_t(i);
      cnt[k] = 1;
      found = true;
    } else {
      i -= a.te[k];
    }
  }
  if (!found && i > 0) return;           // (i == 0: the corner)
  const T* src = a.gp + c[0] * ps[0] + c[1] * ps[1] + c[2];
  const uint32_t c1 = uint32_t(cnt[1]), c2 = uint32_t(cnt[2]), tot = uint32_t(cnt[0]) * c1 * c2;
  T acc = T(0);
  for (uint32_t t0 = lane; t0 < tot; t0 += 64 * kUT) {
    T v[kUT];
#pragma unroll
    for (int u = 0; u < kUT; ++u) {
      const uint32_t t = t0 + 64 * u, r = t / c2, x = t - r * c2, z = r / c1, y = r - z * c1;
      v[u] = t < tot ? src[z * ps[0] + y * ps[1] + x] : T(0);
    }
#pragma unroll
    for (int u = 0; u < kUT; ++u) acc += v[u];
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
  if (lane == 0) a.gx[c[0] * ns[0] + c[1] * ns[1] + c[2]] = acc;
}

template <typename T>
void launch_unpad_ends(const bm_plan_s& p, const void* gp, void* gx, hipStream_t st) {
  UnpadArgs<T> a{};
  a.gp = static_cast<const T*>(gp);
  a.gx = static_cast<T*>(gx);
  bool pad[3];
  for (int k = 0; k < 3; ++k) {
    a.p[k] = p.pdims[k];
    a.n[k] = p.dims[k];
    pad[k] = a.p[k] > a.n[k];
    a.e[k] = a.n[k] - (pad[k] ? 1 : 0);
  }
  uint64_t nf = 0, ne = 0;
  for (int k = 0; k < 3; ++k) {
    const int u = k == 0 ? 1 : 0, v = k == 2 ? 1 : 2;
    a.tf[k] = pad[k] ? uint64_t(a.e[u]) * a.e[v] : 0;
    a.te[k] = pad[u] && pad[v] ? uint64_t(a.e[k]) : 0;
    if (a.tf[k] >= (uint64_t(1) << 32)) fail(BM_EUNSUPPORTED, "grid too large for the pad transpose");
    a.uf[k] = Unflat32(std::max<int64_t>(a.e[u], 1), std::max<int64_t>(a.e[v], 1));
    nf += a.tf[k];
    ne += a.te[k];
  }
  if (pad[0] && pad[1] && pad[2]) ne += 1;
  a.ngf = (nf + NT - 1) / NT;
  const uint64_t g = a.ngf + (ne + NT / 64 - 1) / (NT / 64);
  if (g == 0) return;
  hipLaunchKernelGGL(k_unpad_ends<T>, dim3(unsigned(g)), dim3(NT), 0, st, a);
  BM_HIP(hipGetLastError());
}

template <typename T>
void decompose_adjoint_t(bm_plan_s& p, const void* gcoeff, void* gx, hipStream_t st) {
  const Level& last = p.lv[p.nlev - 1];
  strided_copy(p.esize, coarsest_view(p, const_cast<void*>(gcoeff)), dense_view(p.ws.grid[p.nlev], last.m), st);
  const bool padded = p.dims[0] != p.pdims[0] || p.dims[1] != p.pdims[1] || p.dims[2] != p.pdims[2];
  const bool clamp = p.cfg.pad_mode != 1;
  // a level-1 block level writes nodes below the end of a padded axis straight
  // into gx; only the others go through the padded grid
  void* top = gx;
  if (padded && p.L == 0) {
    top = p.ws.grid[0];
  } else if (padded && clamp) {
    if (!p.ws.gpad) plan_alloc_late(p, &p.ws.gpad, size_t(p.pdims[0] * p.pdims[1] * p.pdims[2]) * p.esize);
    top = p.ws.gpad;
  }
  for (int s = p.nlev; s >= 1; --s) {
    const Level& L = p.lv[s - 1];
    if (!L.local) {
      global_dec_T<T>(p, s, gcoeff, s > 1 ? p.ws.grid[s - 1] : top, st);
      continue;
    }
    NodeOut<T> out{};
    out.a = static_cast<T*>(s > 1 ? p.ws.grid[s - 1] : top);
    for (int k = 0; k < 3; ++k) out.lim[k] = L.n[k];
    const int64_t* d = L.n;
    if (s == 1 && padded) {
      out.a = static_cast<T*>(gx);
      d = p.dims;
      for (int k = 0; k < 3; ++k) out.lim[k] = p.dims[k] - (clamp && p.dims[k] != p.pdims[k] ? 1 : 0);
      if (clamp) {
        out.b = static_cast<T*>(p.ws.gpad);
        out.bs[0] = p.pdims[1] * p.pdims[2];
        out.bs[1] = p.pdims[2];
        out.bs[2] = 1;
      }
    }
    out.as[0] = d[1] * d[2];
    out.as[1] = d[2];
    out.as[2] = 1;
    local_dec_T<T>(p, s, gcoeff, out, st);
  }
  if (!padded) return;
  if (p.L == 0) {
    View3 src = dense_view(top, p.pdims);
    for (int k = 0; k < 3; ++k) src.n[k] = p.dims[k];
    strided_copy(p.esize, src, dense_view(gx, p.dims), st);
  }
  if (clamp) launch_unpad_ends<T>(p, top, gx, st);
}

template <typename T>
void recompose_adjoint_t(bm_plan_s& p, const void* gx, void* gcoeff, hipStream_t st) {
  const bool padded = p.dims[0] != p.pdims[0] || p.dims[1] != p.pdims[1] || p.dims[2] != p.pdims[2];
  for (int s = 1; s <= p.nlev; ++s) {
    const Level& L = p.lv[s - 1];
    if (L.local) {
      // level 1 reads the logical gradient; the crop's transpose is zero beyond it
      const void* gin = s == 1 ? gx : p.ws.grid[s - 1];
      const int64_t* dims = s == 1 ? p.dims : L.n;
      local_rec_T<T>(p, s, gin, dims, dims, gcoeff, st);
    } else {
      const void* gin = p.ws.grid[s - 1];
      if (s == 1) {
        if (padded)
          pad_input(p, gx, p.ws.grid[0], true, st);
        else
          gin = gx;
      }
      global_rec_T<T>(p, s, gin, gcoeff, st);
    }
  }
  const Level& last = p.lv[p.nlev - 1];
  strided_copy(p.esize, dense_view(p.ws.grid[p.nlev], last.m), coarsest_view(p, gcoeff), st);
}

}  // namespace

void decompose_adjoint(bm_plan_s& p, const void* gcoeff, void* gx, hipStream_t st) {
  if (p.cfg.dtype == BM_F32)
    decompose_adjoint_t<float>(p, gcoeff, gx, st);
  else
    decompose_adjoint_t<double>(p, gcoeff, gx, st);
}

void recompose_adjoint(bm_plan_s& p, const void* gx, void* gcoeff, hipStream_t st) {
  if (p.cfg.dtype == BM_F32)
    recompose_adjoint_t<float>(p, gx, gcoeff, st);
  else
    recompose_adjoint_t<double>(p, gx, gcoeff, st);
}

}  // namespace bm
