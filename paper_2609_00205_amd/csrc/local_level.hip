// In-cache Block levels (Sec. IV-A): every b^3 block is decomposed on chip,
// between one coalesced load and one store.
//
// Block geometry: b = 2^k+1 nodes per side; neighbouring blocks share one
// face.  Inside a block the level is the MGARD step of Sec. II-B with the
// correction of the block's surface coarse nodes held at zero
// ("face-fixed"): details d = u - multilinear interpolant of the coarse
// nodes; correction z = (Mc^{-1} P^T M)_x (Mc^{-1} P^T M)_y
// (Mc^{-1} P^T M)_z w over the interior coarse rows; c = u_C + z.  Face values
// depend on face data only, so every node is written once, by its owner.
//
// Mapping to gfx950: one thread owns one z-column (y, x) of a block and keeps
// it in registers.  The multilinear interpolant needs the even-z planes of
// the four neighbouring columns (LDS); the z pass (restriction by P^T M and
// the tridiagonal solve) runs in registers; the y and x passes read short
// LDS lines, one thread per line.  The weights are compile-time constants
// (Sec. IV-A, compile-time index resolution): interior rows of P^T M on a
// unit grid are {1/12, 1/2, 5/6, 1/2, 1/12}; 3 Mc restricted to the interior
// coarse nodes is tridiag(1, 4, 1).  Small blocks are packed several to a
// workgroup so wavefronts stay full.

#include <algorithm>
#include <cstring>

#include "block.h"
#include "internal.h"

namespace bm {
namespace {

// y and x passes of the correction: T1[MI][B][B] -> T2[MI][MI][B] -> Z[MI][MI][MI]
template <typename T, int B>
__device__ inline void pass_y(const T* T1, T* T2, int tb) {
  constexpr int MI = Geo<B>::MI, BB = Geo<B>::BB;
  if (tb < MI * B) {
    const int J = tb / B, x = tb - (tb / B) * B;
    T line[B], o[MI];
#pragma unroll
    for (int y = 0; y < B; ++y) line[y] = T1[J * BB + y * B + x];
    restrict_solve<T, B>(line, o);
#pragma unroll
    for (int I = 0; I < MI; ++I) T2[(J * MI + I) * B + x] = o[I];
  }
}

// (the x pass adds its line z, or subtracts it, at the interior coarse nodes
// of C[MC][MC][MC] itself: no array of z, no pass that picks it up)
template <typename T, int B, bool ADD>
__device__ inline void pass_x(const T* T2, T* C, int tb) {
  constexpr int MI = Geo<B>::MI, MC = Geo<B>::MC;
  if (tb < MI * MI) {
    T line[B], o[MI];
#pragma unroll
    for (int x = 0; x < B; ++x) line[x] = T2[tb * B + x];
    restrict_solve<T, B>(line, o);
    const int J = tb / MI, I = tb - (tb / MI) * MI;
    T* const c = C + ((J + 1) * MC + I + 1) * MC + 1;
#pragma unroll
    for (int K = 0; K < MI; ++K) c[K] = add_rn(c[K], ADD ? o[K] : -o[K]);
  }
}

// The z-column (y, x) of block bl of this lane.  The block kernels are bound
// by how their rows of B values lie in memory, not by arithmetic (without the
// loads and stores left in place they take as long): a wavefront's request is
// worked off 16 lanes at a time and costs by the 64-byte pieces that these
// touch.  B - 1 (16 or 8) columns of a row side by side fill such a group,
// the blocks of a workgroup follow each other, and the columns on the last
// face (which the next block owns and stores) go to the lanes after them.
// Rows of B lanes each made 18 pieces per wavefront and request of the
// recomposition at 512^3 FP32, this 6.  The loads and stores alone, 512^3
// FP32 (a copy of the bytes takes 173 us): one block a workgroup 330 us in
// rows, 275 to 326 in groups; two blocks 265 and 225 to 249.
template <int B, int NB, bool ROWS = false>
struct ColumnLane {
  int y, x, bl;
  __device__ inline ColumnLane(int tid) {
    constexpr int W = NB * (ROWS ? B : B - 1), MAIN = B * W;
    if (ROWS) {
      y = tid / W;
      const int r = tid - y * W;
      bl = y < B ? r / B : NB;
      x = r - (r / B) * B;
      y = y < B ? y : 0;
    } else if (tid < MAIN) {
      y = tid / W;
      const int r = tid - y * W;
      bl = r / (B - 1);
      x = r - bl * (B - 1);
    } else {
      const int e = tid - MAIN;
      bl = e / B;              // (NB and more: idle)
      y = e - bl * B;
      x = B - 1;
    }
  }
};

// The lanes that work on the coarse columns of a workgroup's NB blocks: the
// first NB * MC * MC, along the rows of the blocks side by side.  (The even
// columns' own lanes are a quarter of every wavefront.)
template <int MC, int NB>
struct CoarseLane {
  int p, q, bl;
  bool in;
  __device__ inline CoarseLane(int tid) {
    p = tid / (NB * MC);
    const int r = tid - p * (NB * MC);
    bl = r / MC;
    q = r - bl * MC;
    in = p < MC;
  }
};

template <typename T>
struct DecArgs {
  const T* src;
  int64_t sn[3], ss[3];   // source grid dims and strides (level 1: logical dims)
  uint32_t ss0;           // z stride of the source, 32-bit (within one column)
  int first, zero_pad;    // level 1 reads the unpadded input with clamp / zero fill
  T* coeff;
  int64_t cs[3];          // coefficient strides of this level's grid
  uint32_t cs0;           // z stride of the coefficients, 32-bit
  T* cout;                // compact coarse grid G^s
  int64_t cn[3];
  uint32_t cpl;           // plane size of the coarse grid
  int64_t nb[3], nblocks, nwg, per;
  FastDiv fnb2, fnb1;     // block index -> (bz, by, bx)
  // fused quantization (codes written instead of coefficients)
  int32_t* codes;         // same layout as coeff
  const double* tau;      // this level's block tolerances, kappa of its details and of the
  double kap, kapc;       // coarsest values (last block level when M == 0)
  int coarsest_here;
  int64_t* flag;          // set when a code does not fit in int32
  // last block level followed by a global level: its details are formed
  // here from the block's coarse values (codes with that level's 1/Delta)
  int fuse;
  const double* nqinv;
  double* part;           // per block: the next level's partial load vector [H][H][H] (FP64)
  // nested schedule, next block level in the same launch: the block's coarse
  // values stay in LDS (CC) for it, and nothing is written at them here
  int nest;
};

template <typename T>
struct RecArgs {
  const T* coeff;
  int64_t cs[3];
  uint32_t cs0;
  const T* cin;           // compact coarse grid G^s
  int64_t cn[3];
  uint32_t cpl;
  T* out;                 // output grid view (cropped to on)
  int64_t on[3], os[3];
  uint32_t os0;
  int64_t nb[3], nblocks, nwg, per;
  FastDiv fnb2, fnb1;
  const int32_t* codes;   // fused dequantization: codes instead of coefficients
  const double* tau;      // as in DecArgs
  double kap, kapc;
  int coarsest_here;
  // last block level under a global level: the coarse values of G^s are
  // interpolated here from the next level's coarse grid G^{s+1} plus its
  // details (dequantized with that level's Delta), instead of read from cin
  int fuse;
  const T* cin2;
  int64_t cn2[3];
  const double* nqdel;
};

// Register budget of the block decomposition: FP32 fits 64 VGPRs (8 waves per
// SIMD), so more blocks are in flight to cover HBM latency; FP64 columns need
// more: 5 waves per SIMD (at most 102 VGPRs) fits them without spills and
// leaves four 17^3 workgroups per CU instead of three (512^3 FP64 level 1:
// 0.678 -> 0.574 ms; the recomposition spills at that budget and has none).
template <typename T>
constexpr int kWavesPerEU = sizeof(T) == 4 ? 8 : 5;

// Nested schedule, two block levels in one launch: the finer level (blocks
// of 2B-1 nodes) has each block's B^3 coarse values at `first` of the block's
// LDS region; the coarser level (B-node blocks over the same regions) works
// in the same region after them, 16-byte aligned.
template <typename T, int B>
constexpr int nest_offset(int first) {
  return int(((size_t(first + B * B * B) * sizeof(T) + 15) / 16) * 16 / sizeof(T));
}

// One workgroup's block group g (NBG blocks) of a decomposition level.
// SRC_LDS: the level's input is the coarse values a (2B-1)-node block level
// left in LDS for this group (nested schedule), not the source grid.
template <typename T, int B, bool Q, int NBG = Geo<B, sizeof(T)>::NB, bool SRC_LDS = false>
__device__ __attribute__((always_inline)) inline void decompose_group(const DecArgs<T>& a, int64_t g, T* lds,
                                                                        double (*cls)[NBG * 27]) {
  using G = Geo<B, sizeof(T)>;
  constexpr int BB = G::BB, MC = G::MC, MI = G::MI, NB = NBG;
  constexpr int PREG = SRC_LDS ? Geo<2 * B - 1>::DEC_LDS : G::DEC_LDS;   // LDS elements per block
  constexpr int PCC = Geo<2 * B - 1>::DEC_CC;
  constexpr int NT = SRC_LDS ? Geo<2 * B - 1, sizeof(T)>::NT : G::NT;     // lanes of the workgroup
  constexpr int POFF = SRC_LDS ? nest_offset<T, B>(PCC) : 0;
  static_assert(!SRC_LDS || POFF + G::DEC_LDS <= PREG, "nested level must fit in its parent's LDS region");
  const int tid = threadIdx.x;
  // (a pair of FP32 17^3 blocks makes rows of 34 lanes, which do as well or
  // better here than groups of 16: coefficients / codes 313 / 351 against 325 /
  // 349 us at 512^3 without global levels, 425 / 453 against 438 / 458 at 98 x
  // 1200 x 1200)
  const ColumnLane<B, NB, sizeof(T) == 4 && B == 17> at(tid);
  const int bl = at.bl, y = at.y, x = at.x, tb = y * B + x;
  const int64_t blk = g * NB + bl;
  const bool act = bl < NB && blk < a.nblocks;
  T* UE = lds + (bl < NB ? bl : 0) * PREG + POFF;   // even-z planes [MC][B][B]
  T* T1 = UE + MC * BB;                              // [MI][B][B]
  // after UE is dead: T2 [MI][MI][B] in its place, then the coarse values CC
  T* CC = UE + G::DEC_CC;                            // [MC][MC][MC]
  // region of block b of the group, if there is one
  auto region = [&](int b) { return g * NB + b < a.nblocks ? lds + b * PREG + POFF : nullptr; };
  const bool ecol = ((y | x) & 1) == 0;
  int64_t bz = 0, by = 0, bx = 0;
  if (act) block_coords(uint32_t(blk), a.fnb2, a.fnb1, a.nb, bz, by, bx);
  const int64_t oz = bz * (B - 1), gy = by * (B - 1) + y, gx = bx * (B - 1) + x;
  // a node on a shared face is written by the block that starts on it
  const bool owned = (y < B - 1 || by == a.nb[1] - 1) && (x < B - 1 || bx == a.nb[2] - 1);
  const bool lastz = bz == a.nb[0] - 1;
  // fused quantization: the blocks' 1/Delta classes (read after the barrier)
  if (Q)
    class_table<NB, true>(a.tau, a.kap, a.kapc, a.coarsest_here, g * NB, a.nblocks, a.fnb2, a.fnb1, a.nb, cls);
  T v[B];
  if (act && SRC_LDS) {
    const T* cc = lds + bl * PREG + PCC;             // [B][B][B] coarse values of the finer level
#pragma unroll
    for (int z = 0; z < B; ++z) v[z] = cc[(z * B + y) * B + x];
#pragma unroll
    for (int j = 0; j < MC; ++j) UE[j * BB + tb] = v[2 * j];
  } else if (act) {
    if (!a.first || (oz + B <= a.sn[0] && gy < a.sn[1] && gx < a.sn[2])) {
      const T* col = a.src + oz * a.ss[0] + gy * a.ss[1] + gx * a.ss[2];
#pragma unroll
      for (int z = 0; z < B; ++z) v[z] = col[z * a.ss0];
    } else {
      // level 1 at the far faces: clamp or zero-fill outside the logical input
      const bool yx_in = gy < a.sn[1] && gx < a.sn[2];
      const int64_t ry = gy < a.sn[1] ? gy : a.sn[1] - 1;
      const int64_t rx = gx < a.sn[2] ? gx : a.sn[2] - 1;
      const T* col = a.src + ry * a.ss[1] + rx * a.ss[2];
#pragma unroll
      for (int z = 0; z < B; ++z) {
        const int64_t gz = oz + z;
        const bool in = yx_in && gz < a.sn[0];
        v[z] = (a.zero_pad && !in) ? T(0) : col[(gz < a.sn[0] ? gz : a.sn[0] - 1) * a.ss[0]];
      }
    }
#pragma unroll
    for (int j = 0; j < MC; ++j) UE[j * BB + tb] = v[2 * j];
  }
  __syncthreads();
  if (act) {
    // details: u minus the multilinear interpolant of the coarse nodes.  They
    // are final, so they are stored at once; v keeps u_C on the coarse nodes.
    const int y0 = y & ~1, y1 = y0 + (y & 1) * 2, x0 = x & ~1, x1 = x0 + (x & 1) * 2;
    T I2[MC];
#pragma unroll
    for (int j = 0; j < MC; ++j) {
      const T* pl = UE + j * BB;
      I2[j] = T(0.25) * ((pl[y0 * B + x0] + pl[y0 * B + x1]) + (pl[y1 * B + x0] + pl[y1 * B + x1]));
    }
#pragma unroll
    for (int z = 0; z < B; ++z) {
      if (z & 1)
        v[z] = v[z] - T(0.5) * (I2[z >> 1] + I2[(z >> 1) + 1]);
      else if (!ecol)
        v[z] = v[z] - I2[z >> 1];
    }
    if (owned) {
      // The coarse nodes of an even column get a placeholder (u_C, or code
      // 0): a later level (or the coarsest copy) overwrites them.  The plane
      // z = B-1 belongs to the next block unless this is the last one.
      // (fused with the next level: the coarse nodes are written at the end)
      const bool later = (a.fuse || a.nest) && ecol;
      if (!Q) {
        T* dst = a.coeff + oz * a.cs[0] + gy * a.cs[1] + gx * a.cs[2];
#pragma unroll
        for (int z = 1; z < B - 1; z += 2) dst[z * a.cs0] = v[z];
        if (!later) {
#pragma unroll
          for (int z = 0; z < B - 1; z += 2) dst[z * a.cs0] = v[z];
          if (lastz) dst[(B - 1) * a.cs0] = v[B - 1];
        }
      } else {
        int32_t* dst = a.codes + oz * a.cs[0] + gy * a.cs[1] + gx * a.cs[2];
        double iv[3];
        column_class<B>(cls[0], bl, y, x, iv);
        const double ie[3] = {ecol ? 0.0 : iv[0], ecol ? 0.0 : iv[1], ecol ? 0.0 : iv[2]};   // (placeholder 0)
        bool ok = true;
#pragma unroll
        for (int z = 1; z < B - 1; z += 2) dst[z * a.cs0] = quant_code(v[z], iv[1], ok);
        if (!later) {   // even planes in one branch
#pragma unroll
          for (int z = 0; z < B - 1; z += 2) dst[z * a.cs0] = quant_code(v[z], ie[zcase<B>(z)], ok);
          if (lastz) dst[(B - 1) * a.cs0] = quant_code(v[B - 1], ie[2], ok);
        }
        if (!ok) {   // (or a coarse node that is not finite)
          unsigned bad = 0;
#pragma unroll
          for (int z = 0; z < B; ++z) {
            const bool here = (z & 1) || (!ecol && (z < B - 1 || lastz));
            bad |= here ? quant_flag(v[z], iv[zcase<B>(z)]) : 0u;
          }
          if (bad) atomicOr(reinterpret_cast<unsigned long long*>(a.flag), (unsigned long long)bad);
        }
      }
    }
    // correction, z pass: w is zero on the coarse nodes
    T w[B], o[MI];
#pragma unroll
    for (int z = 0; z < B; ++z) w[z] = ((z & 1) || !ecol) ? v[z] : T(0);
    restrict_solve<T, B>(w, o);
#pragma unroll
    for (int J = 0; J < MI; ++J) T1[J * BB + tb] = o[J];
  }
  __syncthreads();
  if (act && ecol) {
#pragma unroll
    for (int j = 0; j < MC; ++j) CC[(j * MC + (y >> 1)) * MC + (x >> 1)] = v[2 * j];
  }
  if (const int b = tid / (MI * B); b < NB)
    if (T* R = region(b)) pass_y<T, B>(R + MC * BB, R, tid - b * (MI * B));
  __syncthreads();
  // coarse values c = u_C + z (z = 0 on the block surface)
  if (const int b = tid / (MI * MI); b < NB)
    if (T* R = region(b)) pass_x<T, B, true>(R, R + G::DEC_CC, tid - b * (MI * MI));
  __syncthreads();
  // what follows is per coarse column, on lanes of its own
  constexpr int H = (MC + 1) / 2;
  // fused: the next level's load vector, in FP64 (see below): z pass in
  // registers, then y and x passes in LDS after CC
  constexpr int ZOFF = int(((MC * MC * MC * sizeof(T) + 7) / 8) * (8 / sizeof(T)));
  auto Z1 = [&](T* R) { return reinterpret_cast<double*>(R + G::DEC_CC + ZOFF); };   // [H][MC][MC], then Y1 [H][H][MC]
  const CoarseLane<MC, NB> cl(tid);
  if (cl.in && g * NB + cl.bl < a.nblocks && !a.nest) {
    const int p = cl.p, q = cl.q;
    const T* const C = lds + cl.bl * PREG + POFF + G::DEC_CC;
    int64_t cz, cy, cx;
    block_coords(uint32_t(g * NB + cl.bl), a.fnb2, a.fnb1, a.nb, cz, cy, cx);
    const bool own = (p < MC - 1 || cy == a.nb[1] - 1) && (q < MC - 1 || cx == a.nb[2] - 1);
    const bool end = cz == a.nb[0] - 1;
    const int64_t o = cz * (B - 1) * a.cs[0] + (cy * (B - 1) + 2 * p) * a.cs[1] + (cx * (B - 1) + 2 * q) * a.cs[2];
    T c[MC];
#pragma unroll
    for (int j = 0; j < MC; ++j) c[j] = C[(j * MC + p) * MC + q];
    if (a.fuse) {
      double* const Zb = Z1(lds + cl.bl * PREG + POFF);
#pragma unroll
      for (int k = 0; k < H; ++k)
        Zb[(k * MC + p) * MC + q] = restrict_half<double, MC>(k, [&](int t) { return double(c[t]); });
    }
    if (own && Q && a.coarsest_here) {
      // last level of the hierarchy: codes for the coarsest values
      double ci[3];
      column_class<B>(cls[1], cl.bl, 2 * p, 2 * q, ci);
      int32_t* dst = a.codes + o;
      unsigned bad = 0;
#pragma unroll
      for (int j = 0; j < MC - 1; ++j) dst[2 * j * a.cs0] = quant(c[j], ci[zcase<B>(2 * j)], false, bad);
      if (end) dst[(B - 1) * a.cs0] = quant(c[MC - 1], ci[2], false, bad);
      if (bad) atomicOr(reinterpret_cast<unsigned long long*>(a.flag), (unsigned long long)bad);
    } else if (own && !a.fuse) {
      // the compact coarse grid feeds the next level
      T* cdst = a.cout + cz * (MC - 1) * int64_t(a.cpl) + (cy * (MC - 1) + p) * a.cn[2] + cx * (MC - 1) + q;
#pragma unroll
      for (int j = 0; j < MC - 1; ++j) cdst[j * a.cpl] = c[j];
      if (end) cdst[(MC - 1) * a.cpl] = c[MC - 1];
    } else if (own) {
      // details of the next (global) level at this column's coarse nodes: c
      // minus the interpolant over the cell of the next coarse grid (every
      // such cell lies inside the block); its coarse nodes get a placeholder
      // (c, or code 0) that a later level or the coarsest values overwrite
      const int op = p & 1, oq = q & 1;
      const double inv = Q ? *a.nqinv : 0.0;
      T in[MC];
      column_interp<T, MC>(p, q, [&](int J, int P, int K) { return C[((2 * J) * MC + 2 * P) * MC + 2 * K]; }, in);
      unsigned bad = 0;
#pragma unroll
      for (int j = 0; j < MC; ++j) {
        if (j == MC - 1 && !end) continue;
        const bool cn = ((j & 1) | op | oq) == 0;
        const T d = cn ? c[j] : c[j] - in[j];
        const int64_t oj = o + int64_t(2 * j) * a.cs0;
        if (Q)
          a.codes[oj] = quant(d, inv, cn, bad);
        else
          a.coeff[oj] = d;
      }
      if (Q && bad) atomicOr(reinterpret_cast<unsigned long long*>(a.flag), (unsigned long long)bad);
    }
  }
  if (a.fuse) {
    __syncthreads();
    // The next level's load vector 3 P^T M (per axis) at its coarse nodes in
    // this block, from the block's own coarse values only: rows on the block
    // faces take the half of the stencil on this side ({5/12, 1/2, 1/12}, the
    // natural end row), the neighbour adds the other half.  Shrinking passes
    // z (in registers, above), y and x (LDS), in FP64 so that the sum of 125
    // terms and the gather of up to 8 partials round once; the partial sums
    // go to a per-block array that a gather completes, so the global level
    // needs no pass over G^s.
    for (int i = tid; i < NB * H * H * MC; i += NT) {
      const int b = i / (H * H * MC), e = i - b * (H * H * MC);
      if (T* R = region(b)) {
        const int k0 = e / (H * MC), r = e - k0 * (H * MC), k1 = r / MC, q = r - k1 * MC;
        const double* const Z = Z1(R);
        Z1(R)[H * MC * MC + e] = restrict_half<double, MC>(k1, [&](int t) { return Z[(k0 * MC + t) * MC + q]; });
      }
    }
    __syncthreads();
    for (int i = tid; i < NB * H * H * H; i += NT) {
      const int b = i / (H * H * H), e = i - b * (H * H * H);
      if (T* R = region(b)) {
        const int r = e / H, k2 = e - r * H;
        const double* const Y1 = Z1(R) + H * MC * MC;
        a.part[(g * NB + b) * (H * H * H) + e] = restrict_half<double, MC>(k2, [&](int t) { return Y1[r * MC + t]; });
      }
    }
  }
}

// One workgroup's block group g (NBG blocks) of a recomposition level.
// Nested schedule, two block levels in one launch: MODE 1 is the coarser
// level (B-node blocks), which writes all B^3 values of each block to the
// start of the block's LDS region of the finer (2B-1)-node level and works
// after them; MODE 2 is that finer level, which reads its coarse values
// there instead of from the coarse grid.
// (FP64 rows of 17 values are 128 bytes wide in any case and read best as
// rows: 512^3 FP64 446 / 453 us against 463 / 465 in groups of 16 lanes, where
// the decomposition has 602 / 555 against 574 / 524.)
template <typename T, int B, bool Q, int NBG = Geo<B, sizeof(T), false>::NB, int MODE = 0, bool ROWS = sizeof(T) == 8>
__device__ __attribute__((always_inline)) inline void recompose_group(const RecArgs<T>& a, int64_t g, T* lds,
                                                                        double (*cls)[NBG * 27]) {
  using G = Geo<B, sizeof(T), false>;
  constexpr int BB = G::BB, MC = G::MC, MI = G::MI, NB = NBG;
  constexpr int PREG = MODE == 1 ? Geo<2 * B - 1>::REC_LDS : G::REC_LDS;   // LDS elements per block
  constexpr int POFF = MODE == 1 ? nest_offset<T, B>(0) : 0;
  constexpr int BL = MODE == 1 ? 2 * B - 1 : B, NT = (NBG * BL * BL + 63) / 64 * 64;   // lanes of the workgroup
  static_assert(MODE != 1 || POFF + G::REC_LDS <= PREG, "nested level must fit in its parent's LDS region");
  const int tid = threadIdx.x;
  const ColumnLane<B, NB, ROWS> at(tid);
  const int bl = at.bl, y = at.y, x = at.x, tb = y * B + x;
  const int64_t blk = g * NB + bl;
  const bool act = bl < NB && blk < a.nblocks;
  T* UC = lds + (bl < NB ? bl : 0) * PREG + POFF;   // coarse values u_C [MC][MC][MC]
  T* T1 = UC + MC * MC * MC;                         // [MI][B][B]
  constexpr int T2OFF = MC * MC * MC + MI * BB;      // [MI][MI][B]
  constexpr int XOFF = T2OFF + MI * MI * B;          // [H][H][H] the next level's coarse values (fused)
  // region of block b of the group, if there is one
  auto region = [&](int b) { return g * NB + b < a.nblocks ? lds + b * PREG + POFF : nullptr; };
  const bool ecol = ((y | x) & 1) == 0;
  int64_t bz = 0, by = 0, bx = 0;
  if (act) block_coords(uint32_t(blk), a.fnb2, a.fnb1, a.nb, bz, by, bx);
  const int64_t oz = bz * (B - 1), gy = by * (B - 1) + y, gx = bx * (B - 1) + x;
  T w[B];
  int32_t qv[B];
  // the whole column is read (coarse nodes too, then zeroed): one load per
  // node, on its way before anything is waited for
  const int64_t off = oz * a.cs[0] + gy * a.cs[1] + gx * a.cs[2];
  if (act) {
    if (!Q) {
      const T* col = a.coeff + off;
#pragma unroll
      for (int z = 0; z < B; ++z) w[z] = col[z * a.cs0];
    } else {
      const int32_t* col = a.codes + off;
#pragma unroll
      for (int z = 0; z < B; ++z) qv[z] = col[z * a.cs0];
    }
  }
  // fused dequantization: the blocks' Delta classes
  if (Q)
    class_table<NB, false>(a.tau, a.kap, a.kapc, a.coarsest_here, g * NB, a.nblocks, a.fnb2, a.fnb1, a.nb, cls);
  // fused with the next (global) level: its coarse values over this block
  constexpr int H = G::H;
  if (a.fuse) {
    const int64_t h0 = (MC - 1) / 2, pl2 = a.cn2[1] * a.cn2[2];
    for (int i = tid; i < NB * H * H * H; i += NT) {
      const int b = i / (H * H * H), e = i - b * (H * H * H);
      if (T* R = region(b)) {
        int64_t cz, cy, cx;
        block_coords(uint32_t(g * NB + b), a.fnb2, a.fnb1, a.nb, cz, cy, cx);
        const T* src = a.cin2 + cz * h0 * pl2 + cy * h0 * a.cn2[2] + cx * h0;
        const int k0 = e / (H * H), r = e - k0 * H * H, k1 = r / H, k2 = r - k1 * H;
        R[XOFF + e] = src[k0 * pl2 + k1 * a.cn2[2] + k2];
      }
    }
  }
  // the coarse values come from the column itself (coarsest codes, details of
  // the fused next level), from the level's coarse grid, or are there already
  const bool self = a.fuse || (Q && a.coarsest_here);
  const CoarseLane<MC, NB> cl(tid);
  const bool cact = cl.in && g * NB + cl.bl < a.nblocks;
  T ce[MC];
  if (MODE != 2 && !self && cact) {
    int64_t cz, cy, cx;
    block_coords(uint32_t(g * NB + cl.bl), a.fnb2, a.fnb1, a.nb, cz, cy, cx);
    const T* ccol = a.cin + cz * (MC - 1) * int64_t(a.cpl) + (cy * (MC - 1) + cl.p) * a.cn[2] + cx * (MC - 1) + cl.q;
#pragma unroll
    for (int j = 0; j < MC; ++j) ce[j] = ccol[j * a.cpl];
  }
  if (Q || a.fuse) __syncthreads();
  if (MODE != 2 && !self && cact) {
    T* const C = lds + cl.bl * PREG + POFF;
#pragma unroll
    for (int j = 0; j < MC; ++j) C[(j * MC + cl.p) * MC + cl.q] = ce[j];
  }
  if (act) {
    if (Q) {
      // c_hat = (T)(q * Delta); an even column's even planes take Delta of the
      // coarsest values or of the fused next level
      double de[3];
      column_class<B>(cls[ecol && a.coarsest_here ? 1 : 0], bl, y, x, de);
      if (a.fuse && ecol) de[0] = de[1] = de[2] = *a.nqdel;
#pragma unroll
      for (int z = 0; z < B; z += 2) w[z] = T(mul_rn(double(qv[z]), de[zcase<B>(z)]));
      column_class<B>(cls[0], bl, y, x, de);
#pragma unroll
      for (int z = 1; z < B; z += 2) w[z] = T(mul_rn(double(qv[z]), de[1]));
    }
    if (ecol) {
      // c waits in UC through the correction passes instead of in registers
      if (MODE != 2 && self) {
#pragma unroll
        for (int j = 0; j < MC; ++j) UC[(j * MC + (y >> 1)) * MC + (x >> 1)] = w[2 * j];
      }
#pragma unroll
      for (int j = 0; j < MC; ++j) w[2 * j] = T(0);
    }
  }
  if (act) {
    T o[MI];
    restrict_solve<T, B>(w, o);
#pragma unroll
    for (int J = 0; J < MI; ++J) T1[J * BB + tb] = o[J];
  }
  __syncthreads();
  if (const int b = tid / (MI * B); b < NB)
    if (T* R = region(b)) pass_y<T, B>(R + MC * MC * MC, R + T2OFF, tid - b * (MI * B));
  if (a.fuse) {
    // u at the coarse nodes = next level's detail + interpolant of its coarse
    // values (exactly the next level's recomposition), on the last lanes: the
    // y pass is on the first
    const CoarseLane<MC, NB> fl(NT - 1 - tid);
    if (fl.in && g * NB + fl.bl < a.nblocks) {
      T* const C = lds + fl.bl * PREG + POFF;
      const T* const X = C + XOFF;
      const int op = fl.p & 1, oq = fl.q & 1;
      T in[MC];
      column_interp<T, MC>(fl.p, fl.q, [&](int J, int P, int K) { return X[(J * H + P) * H + K]; }, in);
#pragma unroll
      for (int j = 0; j < MC; ++j) {
        T& u = C[(j * MC + fl.p) * MC + fl.q];
        u = ((j & 1) | op | oq) == 0 ? in[j] : u + in[j];   // (the next level's coarse value itself, exact)
      }
    }
  }
  __syncthreads();
  // u_C = c - z (z = 0 on the block surface)
  if (const int b = tid / (MI * MI); b < NB)
    if (T* R = region(b)) pass_x<T, B, false>(R + T2OFF, R, tid - b * (MI * MI));
  __syncthreads();
  if (act) {
    // u = interpolant(u_C) + w
    const int cy0 = y >> 1, cy1 = (y + 1) >> 1, cx0 = x >> 1, cx1 = (x + 1) >> 1;
    T I2[MC];
#pragma unroll
    for (int j = 0; j < MC; ++j) {
      const T* pl = UC + j * MC * MC;
      I2[j] = T(0.25) * ((pl[cy0 * MC + cx0] + pl[cy0 * MC + cx1]) + (pl[cy1 * MC + cx0] + pl[cy1 * MC + cx1]));
    }
    auto val = [&](int z) {
      return (z & 1) ? T(0.5) * (I2[z >> 1] + I2[(z >> 1) + 1]) + w[z] : (ecol ? I2[z >> 1] : I2[z >> 1] + w[z]);
    };
    if (MODE == 1) {
      // every node of the block, faces included: the finer level's coarse values
      T* dst = lds + bl * PREG;
#pragma unroll
      for (int z = 0; z < B; ++z) dst[(z * B + y) * B + x] = val(z);
      return;
    }
    const bool owny = (y < B - 1 || by == a.nb[1] - 1) && gy < a.on[1];
    const bool ownx = (x < B - 1 || bx == a.nb[2] - 1) && gx < a.on[2];
    const bool lastz = bz == a.nb[0] - 1;
    if (owny && ownx) {
      T* dst = a.out + oz * a.os[0] + gy * a.os[1] + gx * a.os[2];
      if (oz + B <= a.on[0]) {
#pragma unroll
        for (int z = 0; z < B - 1; ++z) dst[z * a.os0] = val(z);
        if (lastz) dst[(B - 1) * a.os0] = val(B - 1);
      } else {
        // the block reaches past the (cropped) output
#pragma unroll
        for (int z = 0; z < B; ++z)
          if ((z < B - 1 || lastz) && oz + z < a.on[0]) dst[z * a.os0] = val(z);
      }
    }
  }
}

template <typename T, int B, bool Q>
__global__ __launch_bounds__((Geo<B, sizeof(T)>::NT)) __attribute__((amdgpu_waves_per_eu(kWavesPerEU<T>))) void k_local_decompose(DecArgs<T> a) {
  __shared__ __attribute__((aligned(16))) T lds[Geo<B, sizeof(T)>::NB * Geo<B>::DEC_LDS];   // FP64 scratch inside
  __shared__ double cls[Q ? 2 : 1][Geo<B, sizeof(T)>::NB * 27];   // Delta classes of the blocks
  const int64_t g = xcd_group(blockIdx.x, a.per);
  if (g >= a.nwg) return;
  decompose_group<T, B, Q>(a, g, lds, cls);
}

template <typename T, int B, bool Q, int NB>
__global__ __launch_bounds__((NB * B * B + 63) / 64 * 64) void k_local_recompose(RecArgs<T> a) {
  __shared__ T lds[NB * Geo<B>::REC_LDS];
  __shared__ double cls[Q ? 2 : 1][NB * 27];   // Delta classes of the blocks
  const int64_t g = xcd_group(blockIdx.x, a.per);
  if (g >= a.nwg) return;
  recompose_group<T, B, Q, NB>(a, g, lds, cls);
}

// Nested schedule: block levels of 17- and 9-node blocks over the same
// regions in one launch.  Decomposition: the 17-node level keeps each
// block's 9^3 coarse values in LDS and the 9-node level decomposes them
// there (the level-2 grid never goes through HBM).  Recomposition: the
// 9-node level recomposes each block's 9^3 values into LDS, and the
// 17-node level takes them as its coarse values.
template <typename T, bool Q>
__global__ __launch_bounds__((Geo<17, sizeof(T)>::NT)) __attribute__((amdgpu_waves_per_eu(kWavesPerEU<T>))) void k_local_decompose_nest(DecArgs<T> a1, DecArgs<T> a2) {
  constexpr int NB = Geo<17, sizeof(T)>::NB;
  __shared__ __attribute__((aligned(16))) T lds[NB * Geo<17>::DEC_LDS];   // FP64 scratch inside
  __shared__ double cls[Q ? 2 : 1][NB * 27];   // Delta classes of the blocks
  const int64_t g = xcd_group(blockIdx.x, a1.per);
  if (g >= a1.nwg) return;
  decompose_group<T, 17, Q>(a1, g, lds, cls);
  __syncthreads();
  decompose_group<T, 9, Q, NB, true>(a2, g, lds, cls);
}

// (waves: two levels' arguments take more scalar registers than eight waves a
// SIMD leave, and with seven a third workgroup of 640 lanes does not fit a CU;
// 30 scalars spilled to vector lanes cost less: 512^3 FP32 codes 464 -> 440 us
// a restore with two global levels)
template <typename T, bool Q, int NB, bool ROWS>
__global__ __launch_bounds__((NB * 289 + 63) / 64 * 64) __attribute__((amdgpu_waves_per_eu(kWavesPerEU<T>))) void k_local_recompose_nest(RecArgs<T> a2, RecArgs<T> a1) {
  __shared__ __attribute__((aligned(16))) T lds[NB * Geo<17>::REC_LDS];
  __shared__ double cls[Q ? 2 : 1][NB * 27];   // Delta classes of the blocks
  const int64_t g = xcd_group(blockIdx.x, a1.per);
  if (g >= a1.nwg) return;
  recompose_group<T, 9, Q, NB, 1, ROWS>(a2, g, lds, cls);
  __syncthreads();
  recompose_group<T, 17, Q, NB, 2, ROWS>(a1, g, lds, cls);
}

// Many fields in one launch: workgroup k takes task k, block group
// k - first[f] of field f (first[] ascending, first[nf] = total, task_field),
// in the XCD order of a single field's launch.

// (One workgroup per task and no loop over tasks: in a persistent launch the
// compiler kept the addresses of 17 planes over the loop, 106 to 111 VGPRs
// against 63, which left one FP32 decomposition workgroup per CU.  The field
// index is the same for every lane of the workgroup; said so with
// readfirstlane, and with the argument array read-only and unaliased, the
// record is read by scalar loads.  It is copied before use: read in place, its
// fields were fetched where they were needed, into vector registers: 68 and
// 121 of them in the recompositions against 61 and 92.)
template <typename T, int B, bool Q>
__global__ __launch_bounds__((Geo<B, sizeof(T)>::NT)) __attribute__((amdgpu_waves_per_eu(kWavesPerEU<T>))) void k_batch_decompose(
    const DecArgs<T>* __restrict__ fa, const int64_t* __restrict__ first, int nf, int64_t ntasks) {
  __shared__ __attribute__((aligned(16))) T lds[Geo<B, sizeof(T)>::NB * Geo<B>::DEC_LDS];   // FP64 scratch inside
  __shared__ double cls[Q ? 2 : 1][Geo<B, sizeof(T)>::NB * 27];   // Delta classes of the blocks
  const int64_t k = xcd_group(blockIdx.x, (ntasks + 7) / 8);
  if (k >= ntasks) return;
  const int f = __builtin_amdgcn_readfirstlane(task_field(first, nf, k));
  const DecArgs<T> a = fa[f];
  decompose_group<T, B, Q>(a, k - first[f], lds, cls);
}

template <typename T, int B, bool Q>
__global__ __launch_bounds__((Geo<B, sizeof(T), false>::NT)) void k_batch_recompose(const RecArgs<T>* __restrict__ fa,
                                                                              const int64_t* __restrict__ first, int nf,
                                                                              int64_t ntasks) {
  __shared__ T lds[Geo<B, sizeof(T), false>::NB * Geo<B>::REC_LDS];
  __shared__ double cls[Q ? 2 : 1][Geo<B, sizeof(T), false>::NB * 27];   // Delta classes of the blocks
  const int64_t k = xcd_group(blockIdx.x, (ntasks + 7) / 8);
  if (k >= ntasks) return;
  const int f = __builtin_amdgcn_readfirstlane(task_field(first, nf, k));
  const RecArgs<T> a = fa[f];
  recompose_group<T, B, Q>(a, k - first[f], lds, cls);
}

// The nested schedule of every field in one launch: task k is
// block group k - first[f] of field f at its 17-node level (arguments f1[f]),
// then the same group of its 9-node level (f2[f]) on the coarse values the
// first left in LDS, as k_local_decompose_nest / k_local_recompose_nest do
// for one field.
template <typename T, bool Q>
__global__ __launch_bounds__((Geo<17, sizeof(T)>::NT)) __attribute__((amdgpu_waves_per_eu(kWavesPerEU<T>))) void k_batch_decompose_nest(
    const DecArgs<T>* __restrict__ f1, const DecArgs<T>* __restrict__ f2, const int64_t* __restrict__ first, int nf,
    int64_t ntasks) {
  constexpr int NB = Geo<17, sizeof(T)>::NB;
  __shared__ __attribute__((aligned(16))) T lds[NB * Geo<17>::DEC_LDS];   // FP64 scratch inside
  __shared__ double cls[Q ? 2 : 1][NB * 27];   // Delta classes of the blocks
  const int64_t k = xcd_group(blockIdx.x, (ntasks + 7) / 8);
  if (k >= ntasks) return;
  const int f = __builtin_amdgcn_readfirstlane(task_field(first, nf, k));
  const int64_t g = k - first[f];
  const DecArgs<T> a1 = f1[f];
  decompose_group<T, 17, Q>(a1, g, lds, cls);
  __syncthreads();
  const DecArgs<T> a2 = f2[f];
  decompose_group<T, 9, Q, NB, true>(a2, g, lds, cls);
}

template <typename T, bool Q>
__global__ __launch_bounds__((Geo<17, sizeof(T), false>::NT)) void k_batch_recompose_nest(
    const RecArgs<T>* __restrict__ f1, const RecArgs<T>* __restrict__ f2, const int64_t* __restrict__ first, int nf,
    int64_t ntasks) {
  constexpr int NB = Geo<17, sizeof(T), false>::NB;
  __shared__ T lds[NB * Geo<17>::REC_LDS];
  __shared__ double cls[Q ? 2 : 1][NB * 27];   // Delta classes of the blocks
  const int64_t k = xcd_group(blockIdx.x, (ntasks + 7) / 8);
  if (k >= ntasks) return;
  const int f = __builtin_amdgcn_readfirstlane(task_field(first, nf, k));
  const int64_t g = k - first[f];
  const RecArgs<T> a2 = f2[f];
  recompose_group<T, 9, Q, NB, 1>(a2, g, lds, cls);
  __syncthreads();
  const RecArgs<T> a1 = f1[f];
  recompose_group<T, 17, Q, NB, 2>(a1, g, lds, cls);
}

// 32-bit z stride within one block column
inline uint32_t column_stride(int64_t s, int B) {
  if (s * (B - 1) >= (int64_t(1) << 32)) fail(BM_EUNSUPPORTED, "grid planes too large for 32-bit column offsets");
  return uint32_t(s);
}

template <typename T, int B>
DecArgs<T> dec_args(const bm_plan_s& p, int s, const View3& src, bool first, void* coeff, void* cout, int32_t* codes,
                    const QPrep* q) {
  using G = Geo<B, sizeof(T)>;
  const Level& L = p.lv[s - 1];
  DecArgs<T> a{};
  a.src = static_cast<const T*>(src.ptr);
  for (int k = 0; k < 3; ++k) {
    a.sn[k] = src.n[k];
    a.ss[k] = src.s[k];
    a.cn[k] = L.m[k];
    a.nb[k] = L.nb[k];
  }
  a.ss0 = column_stride(src.s[0], B);
  a.first = first;
  a.zero_pad = p.cfg.pad_mode == 1;
  a.coeff = static_cast<T*>(coeff);
  const View3 cv = level_view(p, s, q ? static_cast<void*>(codes) : coeff);
  for (int k = 0; k < 3; ++k) a.cs[k] = cv.s[k];
  a.cs0 = column_stride(cv.s[0], B);
  a.cout = static_cast<T*>(cout);
  a.cpl = column_stride(L.m[1] * L.m[2], B);
  a.nblocks = L.nb[0] * L.nb[1] * L.nb[2];
  if (a.nblocks >= (int64_t(1) << 32)) fail(BM_EUNSUPPORTED, "too many blocks");
  a.fnb2 = FastDiv(uint32_t(L.nb[2]));
  a.fnb1 = FastDiv(uint32_t(L.nb[1]));
  a.nwg = (a.nblocks + G::NB - 1) / G::NB;
  a.per = (a.nwg + 7) / 8;
  if (q) {
    a.codes = codes;
    a.tau = q->lv[s - 1].tau;
    a.kap = q->lv[s - 1].kap;
    a.coarsest_here = (p.M == 0 && s == p.L) ? 1 : 0;
    if (a.coarsest_here) a.kapc = q->lv[kCoarseSlotHost].kap;
    a.flag = q->flag;
  }
  a.fuse = (p.fuse_next && s == p.L) ? 1 : 0;
  if (a.fuse && q) a.nqinv = q->q + 2 * s + 1;   // 1/Delta of level s+1
  if (a.fuse) a.part = static_cast<double*>(p.ws.part);
  return a;
}

template <typename T, int B>
void launch_dec(const bm_plan_s& p, int s, const View3& src, bool first, void* coeff, void* cout, int32_t* codes,
                const QPrep* q, hipStream_t st) {
  using G = Geo<B, sizeof(T)>;
  const DecArgs<T> a = dec_args<T, B>(p, s, src, first, coeff, cout, codes, q);
  if (q)
    hipLaunchKernelGGL((k_local_decompose<T, B, true>), dim3(unsigned(8 * a.per)), dim3(G::NT), 0, st, a);
  else
    hipLaunchKernelGGL((k_local_decompose<T, B, false>), dim3(unsigned(8 * a.per)), dim3(G::NT), 0, st, a);
  BM_HIP(hipGetLastError());
}

template <typename T, int B>
RecArgs<T> rec_args(const bm_plan_s& p, int s, const void* coeff, const void* cin, void* out, bool last,
                    const int32_t* codes, const QPrep* q, bool crop = true, int nb = Geo<B, sizeof(T), false>::NB) {
  using G = Geo<B, sizeof(T), false>;
  const Level& L = p.lv[s - 1];
  RecArgs<T> a{};
  a.coeff = static_cast<const T*>(coeff);
  const View3 cv = level_view(p, s, q ? const_cast<int32_t*>(codes) : const_cast<void*>(coeff));
  for (int k = 0; k < 3; ++k) {
    a.cs[k] = cv.s[k];
    a.cn[k] = L.m[k];
    a.nb[k] = L.nb[k];
  }
  a.cs0 = column_stride(cv.s[0], B);
  a.cpl = column_stride(L.m[1] * L.m[2], B);
  a.cin = static_cast<const T*>(cin);
  a.out = static_cast<T*>(out);
  // last: writing the caller's output with the logical (unpadded) dims
  const int64_t* on = last ? p.dims : L.n;
  for (int k = 0; k < 3; ++k) a.on[k] = on[k];
  a.os[0] = on[1] * on[2];
  a.os[1] = on[2];
  a.os[2] = 1;
  a.os0 = column_stride(a.os[0], B);
  // planes of blocks that start past the (cropped) output have nothing to
  // write: 98 x 1200 x 1200 with two block levels is padded to 129 planes of
  // nodes, and its last plane of blocks out of eight is left out (level 1 396
  // -> 367 us; left out inside the kernel it idled one XCD and gained nothing)
  const int64_t nbz = crop ? std::min(L.nb[0], (on[0] + B - 2) / (B - 1)) : L.nb[0];
  a.nblocks = nbz * L.nb[1] * L.nb[2];
  if (a.nblocks >= (int64_t(1) << 32)) fail(BM_EUNSUPPORTED, "too many blocks");
  a.fnb2 = FastDiv(uint32_t(L.nb[2]));
  a.fnb1 = FastDiv(uint32_t(L.nb[1]));
  a.nwg = (a.nblocks + nb - 1) / nb;
  a.per = (a.nwg + 7) / 8;
  if (q) {
    a.codes = codes;
    a.tau = q->lv[s - 1].tau;
    a.kap = q->lv[s - 1].kap;
    a.coarsest_here = (p.M == 0 && s == p.L) ? 1 : 0;
    if (a.coarsest_here) a.kapc = q->lv[kCoarseSlotHost].kap;
  }
  a.fuse = (p.fuse_next && s == p.L) ? 1 : 0;
  if (a.fuse) {
    a.cin2 = static_cast<const T*>(p.ws.grid[s + 1]);
    for (int k = 0; k < 3; ++k) a.cn2[k] = p.lv[s].m[k];
    if (q) a.nqdel = q->q + 2 * s;                // Delta of level s+1
  }
  return a;
}

template <typename T, int B, int NB>
void launch_rec_nb(const bm_plan_s& p, int s, const void* coeff, const void* cin, void* out, bool last,
                   const int32_t* codes, const QPrep* q, hipStream_t st) {
  const RecArgs<T> a = rec_args<T, B>(p, s, coeff, cin, out, last, codes, q, true, NB);
  auto* const k = q ? k_local_recompose<T, B, true, NB> : k_local_recompose<T, B, false, NB>;
  hipLaunchKernelGGL(k, dim3(unsigned(8 * a.per)), dim3((NB * B * B + 63) / 64 * 64), 0, st, a);
  BM_HIP(hipGetLastError());
}

// (two FP32 blocks a workgroup share lines along x; where a row has one block
// there is none to share: 2200 x 2200 x 1 one level 130 -> 115 us, with codes
// 101 -> 87)
template <typename T, int B>
void launch_rec(const bm_plan_s& p, int s, const void* coeff, const void* cin, void* out, bool last,
                const int32_t* codes, const QPrep* q, hipStream_t st) {
  constexpr int NB = Geo<B, sizeof(T), false>::NB;
  if constexpr (B == 17 && NB > 1)
    if (p.lv[s - 1].nb[2] == 1)
      return launch_rec_nb<T, B, 1>(p, s, coeff, cin, out, last, codes, q, st);
  launch_rec_nb<T, B, NB>(p, s, coeff, cin, out, last, codes, q, st);
}


// workgroups of a launch over ntasks tasks in XCD order
unsigned task_grid(int64_t ntasks) {
  const int64_t g = 8 * ((ntasks + 7) / 8);
  if (g >= (int64_t(1) << 31)) fail(BM_EUNSUPPORTED, "too many block groups in one batch");
  return unsigned(g);
}

template <typename T, int B>
void launch_batch(bool dec, bool quant, const void* args, const int64_t* first, int nf, int64_t ntasks,
                  hipStream_t st) {
  using G = Geo<B, sizeof(T)>;
  if (ntasks <= 0) return;
  if (dec) {
    const auto* fa = static_cast<const DecArgs<T>*>(args);
    if (quant) {
      auto k = k_batch_decompose<T, B, true>;
      hipLaunchKernelGGL(k, dim3(task_grid(ntasks)), dim3(G::NT), 0, st, fa, first, nf, ntasks);
    } else {
      auto k = k_batch_decompose<T, B, false>;
      hipLaunchKernelGGL(k, dim3(task_grid(ntasks)), dim3(G::NT), 0, st, fa, first, nf, ntasks);
    }
  } else {
    using R = Geo<B, sizeof(T), false>;
    const auto* fa = static_cast<const RecArgs<T>*>(args);
    if (quant) {
      auto k = k_batch_recompose<T, B, true>;
      hipLaunchKernelGGL(k, dim3(task_grid(ntasks)), dim3(R::NT), 0, st, fa, first, nf, ntasks);
    } else {
      auto k = k_batch_recompose<T, B, false>;
      hipLaunchKernelGGL(k, dim3(task_grid(ntasks)), dim3(R::NT), 0, st, fa, first, nf, ntasks);
    }
  }
  BM_HIP(hipGetLastError());
}

template <int B>
void dispatch_dec(const bm_plan_s& p, int s, const View3& src, bool first, void* coeff, void* cout, int32_t* codes,
                  const QPrep* q, hipStream_t st) {
  if (p.cfg.dtype == BM_F32)
    launch_dec<float, B>(p, s, src, first, coeff, cout, codes, q, st);
  else
    launch_dec<double, B>(p, s, src, first, coeff, cout, codes, q, st);
}

template <int B>
void dispatch_rec(const bm_plan_s& p, int s, const void* coeff, const void* cin, void* out, bool last,
                  const int32_t* codes, const QPrep* q, hipStream_t st) {
  if (p.cfg.dtype == BM_F32)
    launch_rec<float, B>(p, s, coeff, cin, out, last, codes, q, st);
  else
    launch_rec<double, B>(p, s, coeff, cin, out, last, codes, q, st);
}

template <typename T>
void launch_dec_nest(const bm_plan_s& p, int s, const View3& src, bool first, void* coeff, int32_t* codes,
                     const QPrep* q, hipStream_t st) {
  using G = Geo<17, sizeof(T)>;
  DecArgs<T> a1 = dec_args<T, 17>(p, s, src, first, coeff, nullptr, codes, q);
  a1.nest = 1;
  const DecArgs<T> a2 = dec_args<T, 9>(p, s + 1, dense_view(p.ws.grid[s], p.lv[s].n), false, coeff,
                                       p.ws.grid[s + 1], codes, q);
  if (a1.fuse || a1.coarsest_here || a2.nblocks != a1.nblocks) fail(BM_EINVAL, "nested pair: inconsistent levels");
  if (q)
    hipLaunchKernelGGL((k_local_decompose_nest<T, true>), dim3(unsigned(8 * a1.per)), dim3(G::NT), 0, st, a1, a2);
  else
    hipLaunchKernelGGL((k_local_decompose_nest<T, false>), dim3(unsigned(8 * a1.per)), dim3(G::NT), 0, st, a1, a2);
  BM_HIP(hipGetLastError());
}

template <typename T, int NB, bool ROWS>
void launch_rec_pairs(const bm_plan_s& p, int s, const void* coeff, const void* cin, void* out, bool last,
                      const int32_t* codes, const QPrep* q, hipStream_t st) {
  const RecArgs<T> a1 = rec_args<T, 17>(p, s, coeff, nullptr, out, last, codes, q, false, NB);
  const RecArgs<T> a2 = rec_args<T, 9>(p, s + 1, coeff, cin, nullptr, false, codes, q, false);
  if (a1.fuse || a1.coarsest_here || a2.nblocks != a1.nblocks) fail(BM_EINVAL, "nested pair: inconsistent levels");
  auto* const k = q ? k_local_recompose_nest<T, true, NB, ROWS> : k_local_recompose_nest<T, false, NB, ROWS>;
  hipLaunchKernelGGL(k, dim3(unsigned(8 * a1.per)), dim3((NB * 289 + 63) / 64 * 64), 0, st, a2, a1);
  BM_HIP(hipGetLastError());
}

// share of a recomposition level's nodes (whole blocks) in its output
inline double whole(const bm_plan_s& p, int s, bool last) {
  double w = 1.0;
  for (int k = 0; k < 3; ++k) w *= last ? double(p.dims[k]) / double(p.lv[s - 1].n[k]) : 1.0;
  return w;
}

// FP32 pairs: two blocks a workgroup share the lines between them, which pays
// where many workgroups write most of what they span; with few blocks, or an
// output cropped to a part of them, workgroups of one block start and end
// sooner; under codes and a global level, whose coarse values come from one
// more grid, one block in plain rows.  us, one block in groups of 16 / one in
// rows / two, without codes; with:
//   257^3, M = 0        34 / 37 / 38;      32 / 33 / 38
//   513^3, M = 0        429 / 393 / 362;   410 / 377 / 362
//   513^3, M = 1        439 / 403 / 377;   435 / 405 / 409
//   98 x 1200^2, M = 1  465 / 449 / 443;   475 / 463 / 487
//   1 x 4096^2, M = 0   471 / 456 / 523;   473 / 475 / 565
//   1 x 4096^2, M = 1   543 / 533 / 620;   600 / 604 / 698
template <typename T>
void launch_rec_nest(const bm_plan_s& p, int s, const void* coeff, const void* cin, void* out, bool last,
                     const int32_t* codes, const QPrep* q, hipStream_t st) {
  if constexpr (sizeof(T) == 8) {
    launch_rec_pairs<T, 1, true>(p, s, coeff, cin, out, last, codes, q, st);
  } else {
    const Level& L = p.lv[s - 1];
    const bool fused = p.fuse_next && s + 1 == p.L;
    if (L.nb[0] * L.nb[1] * L.nb[2] < 8192 || whole(p, s, last) < 0.75)
      launch_rec_pairs<T, 1, false>(p, s, coeff, cin, out, last, codes, q, st);
    else if (q && fused)
      launch_rec_pairs<T, 1, true>(p, s, coeff, cin, out, last, codes, q, st);
    else
      launch_rec_pairs<T, 2, false>(p, s, coeff, cin, out, last, codes, q, st);
  }
}

}  // namespace

bool nest_pair(const bm_plan_s& p, int s) {
  return p.cfg.nested && s >= 1 && s < p.L && p.lv[s - 1].b == 17 && p.lv[s].b == 9;
}

void local_decompose_nest(const bm_plan_s& p, int s, const View3& src, bool first, void* coeff, int32_t* codes,
                          const QPrep* q, hipStream_t st) {
  if (!nest_pair(p, s)) fail(BM_EINVAL, "block levels s, s+1 are not a nested 17/9 pair");
  if (p.cfg.dtype == BM_F32)
    launch_dec_nest<float>(p, s, src, first, coeff, codes, q, st);
  else
    launch_dec_nest<double>(p, s, src, first, coeff, codes, q, st);
}

void local_recompose_nest(const bm_plan_s& p, int s, const void* coeff, const void* cin, void* out, bool last,
                          const int32_t* codes, const QPrep* q, hipStream_t st) {
  if (!nest_pair(p, s)) fail(BM_EINVAL, "block levels s, s+1 are not a nested 17/9 pair");
  if (p.cfg.dtype == BM_F32)
    launch_rec_nest<float>(p, s, coeff, cin, out, last, codes, q, st);
  else
    launch_rec_nest<double>(p, s, coeff, cin, out, last, codes, q, st);
}

void local_decompose(const bm_plan_s& p, int s, const View3& src, bool first, void* coeff, void* coarse_out,
                     hipStream_t st) {
  if (p.lv[s - 1].b == 33)
    wide_decompose(p, s, src, first, coeff, coarse_out, nullptr, nullptr, st);
  else if (p.lv[s - 1].b == 9)
    dispatch_dec<9>(p, s, src, first, coeff, coarse_out, nullptr, nullptr, st);
  else
    dispatch_dec<17>(p, s, src, first, coeff, coarse_out, nullptr, nullptr, st);
}

void local_recompose(const bm_plan_s& p, int s, const void* coeff, const void* coarse_in, void* out, bool last,
                     hipStream_t st) {
  if (p.lv[s - 1].b == 33)
    wide_recompose(p, s, coeff, const_cast<void*>(coarse_in), out, last, nullptr, nullptr, st);
  else if (p.lv[s - 1].b == 9)
    dispatch_rec<9>(p, s, coeff, coarse_in, out, last, nullptr, nullptr, st);
  else
    dispatch_rec<17>(p, s, coeff, coarse_in, out, last, nullptr, nullptr, st);
}

void local_decompose_q(const bm_plan_s& p, int s, const View3& src, bool first, int32_t* codes, void* coarse_out,
                       const QPrep& q, hipStream_t st) {
  if (p.lv[s - 1].b == 33)
    wide_decompose(p, s, src, first, nullptr, coarse_out, codes, &q, st);
  else if (p.lv[s - 1].b == 9)
    dispatch_dec<9>(p, s, src, first, nullptr, coarse_out, codes, &q, st);
  else
    dispatch_dec<17>(p, s, src, first, nullptr, coarse_out, codes, &q, st);
}

void local_recompose_q(const bm_plan_s& p, int s, const int32_t* codes, const void* coarse_in, void* out, bool last,
                       const QPrep& q, hipStream_t st) {
  if (p.lv[s - 1].b == 33)
    wide_recompose(p, s, nullptr, const_cast<void*>(coarse_in), out, last, codes, &q, st);
  else if (p.lv[s - 1].b == 9)
    dispatch_rec<9>(p, s, nullptr, coarse_in, out, last, codes, &q, st);
  else
    dispatch_rec<17>(p, s, nullptr, coarse_in, out, last, codes, &q, st);
}

int64_t block_groups(const bm_plan_s& p, int s, bool dec) {
  const int nbw = p.lv[s - 1].b <= 9 ? Geo<9>::NB
                                   : (p.esize == 4 ? (dec ? Geo<17, 4, true>::NB : Geo<17, 4, false>::NB) : Geo<17, 8>::NB);
  const int64_t* nb = p.lv[s - 1].nb;
  return (nb[0] * nb[1] * nb[2] + nbw - 1) / nbw;
}

size_t block_args_size(const bm_plan_s& p, bool dec) {
  if (p.cfg.dtype == BM_F32) return dec ? sizeof(DecArgs<float>) : sizeof(RecArgs<float>);
  return dec ? sizeof(DecArgs<double>) : sizeof(RecArgs<double>);
}

void block_dec_args(const bm_plan_s& p, int s, const View3& src, bool first, void* coeff, void* cout, int32_t* codes,
                    const QPrep* q, void* out) {
  if (p.cfg.dtype == BM_F32) {
    const auto a = p.lv[s - 1].b == 9 ? dec_args<float, 9>(p, s, src, first, coeff, cout, codes, q)
                                    : dec_args<float, 17>(p, s, src, first, coeff, cout, codes, q);
    std::memcpy(out, &a, sizeof(a));
  } else {
    const auto a = p.lv[s - 1].b == 9 ? dec_args<double, 9>(p, s, src, first, coeff, cout, codes, q)
                                    : dec_args<double, 17>(p, s, src, first, coeff, cout, codes, q);
    std::memcpy(out, &a, sizeof(a));
  }
}

void block_rec_args(const bm_plan_s& p, int s, const void* coeff, const void* cin, void* outp, bool last,
                    const int32_t* codes, const QPrep* q, void* out) {
  if (p.cfg.dtype == BM_F32) {
    const auto a = p.lv[s - 1].b == 9 ? rec_args<float, 9>(p, s, coeff, cin, outp, last, codes, q)
                                    : rec_args<float, 17>(p, s, coeff, cin, outp, last, codes, q);
    std::memcpy(out, &a, sizeof(a));
  } else {
    const auto a = p.lv[s - 1].b == 9 ? rec_args<double, 9>(p, s, coeff, cin, outp, last, codes, q)
                                    : rec_args<double, 17>(p, s, coeff, cin, outp, last, codes, q);
    std::memcpy(out, &a, sizeof(a));
  }
}

void launch_block_batch(int block, int dtype, bool dec, bool quant, const void* args, const int64_t* first, int nf,
                        int64_t ntasks, hipStream_t st) {
  if (dtype == BM_F32) {
    if (block == 9)
      launch_batch<float, 9>(dec, quant, args, first, nf, ntasks, st);
    else
      launch_batch<float, 17>(dec, quant, args, first, nf, ntasks, st);
  } else {
    if (block == 9)
      launch_batch<double, 9>(dec, quant, args, first, nf, ntasks, st);
    else
      launch_batch<double, 17>(dec, quant, args, first, nf, ntasks, st);
  }
}

namespace {

template <typename T>
void nest_dec_pair(const bm_plan_s& p, const View3& src, int32_t* codes, const QPrep* q, void* out1, void* out2) {
  DecArgs<T> a1 = dec_args<T, 17>(p, 1, src, true, nullptr, nullptr, codes, q);
  a1.nest = 1;
  const DecArgs<T> a2 = dec_args<T, 9>(p, 2, dense_view(p.ws.grid[1], p.lv[1].n), false, nullptr, p.ws.grid[2], codes, q);
  if (a1.fuse || a1.coarsest_here || a2.nblocks != a1.nblocks) fail(BM_EINVAL, "nested pair: inconsistent levels");
  std::memcpy(out1, &a1, sizeof(a1));
  std::memcpy(out2, &a2, sizeof(a2));
}

template <typename T>
void nest_rec_pair(const bm_plan_s& p, void* x, const int32_t* codes, const QPrep* q, void* out1, void* out2) {
  const RecArgs<T> a1 = rec_args<T, 17>(p, 1, nullptr, nullptr, x, true, codes, q, false);
  const RecArgs<T> a2 = rec_args<T, 9>(p, 2, nullptr, p.ws.grid[2], nullptr, false, codes, q, false);
  if (a1.fuse || a1.coarsest_here || a2.nblocks != a1.nblocks) fail(BM_EINVAL, "nested pair: inconsistent levels");
  std::memcpy(out1, &a1, sizeof(a1));
  std::memcpy(out2, &a2, sizeof(a2));
}

template <typename T>
void launch_batch_nest(bool dec, const void* a1, const void* a2, const int64_t* first, int nf, int64_t ntasks,
                       hipStream_t st) {
  if (ntasks <= 0) return;
  if (dec) {
    auto k = k_batch_decompose_nest<T, true>;
    const int nt = Geo<17, sizeof(T)>::NT;
    hipLaunchKernelGGL(k, dim3(task_grid(ntasks)), dim3(nt), 0, st, static_cast<const DecArgs<T>*>(a1),
                       static_cast<const DecArgs<T>*>(a2), first, nf, ntasks);
  } else {
    auto k = k_batch_recompose_nest<T, true>;
    const int nt = Geo<17, sizeof(T), false>::NT;
    hipLaunchKernelGGL(k, dim3(task_grid(ntasks)), dim3(nt), 0, st, static_cast<const RecArgs<T>*>(a1),
                       static_cast<const RecArgs<T>*>(a2), first, nf, ntasks);
  }
  BM_HIP(hipGetLastError());
}

}  // namespace

// Arguments of a field's nested pair (17-node level 1, 9-node level 2) for
// the batched nest launch: out1 gets level 1's, out2 level 2's (each
// block_args_size bytes).
void block_nest_args(const bm_plan_s& p, bool dec, const View3& src, void* x, int32_t* codes, const QPrep* q,
                     void* out1, void* out2) {
  if (!nest_pair(p, 1)) fail(BM_EINVAL, "block levels 1, 2 are not a nested 17/9 pair");
  if (dec) {
    if (p.cfg.dtype == BM_F32)
      nest_dec_pair<float>(p, src, codes, q, out1, out2);
    else
      nest_dec_pair<double>(p, src, codes, q, out1, out2);
  } else {
    if (p.cfg.dtype == BM_F32)
      nest_rec_pair<float>(p, x, codes, q, out1, out2);
    else
      nest_rec_pair<double>(p, x, codes, q, out1, out2);
  }
}

void launch_block_batch_nest(int dtype, bool dec, const void* a1, const void* a2, const int64_t* first, int nf,
                             int64_t ntasks, hipStream_t st) {
  if (dtype == BM_F32)
    launch_batch_nest<float>(dec, a1, a2, first, nf, ntasks, st);
  else
    launch_batch_nest<double>(dec, a1, a2, first, nf, ntasks, st);
}

}  // namespace bm
