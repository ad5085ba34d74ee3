// Lossless stage: canonical Huffman coding of the quantization codes
// (the paper's pipeline ends with Huffman stages for outliers, histogram,
// codebook, encoding; Sec. IV-B).
//
// Symbols: q + 2^15 for |q| < 2^15, else the escape symbol 0 with the
// value q kept as an outlier, in raster order: an outlier's position is
// that of its escape symbol, and per-chunk outlier offsets locate the
// outliers of each chunk (stream version 3).  Code lengths come from
// Huffman's algorithm merging the two smallest (weight, smallest symbol in
// the subtree) keys, so the tree is unique; lengths above 32 are cut to 32
// and the longest codes below 32 are lengthened (largest symbol first) until
// Kraft's sum is <= 1.  Codes are canonical in (length, symbol) order.
// The stream is cut into chunks of 4096 symbols, each packed MSB-first into
// 32-bit words and starting on a word boundary.
//
// GPU work: an LDS-privatised histogram; bit counts and encode with a
// workgroup of 256 threads per chunk (16 consecutive symbols per thread,
// their bit offsets from a workgroup scan, LDS atomic ORs into the chunk's
// words); decode with four wavefronts per chunk.  Decoding a chunk is split
// over its 256 lanes by bit position: lane l owns the codewords that start in
// the l-th 1/256 of the chunk's bits.  Where that first codeword starts is
// only known once lane l - 1 has decoded, so every lane first decodes its part
// from a guessed start (the part's first bit) and hands its end position to
// the next lane; the hand-over is repeated, re-decoding only the lanes whose
// start changed, until no start changes, which is the exact decomposition
// (the fixed point of "start of lane l + 1 = end of lane l from the start of
// lane l", reached in at most 256 rounds).  Huffman codes resynchronise within
// a few codewords from a wrong start, so a few rounds are the rule
// (self-synchronising parallel decoding, as in Weissenberger and Schmidt,
// ICPP 2018).  The codebook is built on the host.

#include <algorithm>
#include <chrono>
#include <cstring>
#include <functional>
#include <memory>
#include <mutex>

#include "internal.h"

namespace bm {
namespace {

constexpr int R = 1 << 15;
constexpr int NSYM = 2 * R;
constexpr int CHUNK = 4096;
constexpr int LMAX = 32;
constexpr int HW = 4096;             // LDS histogram window: symbols [R - HW, R + HW)
constexpr int DLB = 11;              // decode lookup bits
constexpr int ET = 256;              // threads per chunk in the bit count and the encode
constexpr int EPT = CHUNK / ET;      // consecutive symbols per thread there
constexpr uint32_t kNoPos = 0xFFFFFFFFu;   // decode position after an invalid code
constexpr size_t kLdsCap = 64 * 1024;      // LDS bytes a decode workgroup may take

using clk = std::chrono::steady_clock;
inline double ms_since(clk::time_point t0) {
  return std::chrono::duration<double, std::milli>(clk::now() - t0).count();
}

__device__ inline uint32_t sym_of(int32_t q) { return (q > -R && q < R) ? uint32_t(q + R) : 0u; }

// LDS bins: [0, 2 HW) for symbols R-HW .. R+HW-1, bin 2 HW for the escape
// symbol; everything else (rare) goes straight to the global histogram.
// Atomics bound it: in LDS, where neighbouring codes often share a bin (even
// and odd lanes count apart), and at the end, when every workgroup adds its
// bins to the same global ones (so two workgroups of 1024 lanes per CU
// instead of eight of 256).  Codes are read 16 bytes a lane (VEC: the array
// is 16-byte aligned).  135 M codes of the 512^3 ROI field: 0.340 -> 0.144 ms.
constexpr int kHistNT = 1024, kHistGroups = 512;

template <bool VEC>
__global__ __launch_bounds__(kHistNT) void k_hist(const int32_t* codes, int64_t n, unsigned long long* hist) {
  __shared__ uint32_t h[2][2 * HW + 1];
  for (int i = threadIdx.x; i < 2 * (2 * HW + 1); i += kHistNT) (&h[0][0])[i] = 0;
  __syncthreads();
  uint32_t* const mine = h[threadIdx.x & 1];
  auto count = [&](int32_t q) {
    const uint32_t s = sym_of(q);
    const uint32_t k = s - uint32_t(R - HW);
    if (s == 0)
      atomicAdd(&mine[2 * HW], 1u);
    else if (k < 2 * HW)
      atomicAdd(&mine[k], 1u);
    else
      atomicAdd(&hist[s], 1ull);
  };
  const int64_t t = int64_t(blockIdx.x) * kHistNT + threadIdx.x, nt = int64_t(gridDim.x) * kHistNT;
  const int64_t n4 = VEC ? n / 4 : 0;
  const int4* v = reinterpret_cast<const int4*>(codes);
  int64_t i = t;
  for (; i + nt < n4; i += 2 * nt) {
    const int4 a = v[i], b = v[i + nt];
    count(a.x);
    count(a.y);
    count(a.z);
    count(a.w);
    count(b.x);
    count(b.y);
    count(b.z);
    count(b.w);
  }
  for (; i < n4; i += nt) {
    const int4 a = v[i];
    count(a.x);
    count(a.y);
    count(a.z);
    count(a.w);
  }
  for (i = 4 * n4 + t; i < n; i += nt) count(codes[i]);
  __syncthreads();
  for (int k = threadIdx.x; k <= 2 * HW; k += kHistNT) {
    const uint32_t c = h[0][k] + h[1][k];
    if (c) atomicAdd(&hist[k == 2 * HW ? 0 : R - HW + k], (unsigned long long)c);
  }
}

__global__ void k_zero_u64(unsigned long long* p, int64_t n) {
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256) p[i] = 0;
}

__device__ inline uint32_t wave_incl_scan(uint32_t v, int lane) {
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t t = __shfl_up(v, off, 64);
    if (lane >= off) v += t;
  }
  return v;
}

__device__ inline uint32_t wave_excl_scan(uint32_t v, int lane) { return wave_incl_scan(v, lane) - v; }

// The EPT consecutive codes [i0, i0 + EPT) of a chunk of cnt codes at p
// (0 past cnt); VEC: 16-byte loads (p is 16-byte aligned).
template <bool VEC>
__device__ inline void load_run(const int32_t* p, int i0, int cnt, int32_t (&q)[EPT]) {
  if (VEC && i0 + EPT <= cnt) {
    const int4* v = reinterpret_cast<const int4*>(p + i0);
#pragma unroll
    for (int k = 0; k < EPT / 4; ++k) {
      const int4 w = v[k];
      q[4 * k] = w.x;
      q[4 * k + 1] = w.y;
      q[4 * k + 2] = w.z;
      q[4 * k + 3] = w.w;
    }
  } else {
#pragma unroll
    for (int k = 0; k < EPT; ++k) q[k] = i0 + k < cnt ? p[i0 + k] : 0;
  }
}

// bits and escapes of each chunk (a workgroup per chunk)
template <bool VEC>
__global__ __launch_bounds__(ET) void k_chunk_bits(const int32_t* codes, int64_t n, const uint8_t* len,
                                                   uint32_t* bits, uint32_t* esc) {
  __shared__ uint32_t part[2][ET / 64];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t c = blockIdx.x, b0 = c * CHUNK;
  const int cnt = int(b0 + CHUNK < n ? CHUNK : n - b0);
  int32_t q[EPT];
  load_run<VEC>(codes + b0, EPT * t, cnt, q);
  uint32_t nb = 0, ne = 0;
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    if (EPT * t + k < cnt) {
      const uint32_t s = sym_of(q[k]);
      nb += len[s];
      ne += s == 0;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    nb += __shfl_down(nb, off, 64);
    ne += __shfl_down(ne, off, 64);
  }
  if (lane == 0) {
    part[0][wave] = nb;
    part[1][wave] = ne;
  }
  __syncthreads();
  if (t == 0) {
    uint32_t sb = 0, se = 0;
    for (int w = 0; w < ET / 64; ++w) {
      sb += part[0][w];
      se += part[1][w];
    }
    bits[c] = sb;
    esc[c] = se;
  }
}

// a 32-bit little-endian store; BYTES: four byte stores (a destination that
// is not 4-byte aligned)
template <bool BYTES>
__device__ inline void store32(void* base, uint64_t i, uint32_t v) {
  if (BYTES) {
    uint8_t* p = static_cast<uint8_t*>(base) + 4 * i;
    p[0] = uint8_t(v);
    p[1] = uint8_t(v >> 8);
    p[2] = uint8_t(v >> 16);
    p[3] = uint8_t(v >> 24);
  } else {
    static_cast<uint32_t*>(base)[i] = v;
  }
}

// A workgroup per chunk; thread t codes symbols [16 t, 16 t + 16) of the
// chunk at the bit offset a workgroup scan of the code lengths gives, OR-ing
// each code into the chunk's words in LDS (dynamic size: the longest chunk's
// words).  Code lengths and codes are looked up for all 16 symbols before any
// is placed, so the table reads overlap.
template <bool BYTES, bool VEC>
__global__ __launch_bounds__(ET) void k_encode(const int32_t* codes, int64_t n, const uint8_t* len,
                                               const uint32_t* cw, const uint64_t* woff, const uint64_t* ooff,
                                               void* words, void* oval) {
  extern __shared__ uint32_t out[];
  __shared__ uint32_t part[2][ET / 64];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t c = blockIdx.x, b0 = c * CHUNK;
  const int cnt = int(b0 + CHUNK < n ? CHUNK : n - b0);
  const uint64_t w0 = woff[c];
  const uint32_t nw = uint32_t(woff[c + 1] - w0);
  for (uint32_t i = t; i < nw; i += ET) out[i] = 0;
  int32_t q[EPT];
  load_run<VEC>(codes + b0, EPT * t, cnt, q);
  uint32_t l[EPT], v[EPT];
  uint32_t nb = 0, ne = 0;
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    l[k] = 0;
    v[k] = 0;
    if (EPT * t + k < cnt) {
      const uint32_t s = sym_of(q[k]);
      l[k] = len[s];
      v[k] = cw[s];
      ne += s == 0;
    }
    nb += l[k];
  }
  const uint32_t ib = wave_incl_scan(nb, lane), ie = wave_incl_scan(ne, lane);
  if (lane == 63) {
    part[0][wave] = ib;
    part[1][wave] = ie;
  }
  __syncthreads();
  uint32_t p = ib - nb, pe = ie - ne;
  for (int w = 0; w < wave; ++w) {
    p += part[0][w];
    pe += part[1][w];
  }
  uint64_t e = ooff[c] + pe;
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    if (l[k] == 0) break;   // past the chunk's end (a coded symbol has a length >= 1)
    const uint32_t w = p >> 5, o = p & 31;
    if (o + l[k] <= 32) {
      atomicOr(&out[w], v[k] << (32 - o - l[k]));
    } else {
      atomicOr(&out[w], v[k] >> (o + l[k] - 32));
      atomicOr(&out[w + 1], v[k] << (64 - o - l[k]));
    }
    p += l[k];
    if (q[k] <= -R || q[k] >= R) store32<BYTES>(oval, e++, uint32_t(q[k]));
  }
  __syncthreads();
  for (uint32_t i = t; i < nw; i += ET) store32<BYTES>(words, w0 + i, out[i]);
}

// ------------------------------------------------------------------ decode
// Tables (built on the host from the code lengths):
// * lut[2^DLB], indexed by the next DLB bits: for a code of l <= DLB bits,
//   its symbol | l << 16; for a prefix whose codes all
//   have one length l > DLB and fill it, kOne | the index of its first code
//   | l << 16 (the code's index is that plus the l - DLB bits after the
//   prefix); for any other prefix of longer codes, kLong | Lmin << 16 |
//   Lmax << 24, the shortest and longest code lengths with that prefix; 0 for
//   a prefix of no code;
// * lastc[L]: the largest 32-bit left-justified code value of length <= L
//   (codes are canonical, so a code of length L is the 32-bit window w with
//   lastc[L - 1] < w <= lastc[L]);
// * offs[L]: index in canonical order of a code of length L minus its value;
// * sorted16: the coded symbols in canonical order (device memory).
constexpr uint32_t kLong = 0x80000000u;
constexpr uint32_t kOne = 0x40000000u;
constexpr int kDecHdrWords = (1 << DLB) + 2 * (LMAX + 1);

struct DecTables {
  const uint32_t* hdr;        // [kDecHdrWords]: lut, lastc, offs
  const uint16_t* sorted16;   // coded symbols in (length, symbol) order
  uint32_t nsorted;           // their count (>= 1)
  uint32_t escidx;            // index of the escape symbol in canonical order (nsorted: none)
};

struct DecLds {
  const uint32_t* lut;
  const uint32_t* lastc;
  const uint32_t* offs;
};

// Decodes the codewords of a chunk that start at x and after, while they
// start before hi.  wl: the chunk's words in LDS followed by two zero words.
// Returns the position of the first codeword at or past hi (x itself when
// x >= hi), or kNoPos at an invalid code; ns counts the codewords decoded.
// With EMIT, emit(k, v, lng, e) receives for the k-th code its symbol (lng
// false: a code of at most DLB bits) or its index in canonical order (lng
// true) and the position where it ends.  Each step reads the two words under
// the position (one LDS instruction) and shifts them, so a step is a dozen
// vector instructions; an invalid code ends the loop through its condition
// (pos = kNoPos), so the loop has a single exit and the common path no branch
// but the rare long-code one.
template <bool EMIT, typename Emit>
__device__ inline uint32_t decode_run(const uint32_t* wl, const DecLds& d, uint32_t x, uint32_t hi, uint32_t& ns,
                                      Emit emit) {
  ns = 0;
  uint32_t pos = x;
  while (pos < hi) {
    const uint32_t i = pos >> 5;   // i + 1 <= nw while pos < hi <= 32 nw
    const uint64_t win = (uint64_t(wl[i]) << 32) | wl[i + 1];
    const uint32_t top = uint32_t((win << (pos & 31)) >> 32);
    const uint32_t lu = d.lut[top >> (32 - DLB)];
    uint32_t l = (lu >> 16) & 63u, v = lu & 0xFFFFu;
    if (lu & kLong) {   // a prefix of codes of several lengths, or one they do not fill (rare)
      const uint32_t lmax = (lu >> 24) & 63u;
      uint32_t lc = d.lastc[l];
      while (top > lc && l < lmax) lc = d.lastc[++l];
      if (EMIT) v = d.offs[l] + (top >> (32 - l));
      if (top > lc) l = 0;
    } else if (EMIT && (lu & kOne)) {
      v += (top << DLB) >> (32 - l + DLB);
    }
    const bool valid = l != 0;
    if (EMIT && valid) emit(ns, v, l > DLB, pos + l);
    ns += valid;
    pos = valid ? pos + l : kNoPos;
  }
  return pos;
}

// Decode: CPW chunks per workgroup, WPC wavefronts (NL = 64 WPC lanes) per
// chunk; chunk lane L owns the codewords that start in the L-th 1/NL of the
// chunk's bits.  LDS: the tables (shared), then per chunk its words
// (wcap + 2), a bit mask of the tile's long codes, a tile of its 4096 symbols
// (uint16; for a code longer than DLB bits its index in canonical order) and
// a small control block.  Rounds of the start hand-over end with workgroup
// barriers (lane 63 of a wavefront hands its end to lane 0 of the next
// through LDS).  The tile is turned into codes by the chunk's wavefronts, a
// segment of 4096 / WPC positions each, 256 at a time: the long codes'
// symbols gathered from sorted16 (only the lanes that hold one load), then
// stored 64 consecutive codes per instruction; an escape's position in the
// chunk goes to rel (in outlier order) and k_outliers puts the outlier values
// in place afterwards, so no lane waits for a load from the outlier array.
// A chunk whose symbols do not decode from its own words (an invalid code,
// too few codewords, a codeword that runs past the chunk's last word) or
// whose escapes do not match its outlier count raises the flag (the caller
// then fails); bits after the chunk's last symbol are not read as symbols.
constexpr int kCtl = 20;   // control words per chunk: hand-over [4], first bad lane [4], wave totals [8], escapes [4]

template <int WPC, int CPW>
__global__ __launch_bounds__(64 * WPC * CPW) void k_decode(const uint32_t* words, const uint64_t* woff, int64_t nch,
                                                           int64_t n, DecTables t, const uint64_t* ooff,
                                                           uint16_t* rel, int32_t* codes, int* err, int wcap) {
  static_assert(WPC == 1 || WPC == 2 || WPC == 4, "1, 2 or 4 wavefronts per chunk");
  constexpr int NL = 64 * WPC, SEG = CHUNK / WPC;
  extern __shared__ uint32_t smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int slot = wave / WPC, wic = wave % WPC, L = wic * 64 + lane;
  const int per = wcap + 2 + CHUNK / 32 + CHUNK / 2 + kCtl;
  uint32_t* flag = smem + kDecHdrWords;                     // [2] workgroup: a start changed in the round
  uint32_t* wl = smem + kDecHdrWords + 2 + slot * per;      // chunk words, two zero words
  uint32_t* lmask = wl + wcap + 2;
  uint16_t* tile = reinterpret_cast<uint16_t*>(lmask + CHUNK / 32);
  uint32_t* ctl = lmask + CHUNK / 32 + CHUNK / 2;
  uint32_t* xch = ctl;        // [WPC] end of each wavefront's lane 63
  uint32_t* fbad = ctl + 4;   // [WPC] first lane of each wavefront that met an invalid code (64: none)
  uint32_t* wtot = ctl + 8;   // [WPC] codewords of each wavefront; [WPC] of lanes up to the first bad one
  uint32_t* esc = ctl + 16;   // [WPC] escapes in each tile segment
  for (int i = tid; i < kDecHdrWords; i += 64 * WPC * CPW) smem[i] = t.hdr[i];
  if (tid < 2) flag[tid] = 0;
  const int64_t c = int64_t(blockIdx.x) * CPW + slot;
  const bool valid = c < nch;   // uniform over the chunk's wavefronts
  uint64_t w0 = 0;
  uint32_t nw = 0;
  if (valid) {
    w0 = woff[c];
    nw = uint32_t(woff[c + 1] - w0);   // <= wcap (checked on the host)
  }
  for (uint32_t i = L; i < nw + 2; i += NL) wl[i] = i < nw ? words[w0 + i] : 0u;
  for (int i = L; i < CHUNK / 32; i += NL) lmask[i] = 0;
  if (L < kCtl) ctl[L] = 0;
  __syncthreads();
  const DecLds d{smem, smem + (1 << DLB), smem + (1 << DLB) + (LMAX + 1)};
  const int64_t b0 = c * CHUNK;
  const uint32_t cnt = valid ? uint32_t(b0 + CHUNK < n ? CHUNK : n - b0) : 0u;
  const uint32_t NB = nw * 32, S = max((NB + NL - 1) / NL, 32u);
  const uint32_t lo = min(uint32_t(L) * S, NB), hi = min(lo + S, NB);
  auto none = [](uint32_t, uint32_t, bool, uint32_t) {};
  // The lanes' start positions: guessed, then handed over until they hold.
  // A lane whose predecessor met an invalid code keeps its own start (a
  // wrong start of the predecessor is the likely cause); lanes up to the
  // first one that ends in an invalid code hold exact starts at the fixed
  // point, and only their symbols are used.
  // Later rounds decode only the lanes whose start changed.
  uint32_t x = lo, ns = 0, end = 0;
  bool ok = false, dirty = true;
  for (int round = 0; round <= NL; ++round) {
    if (dirty) end = decode_run<false>(wl, d, x, hi, ns, none);
    if (lane == 63) xch[wic] = end;
    __syncthreads();
    uint32_t xn = __shfl_up(end, 1, 64);
    if (lane == 0) xn = wic ? xch[wic - 1] : 0u;
    if (xn == kNoPos) xn = x;
    dirty = xn != x;
    if (__any(dirty) && lane == 0) atomicOr(&flag[round & 1], 1u);
    __syncthreads();
    const bool again = flag[round & 1] != 0;
    if (tid == 0) flag[(round + 1) & 1] = 0;
    x = xn;
    if (!again) {
      ok = true;
      break;
    }
  }
  // lanes past the chunk's first one that ends in an invalid code are not used
  const uint64_t badm = __ballot(end == kNoPos);
  const uint32_t fb = badm ? uint32_t(__ffsll((unsigned long long)badm) - 1) : 64u;
  const uint32_t incl = wave_incl_scan(ns, lane);
  if (lane == 63) {
    fbad[wic] = fb;
    wtot[wic] = incl;
  }
  if (fb < 64 && uint32_t(lane) == fb) wtot[4 + wic] = incl;
  __syncthreads();
  uint32_t before = 0, total = 0, lastw = WPC;
  for (int w = 0; w < WPC; ++w) {
    if (lastw == WPC && fbad[w] < 64) lastw = uint32_t(w);
    if (w < wic) before += wtot[w];
  }
  for (int w = 0; w < WPC; ++w) {
    if (uint32_t(w) < lastw) total += wtot[w];
    if (uint32_t(w) == lastw) total += wtot[4 + w];
  }
  const bool used = uint32_t(wic) < lastw || (uint32_t(wic) == lastw && uint32_t(lane) <= fbad[wic]);
  const uint32_t start = before + incl - ns;
  const bool good = valid && ok && total >= cnt;   // uniform over the chunk
  if (valid && !good && L == 0) atomicOr(err, 1);
  bool over = false;   // a codeword of the chunk's symbols runs past its words
  uint32_t ne[WPC] = {};
  if (good && used)
    decode_run<true>(wl, d, x, hi, ns, [&](uint32_t k, uint32_t v, bool lng, uint32_t e) {
      const uint32_t i = start + k;
      if (i < cnt) {
        tile[i] = uint16_t(v);
        if (lng) atomicOr(&lmask[i >> 5], 1u << (i & 31));
        over |= e > NB;
        if (lng ? v == t.escidx : v == 0) {
#pragma unroll
          for (int w = 0; w < WPC; ++w) ne[w] += i / SEG == uint32_t(w);
        }
      }
    });
#pragma unroll
  for (int w = 0; w < WPC; ++w)
    if (ne[w]) atomicAdd(&esc[w], ne[w]);
  if (__any(over) && lane == 0) atomicOr(err, 1);
  __syncthreads();
  if (!good) return;   // no barrier follows
  uint64_t run = ooff[c];
  for (int w = 0; w < wic; ++w) run += esc[w];
  const uint64_t e1 = ooff[c + 1];
  const uint32_t s0 = uint32_t(wic) * SEG, s1 = min(s0 + SEG, cnt);
  for (uint32_t k0 = s0; k0 < s1; k0 += 256) {
    uint32_t s[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t i = k0 + 64 * j + lane;
      s[j] = 1u;
      if (i < s1) {
        s[j] = tile[i];
        if ((lmask[i >> 5] >> (i & 31)) & 1u) s[j] = t.sorted16[min(s[j], t.nsorted - 1)];
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t i = k0 + 64 * j + lane;
      const uint64_t m = __ballot(s[j] == 0);
      if (s[j] == 0) {
        const uint64_t ei = run + __popcll(m & ((uint64_t(1) << lane) - 1));
        if (ei < e1) rel[ei] = uint16_t(i);
      }
      if (i < s1) codes[b0 + i] = int32_t(s[j]) - R;
      run += __popcll(m);
    }
  }
  // the segment's escapes as counted in the write pass, and all of them the chunk's count
  uint64_t upto = ooff[c];
  for (int w = 0; w <= wic; ++w) upto += esc[w];
  if (lane == 0 && (run != upto || (wic == WPC - 1 && upto != e1))) atomicOr(err, 1);
}

// The outlier values of each chunk to their positions (a workgroup per
// chunk).  Positions are bounded by the chunk's length: a chunk that failed
// to decode may have left its entries of rel unset (the call then fails).
__global__ __launch_bounds__(256) void k_outliers(const uint64_t* ooff, const uint16_t* rel, const int32_t* oval,
                                                  int32_t* codes, int64_t n) {
  const int64_t c = blockIdx.x, b0 = c * CHUNK;
  const uint32_t cnt = uint32_t(b0 + CHUNK < n ? CHUNK : n - b0);
  const uint64_t e0 = ooff[c], e1 = ooff[c + 1];
  for (uint64_t e = e0 + threadIdx.x; e < e1; e += 256) {
    const uint32_t r = rel[e];
    if (r < cnt) codes[b0 + r] = oval[e];
  }
}

// ------------------------------------------------------------------ host codebook
// The codebook is built in fixed arrays (no allocation), so the same code
// serves the entry point that may not allocate.

// Work arrays of the code-length construction: keys (weight << 16 | smallest
// symbol in the subtree) of the leaves in order and of the merged nodes in the
// order they are made, parents and depths of the merge tree.  Node ids: a
// leaf's symbol, NSYM + merge number.
template <typename K>
struct LenWorkOf {
  K leaf[NSYM + 1], tmp[NSYM + 1], node[NSYM + 1];
  uint32_t digit[4][2048];
  int32_t parent[2 * NSYM], depth[2 * NSYM], L[NSYM], present[NSYM];
};
using LenWork = LenWorkOf<uint64_t>;

// Stable sort by weight of np keys in symbol order, 11 bits a pass; wmax: the
// largest weight.  Each pass runs over the four quarters side by side with
// bucket positions of their own: neighbouring symbols have similar counts, so
// one run would wait at almost every key for the position it just moved.
template <typename K>
K* sort_leaves(LenWorkOf<K>& w, int np, uint64_t wmax) {
  K *A = w.leaf, *T = w.tmp;
  int q[5];
  for (int k = 0; k <= 4; ++k) q[k] = int(int64_t(np) * k / 4);
  const int run = q[1] - q[0];                          // (quarters differ by at most one)
  for (int sh = 0; sh < 64 && (wmax >> sh) != 0; sh += 11) {
    auto dig = [&](K k) { return uint32_t(uint64_t(k >> 16) >> sh) & 2047u; };
    std::memset(w.digit, 0, sizeof(w.digit));
    for (int k = 0; k < run; ++k)
      for (int j = 0; j < 4; ++j) ++w.digit[j][dig(A[q[j] + k])];
    for (int j = 0; j < 4; ++j)
      for (int k = q[j] + run; k < q[j + 1]; ++k) ++w.digit[j][dig(A[k])];
    uint32_t sum = 0;
    for (int d = 0; d < 2048; ++d)
      for (int j = 0; j < 4; ++j) {
        const uint32_t c = w.digit[j][d];
        w.digit[j][d] = sum;
        sum += c;
      }
    for (int k = 0; k < run; ++k)
      for (int j = 0; j < 4; ++j) T[w.digit[j][dig(A[q[j] + k])]++] = A[q[j] + k];
    for (int j = 0; j < 4; ++j)
      for (int k = q[j] + run; k < q[j + 1]; ++k) T[w.digit[j][dig(A[k])]++] = A[k];
    std::swap(A, T);
  }
  return A;
}

// Huffman code lengths of the symbols with hist[s] > 0 (len[s] = 0 for the
// others): merge the two smallest (weight, smallest symbol in the subtree)
// keys until one tree remains; lengths above 32 are cut to 32 and the
// longest codes below 32 are lengthened (largest symbol first) until Kraft's
// sum is <= 1.  The keys are unique, so the tree is.  Two sorted queues give
// the smallest keys in O(n): the leaves sorted by key (a stable radix sort by
// weight of the symbols in ascending order), and the merged nodes in the
// order they are made, which is key order too: merges take keys in
// increasing order, so merged weights do not decrease, and two merged nodes
// of one weight 2w both come from pairs of weight-w nodes taken in
// increasing symbol order, so their smallest symbols increase.  A queue's head
// is taken by conditional moves (which one it is cannot be predicted), an
// entry above every key behind each queue's end.
template <typename K>
void code_lengths_of(const uint64_t* hist, uint8_t* len, LenWorkOf<K>& w, int np, uint64_t wmax) {
  for (int k = 0; k < np; ++k) w.leaf[k] = K(hist[w.present[k]]) << 16 | K(w.present[k]);
  K* const A = sort_leaves(w, np, wmax);
  K* const B = w.node;
  A[np] = B[0] = ~K(0);
  int ai = 0, bi = 0, next = NSYM;
  auto pop = [&](K& key) -> int {
    const K a = A[ai], b = B[bi];
    const bool leaf = a < b;
    key = leaf ? a : b;
    const int id = leaf ? int(a & 0xFFFFu) : NSYM + bi;
    ai += leaf;
    bi += !leaf;
    return id;
  };
  for (int k = 0; k < np - 1; ++k) {
    K a, b;
    w.parent[pop(a)] = next;
    w.parent[pop(b)] = next;
    B[k] = ((a >> 16) + (b >> 16)) << 16 | std::min(a & 0xFFFFu, b & 0xFFFFu);
    B[k + 1] = ~K(0);
    ++next;
  }
  w.depth[next - 1] = 0;
  for (int v = next - 2; v >= NSYM; --v) w.depth[v] = w.depth[w.parent[v]] + 1;  // parents come after children
  int maxl = 0;
  for (int k = 0; k < np; ++k) {
    const int s = w.present[k];
    w.L[s] = w.depth[w.parent[s]] + 1;
    maxl = std::max(maxl, w.L[s]);
  }
  if (maxl > LMAX) {
    uint64_t kraft = 0;
    for (int k = 0; k < np; ++k) {
      const int s = w.present[k];
      if (w.L[s] > LMAX) w.L[s] = LMAX;
      kraft += uint64_t(1) << (LMAX - w.L[s]);
    }
    while (kraft > (uint64_t(1) << LMAX)) {
      int best = -1;
      for (int k = 0; k < np; ++k) {
        const int s = w.present[k];
        if (w.L[s] < LMAX && (best < 0 || w.L[s] > w.L[best] || (w.L[s] == w.L[best] && s > best))) best = s;
      }
      kraft -= uint64_t(1) << (LMAX - w.L[best] - 1);
      w.L[best] += 1;
    }
  }
  for (int k = 0; k < np; ++k) len[w.present[k]] = uint8_t(w.L[w.present[k]]);
}

void code_lengths(const uint64_t* hist, uint8_t* len, LenWork& w) {
  std::memset(len, 0, NSYM);
  int np = 0;
  uint64_t wmax = 0;
  for (int s = 0; s < NSYM; ++s)
    if (hist[s]) {
      w.present[np++] = s;
      wmax = std::max(wmax, hist[s]);
    }
  if (np == 0) return;
  if (np == 1) {
    len[w.present[0]] = 1;
    return;
  }
  if (wmax < (uint64_t(1) << 47) / uint64_t(np)) {      // every sum of weights fits above the symbol
    code_lengths_of(hist, len, w, np, wmax);
  } else {                                              // (counts of more codes than a call can hold)
    using K = unsigned __int128;
    std::unique_ptr<LenWorkOf<K>> big{new LenWorkOf<K>};
    std::copy(w.present, w.present + np, big->present);
    code_lengths_of(hist, len, *big, np, wmax);
  }
}

// Canonical codes in (length, symbol) order; sorted receives the coded
// symbols in that order (a counting sort by length), *nsorted their count.
void canonical(const uint8_t* len, uint32_t* code, uint32_t* sorted, int* nsorted) {
  std::memset(code, 0, NSYM * sizeof(uint32_t));
  uint32_t at[LMAX + 2] = {};
  for (int s = 0; s < NSYM; ++s)
    if (len[s]) ++at[len[s] + 1];
  for (int l = 1; l <= LMAX; ++l) at[l + 1] += at[l];
  const int n = int(at[LMAX + 1]);
  for (int s = 0; s < NSYM; ++s)
    if (len[s]) sorted[at[len[s]]++] = uint32_t(s);
  uint64_t c = 0;
  int prev = 0;
  for (int i = 0; i < n; ++i) {
    const int l = len[sorted[i]];
    if (i) c = (c + 1) << (l - prev);
    code[sorted[i]] = uint32_t(c);
    prev = l;
  }
  *nsorted = n;
}

// stream header; the code-length table lists present symbols only:
// uint16 symbol[npresent] (ascending), then uint8 length[npresent]
struct HuffHeader {
  uint32_t magic, version;
  int64_t n, nchunks, nwords, noutliers, npresent;
};
constexpr uint32_t kHuffMagic = 0x46484D42u;   // "BMHF"

struct EventPair {
  hipEvent_t a = nullptr, b = nullptr;
  EventPair() {
    BM_HIP(hipEventCreate(&a));
    BM_HIP(hipEventCreate(&b));
  }
  ~EventPair() {
    if (a) (void)hipEventDestroy(a);
    if (b) (void)hipEventDestroy(b);
  }
  double ms() const {
    BM_HIP(hipEventSynchronize(b));
    float t = 0.f;
    BM_HIP(hipEventElapsedTime(&t, a, b));
    return double(t);
  }
};

thread_local bm_lossless_times g_times{};

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

void launch_hist(const int32_t* codes, int64_t n, unsigned long long* hist, hipStream_t st) {
  hipLaunchKernelGGL(k_zero_u64, dim3(64), dim3(256), 0, st, hist, int64_t(NSYM));
  if (n) {
    const dim3 g{unsigned(std::min<int64_t>(kHistGroups, (n + 8 * kHistNT - 1) / (8 * kHistNT)))};
    if (aligned16(codes))
      hipLaunchKernelGGL(k_hist<true>, g, dim3(kHistNT), 0, st, codes, n, hist);
    else
      hipLaunchKernelGGL(k_hist<false>, g, dim3(kHistNT), 0, st, codes, n, hist);
  }
  BM_HIP(hipGetLastError());
}

void launch_chunk_bits(const int32_t* codes, int64_t n, int64_t nch, const uint8_t* len, uint32_t* bits,
                       uint32_t* esc, hipStream_t st) {
  if (!nch) return;
  if (aligned16(codes))
    hipLaunchKernelGGL(k_chunk_bits<true>, dim3(unsigned(nch)), dim3(ET), 0, st, codes, n, len, bits, esc);
  else
    hipLaunchKernelGGL(k_chunk_bits<false>, dim3(unsigned(nch)), dim3(ET), 0, st, codes, n, len, bits, esc);
  BM_HIP(hipGetLastError());
}

void launch_encode(const int32_t* codes, int64_t n, int64_t nch, const uint8_t* len, const uint32_t* cw,
                   const uint64_t* woff, const uint64_t* ooff, uint64_t wmax, void* words, void* oval,
                   hipStream_t st) {
  if (!nch) return;
  const size_t shm = size_t(wmax) * 4;
  const bool bytes = (reinterpret_cast<uintptr_t>(words) & 3) != 0;   // oval - words is a multiple of 4
  const bool vec = aligned16(codes);
  const dim3 g{unsigned(nch)}, b{unsigned(ET)};
  if (bytes && vec)
    hipLaunchKernelGGL((k_encode<true, true>), g, b, shm, st, codes, n, len, cw, woff, ooff, words, oval);
  else if (bytes)
    hipLaunchKernelGGL((k_encode<true, false>), g, b, shm, st, codes, n, len, cw, woff, ooff, words, oval);
  else if (vec)
    hipLaunchKernelGGL((k_encode<false, true>), g, b, shm, st, codes, n, len, cw, woff, ooff, words, oval);
  else
    hipLaunchKernelGGL((k_encode<false, false>), g, b, shm, st, codes, n, len, cw, woff, ooff, words, oval);
  BM_HIP(hipGetLastError());
}

constexpr int kDecWpc = 4;   // wavefronts per chunk in the decode
constexpr int kDecCpw = 2;   // chunks per decode workgroup

template <int WPC, int CPW>
void launch_decode(const uint32_t* words, const uint64_t* woff, int64_t nch, int64_t n, const DecTables& t,
                   const uint64_t* ooff, uint16_t* rel, int32_t* codes, int* err, int wcap, hipStream_t st) {
  // LDS: tables, two flags, then per chunk its words (+2), long-code mask, tile and control block
  const size_t per = size_t(wcap) + 2 + CHUNK / 32 + CHUNK / 2 + kCtl;
  const size_t bytes = (size_t(kDecHdrWords) + 2 + CPW * per) * 4;
  if (bytes > kLdsCap) fail(BM_EUNSUPPORTED, "decode workgroup does not fit in LDS");
  hipLaunchKernelGGL((k_decode<WPC, CPW>), dim3(unsigned((nch + CPW - 1) / CPW)), dim3(64 * WPC * CPW), bytes, st,
                     words, woff, nch, n, t, ooff, rel, codes, err, wcap);
}

// CRC-32 (the reflected polynomial 0xEDB88320 with pre- and post-inversion,
// as zlib) of every 16 KiB block of the code words: each lane takes 64
// consecutive bytes with a four-table byte-slicing update, then the
// workgroup folds its 256 lane CRCs in order by a tree whose level k moves
// the left CRC over the right part's 64 * 2^k bytes (crc(A B) = Z(crc(A)) ^
// crc(B), Z linear over GF(2): its 32 columns come with the launch).
struct CrcTree {
  uint32_t m[8][32];
};

__device__ inline uint32_t gf2_mul(const uint32_t (&m)[32], uint32_t v) {
  uint32_t r = 0;
#pragma unroll
  for (int i = 0; i < 32; ++i)
    if ((v >> i) & 1u) r ^= m[i];
  return r;
}

__global__ __launch_bounds__(256) void k_crc_blocks(const uint4* words, CrcTree t, uint32_t* out) {
  static_assert(kCrcBlock == 256 * 64, "one 64-byte run per lane");
  __shared__ uint32_t tab[4][256];
  __shared__ uint32_t s[256];
  const int tid = threadIdx.x;
  const uint4* q = words + (size_t(blockIdx.x) * 256 + tid) * 4;
  uint4 v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = q[k];
  uint32_t c = uint32_t(tid);
#pragma unroll
  for (int k = 0; k < 8; ++k) c = (c & 1u) ? 0xEDB88320u ^ (c >> 1) : c >> 1;
  tab[0][tid] = c;
  __syncthreads();
#pragma unroll
  for (int k = 1; k < 4; ++k) {
    c = (c >> 8) ^ tab[0][c & 0xFFu];
    tab[k][tid] = c;
  }
  __syncthreads();
  uint32_t crc = 0xFFFFFFFFu;
  auto step = [&](uint32_t w) {
    crc ^= w;
    crc = tab[3][crc & 0xFFu] ^ tab[2][(crc >> 8) & 0xFFu] ^ tab[1][(crc >> 16) & 0xFFu] ^ tab[0][crc >> 24];
  };
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    step(v[k].x);
    step(v[k].y);
    step(v[k].z);
    step(v[k].w);
  }
  s[tid] = ~crc;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int w = 1 << k;
    if ((tid & (2 * w - 1)) == 0) s[tid] = gf2_mul(t.m[k], s[tid]) ^ s[tid + w];
    __syncthreads();
  }
  if (tid == 0) out[blockIdx.x] = s[0];
}

}  // namespace

// ------------------------------------------------------------------ encoder
// One plan per code array: histogram (device), code lengths and canonical
// codes (host), per-chunk bit and escape counts (device), word and outlier
// offsets (host).  write() encodes with that plan.  Every copy between the
// host and the device goes through pinned memory, so a call waits for its
// stream three times (counts, sizes, stream) and not at each copy.
namespace {
// The calling thread's work arrays (4 MiB of ordinary memory, freed with the
// thread: clearing and first touching them cost as much as the construction,
// and pinned memory may lie on another node than the thread)
struct TableWork {
  LenWork lw;
  uint64_t hist[NSYM];
  uint8_t len[NSYM];
  uint32_t cw[NSYM], sorted[NSYM];
};
TableWork& table_work() {
  thread_local std::unique_ptr<TableWork> w{new TableWork};
  return *w;
}
}  // namespace

struct HuffmanEncoder::Impl {
  const int32_t* codes;
  int64_t n, nch;
  hipStream_t st;
  HostBuf<uint64_t> hist{NSYM}, woff, ooff;
  HostBuf<uint8_t> len{NSYM}, plen{NSYM};
  HostBuf<uint32_t> cw{NSYM}, sizes, crc;
  HostBuf<uint16_t> psym{NSYM};
  int64_t np = 0;
  uint64_t wmax = 0;
  size_t bytes = 0;
  CrcSpan span[2];      // the last write's words and outlier values
  uint32_t head = 0;    // CRC-32 of its bytes before them
  DevBuf<unsigned long long> dhist{NSYM};
  DevBuf<uint8_t> dlen{NSYM};
  DevBuf<uint32_t> dcw{NSYM};
  EventPair eh;
  IdleOnError idle;
  Impl(const int32_t* c, int64_t n_, hipStream_t s)
      : codes(c), n(n_), nch((n_ + CHUNK - 1) / CHUNK), st(s), woff(size_t(nch + 1)), ooff(size_t(nch + 1)), idle(s) {}
};

HuffmanEncoder::HuffmanEncoder(const int32_t* codes, int64_t n, hipStream_t st) {
  if (n < 0 || (n > 0 && !codes)) fail(BM_EINVAL, "bad code array");
  d_ = std::make_unique<Impl>(codes, n, st);
  Impl& I = *d_;
  bm_lossless_times& T = g_times;
  T.enc_n = n;
  T.enc_hist_ms = T.enc_table_ms = T.enc_sizes_ms = T.enc_encode_ms = T.enc_copy_ms = T.enc_crc_ms = 0.0;
  BM_HIP(hipEventRecord(I.eh.a, st));
  launch_hist(codes, n, I.dhist.p, st);
  BM_HIP(hipEventRecord(I.eh.b, st));
  BM_HIP(hipMemcpyAsync(I.hist.p, I.dhist.p, NSYM * sizeof(uint64_t), hipMemcpyDeviceToHost, st));
}

void HuffmanEncoder::plan() {
  Impl& I = *d_;
  bm_lossless_times& T = g_times;
  const int64_t nch = I.nch;
  const hipStream_t st = I.st;
  BM_HIP(hipStreamSynchronize(st));
  T.enc_hist_ms = I.eh.ms();
  const auto t1 = clk::now();
  {
    TableWork& W = table_work();
    std::memcpy(W.hist, I.hist.p, sizeof(W.hist));
    code_lengths(W.hist, W.len, W.lw);
    int ns = 0;
    canonical(W.len, W.cw, W.sorted, &ns);
    std::memcpy(I.len.p, W.len, sizeof(W.len));
    std::memcpy(I.cw.p, W.cw, sizeof(W.cw));
    uint16_t* const psym = I.psym.p;
    uint8_t* const plen = I.plen.p;
    int64_t np = 0;
    for (int s = 0; s < NSYM; ++s)
      if (W.len[s]) {
        psym[np] = uint16_t(s);
        plen[np++] = W.len[s];
      }
    I.np = np;
  }
  T.enc_table_ms = ms_since(t1);
  const auto t2 = clk::now();
  const size_t nc = size_t(std::max<int64_t>(nch, 1));
  I.sizes.reset(2 * nc);
  DevBuf<uint32_t> dsizes(2 * nc);
  IdleOnError idle(st);
  BM_HIP(hipMemcpyAsync(I.dlen.p, I.len.p, NSYM, hipMemcpyHostToDevice, st));
  BM_HIP(hipMemcpyAsync(I.dcw.p, I.cw.p, NSYM * sizeof(uint32_t), hipMemcpyHostToDevice, st));
  launch_chunk_bits(I.codes, I.n, nch, I.dlen.p, dsizes.p, dsizes.p + nc, st);
  if (nch) BM_HIP(hipMemcpyAsync(I.sizes.p, dsizes.p, 2 * nc * sizeof(uint32_t), hipMemcpyDeviceToHost, st));
  BM_HIP(hipStreamSynchronize(st));
  I.woff[0] = I.ooff[0] = 0;
  for (int64_t c = 0; c < nch; ++c) {
    const uint64_t w = (uint64_t(I.sizes[c]) + 31) / 32;
    I.wmax = std::max(I.wmax, w);
    I.woff[c + 1] = I.woff[c] + w;
    I.ooff[c + 1] = I.ooff[c] + I.sizes[nc + c];
  }
  T.enc_sizes_ms = ms_since(t2);
  I.bytes = sizeof(HuffHeader) + size_t(I.np) * 3 + size_t(nch + 1) * 16 + size_t(I.woff[nch]) * 4 +
            size_t(I.ooff[nch]) * 4;
}

HuffmanEncoder::~HuffmanEncoder() = default;

size_t HuffmanEncoder::bytes() const { return d_->bytes; }
const CrcSpan (&HuffmanEncoder::device_spans() const)[2] { return d_->span; }
uint32_t HuffmanEncoder::head_crc() const { return d_->head; }

namespace {
// the columns of the tree's shifts over 64, 128, ..., 8192 zero bytes
const CrcTree& crc_tree() {
  static const CrcTree t = [] {
    CrcTree r{};
    for (int k = 0; k < 8; ++k) crc32_shift_matrix(uint64_t(64) << k, r.m[k]);
    return r;
  }();
  return t;
}

// Launches the CRC-32 of every whole kCrcBlock of the spans' device copies
// and its copy to host (pinned): stream-ordered.
void launch_span_crcs(CrcSpan (&span)[2], const void* const (&src)[2], DevBuf<uint32_t>& dev, HostBuf<uint32_t>& host,
                      hipStream_t st) {
  for (CrcSpan& c : span) {
    c.nblk = c.bytes / kCrcBlock;
    if (c.nblk >= (size_t(1) << 31)) fail(BM_EUNSUPPORTED, "Huffman stream too large");
  }
  const size_t tot = span[0].nblk + span[1].nblk;
  if (!tot) return;
  dev.reset(tot);
  host.reset(tot);
  size_t at = 0;
  for (int k = 0; k < 2; ++k) {
    span[k].block_crc = host.p + at;
    if (span[k].nblk)
      hipLaunchKernelGGL(k_crc_blocks, dim3(unsigned(span[k].nblk)), dim3(256), 0, st,
                         static_cast<const uint4*>(src[k]), crc_tree(), dev.p + at);
    BM_HIP(hipGetLastError());
    at += span[k].nblk;
  }
  BM_HIP(hipMemcpyAsync(host.p, dev.p, tot * 4, hipMemcpyDeviceToHost, st));
}
}  // namespace

void HuffmanEncoder::write(uint8_t* dst, size_t capacity, const std::function<void()>& meanwhile) {
  Impl& I = *d_;
  bm_lossless_times& T = g_times;
  if (I.bytes > capacity) fail(BM_ECAPACITY, "Huffman stream larger than its buffer");
  const int64_t nch = I.nch, nw = int64_t(I.woff[nch]), nout = int64_t(I.ooff[nch]);
  const int64_t np = I.np;
  DevBuf<uint64_t> doff(size_t(2 * (nch + 1)));
  uint64_t *const dwoff = doff.p, *const dooff = doff.p + nch + 1;
  DevBuf<uint32_t> dwords(size_t(std::max<int64_t>(nw, 1))), dcrc;
  DevBuf<int32_t> doval(size_t(std::max<int64_t>(nout, 1)));
  EventPair ee, ec;
  IdleOnError idle(I.st);
  BM_HIP(hipMemcpyAsync(dwoff, I.woff.p, (nch + 1) * sizeof(uint64_t), hipMemcpyHostToDevice, I.st));
  BM_HIP(hipMemcpyAsync(dooff, I.ooff.p, (nch + 1) * sizeof(uint64_t), hipMemcpyHostToDevice, I.st));
  BM_HIP(hipEventRecord(ee.a, I.st));
  launch_encode(I.codes, I.n, nch, I.dlen.p, I.dcw.p, dwoff, dooff, I.wmax, dwords.p, doval.p, I.st);
  uint8_t* o = dst + sizeof(HuffHeader) + size_t(np) * 3 + size_t(nch + 1) * 16;
  I.span[0] = CrcSpan{size_t(o - dst), size_t(nw) * 4};
  I.span[1] = CrcSpan{I.span[0].offset + I.span[0].bytes, size_t(nout) * 4};
  // the CRC-32 of every whole 16 KiB block of the words and of the outlier
  // values, while they are on the device
  launch_span_crcs(I.span, {dwords.p, doval.p}, dcrc, I.crc, I.st);
  BM_HIP(hipEventRecord(ee.b, I.st));
  BM_HIP(hipEventRecord(ec.a, I.st));
  if (nw) BM_HIP(hipMemcpyAsync(dst + I.span[0].offset, dwords.p, I.span[0].bytes, hipMemcpyDeviceToHost, I.st));
  if (nout) BM_HIP(hipMemcpyAsync(dst + I.span[1].offset, doval.p, I.span[1].bytes, hipMemcpyDeviceToHost, I.st));
  BM_HIP(hipEventRecord(ec.b, I.st));
  // the rest of the stream and its CRC, while the copies run
  HuffHeader hh{kHuffMagic, 3, I.n, nch, nw, nout, np};
  o = dst;
  std::memcpy(o, &hh, sizeof(hh));
  o += sizeof(hh);
  if (np) std::memcpy(o, I.psym.p, size_t(np) * 2);
  o += size_t(np) * 2;
  if (np) std::memcpy(o, I.plen.p, size_t(np));
  o += size_t(np);
  std::memcpy(o, I.woff.p, (nch + 1) * 8);
  o += (nch + 1) * 8;
  std::memcpy(o, I.ooff.p, (nch + 1) * 8);
  I.head = container_crc(dst, I.span[0].offset);
  if (meanwhile) meanwhile();
  BM_HIP(hipStreamSynchronize(I.st));
  T.enc_encode_ms = ee.ms();
  T.enc_copy_ms = ec.ms();
}

size_t huffman_size(const int32_t* codes, int64_t n, hipStream_t st) {
  HuffmanEncoder e(codes, n, st);
  e.plan();
  return e.bytes();
}

size_t huffman_encode(const int32_t* codes, int64_t n, std::vector<uint8_t>& out, hipStream_t st) {
  HuffmanEncoder e(codes, n, st);
  e.plan();
  out.resize(e.bytes());
  e.write(out.data(), out.size());
  return out.size();
}

void set_lossless_crc_ms(double ms) { g_times.enc_crc_ms = ms; }

void huffman_code_lengths(const uint64_t* hist, uint8_t* len) { code_lengths(hist, len, table_work().lw); }

bm_lossless_times lossless_times() { return g_times; }

// ------------------------------------------------------------------ decode (host)
struct DecHost {
  uint8_t len[NSYM];
  uint32_t cw[NSYM], sorted[NSYM];
  uint32_t hdr[kDecHdrWords];
  uint16_t psym[NSYM], sorted16[NSYM];
};

struct HuffmanDecoder::Impl {
  hipStream_t st;
  const uint8_t* in;
  size_t in_bytes;
  int64_t n = 0, nch = 0, nw = 0, nout = 0;
  uint64_t wcap = 0;
  CrcSpan span[2];
  uint32_t nsorted = 1, escidx = 0;
  HostBuf<DecHost> host{1};
  HostBuf<uint64_t> off;             // word offsets, then outlier offsets
  HostBuf<uint32_t> crc;
  HostBuf<int> err{1};
  DevBuf<uint32_t> dhdr{kDecHdrWords}, dwords, dcrc;
  DevBuf<uint16_t> dsorted{NSYM}, drel;
  DevBuf<uint64_t> doff;
  DevBuf<int32_t> doval;
  DevBuf<unsigned long long> derr{1};
  EventPair eu, et;                  // around the copies of words and outliers, of tables and offsets
  IdleOnError idle;
  Impl(const uint8_t* i, size_t ib, hipStream_t s) : st(s), in(i), in_bytes(ib), idle(s) {}
};

HuffmanDecoder::~HuffmanDecoder() = default;

HuffmanDecoder::HuffmanDecoder(const uint8_t* in, size_t in_bytes, hipStream_t st) {
  d_ = std::make_unique<Impl>(in, in_bytes, st);
  Impl& I = *d_;
  bm_lossless_times& T = g_times;
  T.dec_parse_ms = T.dec_upload_ms = T.dec_decode_ms = 0.0;
  const auto t0 = clk::now();
  if (!in || in_bytes < sizeof(HuffHeader)) fail(BM_ECORRUPT, "Huffman stream too short");
  HuffHeader hh;
  std::memcpy(&hh, in, sizeof(hh));
  if (hh.magic != kHuffMagic || hh.version != 3) fail(BM_ECORRUPT, "bad Huffman stream header");
  const int64_t n = hh.n;
  if (n < 0 || hh.nchunks != (n + CHUNK - 1) / CHUNK || hh.nwords < 0 || hh.noutliers < 0 || hh.noutliers > n ||
      hh.npresent < 0 || hh.npresent > NSYM || hh.nwords > (int64_t(1) << 40))
    fail(BM_ECORRUPT, "inconsistent Huffman stream header");
  const int64_t nch = hh.nchunks, nw = hh.nwords, nout = hh.noutliers, np = hh.npresent;
  const size_t need = sizeof(hh) + size_t(np) * 3 + size_t(nch + 1) * 16 + size_t(nw) * 4 + size_t(nout) * 4;
  if (in_bytes < need) fail(BM_ECORRUPT, "Huffman stream truncated");
  I.n = n;
  I.nch = nch;
  I.nw = nw;
  I.nout = nout;
  I.span[0] = CrcSpan{sizeof(hh) + size_t(np) * 3 + size_t(nch + 1) * 16, size_t(nw) * 4};
  I.span[1] = CrcSpan{I.span[0].offset + I.span[0].bytes, size_t(nout) * 4};
  // the code words and outlier values start on their way while the rest is
  // parsed here
  I.dwords.reset(size_t(std::max<int64_t>(nw, 1)));
  I.doval.reset(size_t(std::max<int64_t>(nout, 1)));
  I.drel.reset(size_t(std::max<int64_t>(nout, 1)));
  I.doff.reset(size_t(2 * (nch + 1)));
  I.off.reset(size_t(2 * (nch + 1)));
  BM_HIP(hipEventRecord(I.eu.a, st));
  const auto tc = clk::now();   // (a copy from ordinary memory holds the host up: part of the upload)
  if (nw) BM_HIP(hipMemcpyAsync(I.dwords.p, in + I.span[0].offset, I.span[0].bytes, hipMemcpyHostToDevice, st));
  if (nout) BM_HIP(hipMemcpyAsync(I.doval.p, in + I.span[1].offset, I.span[1].bytes, hipMemcpyHostToDevice, st));
  BM_HIP(hipEventRecord(I.eu.b, st));
  const double held = ms_since(tc);
  const uint8_t* p = in + sizeof(hh);
  DecHost& H = I.host[0];
  uint8_t* const len = H.len;
  std::memset(len, 0, NSYM);
  if (np) std::memcpy(H.psym, p, size_t(np) * 2);
  for (int64_t k = 0; k < np; ++k) {
    if (k && H.psym[k] <= H.psym[k - 1]) fail(BM_ECORRUPT, "code table symbols out of order");
    len[H.psym[k]] = p[size_t(np) * 2 + k];
    if (len[H.psym[k]] == 0) fail(BM_ECORRUPT, "zero code length in the table");
  }
  p += size_t(np) * 3;
  std::memcpy(I.off.p, p, size_t(nch + 1) * 16);
  const uint64_t *woff = I.off.p, *ooff = I.off.p + nch + 1;
  if (woff[0] != 0 || ooff[0] != 0 || ooff[nch] != uint64_t(nout)) fail(BM_ECORRUPT, "bad chunk offsets");
  uint64_t wcap = 0;
  for (int64_t c = 0; c < nch; ++c) {
    const uint64_t cnt = uint64_t(std::min<int64_t>(CHUNK, n - c * CHUNK));
    // a chunk of cnt symbols has at most 32 cnt bits
    if (woff[c + 1] < woff[c] || woff[c + 1] > uint64_t(nw) || woff[c + 1] - woff[c] > cnt ||
        ooff[c + 1] < ooff[c] || ooff[c + 1] - ooff[c] > cnt)
      fail(BM_ECORRUPT, "bad chunk offsets");
    wcap = std::max(wcap, woff[c + 1] - woff[c]);
  }
  I.wcap = wcap;
  uint64_t kraft = 0;
  for (int s = 0; s < NSYM; ++s) {
    if (len[s] > LMAX) fail(BM_ECORRUPT, "code length above 32");
    if (len[s]) kraft += uint64_t(1) << (LMAX - len[s]);
  }
  if (kraft > (uint64_t(1) << LMAX)) fail(BM_ECORRUPT, "code lengths violate Kraft's inequality");
  const uint32_t *const cw = H.cw, *const sorted = H.sorted;
  int ns = 0;
  canonical(len, H.cw, H.sorted, &ns);
  // decode tables (layout at k_decode)
  std::memset(H.hdr, 0, sizeof(H.hdr));
  H.sorted16[0] = 0;
  I.nsorted = uint32_t(std::max(ns, 1));
  {
    uint32_t* lut = H.hdr;
    uint32_t* lastc = lut + (1 << DLB);
    uint32_t* offs = lastc + (LMAX + 1);
    uint32_t first[LMAX + 1] = {}, count[LMAX + 1] = {}, base[LMAX + 1] = {};
    for (int i = 0; i < ns; ++i) {
      const uint32_t s = sorted[i], l = len[s];
      H.sorted16[i] = uint16_t(s);
      if (count[l] == 0) {
        first[l] = cw[s];
        base[l] = uint32_t(i);
      }
      ++count[l];
      if (l <= DLB) {
        const uint32_t lo = cw[s] << (DLB - l), span = 1u << (DLB - l);
        for (uint32_t k = 0; k < span; ++k) lut[lo + k] = s | (l << 16);
      } else {
        uint32_t& e = lut[cw[s] >> (l - DLB)];
        e = e ? ((e & ~(63u << 24)) | (l << 24)) : (kLong | (l << 16) | (l << 24) | uint32_t(i));
      }
    }
    // prefixes of one code length whose codes fill them: length and first index in the entry
    for (uint32_t pf = 0; pf < (1u << DLB); ++pf) {
      const uint32_t e = lut[pf];
      if (!(e & kLong)) continue;
      const uint32_t lmin = (e >> 16) & 63u, lmax = (e >> 24) & 63u, i0 = e & 0xFFFFu;
      if (lmin != lmax || i0 + (1u << (lmin - DLB)) > uint32_t(ns)) continue;
      const uint32_t s0 = sorted[i0], sl = sorted[i0 + (1u << (lmin - DLB)) - 1];
      // the prefix's first code starts it; the 2^(l - DLB)-th code of length l from there ends it
      if (len[sl] == lmin && (cw[s0] >> (lmin - DLB)) == pf && (cw[sl] >> (lmin - DLB)) == pf)
        lut[pf] = kOne | i0 | (lmin << 16);
    }
    uint64_t end = 0;   // left-justified end of the codes of length <= L
    for (int l = 1; l <= LMAX; ++l) {
      if (count[l]) end = (uint64_t(first[l]) + count[l]) << (LMAX - l);
      lastc[l] = end ? uint32_t(end - 1) : 0u;
      offs[l] = base[l] - first[l];
    }
  }
  I.escidx = I.nsorted;
  for (int i = 0; i < ns; ++i)
    if (sorted[i] == 0) I.escidx = uint32_t(i);
  T.dec_parse_ms = ms_since(t0) - held;
  BM_HIP(hipEventRecord(I.et.a, st));
  BM_HIP(hipMemcpyAsync(I.dhdr.p, H.hdr, sizeof(H.hdr), hipMemcpyHostToDevice, st));
  BM_HIP(hipMemcpyAsync(I.dsorted.p, H.sorted16, size_t(I.nsorted) * 2, hipMemcpyHostToDevice, st));
  BM_HIP(hipMemcpyAsync(I.doff.p, I.off.p, size_t(nch + 1) * 16, hipMemcpyHostToDevice, st));
  BM_HIP(hipEventRecord(I.et.b, st));
}

uint32_t HuffmanDecoder::crc(uint32_t crc) {
  Impl& I = *d_;
  launch_span_crcs(I.span, {I.dwords.p, I.doval.p}, I.dcrc, I.crc, I.st);
  const uint32_t head = container_crc(I.in, I.span[0].offset);   // while the stream is on its way
  BM_HIP(hipStreamSynchronize(I.st));
  return crc_with_spans(I.in, I.in_bytes, crc, head, I.span, 2);
}

void HuffmanDecoder::decode(int32_t* codes, int64_t n) {
  Impl& I = *d_;
  bm_lossless_times& T = g_times;
  if (I.n != n) fail(BM_EINVAL, "symbol count does not match the destination");
  T.dec_n = n;
  const int64_t nch = I.nch;
  const DecTables t{I.dhdr.p, I.dsorted.p, I.nsorted, I.escidx};
  int* const derr = reinterpret_cast<int*>(I.derr.p);
  const uint64_t *const dwoff = I.doff.p, *const dooff = I.doff.p + nch + 1;
  hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(64), 0, I.st, I.derr.p, int64_t(1));
  BM_HIP(hipGetLastError());
  EventPair ed;
  BM_HIP(hipEventRecord(ed.a, I.st));
  if (nch) {
    launch_decode<kDecWpc, kDecCpw>(I.dwords.p, dwoff, nch, n, t, dooff, I.drel.p, codes, derr,
                                    int(I.wcap), I.st);
    BM_HIP(hipGetLastError());
    if (I.nout)
      hipLaunchKernelGGL(k_outliers, dim3(unsigned(nch)), dim3(256), 0, I.st, dooff, I.drel.p, I.doval.p, codes,
                         n);
    BM_HIP(hipGetLastError());
  }
  BM_HIP(hipEventRecord(ed.b, I.st));
  BM_HIP(hipMemcpyAsync(I.err.p, derr, sizeof(int), hipMemcpyDeviceToHost, I.st));
  BM_HIP(hipStreamSynchronize(I.st));
  T.dec_upload_ms = I.eu.ms() + I.et.ms();
  T.dec_decode_ms = ed.ms();
  if (I.err[0]) fail(BM_ECORRUPT, "Huffman stream does not decode");
}

void huffman_decode(const uint8_t* in, size_t in_bytes, int32_t* codes, int64_t n, hipStream_t st) {
  if (!in || in_bytes < sizeof(HuffHeader)) fail(BM_ECORRUPT, "Huffman stream too short");
  HuffHeader hh;
  std::memcpy(&hh, in, sizeof(hh));
  if (hh.magic == kHuffMagic && hh.version == 3 && hh.n != n)
    fail(BM_EINVAL, "symbol count does not match the destination");
  HuffmanDecoder d(in, in_bytes, st);
  d.decode(codes, n);
}

// ------------------------------------------------------------------ stage times
// The encoder's stages timed one by one (the lossless part of the time model
// of Algorithm 1): histogram, code table, chunk sizes + encode, copy-out + CRC.
void huffman_stage_times(const int32_t* codes, int64_t n, hipStream_t st, double ms[4]) {
  HuffmanEncoder e(codes, n, st);
  e.plan();
  std::vector<uint8_t> out(e.bytes());
  e.write(out.data(), out.size());
  const auto t0 = clk::now();
  volatile uint32_t crc = stream_crc(e, out.data(), out.size(), 0);
  (void)crc;
  const double crc_ms = ms_since(t0);
  const bm_lossless_times& T = g_times;
  ms[0] = T.enc_hist_ms;
  ms[1] = T.enc_table_ms;
  ms[2] = T.enc_sizes_ms + T.enc_encode_ms;
  ms[3] = T.enc_copy_ms + crc_ms;
}

// ------------------------------------------------------------------ no allocation
// Huffman encoding into a device buffer with every work array fixed in size:
// device scratch in one file-scope array (per GPU, held until the process
// ends), host work arrays static.  Calls share both, so they are serialised
// by a mutex on the host; calls on one GPU must not overlap in time (they
// share that GPU's scratch).

namespace {

constexpr int64_t kNoAllocMaxCh = kNoAllocMaxCodes / CHUNK;
constexpr size_t kScrHist = 0;                                         // uint64 [NSYM]
constexpr size_t kScrLen = kScrHist + size_t(NSYM) * 8;                // uint8  [NSYM]
constexpr size_t kScrCw = kScrLen + size_t(NSYM);                      // uint32 [NSYM]
constexpr size_t kScrBits = kScrCw + size_t(NSYM) * 4;                 // uint32 [chunks]
constexpr size_t kScrEsc = kScrBits + size_t(kNoAllocMaxCh) * 4;       // uint32 [chunks]
constexpr size_t kScrWoff = kScrEsc + size_t(kNoAllocMaxCh) * 4;       // uint64 [chunks + 1]
constexpr size_t kScrOoff = kScrWoff + size_t(kNoAllocMaxCh + 1) * 8;  // uint64 [chunks + 1]
constexpr size_t kScratchBytes = kScrOoff + size_t(kNoAllocMaxCh + 1) * 8;
static_assert(kScrCw % 4 == 0 && kScrWoff % 8 == 0 && kScrOoff % 8 == 0, "scratch alignment");

__device__ __align__(256) unsigned char scratch[kScratchBytes];

struct NoAllocHost {
  uint64_t hist[NSYM];
  uint8_t len[NSYM];
  uint32_t cw[NSYM], sorted[NSYM];
  uint16_t psym[NSYM];
  uint8_t plen[NSYM];
  uint32_t bits[kNoAllocMaxCh], esc[kNoAllocMaxCh];
  uint64_t woff[kNoAllocMaxCh + 1], ooff[kNoAllocMaxCh + 1];
  LenWork work;
};
NoAllocHost g_na;
std::mutex g_na_mu;
constexpr int kMaxDevices = 64;
unsigned char* g_scratch[kMaxDevices] = {};   // each GPU's copy of `scratch` (device address)

unsigned char* scratch_ptr() {
  int dev = 0;
  BM_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) fail(BM_EUNSUPPORTED, "device index beyond 63");
  if (!g_scratch[dev]) {
    void* p = nullptr;
    BM_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    g_scratch[dev] = static_cast<unsigned char*>(p);
  }
  return g_scratch[dev];
}

}  // namespace

size_t huffman_encode_noalloc(const int32_t* codes, int64_t n, void* out, size_t capacity, size_t* out_bytes,
                              hipStream_t st) {
  if (n < 0 || n > kNoAllocMaxCodes) fail(BM_EINVAL, "n outside [0, 2^28] for the entry point that does not allocate");
  if (n > 0 && !codes) fail(BM_EINVAL, "null codes");
  std::lock_guard<std::mutex> lock(g_na_mu);
  NoAllocHost& H = g_na;
  unsigned char* scr = scratch_ptr();
  auto* hist = reinterpret_cast<unsigned long long*>(scr + kScrHist);
  auto* dlen = scr + kScrLen;
  auto* dcw = reinterpret_cast<uint32_t*>(scr + kScrCw);
  auto* bits = reinterpret_cast<uint32_t*>(scr + kScrBits);
  auto* esc = reinterpret_cast<uint32_t*>(scr + kScrEsc);
  auto* dwoff = reinterpret_cast<uint64_t*>(scr + kScrWoff);
  auto* dooff = reinterpret_cast<uint64_t*>(scr + kScrOoff);
  const int64_t nch = (n + CHUNK - 1) / CHUNK;
  launch_hist(codes, n, hist, st);
  BM_HIP(hipMemcpyAsync(H.hist, hist, sizeof(H.hist), hipMemcpyDeviceToHost, st));
  BM_HIP(hipStreamSynchronize(st));
  code_lengths(H.hist, H.len, H.work);
  int ns = 0;
  canonical(H.len, H.cw, H.sorted, &ns);
  BM_HIP(hipMemcpyAsync(dlen, H.len, sizeof(H.len), hipMemcpyHostToDevice, st));
  BM_HIP(hipMemcpyAsync(dcw, H.cw, sizeof(H.cw), hipMemcpyHostToDevice, st));
  launch_chunk_bits(codes, n, nch, dlen, bits, esc, st);
  if (nch) {
    BM_HIP(hipMemcpyAsync(H.bits, bits, size_t(nch) * 4, hipMemcpyDeviceToHost, st));
    BM_HIP(hipMemcpyAsync(H.esc, esc, size_t(nch) * 4, hipMemcpyDeviceToHost, st));
  }
  BM_HIP(hipStreamSynchronize(st));
  H.woff[0] = 0;
  H.ooff[0] = 0;
  uint64_t wmax = 0;
  for (int64_t c = 0; c < nch; ++c) {
    const uint64_t w = (uint64_t(H.bits[c]) + 31) / 32;
    wmax = std::max(wmax, w);
    H.woff[c + 1] = H.woff[c] + w;
    H.ooff[c + 1] = H.ooff[c] + H.esc[c];
  }
  int64_t np = 0;
  for (int s = 0; s < NSYM; ++s)
    if (H.len[s]) {
      H.psym[np] = uint16_t(s);
      H.plen[np] = H.len[s];
      ++np;
    }
  const int64_t nw = int64_t(H.woff[nch]), nout = int64_t(H.ooff[nch]);
  HuffHeader hh{kHuffMagic, 3, n, nch, nw, nout, np};
  const size_t off_tab = sizeof(hh), off_off = off_tab + size_t(np) * 3;
  const size_t off_words = off_off + size_t(nch + 1) * 16, off_out = off_words + size_t(nw) * 4;
  const size_t bytes = off_out + size_t(nout) * 4;
  *out_bytes = bytes;
  if (!out || capacity < bytes) fail(BM_ECAPACITY, "output buffer too small");
  uint8_t* o = static_cast<uint8_t*>(out);
  BM_HIP(hipMemcpyAsync(o, &hh, sizeof(hh), hipMemcpyHostToDevice, st));
  if (np) {
    BM_HIP(hipMemcpyAsync(o + off_tab, H.psym, size_t(np) * 2, hipMemcpyHostToDevice, st));
    BM_HIP(hipMemcpyAsync(o + off_tab + size_t(np) * 2, H.plen, size_t(np), hipMemcpyHostToDevice, st));
  }
  BM_HIP(hipMemcpyAsync(o + off_off, H.woff, size_t(nch + 1) * 8, hipMemcpyHostToDevice, st));
  BM_HIP(hipMemcpyAsync(o + off_off + size_t(nch + 1) * 8, H.ooff, size_t(nch + 1) * 8, hipMemcpyHostToDevice, st));
  BM_HIP(hipMemcpyAsync(dwoff, H.woff, size_t(nch + 1) * 8, hipMemcpyHostToDevice, st));
  BM_HIP(hipMemcpyAsync(dooff, H.ooff, size_t(nch + 1) * 8, hipMemcpyHostToDevice, st));
  launch_encode(codes, n, nch, dlen, dcw, dwoff, dooff, wmax, o + off_words, o + off_out, st);
  BM_HIP(hipStreamSynchronize(st));
  return bytes;
}

}  // namespace bm
