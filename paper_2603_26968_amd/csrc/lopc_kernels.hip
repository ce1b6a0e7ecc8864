// lopc_kernels.hip -- gfx950 kernels of liblopc.so (LOPC, arXiv 2603.26968).
//
// Range, error bound, first tile pass and subbin repair (lopc_codec.hip has the
// chunk encoder and decoder).  Wave64 throughout: order flags from comparison
// masks joined on the scalar side, list places from ballots and mbcnt.  No
// MFMA: nothing here is a dense contraction.
//
// Paper map: error bound and quantizer Sec. IV-A; neighbour order flags and
// subbin raising Alg. 1 / Alg. 2 / Sec. IV-B.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "lopc_tile.h"

namespace lopc {
namespace {

// ------------------------------------------------------------------ a0
template <int K>
__device__ __forceinline__ void minmax_body(const typename Traits<K>::Raw* x, uint32_t n,
                                            int64_t* part, uint32_t blk, uint32_t nblk) {
  using Tr = Traits<K>;
  using Raw = typename Tr::Raw;
  constexpr int V = 16 / K;  // values per 16-byte vector
  constexpr int U = 4;       // vectors in flight per thread
  // non-finite values are flagged by the tile pass, which sees every point
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  auto take = [&](Raw u) {
    const int64_t k = Tr::key(u);
    lo = k < lo ? k : lo;
    hi = k > hi ? k : hi;
  };
  const uint32_t nv = n / V, stride = nblk * kThreads;
  uint32_t i = blk * kThreads + threadIdx.x;
  for (; i + (U - 1) * stride < nv; i += U * stride) {
    Raw u[U][V];
#pragma unroll
    for (int q = 0; q < U; ++q) *(uint4*)u[q] = ((const uint4*)x)[i + q * stride];
#pragma unroll
    for (int q = 0; q < U; ++q)
#pragma unroll
      for (int k = 0; k < V; ++k) take(u[q][k]);
  }
  for (; i < nv; i += stride) {
    Raw u[V];
    *(uint4*)u = ((const uint4*)x)[i];
#pragma unroll
    for (int k = 0; k < V; ++k) take(u[k]);
  }
  for (uint32_t t = nv * V + blk * kThreads + threadIdx.x; t < n; t += stride) take(x[t]);
  lo = wave_reduce(lo, OpMin{});
  hi = wave_reduce(hi, OpMax{});
  __shared__ int64_t slo[kWaves], shi[kWaves];
  if (lane() == 0) {
    slo[wave()] = lo;
    shi[wave()] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kWaves; ++w) {
      lo = slo[w] < lo ? slo[w] : lo;
      hi = shi[w] > hi ? shi[w] : hi;
    }
    part[2 * blk] = lo;
    part[2 * blk + 1] = hi;
  }
}

template <int K>
__global__ __launch_bounds__(kThreads) void k_minmax(
    const typename Traits<K>::Raw* x, uint32_t n, int64_t* part, uint4* zero, uint32_t nzero) {
  // the zeroed prefix of the workspace (Params, counters, stamps, look-back
  // words), which no earlier work of the call touches, is cleared here
  // rather than by a separate fill
  for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < nzero; i += gridDim.x * kThreads)
    zero[i] = make_uint4(0, 0, 0, 0);
  minmax_body<K>(x, n, part, blockIdx.x, gridDim.x);
}


template <int K>
__device__ __forceinline__ void params_body(int mode, double eb, const int64_t* part, int nblocks,
                            Params* prm, uint8_t* stream, uint64_t cap, int ndim,
                            int64_t d0, int64_t d1, int64_t d2) {
  using Tr = Traits<K>;
  __shared__ int64_t slo[kWaves], shi[kWaves];
  __shared__ uint32_t hw[kHeaderBytes / 4];
  int64_t lo = INT64_MAX, hi = INT64_MIN;
  if (mode == 1)
    for (int b = threadIdx.x; b < nblocks; b += kThreads) {
      const longlong2 p = ((const longlong2*)part)[b];
      lo = min(lo, (int64_t)p.x);
      hi = max(hi, (int64_t)p.y);
    }
  lo = wave_reduce(lo, OpMin{});
  hi = wave_reduce(hi, OpMax{});
  if (lane() == 0) {
    slo[wave()] = lo;
    shi[wave()] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kWaves; ++w) {
      lo = min(lo, slo[w]);
      hi = max(hi, shi[w]);
    }
    double e = eb;
    if (mode == 1) {
      // NOA: eps = eb * (max - min), all in binary64 (Sec. IV-A)
      double vlo = Tr::to_double(Tr::unkey(lo));
      double vhi = Tr::to_double(Tr::unkey(hi));
      double range = vhi - vlo;
      e = eb * range;
      prm->kmin = lo;
      prm->kmax = hi;
    }
    double v = 1.0 / e;
    bool ok = (e > 0.0) && finite64((uint64_t)__double_as_longlong(e)) &&
              finite64((uint64_t)__double_as_longlong(v));
    if (ok && fma(v, e, -1.0) < 0.0)
      v = __longlong_as_double(__double_as_longlong(v) + 1);  // next up
    ok = ok && finite64((uint64_t)__double_as_longlong(v));
    if (!ok) {
      set_status(prm, ST_BOUND);
      e = 1.0;
      v = 1.0;
    }
    prm->eb = eb;
    prm->eps = e;
    prm->inv = v;
    prm->winv = 1.0 / v;
    // the stream header as 16 little-endian words
    const uint64_t q[8] = {(uint64_t)kMagic | (uint64_t)(kVersion | (K == 4 ? 0u : 1u) << 16 |
                                                           (uint32_t)ndim << 24) << 32,
                           (uint64_t)d0, (uint64_t)d1, (uint64_t)d2,
                           (uint64_t)(uint32_t)mode | (uint64_t)kChunkBytes << 32,
                           (uint64_t)__double_as_longlong(eb), (uint64_t)__double_as_longlong(e),
                           (uint64_t)__double_as_longlong(v)};
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      hw[2 * w] = (uint32_t)q[w];
      hw[2 * w + 1] = (uint32_t)(q[w] >> 32);
    }
  }
  __syncthreads();
  if (threadIdx.x < kHeaderBytes / 4) {
    ((uint32_t*)prm->header)[threadIdx.x] = hw[threadIdx.x];
    if (cap >= kHeaderBytes) ((uint32_t*)stream)[threadIdx.x] = hw[threadIdx.x];
  }
}

template <int K>
__global__ __launch_bounds__(kThreads) void k_params(
    int mode, double eb, const int64_t* part, int nblocks, Params* prm,
    uint8_t* stream, uint64_t cap, int ndim, int64_t d0, int64_t d1,
    int64_t d2) {
  params_body<K>(mode, eb, part, nblocks, prm, stream, cap, ndim, d0, d1, d2);
}


// ------------------------------------------------------------------ a3
// Tiles of the subbin repair.  A workgroup owns a TZ x TY x TX tile and keeps
// the subbins of the tile plus a one-point halo in LDS.  It relaxes them in
// place until nothing changes (the raising rule of Alg. 2 with the halo held
// fixed; every value only grows and stays below the least fixed point, so
// concurrent reads of stale values are harmless), writes back what changed,
// and, if a boundary value changed, marks the 26 neighbour tiles for the next
// sweep.  Sweeps repeat until no tile is marked; the result is the least
// fixed point whatever the order in which tiles run.

// Neighbour tiles reached from owned point i along the stencil offsets in
// `bits` (a subset of the point's 14 / 6 offsets), as a 27-bit set: bit
// (dz + 1) * 9 + (dy + 1) * 3 + (dx + 1) for tile offset (dz, dy, dx).
// Offsets that stay inside the tile add nothing.
template <int TZ, int TY, int TX>
__device__ __forceinline__ uint32_t out_dirs(int i, uint32_t bits) {
  const int iz = i / (TY * TX), iy = (i / TX) % TY, ix = i % TX;
  uint32_t d = 0;
  while (bits) {
    const int j = __builtin_ctz(bits);
    bits &= bits - 1;
    const int z = iz + off_z(j), y = iy + off_y(j), x = ix + off_x(j);
    const int dz = z < 0 ? -1 : (z >= TZ ? 1 : 0), dy = y < 0 ? -1 : (y >= TY ? 1 : 0),
              dx = x < 0 ? -1 : (x >= TX ? 1 : 0);
    if (dz | dy | dx) d |= 1u << ((dz + 1) * 9 + (dy + 1) * 3 + (dx + 1));
  }
  return d;
}

// OR of v over the workgroup (every thread gets it)
__device__ __forceinline__ uint64_t block_or64(uint64_t v) {
  __shared__ uint64_t w[kWaves];
  v = wave_reduce(v, OpOr{});
  if (lane() == 0) w[wave()] = v;
  __syncthreads();
  uint64_t r = 0;
#pragma unroll
  for (int q = 0; q < kWaves; ++q) r |= w[q];
  __syncthreads();
  return r;
}

// Workgroups are dealt to the 8 XCDs (each with its own L2) round-robin by
// index.  Give each XCD a contiguous range of tiles instead, so that tiles
// that share halo data share an L2: workgroup b (of n) takes tile
// start(b % 8) + b / 8.  A bijection of [0, n); only locality depends on
// the dealing order.
__device__ __forceinline__ uint32_t xcd_tile(uint32_t b, uint32_t n) {
  const uint32_t x = b & 7u, per = n >> 3, rem = n & 7u;
  return x * per + (x < rem ? x : rem) + (b >> 3);
}

// Colour of a tile: the parity of the sum of its tile coordinates (a
// checkerboard: face and corner neighbours have the other colour, edge
// neighbours the same).
__device__ __forceinline__ uint32_t tile_colour(int tz, int ty, int tx) {
  return (uint32_t)((tz + ty + tx) & 1);
}

// neighbour directions (27-direction set, bit (dz+1)*9 + (dy+1)*3 + dx+1)
// towards a tile of the same colour: two nonzero offsets
constexpr uint32_t same_colour_dirs() {
  uint32_t m = 0;
  for (int d = 0; d < 27; ++d) {
    const int nz = (d / 9 != 1) + ((d / 3) % 3 != 1) + (d % 3 != 1);
    if (nz == 2) m |= 1u << d;
  }
  return m;
}

// Tile of block b in a launch over the tiles of one colour: the (b mod hx)-th
// tile of that colour in tile row b / hx (hx: half a row, rounded up); none
// (ntiles) for the last block of a row that has one tile fewer.
__device__ __forceinline__ uint32_t colour_tile(uint32_t b, uint32_t colour, const Tiling& tl) {
  const uint32_t hx = (uint32_t)(tl.ntx + 1) / 2;
  const uint32_t row = b / hx, tz = row / (uint32_t)tl.nty, ty = row % (uint32_t)tl.nty;
  const uint32_t tx = ((colour + tz + ty) & 1u) + 2 * (b % hx);
  return tx < (uint32_t)tl.ntx ? (tz * tl.nty + ty) * tl.ntx + tx : tl.ntiles;
}

struct TileCoord {
  int tz, ty, tx, z0, y0, x0;
};

template <int TZ, int TY, int TX>
__device__ __forceinline__ TileCoord tile_coord(uint32_t t, const Tiling& tl) {
  TileCoord c;
  c.tz = (int)(t / (uint32_t)(tl.nty * tl.ntx));
  c.ty = (int)((t / (uint32_t)tl.ntx) % (uint32_t)tl.nty);
  c.tx = (int)(t % (uint32_t)tl.ntx);
  c.z0 = c.tz * TZ;
  c.y0 = c.ty * TY;
  c.x0 = c.tx * TX;
  return c;
}

// the relaxation-iteration slots of the single-field counters block
__device__ __forceinline__ unsigned long long* relax_total(uint32_t* counters) {
  return (unsigned long long*)(counters + kRelaxWord);
}

// Lower neighbours of a point as LDS offsets for the relaxation: up to three
// 10-bit fields (offset + 512; an unused field holds 512, the point itself),
// the count in bits 30-31; more than three: kDense (the full mask is used).
constexpr uint32_t kDense = 0xffffffffu;
template <int TZ, int TY, int TX>
__device__ __forceinline__ uint32_t walk_code(uint32_t m) {
  using G = TileGeom<TZ, TY, TX>;
  const uint32_t n = (uint32_t)__popc(m);
  if (n > 3) return kDense;
  uint32_t code = n << 30 | 512u | 512u << 10 | 512u << 20;
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    if (m) {
      const int j = __builtin_ctz(m);
      m &= m - 1;
      code += (uint32_t)off_lin(j, G::HX, G::HY * G::HX) << (10 * f);
    }
  }
  return code;
}

// The best raise of the point at LDS index li from all its stencil
// neighbours, selected by its lower-neighbour mask m without branches or
// compares: bit j of m widened to an all-ones / zero word masks the
// neighbour's subbin, and for an even j (a neighbour of higher index, weight
// 1) subtracting the widened bit adds the weight only where the bit is set.
// The maxima fold three at a time.
template <int NJ, int HX, int HXY>
__device__ __forceinline__ uint32_t dense_best(const uint32_t* S, int li, uint32_t m,
                                               uint32_t cur) {
  uint32_t c[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const uint32_t v = S[li + kOff[j][0] * HXY + kOff[j][1] * HX + kOff[j][2]];
    const uint32_t w = (uint32_t)((int32_t)(m << (31 - j)) >> 31);
    // one AND (kept as written: the compiler would otherwise turn the masked
    // maximum back into a compare and a select)
    uint32_t vw;
    asm("v_and_b32 %0, %1, %2" : "=v"(vw) : "v"(v), "v"(w));
    c[j] = (j & 1) ? vw : vw - w;
  }
  uint32_t a = max(max(cur, c[0]), c[1]);
  uint32_t b = max(max(c[2], c[3]), c[4]);
  uint32_t r = max(max(a, b), c[5]);
  if constexpr (NJ > 6) {
    const uint32_t d = max(max(c[6], c[7]), c[8]);
    const uint32_t e = max(max(c[9], c[10]), c[11]);
    const uint32_t f = max(max(c[12], c[13]), d);
    r = max(max(r, e), f);
  }
  return r;
}

// ---------------------------------------------------------------- LDS words
// A tile run keeps one 32-bit word per halo point in LDS: the subbin in the
// low half, the point's order flags inverted in bits 16..29 (bit 16 + j clear:
// the neighbour at stencil offset j is a same-bin lower neighbour; points
// outside the tile in the first pass, and points outside the grid, have them
// all set), kRose once the run has raised it, kHalo if it lies outside the
// tile.  So one LDS read of a neighbour gives both its subbin and whether it
// depends on the point that reads it, and the maximum of two words of one
// point is the word of its larger subbin.  Subbins above kPackMax go the
// 32-bit way (relax_wide): a run raises a point by at most the points of its
// tile, so 16 bits suffice below it.
constexpr uint32_t kRose = 1u << 30, kNoFlags = 0x3fffu << 16;  // kHalo: 1 << 31
constexpr uint32_t kPackMax = 60000;

// Mask bits j of a point's flags spread over bytes: byte b of word r is
// 0xff when bit 4r + b is set, so that an SDWA operand sign-extends byte b
// to the all-ones / zero word that masks a neighbour's subbin.
template <int NW>
__device__ __forceinline__ void spread_mask(uint32_t m, uint32_t (&pk)[NW]) {
#pragma unroll
  for (int r = 0; r < NW; ++r) {
    const uint32_t x = (m >> (4 * r)) & 0xfu;
    const uint32_t y = (x * 0x00204081u) & 0x01010101u;  // bit b of x to bit 8b
    pk[r] = (y << 8) - y;                                  // 0x01 -> 0xff
  }
}
// the subbin of word v & sext(byte B of p)
template <int B>
__device__ __forceinline__ uint32_t and_sext(uint32_t v, uint32_t p) {
  uint32_t r;
  if constexpr (B == 0)
    asm("v_and_b32_sdwa %0, %1, sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:BYTE_0" : "=v"(r) : "v"(v), "v"(p));
  else if constexpr (B == 1)
    asm("v_and_b32_sdwa %0, %1, sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:BYTE_1" : "=v"(r) : "v"(v), "v"(p));
  else if constexpr (B == 2)
    asm("v_and_b32_sdwa %0, %1, sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:BYTE_2" : "=v"(r) : "v"(v), "v"(p));
  else
    asm("v_and_b32_sdwa %0, %1, sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:BYTE_3" : "=v"(r) : "v"(v), "v"(p));
  return r;
}
// the subbin of word v & mask w
__device__ __forceinline__ uint32_t and_word(uint32_t v, uint32_t w) {
  uint32_t r;
  asm("v_and_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:DWORD" : "=v"(r) : "v"(v), "v"(w));
  return r;
}
// the masked subbins of neighbours J.. (J a compile-time constant)
template <int J, int NJ, int HX, int HXY, int NW>
__device__ __forceinline__ void pk_cands(const uint32_t* P, int li, const uint32_t (&pk)[NW],
                                         uint32_t* c) {
  if constexpr (J < NJ) {
    const uint32_t v = P[li + kOff[J][0] * HXY + kOff[J][1] * HX + kOff[J][2]];
    c[J] = and_sext<J & 3>(v, pk[J >> 2]);
    pk_cands<J + 1, NJ, HX, HXY, NW>(P, li, pk, c);
  }
}
// The larger of cur and the best raise from masked neighbours c (0 where the
// flag is clear): the neighbours of higher index (even j) weigh 1, added once
// to their maximum if any of them is flagged.
template <int NJ>
__device__ __forceinline__ uint32_t fold_cands(const uint32_t* c, uint32_t m, uint32_t cur) {
  const uint32_t up = min(m & (NJ > 6 ? 0x1555u : 0x15u), 1u);
  uint32_t e = max(max(c[0], c[2]), c[4]), o = max(max(c[1], c[3]), c[5]);
  if constexpr (NJ > 6) {
    e = max(max(e, c[6]), c[8]);
    e = max(max(e, c[10]), c[12]);
    o = max(max(o, c[7]), c[9]);
    o = max(max(o, c[11]), c[13]);
  }
  return max(max(cur, o), e + up);
}
// The best raise of the point at LDS index li with lower-neighbour mask m
// from the words of all its stencil neighbours, one masking instruction per
// neighbour where the mask is spread (pk).
template <int NJ, int HX, int HXY, int NW>
__device__ __forceinline__ uint32_t pull_best_pk(const uint32_t* P, int li, uint32_t m,
                                                 const uint32_t (&pk)[NW], uint32_t cur) {
  uint32_t c[NJ];
  pk_cands<0, NJ, HX, HXY, NW>(P, li, pk, c);
  return fold_cands<NJ>(c, m, cur);
}
template <int NJ, int HX, int HXY>
__device__ __forceinline__ uint32_t pull_best(const uint32_t* P, int li, uint32_t m,
                                              uint32_t cur) {
  uint32_t c[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const uint32_t v = P[li + kOff[j][0] * HXY + kOff[j][1] * HX + kOff[j][2]];
    c[j] = and_word(v, (uint32_t)((int32_t)(m << (31 - j)) >> 31));
  }
  return fold_cands<NJ>(c, m, cur);
}

// A pass of the first run that raises at most this many of a tile's NPT points
// hands over to event rounds.
template <int NPT>
constexpr uint32_t kEventShare = NPT / 16;
// Cost of the events of a 2D run after which the rest of it goes by levels
// (whole_run): a round of few events counts 1 (0.31 us), 64 events of another 3.
// A run by levels takes 5 us and 0.1 us a level.  us a call at 24 / 36 / 48:
// 2048^2 bumps at bound 1e-2 353 / 308 / 313, 1800 x 3600 fronts at 1e-3 359 /
// 352 / 352, at 1e-1 1,907 / 1,997 / 2,100; with no limit and passes after full
// lists 302, 366 and 8,830.
constexpr uint32_t kEventCost = 36;
// Events of a round up to which each gets a lane per neighbour.
constexpr uint32_t kNarrow = 32;

// Event lists of a tile run (LDS indices of raised points; two alternating
// lists per wave) and its block-wide words.
template <int NPT>
struct EventLds {
  static constexpr uint32_t kCap = NPT / kWaves;  // entries of one list: a wave's slots
  uint16_t list[kWaves][2][kCap];
  uint32_t over;     // points were left out of a full list, or the events cost too much
  uint32_t big;      // a loaded subbin exceeds kPackMax
  uint32_t dirs;     // neighbour tiles to mark (27-direction set)
  uint32_t rose[3];  // points raised by pass p in slot p % 3
};

// Append the lanes' points (where `go`) to one of the wave's lists of n
// entries (wave-uniform; slots of a wave always fit).
__device__ __forceinline__ void list_points(uint16_t* list, uint32_t& n, bool go, int li) {
  const uint64_t b = __ballot(go);
  if (go) list[n + lane_prefix(b)] = (uint16_t)li;
  n += (uint32_t)__popcll(b);
}

// An LDS word rises to subbin nv where `hit` (q: the word as read); returns
// the word before, ~0 where not.  The maximum of the words keeps the larger
// subbin: their flags agree, and a word without kRose has not changed since it
// was read.
__device__ __forceinline__ uint32_t raise_word(uint32_t* w, bool hit, uint32_t q, uint32_t nv) {
  uint32_t old = ~0u;
  if (hit)
    old = __hip_atomic_fetch_max(w, (q & 0xffff0000u) | kRose | nv, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
  return old;
}

// The points that rose to nv (old: the word before) and lie in the tile join
// the wave's list of n entries; a full list sets E.over.
template <int NPT>
__device__ __forceinline__ void list_risen(EventLds<NPT>& E, uint16_t* list, uint32_t& n,
                                           uint32_t old, int li, uint32_t nv) {
  const bool up = (old & (0xffffu | kHalo)) < nv;
  const uint64_t b = __ballot(up);
  if (!b) return;
  const uint32_t c = (uint32_t)__popcll(b);
  if (n + c > EventLds<NPT>::kCap) {
    E.over = 1;
    return;
  }
  if (up) list[n + lane_prefix(b)] = (uint16_t)li;
  n += c;
}

// Event rounds of one wave, from the n points of its list[0]: every listed
// point pushes its subbin to its stencil neighbours that depend on it, and
// those that rise push in turn until none does.  A round costs its events, not
// the points of the tile: in a later run about one point in twenty rises from
// the halo, and fewer in every round after.  A wave keeps the points it raises
// in lists of its own, so the waves need no barriers (a point raised by one
// while another pushes it is pushed again by the one that raised it).  All
// words of a round are read at once (one LDS round trip), then the raises are
// LDS maxima issued together.  Rounds of few events give each event a lane per
// neighbour instead of a lane in all.  Halo words rise too (kRose marks them),
// but push nothing.  A point raised twice in a round is listed twice (its
// second event finds nothing to raise).  Sets E.over and leaves off where the
// events cost more than the other way (2D, kEventCost).  Returns the rounds.
// Bound by vector issue on large fields and by the latency of the rounds on
// small ones.  Against passes over all points until none rises: the 24 sweep
// launches on a 512^3 float64 lognormal field 8.3 -> 6.1 ms (vector
// instructions of the first 2971 -> 1790 per wave, of the sixth 1298 -> 550),
// 2D 1800 x 3600 float32 sweeps 300 -> 170 us (145 with the runs by levels).
template <int TZ, int TY, int TX>
__device__ __forceinline__ int push_rounds(uint32_t* P, EventLds<TZ * TY * TX>& E, uint32_t n) {
  using G = TileGeom<TZ, TY, TX>;
  constexpr int NJ = TZ == 1 ? 6 : 14;
  constexpr int HX = G::HX, HXY = G::HY * G::HX;
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane(wave());
  // narrow rounds: kPer lanes to an event, one neighbour each
  constexpr int kPer = NJ == 6 ? 8 : 16, kPerWave = 64 / kPer;
  const int jl = lane() % kPer;
  const int offl = jl < NJ ? off_lin(jl, HX, HXY) : 0;
  const uint32_t keepl = 0xffffu | 1u << (16 + ((jl < NJ ? jl : 0) ^ 1));
  int r = 0;
  uint32_t cost = 0;
  while (n) {
    if constexpr (TZ == 1) {
      cost += n > kNarrow ? 3 * ((n + 63) / 64) : 1u;
      if (cost > kEventCost) {
        E.over = 1;
        break;
      }
    }
    const uint16_t* in = E.list[w][r & 1];
    uint16_t* out = E.list[w][(r + 1) & 1];
    uint32_t made = 0;
    auto narrow = [&](auto U_, uint32_t b) {
      constexpr int U = decltype(U_)::value;
      int l[U];
      uint32_t v[U], q[U], old[U];
      bool act[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t e = b + (uint32_t)(u * kPerWave + lane() / kPer);
        act[u] = e < n && jl < NJ;
        l[u] = act[u] ? (int)in[e] : G::local(0);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        v[u] = P[l[u]];
        l[u] += offl;
        q[u] = P[l[u]];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        v[u] = act[u] ? (v[u] & 0xffffu) + (uint32_t)(jl & 1) : 0u;
        old[u] = raise_word(&P[l[u]], (q[u] & keepl) < v[u], q[u], v[u]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) list_risen(E, out, made, old[u], l[u], v[u]);
    };
    if (n <= kPerWave) {
      narrow(std::integral_constant<int, 1>{}, 0u);
    } else if (n <= kNarrow) {
      for (uint32_t b = 0; b < n; b += 4 * kPerWave) narrow(std::integral_constant<int, 4>{}, b);
    } else {
      for (uint32_t b = 0; b < n; b += 64) {
        const bool act = b + (uint32_t)lane() < n;
        const int p = act ? (int)in[b + lane()] : G::local(0);
        const uint32_t v = P[p] & 0xffffu;
        uint32_t q[NJ], old[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          q[j] = P[p + kOff[j][0] * HXY + kOff[j][1] * HX + kOff[j][2]];
        // neighbour j sees p at offset j ^ 1, with weight 1 for odd j (p has
        // the higher index): a hit if its flag bit is clear and its subbin is
        // lower
        const uint32_t nv[2] = {act ? v : 0u, act ? v + 1 : 0u};
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          old[j] = raise_word(&P[p + kOff[j][0] * HXY + kOff[j][1] * HX + kOff[j][2]],
                              (q[j] & (0xffffu | 1u << (16 + (j ^ 1)))) < nv[j & 1], q[j],
                              nv[j & 1]);
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          list_risen(E, out, made, old[j], p + kOff[j][0] * HXY + kOff[j][1] * HX + kOff[j][2],
                     nv[j & 1]);
      }
    }
    n = made;
    ++r;
    __builtin_amdgcn_wave_barrier();
  }
  return r;
}

// One pass over the owned points, flags and subbins from the LDS words, slots
// in ascending or descending order; returns the slots that rose (bit k).
template <int TZ, int TY, int TX>
__device__ __forceinline__ uint32_t word_pass(uint32_t* P, bool rev) {
  using G = TileGeom<TZ, TY, TX>;
  constexpr int NJ = TZ == 1 ? 6 : 14;
  const int li0 = G::local(threadIdx.x);
  uint32_t changed = 0;
#pragma unroll 2
  for (int kk = 0; kk < G::PER; ++kk) {
    const int k = rev ? G::PER - 1 - kk : kk;
    const int li = li0 + k * G::kSlot;
    const uint32_t w = P[li], m = (~w >> 16) & (TZ == 1 ? 0x3fu : 0x3fffu), cur = w & 0xffffu;
    if (!m) continue;
    const uint32_t best = pull_best<NJ, G::HX, G::HY * G::HX>(P, li, m, cur);
    if (best > cur) {
      P[li] = (w + (best - cur)) | kRose;
      changed |= 1u << k;
    }
  }
  return changed;
}

// adds the points that rose (bit k of changed: slot k) to E.rose[slot]
template <int PER, int NPT>
__device__ __forceinline__ void count_rose(EventLds<NPT>& E, uint32_t changed, int slot) {
  uint32_t rose = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) rose += (uint32_t)__popcll(__ballot((changed >> k) & 1u));
  if (rose && lane() == 0) atomicAdd(&E.rose[slot], rose);
}

// Passes until no owned point rises (after a full event list).  Every thread
// calls it past a block barrier; returns the passes.
template <int TZ, int TY, int TX>
__device__ __forceinline__ int word_passes(uint32_t* P, EventLds<TZ * TY * TX>& E,
                                           uint32_t* counters) {
  using G = TileGeom<TZ, TY, TX>;
  if (threadIdx.x < 3) E.rose[threadIdx.x] = 0;
  __syncthreads();
  int iters = 0;
  for (;;) {
    if (threadIdx.x == 0) E.rose[(iters + 1) % 3] = 0;
    const uint32_t changed = word_pass<TZ, TY, TX>(P, iters & 1);
    count_rose<G::PER>(E, changed, iters % 3);
    __syncthreads();
    if (!E.rose[iters % 3]) return iters + 1;
    if (++iters > G::NPT + 2) {  // unreachable: the order inside a tile is acyclic
      if (threadIdx.x == 0) atomicOr(&counters[0], 1u);
      return iters;
    }
  }
}

// Local fixed point of a tile in the first pass: Gauss-Seidel passes over the
// owned points, then event rounds; the halo is fixed.  Only points with a
// same-bin lower neighbour can rise; a wave whose slots hold at most 64 of
// them first gathers them into one lane each (a per-wave list in LDS), so that
// a pass costs one step per wave instead of one per slot, and each listed
// point with at most three lower neighbours reads them at precomputed offsets
// (walk_code: three loads issued back to back).  Other waves visit their slots
// and read every stencil neighbour at once, masked.  Once a pass raises at
// most a sixteenth of the points (kEventShare; and some wave is not listed), those
// points become the first event list.  On a lognormal field (91% of the points in
// one bin) the passes raise 77, 54, 40, 31, 25, 19, 15, 12% ... of the points,
// fifteen in all: the later ones cost far less as events.  Adds the pass count
// to one of 64 statistics slots itot[t % 64].  PK: the slots' masks are spread
// over bytes once (spread_mask) and a visit masks with one SDWA instruction
// per neighbour: fewer vector instructions, 16 more registers (the float64
// first pass; the float32 one loses more occupancy than it saves).
template <int TZ, int TY, int TX, bool PK = false>
__device__ void relax(uint32_t* P, EventLds<TZ * TY * TX>& E, const uint16_t* mk,
                      uint32_t* counters, unsigned long long* itot, uint32_t t) {
  using G = TileGeom<TZ, TY, TX>;
  static_assert(TZ > 1, "2D tiles peel");
  constexpr int NJ = 14;
  static_assert(G::H < 4096, "halo index in 12 bits");
  // the candidates of a listed wave, in the room of its event lists (64 each)
  const int w = __builtin_amdgcn_readfirstlane(wave());
  uint32_t* wl_pt = (uint32_t*)&E.list[w][0][0];
  static_assert(sizeof(E.list[0]) >= 256, "the candidates fit the event lists");
  __shared__ uint32_t dense;  // some wave is not listed
  // a listed point: rise to the best of its lower neighbours (a positive
  // offset, even j, reaches a higher index and adds one)
  auto step = [&](int li, uint32_t m, uint32_t cd) -> bool {
    const uint32_t w = P[li], cur = w & 0xffffu;
    uint32_t best = cur;
    if (__ballot(cd == kDense)) {
      best = pull_best<NJ, G::HX, G::HY * G::HX>(P, li, m, cur);
    } else {
      const int o0 = (int)(cd & 1023u) - 512, o1 = (int)((cd >> 10) & 1023u) - 512,
                o2 = (int)((cd >> 20) & 1023u) - 512;
      const uint32_t c0 = (P[li + o0] & 0xffffu) + (o0 > 0), c1 = (P[li + o1] & 0xffffu) + (o1 > 0),
                     c2 = (P[li + o2] & 0xffffu) + (o2 > 0);
      best = max(max(best, c0), max(c1, c2));
    }
    if (best > cur) {
      P[li] = w + (best - cur);
      return true;
    }
    return false;
  };
  // gather this wave's candidate points
  uint64_t act[G::PER];  // wave-uniform
  uint32_t n = 0;
#pragma unroll
  for (int k = 0; k < G::PER; ++k) {
    act[k] = __ballot(mk[k] != 0);
    n += (uint32_t)__popcll(act[k]);
  }
  const bool listed = n <= 64;
  if (listed) {
    uint32_t base = 0;
#pragma unroll
    for (int k = 0; k < G::PER; ++k) {
      if (mk[k]) {
        const uint32_t pos = base + (uint32_t)__popcll(act[k] & ((1ull << lane()) - 1ull));
        wl_pt[pos] =
            (uint32_t)G::local(threadIdx.x + k * kThreads) | (uint32_t)mk[k] << 12;
      }
      base += (uint32_t)__popcll(act[k]);
    }
  }
  uint32_t my_pt = 0, my_cd = 0;
  __builtin_amdgcn_wave_barrier();
  if (listed && (uint32_t)lane() < n) {
    my_pt = wl_pt[lane()];
    my_cd = walk_code<TZ, TY, TX>(my_pt >> 12);
  }
  // slot k of this thread lies kSlot LDS words after slot 0
  const int li0 = G::local(threadIdx.x);
  // points that rose in pass p: E.rose[p % 3], added to by the waves, read by
  // all after the pass's barrier; thread 0 clears slot (p + 1) % 3 during pass
  // p (last read after the barrier of pass p - 2, next added to in pass
  // p + 1), so one barrier per pass suffices
  if (threadIdx.x < 3) E.rose[threadIdx.x] = 0;
  if (threadIdx.x == 0) {
    dense = 0;
    E.over = 0;
  }
  __syncthreads();
  if (!listed && lane() == 0) dense = 1;
  constexpr int NW = (NJ + 3) / 4;
  uint32_t pk[PK ? G::PER : 1][NW];
  if constexpr (PK) {
#pragma unroll
    for (int k = 0; k < G::PER; ++k) spread_mask<NW>(mk[k], pk[k]);
  }
  int iters = 0, total = 0;
  bool events = false;
  uint32_t nev = 0;  // the wave's first events
  for (;;) {
    uint32_t changed = 0;  // bit k: slot k rose (a listed wave: bit 0)
    if (threadIdx.x == 0) E.rose[(iters + 1) % 3] = 0;
    if (listed) {
      if (my_pt && step((int)(my_pt & 4095u), my_pt >> 12, my_cd)) changed = 1;
    } else {
      // Gauss-Seidel along the thread's slots (one column of points along
      // z), in alternating directions from pass to pass, so a chain along
      // that axis crosses the tile in a pass or two whichever way it runs
      auto visit = [&](int k) {
        const uint32_t m = mk[k];
        if (!m) return;
        const int li = li0 + k * G::kSlot;
        const uint32_t w = P[li], cur = w & 0xffffu;
        uint32_t best;
        if constexpr (PK) best = pull_best_pk<NJ, G::HX, G::HY * G::HX>(P, li, m, pk[k], cur);
        else best = pull_best<NJ, G::HX, G::HY * G::HX>(P, li, m, cur);
        if (best > cur) {
          P[li] = w + (best - cur);
          changed |= 1u << k;
        }
      };
      if constexpr (PK) {
        // slot order fixed at compile time in both directions
        if (iters & 1) {
#pragma unroll
          for (int kk = 0; kk < G::PER; ++kk) visit(G::PER - 1 - kk);
        } else {
#pragma unroll
          for (int kk = 0; kk < G::PER; ++kk) visit(kk);
        }
      } else {
        const bool rev = iters & 1;
#pragma unroll 2
        for (int kk = 0; kk < G::PER; ++kk) visit(rev ? G::PER - 1 - kk : kk);
      }
    }
    count_rose<G::PER>(E, changed, iters % 3);
    __syncthreads();
    const uint32_t c = E.rose[iters % 3];
    ++total;
    if (!c) break;
    if (++iters > G::NPT + 2) {  // unreachable: the order inside a tile is acyclic
      if (threadIdx.x == 0) atomicOr(&counters[0], 1u);
      break;
    }
    if (c <= kEventShare<G::NPT> && dense) {
      uint16_t* l0 = E.list[w][0];
      if (listed) {
        list_points(l0, nev, changed != 0u, (int)(my_pt & 4095u));
      } else {
#pragma unroll
        for (int k = 0; k < G::PER; ++k)
          list_points(l0, nev, (changed >> k) & 1u, li0 + k * G::kSlot);
      }
      events = true;
      break;
    }
  }
  if (events) {
    total += push_rounds<TZ, TY, TX>(P, E, nev);
    __syncthreads();
    if (E.over) total += word_passes<TZ, TY, TX>(P, E, counters);
  }
  if (threadIdx.x == 0) atomicAdd(&itot[t % 64], (unsigned long long)total);
}

// Local fixed point of a tile whose subbins may not fit the 16 bits of an LDS
// word: passes over the owned points (S: subbins, 32 bits; M: flags), slots in
// alternating order, until none rises.  Returns the passes.
template <int TZ, int TY, int TX>
__device__ __forceinline__ int relax_wide(uint32_t* S, const uint16_t* M,
                                          uint32_t* counters) {
  using G = TileGeom<TZ, TY, TX>;
  constexpr int NJ = TZ == 1 ? 6 : 14;
  const int li0 = G::local(threadIdx.x);
  // flag[p % 3]: some point rose in pass p (rotating as E.rose in relax)
  __shared__ uint32_t flag[3];
  if (threadIdx.x < 3) flag[threadIdx.x] = 0;
  __syncthreads();
  int iters = 0;
  for (;;) {
    bool changed = false;
    if (threadIdx.x == 0) flag[(iters + 1) % 3] = 0;
    const bool rev = iters & 1;
#pragma unroll 1
    for (int kk = 0; kk < G::PER; ++kk) {
      const int k = rev ? G::PER - 1 - kk : kk;
      const int li = li0 + k * G::kSlot;
      const uint32_t m = M[li];
      if (!m) continue;
      const uint32_t cur = S[li];
      const uint32_t best = dense_best<NJ, G::HX, G::HY * G::HX>(S, li, m, cur);
      if (best > cur) {
        S[li] = best;
        changed = true;
      }
    }
    if (__ballot(changed) && lane() == 0) flag[iters % 3] = 1;
    __syncthreads();
    if (!flag[iters % 3]) break;
    if (++iters > G::NPT + 2) {  // unreachable: the order inside a tile is acyclic
      if (threadIdx.x == 0) atomicOr(&counters[0], 1u);
      break;
    }
  }
  return iters + 1;
}

// ------------------------------------------------------------------ peeling
// First pass of a 2D tile.  2D fields are smooth on the scale of a tile and
// most of their points have same-bin neighbours, so relaxation passes would
// visit every point many times.  The points are taken in a topological order
// of the tile's part of the order graph instead (Kahn's order): a point is
// ready once all its lower neighbours inside the tile are done, and then takes
// its final value at once (the raising rule of Alg. 2 for a fixed halo).
// The LDS word of an owned point counts its unfinished lower neighbours inside
// the tile in bits 22..24, and holds its level in bits 22..29 once it is done.  A ready point reads its six neighbours' words at
// once (one LDS round trip): its own raise from those its flags name, and the
// dependents, whose flags name it, are counted down by LDS atomics issued
// together; those that reach zero are listed for the next level.  The list
// holds every point once.  Levels of at most 64 points, and those after them,
// run on wave 0 alone without block barriers.  Returns the levels of this
// wave; ends with a block barrier.
constexpr int kLeftShift = 22;
// In memory the order flags of a 2D point (six bits) share their 16 bits with
// its level inside its tile (255: that or more).
constexpr int kLevelShift = 8;
template <int TZ>
__device__ __forceinline__ uint32_t flags_of(uint32_t m) {
  return TZ == 1 ? m & 0x3fu : m;
}
template <int TZ, int TY, int TX>
__device__ __forceinline__ int peel(uint32_t* P, uint16_t* list, uint32_t* tail) {
  using G = TileGeom<TZ, TY, TX>;
  static_assert(TZ == 1, "2D tiles");
  constexpr int NJ = 6, HX = G::HX, HXY = G::HY * G::HX;
  const int li0 = G::local(threadIdx.x);
  if (threadIdx.x == 0) *tail = 0;
  __syncthreads();  // the words, too
  // level 0: nothing below inside the tile
#pragma unroll
  for (int k = 0; k < G::PER; ++k) {
    const int li = li0 + k * G::kSlot;
    const bool go = (P[li] >> kLeftShift & 7u) == 0;
    const uint64_t b = __ballot(go);
    if (!b) continue;
    uint32_t base = 0;
    if (lane() == 0) base = atomicAdd(tail, (uint32_t)__popcll(b));
    base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
    if (go) list[base + lane_prefix(b)] = (uint16_t)li;
  }
  __syncthreads();
  uint32_t beg = 0, end = (uint32_t)__builtin_amdgcn_readfirstlane((int)*tail);
  bool narrow = false;
  int level = 0;
  while (beg < end) {
    narrow = narrow || end - beg <= 64;
    if (narrow && wave() != 0) break;
    if (!narrow) __syncthreads();  // every wave has read *tail
    uint32_t made = 0;             // narrow: points listed by this level
    for (uint32_t b = beg + (narrow ? 0u : (uint32_t)wave() * 64); b < end;
         b += narrow ? 64u : (uint32_t)kThreads) {
      const bool act = b + (uint32_t)lane() < end;
      const int p = act ? (int)list[b + lane()] : li0;
      const uint32_t wp = P[p];
      uint32_t q[NJ], c[NJ], old[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) q[j] = P[p + kOff[j][0] * HXY + kOff[j][1] * HX + kOff[j][2]];
      const uint32_t m = (~wp >> 16) & 0x3fu;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        c[j] = and_word(q[j], (uint32_t)((int32_t)(m << (31 - j)) >> 31));
      const uint32_t best = fold_cands<NJ>(c, m, wp & 0xffffu);
      if (act)
        P[p] = (wp & 0xffff0000u) | best | (uint32_t)min(level, 255) << kLeftShift;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        // neighbour j names p in its flag j ^ 1 (clear) and lies in the tile
        old[j] = 0;
        if (act && !(q[j] & (kHalo | 1u << (16 + (j ^ 1)))))
          old[j] = atomicSub(&P[p + kOff[j][0] * HXY + kOff[j][1] * HX + kOff[j][2]],
                             1u << kLeftShift);
      }
      uint64_t rb[NJ];
      uint32_t tot = 0;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        rb[j] = __ballot((old[j] >> kLeftShift & 7u) == 1u);
        tot += (uint32_t)__popcll(rb[j]);
      }
      if (!tot) continue;
      uint32_t pos = end + made;
      if (narrow) {
        made += tot;
      } else {
        if (lane() == 0) pos = atomicAdd(tail, tot);
        pos = (uint32_t)__builtin_amdgcn_readfirstlane((int)pos);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        if ((rb[j] >> lane()) & 1u)
          list[pos + lane_prefix(rb[j])] =
              (uint16_t)(p + kOff[j][0] * HXY + kOff[j][1] * HX + kOff[j][2]);
        pos += (uint32_t)__popcll(rb[j]);
      }
    }
    beg = end;
    if (narrow) {
      end += made;
      __builtin_amdgcn_wave_barrier();
    } else {
      __syncthreads();
      end = (uint32_t)__builtin_amdgcn_readfirstlane((int)*tail);
    }
    ++level;
  }
  __syncthreads();
  return level;
}

// mark the neighbour tiles in `dirs` (27-bit set, see out_dirs) for sweep
// `next`; one atomic per block adds the number of newly marked tiles to
// counters[1 + next % 64]
__device__ void mark_neighbours(uint32_t dirs, const TileCoord& c, const Tiling& tl,
                                uint32_t* stamp, uint32_t* counters,
                                uint32_t next) {
  bool newly = false;
  if (threadIdx.x < 27 && ((dirs >> threadIdx.x) & 1u)) {
    int dz = (int)threadIdx.x / 9 - 1, dy = ((int)threadIdx.x / 3) % 3 - 1,
        dx = (int)threadIdx.x % 3 - 1;
    int nz = c.tz + dz, ny = c.ty + dy, nx = c.tx + dx;
    if ((dz | dy | dx) != 0 && nz >= 0 && nz < tl.ntz && ny >= 0 &&
        ny < tl.nty && nx >= 0 && nx < tl.ntx) {
      uint32_t u = ((uint32_t)nz * tl.nty + ny) * tl.ntx + nx;
      uint32_t prev = atomicMax(&stamp[u], next);
      newly = prev < next;
    }
  }
  if (threadIdx.x < 64) {
    uint64_t m = __ballot(newly);
    if (threadIdx.x == 0 && m)
      atomicAdd(&counters[1 + (next & 63)], (uint32_t)__popcll(m));
  }
}

// mark_neighbours, and also append the newly marked tiles to the work list
// of sweep `next` (lists: two arrays of tl.ntiles items, sweep parity; each
// tile is listed at most once per sweep, so a list never overflows)
__device__ void mark_list1(uint32_t dirs, const TileCoord& c, const Tiling& tl, uint32_t* stamp,
                           uint32_t* counters, uint32_t* lists, uint32_t next) {
  if (threadIdx.x >= 64) return;
  bool newly = false;
  uint32_t u = 0;
  if (threadIdx.x < 27 && ((dirs >> threadIdx.x) & 1u)) {
    const int dz = (int)threadIdx.x / 9 - 1, dy = ((int)threadIdx.x / 3) % 3 - 1,
              dx = (int)threadIdx.x % 3 - 1;
    const int nz = c.tz + dz, ny = c.ty + dy, nx = c.tx + dx;
    if ((dz | dy | dx) != 0 && nz >= 0 && nz < tl.ntz && ny >= 0 && ny < tl.nty && nx >= 0 &&
        nx < tl.ntx) {
      u = ((uint32_t)nz * tl.nty + ny) * tl.ntx + nx;
      newly = atomicMax(&stamp[u], next) < next;
    }
  }
  const uint64_t m = __ballot(newly);
  if (!m) return;
  uint32_t pos = 0;
  if (threadIdx.x == 0) pos = atomicAdd(&counters[1 + (next & 63)], (uint32_t)__popcll(m));
  pos = __shfl(pos, 0, 64);
  if (newly) lists[(next & 1) * tl.ntiles + pos + lane_prefix(m)] = u;
}

// ------------------------------------------------------------- repair queue
// Tile item of the neighbour in direction bit `d` (27-direction set) of the
// tile at c, in a field whose tile items start at t0.
__device__ __forceinline__ uint32_t dir_tile(int d, const TileCoord& c, const Tiling& tl,
                                             uint32_t t0) {
  const int nz = c.tz + d / 9 - 1, ny = c.ty + (d / 3) % 3 - 1, nx = c.tx + d % 3 - 1;
  return t0 + ((uint32_t)nz * tl.nty + ny) * tl.ntx + nx;
}
__device__ __forceinline__ bool dir_inside(int d, const TileCoord& c, const Tiling& tl) {
  const int nz = c.tz + d / 9 - 1, ny = c.ty + (d / 3) % 3 - 1, nx = c.tx + d % 3 - 1;
  return d != 13 && nz >= 0 && nz < tl.ntz && ny >= 0 && ny < tl.nty && nx >= 0 &&
         nx < tl.ntx;
}

// Publish a listed tile item in the ring (any lane): a tail ticket, then
// wait until the slot's previous item has been taken (never long: at most
// as many items as tiles are in the ring at once).  Release: what the
// caller did before (counting the item as pending) is visible to the worker
// that takes it.
// Watchdog of a queue wait: true once the queue has shown no progress (tail
// and pending unchanged) for kQueueStall ticks, or another wait gave up.
struct QueueWatch {
  unsigned long long tail = ~0ull, since = 0;
  int32_t pending = -1;
  __device__ bool stalled(const QueueRef& Q) {
    if (__hip_atomic_load(&Q.q->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return true;
    const unsigned long long tl =
        __hip_atomic_load(&Q.q->tail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int32_t pd = __hip_atomic_load(&Q.q->pending, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long now = wall_clock64();
    if (tl != tail || pd != pending) {
      tail = tl;
      pending = pd;
      since = now;
      return false;
    }
    if (now - since < kQueueStall) return false;
    atomicOr(&Q.q->err, 1u);
    return true;
  }
};

__device__ void q_publish(const QueueRef& Q, uint32_t item) {
  const unsigned long long pos = atomicAdd(&Q.q->tail, 1ull);
  unsigned long long* slot = Q.ring + (pos & ((1ull << Q.cap_log2) - 1ull));
  const uint32_t lap2 = (uint32_t)(pos >> Q.cap_log2) * 2u;
  QueueWatch w;
  for (uint32_t k = 0;
       (uint32_t)(__hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 32) !=
       lap2;
       ++k) {
    if ((k & 63u) == 63u && w.stalled(Q)) return;
    __builtin_amdgcn_s_sleep(2);
  }
  __hip_atomic_store(slot, (unsigned long long)(lap2 + 1u) << 32 | item, __ATOMIC_RELEASE,
                     __HIP_MEMORY_SCOPE_AGENT);
}

// List tile item `item` (any lane): nothing if it is listed already, else
// count it as pending and publish it.  The caller has released the subbins
// it wrote (a fence at agent scope) before listing; the worker that runs the
// item acquires them through its state word.
__device__ void q_push(const QueueRef& Q, uint32_t item, uint32_t depth) {
  atomicMax(&Q.depth[item], depth);
  if (__hip_atomic_fetch_or(&Q.st[item], TS_LISTED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
      TS_LISTED)
    return;
  atomicAdd(&Q.q->pending, 1);
  q_publish(Q, item);
}

// Take the next item from the ring (one thread of a workgroup): a head
// ticket, then wait for its slot to be filled; kNoTile once nothing is
// listed or running (nothing can be listed after that: only running tiles
// list others).
__device__ uint32_t q_pop(const QueueRef& Q) {
  const unsigned long long pos = atomicAdd(&Q.q->head, 1ull);
  unsigned long long* slot = Q.ring + (pos & ((1ull << Q.cap_log2) - 1ull));
  const uint32_t full = (uint32_t)(pos >> Q.cap_log2) * 2u + 1u;
  unsigned long long v;
  QueueWatch w;
  // back off while waiting: a thousand idle workers polling at full rate
  // would crowd the memory channel of the words they poll
  uint32_t nap = 1;
  for (uint32_t k = 0;; ++k) {
    v = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((uint32_t)(v >> 32) == full) break;
    if ((k & 3u) == 3u &&
        __hip_atomic_load(&Q.q->pending, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)
      return kNoTile;
    if ((k & 255u) == 255u && w.stalled(Q)) return kNoTile;
    for (uint32_t z = 0; z < nap; ++z) __builtin_amdgcn_s_sleep(8);
    nap = nap < 16u ? nap * 2u : 16u;
  }
  // what the publisher did before is visible from here on.  (An acquire load in
  // the loop above invalidates the caches under the running tiles at every
  // poll; queue alone, that way / this: a falling chain of 2^18 points in a row
  // 274 / 114 ms, 128^3 float64 lognormal 31.0 / 9.1 ms, 1800 x 3600 fronts at
  // bound 1e-2 2.5 / 1.6 ms.)
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  __hip_atomic_store(slot, (unsigned long long)(full + 1u) << 32, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
  return (uint32_t)v;
}

// Decide what to do with a taken item t (one thread): true = run it now.
// * t is running on another worker (it was listed again during that run):
//   it parks on itself (direction 13) and is published again when that run
//   ends, so two runs of one tile never overlap (a slower run could
//   otherwise store smaller values over a faster one's).
// * t ran before in this repair: it parks on the first listed or running
//   neighbour of higher index that it depends on (its blockers, stored by
//   its first run), and is published again when that neighbour's run ends.
// * otherwise it runs (`first`: its first run in this repair): it clears
//   its listed bit, acquiring the subbins released by every worker that
//   listed it; a change after that lists it again.
// The parking handshakes (parked bit, then the other tile's state; the
// other tile at the end of its run: its state, then its parked word) are
// sequentially consistent, so no wake-up is lost; a parker that finds the
// other tile idle takes its bit back and publishes itself.
__device__ bool q_park(const QueueRef& Q, uint32_t t, uint32_t v, uint32_t bit) {
  __hip_atomic_fetch_or(&Q.parked[v], bit, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_AGENT);
  if (!(__hip_atomic_fetch_or(&Q.st[v], 0u, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_AGENT) &
        (v == t ? TS_RUNNING : (TS_LISTED | TS_RUNNING)))) {
    if (__hip_atomic_fetch_and(&Q.parked[v], ~bit, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_AGENT) &
        bit)
      q_publish(Q, t);
  }
  return false;
}

__device__ bool q_claim(const QueueRef& Q, uint32_t t, const TileCoord& c, const Tiling& tl,
                        uint32_t t0, unsigned long long& parks, bool& first) {
  const uint32_t old =
      __hip_atomic_fetch_or(&Q.st[t], TS_RUNNING, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_AGENT);
  if (old & TS_RUNNING) {
    ++parks;
    return q_park(Q, t, t, 1u << 13);
  }
  if (old & TS_RAN) {
    uint32_t bl = __hip_atomic_load(&Q.blockers[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    while (bl) {
      const int d = 31 - __builtin_clz(bl);  // the farthest in index first
      bl &= ~(1u << d);
      if (!dir_inside(d, c, tl)) continue;
      const uint32_t v = dir_tile(d, c, tl, t0);
      if (!(__hip_atomic_load(&Q.st[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) &
            (TS_LISTED | TS_RUNNING)))
        continue;
      __hip_atomic_fetch_and(&Q.st[t], ~TS_RUNNING, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_AGENT);
      ++parks;
      return q_park(Q, t, v, 1u << (26 - d));
    }
  }
  first = !(old & TS_RAN);
  __hip_atomic_fetch_and(&Q.st[t], ~TS_LISTED, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
  if (first)
    __hip_atomic_fetch_or(&Q.st[t], TS_RAN, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

// End of a run of tile t (wave 0 of its block, whose waves have each waited for
// their subbin stores before the block's last barrier): list the neighbour
// tiles in `dirs` (27-bit set, see out_dirs), stop running, publish the tiles
// parked on t, and stop counting the run as pending.
__device__ void q_finish(uint32_t dirs, uint32_t t, const TileCoord& c, const Tiling& tl,
                         const QueueRef& Q, uint32_t t0, uint32_t depth) {
  if (dirs) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  if (threadIdx.x < 27 && ((dirs >> threadIdx.x) & 1u) && dir_inside((int)threadIdx.x, c, tl))
    q_push(Q, dir_tile((int)threadIdx.x, c, tl, t0), depth);
  uint32_t woke = 0;
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_and(&Q.st[t], ~TS_RUNNING, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_AGENT);
    woke = __hip_atomic_exchange(&Q.parked[t], 0u, __ATOMIC_SEQ_CST, __HIP_MEMORY_SCOPE_AGENT);
  }
  woke = __shfl(woke, 0, 64);
  if (threadIdx.x < 27 && ((woke >> threadIdx.x) & 1u))
    q_publish(Q, dir_tile((int)threadIdx.x, c, tl, t0));
  if (threadIdx.x == 0)
    __hip_atomic_fetch_add(&Q.q->pending, -1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

template <int TZ, int TY, int TX>
__constant__ const Faces<TZ, TY, TX> kFaces{};

// A lane's point on face slot f of the tile at c: its LDS index (-1: none),
// offset from the field's first point (g00: the tile's first point) and
// whether it lies in the grid.
struct FacePoint {
  int li;
  int64_t g;
  bool in;
};
__device__ __forceinline__ FacePoint face_point(const FaceSlot& f, int ln, const TileCoord& c,
                                                const Box& box, int64_t g00) {
  // (a plane has fewer than 2^32 points, so steps are 32-bit factors)
  const uint32_t nx = (uint32_t)box.nx, nyx = (uint32_t)box.ny * (uint32_t)box.nx;
  const uint32_t r = (uint32_t)f.r0 + (uint32_t)ln;
  const uint32_t u = __umul24(r, (uint32_t)f.magic) >> 16, v = r - __umul24(u, (uint32_t)f.width);
  const bool uz = f.ua == 2, vy = f.va == 1;
  const uint32_t lz = (uint32_t)box.nz, ly = (uint32_t)box.ny;
  const uint32_t bz = (uint32_t)(c.z0 + f.z), by = (uint32_t)(c.y0 + f.y),
                 bx = (uint32_t)(c.x0 + f.x);
  const uint32_t gu = uz ? nyx : nx, gv = vy ? nx : 1u;
  const uint32_t lu = uz ? lz : ly, lv = vy ? ly : nx, bu = uz ? bz : by, bv = vy ? by : bx;
  // the axis the face is normal to (neither u's nor v's): in the grid for all
  // of it or none
  const uint32_t pn = vy ? bx : uz ? by : bz, pl = vy ? nx : uz ? ly : lz;
  // lanes of the slot past the face, or none where the face is outside
  const uint32_t lim = pn < pl ? (uint32_t)f.cnt : 0u;
  FacePoint p;
  p.in = (r < lim) & (bu + u < lu) & (bv + v < lv);
  const int64_t g0 = g00 + (int64_t)f.z * (int64_t)nyx + (int64_t)f.y * (int64_t)nx + f.x;
  p.g = (int64_t)((uint64_t)g0 + (uint64_t)v * gv + (uint64_t)u * gu);
  p.li = r < (uint32_t)f.cnt ? f.li + (int)__umul24(u, (uint32_t)f.lu) + (int)__umul24(v, (uint32_t)f.lv)
                             : -1;
  return p;
}
// The neighbour tile of halo cell li as its bit of the 27-direction set.
template <int TZ, int TY, int TX>
__device__ __forceinline__ uint32_t cell_dir(int li) {
  using G = TileGeom<TZ, TY, TX>;
  const int hz = li / (G::HY * G::HX), hy = (li / G::HX) % G::HY, hx = li % G::HX;
  const int dz = G::ZO ? (hz == 0 ? 0 : hz == G::HZ - 1 ? 2 : 1) : 1,
            dy = hy == 0 ? 0 : hy == G::HY - 1 ? 2 : 1, dx = hx == 0 ? 0 : hx == G::HX - 1 ? 2 : 1;
  return 1u << (dz * 9 + dy * 3 + dx);
}

// m becomes 2m + (a and b of the lane): the conditions as lane masks, joined on
// the scalar side, shifted in by one add with carry.
__device__ __forceinline__ uint32_t shift_in(uint32_t m, uint64_t a, uint64_t b) {
  uint32_t r;
  asm("s_and_b64 vcc, %2, %3\n\tv_addc_co_u32_e32 %0, vcc, %1, %1, vcc"
      : "=v"(r) : "v"(m), "s"(a), "s"(b) : "vcc", "scc");
  return r;
}

// First pass of a tile, fused: quantize (a1), the order flags of the owned
// points (a2, the flags of Alg. 1), and the first relaxation (the first sweep
// of a3) with halo subbins 0 or, for hc >= 0, those of the neighbour tiles of
// colour hc.  Returns (block-uniform) the neighbour tiles to sweep next.
// The values of the owned points and of the face points around them come in
// once, all loads in flight together; each is quantized once (Sec. IV-A).  In LDS a point holds its value
// and its bin (float64: the low 32 bits of the bin's distance from the tile's
// first bin, which decide equality whenever no bin is 2^30 or more from it,
// else the tile is wide and re-quantizes); a point outside the grid holds a
// bin that no point has, so no comparison needs a bounds check.  An order flag
// is two comparisons, their conjunction on the scalar side and one add with
// carry.  The neighbour tiles to sweep next are found at the end from the
// face points: those with a same-bin lower neighbour in the tile that rose and
// would raise them.
// Bound by vector issue in 3D (0.7 to 0.8 of its rate), by the chains of its
// rounds in 2D: 512^3 binary64 2 x 2.69 -> 2 x 1.85 ms, 256^3 binary32 147 ->
// 128 us, 1800 x 3600 binary32 167 -> 119 us against flags from both keys and
// bins per neighbour and passes to the end.
template <int NPT>
struct ReadyLds {
  uint16_t list[NPT];
  uint32_t tail;
};
template <int K, int TZ, int TY, int TX>
struct FirstLds {
  using G = TileGeom<TZ, TY, TX>;
  typename Traits<K>::Raw x[G::H];  // values
  int32_t b[G::H];                  // bins
  uint32_t P[G::H];                 // LDS words of the relaxation
  // 3D: relaxation; 2D: peeling
  std::conditional_t<(TZ > 1), EventLds<G::NPT>, ReadyLds<G::NPT>> E;
  uint32_t wide, dirs;
};
template <int K, int TZ, int TY, int TX>
__device__ __forceinline__ uint32_t tile0_body(
    const typename Traits<K>::Raw* __restrict__ x, Box box, Tiling tl, Params* prm,
    typename Traits<K>::Bin* __restrict__ bins, uint16_t* __restrict__ mask,
    uint32_t* __restrict__ sub, uint32_t* counters, unsigned long long* itot, uint32_t t,
    TileCoord& c, int hc = -1) {
  using Tr = Traits<K>;
  using Raw = typename Tr::Raw;
  using Val = std::conditional_t<K == 4, float, double>;
  using G = TileGeom<TZ, TY, TX>;
  using F = Faces<TZ, TY, TX>;
  constexpr int HXY = G::HY * G::HX, NJ = TZ == 1 ? 6 : 14;
  __shared__ __attribute__((aligned(16))) FirstLds<K, TZ, TY, TX> lds;
  const Val* X = (const Val*)lds.x;
  int32_t* B = lds.b;
  uint32_t* P = lds.P;
  auto val = [](Raw u) -> Val {
    if constexpr (K == 4) return __uint_as_float(u);
    else return __longlong_as_double((long long)u);
  };
  c = tile_coord<TZ, TY, TX>(t, tl);
  const int w = __builtin_amdgcn_readfirstlane(wave());
  const int li0 = G::local(threadIdx.x);
  const int64_t nyx = (int64_t)box.ny * box.nx;
  const int64_t g00 = ((int64_t)c.z0 * box.ny + c.y0) * box.nx + c.x0;
  // slot k of a thread: k planes (2D: k times kRows rows) after slot 0
  constexpr int PZ = G::PER, kRows = kThreads / TX;
  const int iy = (int)threadIdx.x / TX, ix = (int)threadIdx.x % TX;
  const int64_t g0 = g00 + (int64_t)iy * box.nx + ix;
  const int64_t gstep = TZ > 1 ? nyx : (int64_t)kRows * box.nx;
  const bool in0 = (TZ == 1 || c.y0 + iy < box.ny) && c.x0 + ix < box.nx;
  auto in = [&](int k) {
    return in0 && (TZ > 1 ? c.z0 + k < box.nz : c.y0 + iy + k * kRows < box.ny);
  };
  // values: the owned points, the face points (points outside the grid read
  // the tile's first)
  Raw u[PZ], hu[F::kPer];
  int hl[F::kPer];
  uint32_t hin = 0;  // bit q: face point q lies in the grid
#pragma unroll
  for (int k = 0; k < PZ; ++k) u[k] = x[in(k) ? g0 + k * gstep : g00];
  uint32_t hs[F::kPer];  // subbins of the face points of colour hc
#pragma unroll
  for (int q = 0; q < F::kPer; ++q) {
    hl[q] = -1;
    hu[q] = 0;
    hs[q] = 0;
    if (w + q * kWaves >= F::kSlots) continue;
    const FacePoint f = face_point(kFaces<TZ, TY, TX>.s[w + q * kWaves], lane(), c, box, g00);
    hu[q] = x[f.in ? f.g : g00];
    hin |= (uint32_t)f.in << q;
    hl[q] = f.li;
    if (hc >= 0) {
      // tiles across one face or one corner have the other colour, across an
      // edge the same; those of colour hc are final from an earlier launch
      const uint32_t d = cell_dir<TZ, TY, TX>(f.li < 0 ? 0 : f.li);
      const bool take = f.in && !(d & same_colour_dirs());
      const uint32_t v = sub[take ? f.g : g00];
      hs[q] = take ? v : 0u;
    }
  }
  if (threadIdx.x == 0) {
    lds.wide = 0;
    lds.dirs = 0;
  }
  const double inv = prm->inv;
  bool bad_v = false, bad_r = false, far = false;
  const int64_t bref =
      K == 8 ? first_bin<K>(Tr::to_double(x[g00]), inv, bad_r) : 0;
  auto low = [&](int64_t b) -> int32_t {
    if constexpr (K == 4) return (int32_t)b;
    const uint64_t d = (uint64_t)b - (uint64_t)bref;
    far |= d + (1ull << 30) >= (1ull << 31);
    return (int32_t)(uint32_t)d;
  };
  __syncthreads();  // lds.wide
  int32_t bo[PZ];
#pragma unroll
  for (int k = 0; k < PZ; ++k) {
    bad_v |= !Tr::finite(u[k]);
    const int64_t b = first_bin<K>(Tr::to_double(u[k]), inv, bad_r);
    bo[k] = in(k) ? low(b) : kNoBin;
    if (in(k)) bins[g0 + k * gstep] = (typename Tr::Bin)b;  // for the encoder
    lds.x[li0 + k * G::kSlot] = u[k];
    B[li0 + k * G::kSlot] = bo[k];
  }
#pragma unroll
  for (int q = 0; q < F::kPer; ++q) {
    const int64_t b = first_bin<K>(Tr::to_double(hu[q]), inv, bad_r);
    const int32_t lb = (hin >> q) & 1u ? low(b) : kNoBin;
    if (hl[q] >= 0) {
      lds.x[hl[q]] = hu[q];
      B[hl[q]] = lb;
    }
  }
  if (bad_v) set_status(prm, ST_NONFINITE);
  if (bad_r) set_status(prm, ST_RANGE);
  if (K == 8 && __ballot(far) && lane() == 0) lds.wide = 1;
  __syncthreads();
  const bool wide = K == 8 && lds.wide;
  // order flags: same bin and lower in (value, index) order
  uint16_t mk[PZ];
#pragma unroll
  for (int k = 0; k < PZ; ++k) {
    const int li = li0 + k * G::kSlot;
    const Val vp = val(u[k]);
    uint32_t m = 0;
#pragma unroll
    for (int j = NJ - 1; j >= 0; --j) {
      const int ln = li + kOff[j][0] * HXY + kOff[j][1] * G::HX + kOff[j][2];
      const Val vq = X[ln];
      m = shift_in(m, __ballot(B[ln] == bo[k]), __ballot(flag_lower(j, vq, vp)));
    }
    if (wide && in(k)) {
      uint32_t lm = 0;
      const int z = c.z0 + (TZ > 1 ? k : 0), y = c.y0 + iy + (TZ > 1 ? 0 : k * kRows),
                xx = c.x0 + ix;
#pragma unroll 1
      for (int j = 0; j < NJ; ++j) {
        const int zz = z + off_z(j), yy = y + off_y(j), xq = xx + off_x(j);
        if (zz < 0 || zz >= box.nz || yy < 0 || yy >= box.ny || xq < 0 || xq >= box.nx) continue;
        const Val vq = X[li + off_lin(j, G::HX, HXY)];
        const bool same = q_bin((double)vq, inv) == q_bin((double)vp, inv);
        lm |= (uint32_t)(same && (vq < vp || (vq == vp && (j & 1)))) << j;
      }
      m = lm;
    }
    mk[k] = in(k) ? (uint16_t)m : (uint16_t)0;
    if constexpr (TZ > 1) {
      if (in(k)) mask[g0 + k * gstep] = (uint16_t)m;
      P[li] = kNoFlags & ~((uint32_t)mk[k] << 16);
    } else {
      // the count of lower neighbours inside the tile
      const int ry = iy + k * kRows;
      const uint32_t inb = (ry == 0 ? ~0x28u : ~0u) & (ry == TY - 1 ? ~0x14u : ~0u) &
                           (ix == 0 ? ~0x22u : ~0u) & (ix == TX - 1 ? ~0x11u : ~0u);
      P[li] = ((0x3fu & ~(uint32_t)mk[k]) << 16) |
              (uint32_t)__popc(mk[k] & inb) << kLeftShift;
    }
  }
#pragma unroll
  for (int q = 0; q < F::kPer; ++q)
    if (hl[q] >= 0) P[hl[q]] = kNoFlags | kHalo | hs[q];
  for (int i = threadIdx.x; i < Blind<TZ, TY, TX>::kCells; i += kThreads)
    P[Blind<TZ, TY, TX>::cell(i)] = kNoFlags | kHalo;
  // (a first run's subbins stay below twice the points of a tile: 16 bits)
  if constexpr (TZ > 1) {
    relax<TZ, TY, TX, K == 8>(P, lds.E, mk, counters, itot, t);
  } else {
    const int levels = peel<TZ, TY, TX>(P, lds.E.list, &lds.E.tail);
    if (threadIdx.x == 0) atomicAdd(&itot[t % 64], (unsigned long long)(levels + 1));
  }
#pragma unroll
  for (int k = 0; k < PZ; ++k)
    if (in(k)) {
      const uint32_t v = P[li0 + k * G::kSlot];
      sub[g0 + k * gstep] = v & 0xffffu;
      if constexpr (TZ == 1)
        mask[g0 + k * gstep] = (uint16_t)(mk[k] | (v >> kLeftShift & 0xffu) << kLevelShift);
    }
  uint32_t dirs = 0;
#pragma unroll
  for (int q = 0; q < F::kPer; ++q) {
    if (w + q * kWaves >= F::kSlots) continue;
    const FaceSlot& f = kFaces<TZ, TY, TX>.s[w + q * kWaves];
    const bool on = (hin >> q) & 1u;
    const int l = on ? hl[q] : f.li;
    // a target's subbin above th raises the point beyond what it has (what
    // its tile took from a subbin of 0 it already has); the target has the
    // higher index, weight 1, on low faces
    const uint32_t wt = 1u - f.weight;
    const uint32_t th = !on ? 0xffffu : hs[q] > wt ? hs[q] - wt : 0u;
    uint64_t up[F::ND], any = 0;
#pragma unroll
    for (int k = 0; k < F::ND; ++k) {
      up[k] = __ballot((P[l + f.d[k]] & (0xffffu | kHalo)) - th - 1u < 0xffffu);
      any |= up[k];
    }
    if (!any) continue;
    const Val vh = val(hu[q]);
    const int32_t bh = B[l];
    any = 0;
#pragma unroll
    for (int k = 0; k < F::ND; ++k) {
      const Val vq = X[l + f.d[k]];
      const uint64_t lt = __ballot(vq < vh), le = __ballot(vq <= vh);
      uint64_t same = __ballot(B[l + f.d[k]] == bh);
      if (wide) same = __ballot(q_bin((double)vq, inv) == q_bin((double)vh, inv));
      any |= up[k] & (f.weight ? le : lt) & same;
    }
    if ((any >> lane()) & 1u) dirs |= cell_dir<TZ, TY, TX>(l);
  }
  if (__ballot(dirs != 0u)) {
    dirs = wave_reduce(dirs, OpOr{});
    if (lane() == 0) atomicOr(&lds.dirs, dirs);
  }
  __syncthreads();
  return lds.dirs;
}

// Waves per SIMD the first pass is held to (its register budget).
template <int K, int TZ, int TY, int TX>
constexpr int kTile0Waves = TZ * TY * TX > 1024 && TZ > 1 ? (K == 4 ? 3 : 2) : K == 4 ? 5 : TZ > 1 ? 4 : 3;

// Q.q null: mark the tiles to sweep next (and append them to the work list
// of sweep 1 when lists is given); else list them in the repair queue (the
// kernel boundary publishes the subbins).
template <int K, int TZ, int TY, int TX>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(kTile0Waves<K, TZ, TY, TX>, 8))) void k_tile0(
    const typename Traits<K>::Raw* __restrict__ x, Box box, Tiling tl, Params* prm,
    typename Traits<K>::Bin* __restrict__ bins,
    uint16_t* __restrict__ mask, uint32_t* __restrict__ sub, uint32_t* stamp,
    uint32_t* counters, uint32_t* lists, QueueRef Q, uint32_t colour) {
  TileCoord c;
  // colour 2: every tile; 0 / 1: the tiles of that colour, those of colour 1
  // taking the subbins of their neighbours of colour 0 as halo
  const uint32_t b = xcd_tile(blockIdx.x, gridDim.x);
  const uint32_t t = colour < 2 ? colour_tile(b, colour, tl) : b;
  if (t >= tl.ntiles) return;
  uint32_t dirs = tile0_body<K, TZ, TY, TX>(x, box, tl, prm, bins, mask, sub, counters,
                                            relax_total(counters), t, c, colour == 1 ? 0 : -1);
  // tiles of colour 1 read the results of colour 0 in the next launch
  if (colour == 0) dirs &= same_colour_dirs();
  if (Q.q) {
    if (threadIdx.x < 27 && ((dirs >> threadIdx.x) & 1u) && dir_inside((int)threadIdx.x, c, tl))
      q_push(Q, dir_tile((int)threadIdx.x, c, tl, 0), 1);
  } else if (lists) {
    mark_list1(dirs, c, tl, stamp, counters, lists, 1);
  } else {
    mark_neighbours(dirs, c, tl, stamp, counters, 1);
  }
}


// LDS of a run, handed in by the kernel (one buffer where it runs 2D and 3D
// tiles).
template <int TZ, int TY, int TX>
struct RunLds {
  uint32_t P[TileGeom<TZ, TY, TX>::H];  // LDS words (32-bit way: subbins)
  EventLds<TZ * TY * TX> E;
  alignas(16) uint32_t hist[TZ == 1 ? 256 : 4];  // 2D: points of each level
  uint32_t go;
};

// The owned points of a 2D tile level by level (P: LDS words; WIDE: subbins
// in 32 bits; flags(k): those of slot k): a point's level is the longest path
// of its lower neighbours inside the tile, kept by the first pass (level(k)),
// so one visit in this order, the halo fixed, gives every point its final
// value.  The points with flags are sorted into `list` (a counting sort; LDS
// index, flags and level to an entry), then the first wave takes them, up to 64
// of one level at a time: per step one LDS round trip, with the next entries
// already on their way, no atomics and no barriers.  Returns the steps
// (block-uniform), -1 before it has touched P if a level is not known (255).
template <int TZ, int TY, int TX, bool WIDE, typename Flags, typename Level>
__device__ __forceinline__ int level_run(RunLds<TZ, TY, TX>& lds, int tid, const Flags& flags,
                                         const Level& level) {
  using G = TileGeom<TZ, TY, TX>;
  static_assert(TZ == 1, "2D tiles");
  constexpr int NJ = 6, HX = G::HX, HXY = G::HY * G::HX;
  uint32_t* const P = lds.P;
  uint32_t* const list = (uint32_t*)&lds.E.list[0][0][0];
  static_assert(sizeof(lds.E.list) >= G::NPT * 4 && G::H <= 4096, "the entries fit");
  uint32_t* const unknown = &lds.E.rose[0];
  uint32_t lv[G::PER / 4] = {};  // four levels to a word
#pragma unroll
  for (int k = 0; k < G::PER; ++k) lv[k / 4] |= level(k) << (8 * (k % 4));
  static_assert(kThreads == 256 && G::PER % 4 == 0, "a counter per thread");
  lds.hist[tid] = 0;
  if (tid == 0) *unknown = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < G::PER; ++k) {
    const uint32_t l = (lv[k / 4] >> (8 * (k % 4))) & 255u;
    if (flags(k)) {
      if (l == 255u) *unknown = 1;
      atomicAdd(&lds.hist[l], 1u);
    }
  }
  __syncthreads();
  const bool none = *unknown != 0;
  // the counts become starts
  if (tid < 64) {
    const uint4 v = ((const uint4*)lds.hist)[tid & 63];
    const uint32_t t = v.x + v.y + v.z + v.w, b = wave_scan_u32(t) - t;
    ((uint4*)lds.hist)[tid & 63] = make_uint4(b, b + v.x, b + v.x + v.y, b + v.x + v.y + v.z);
  }
  __syncthreads();
  if (none) return -1;
  // no point has level 255: its start is the number of points
  const uint32_t total = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds.hist[255]);
#pragma unroll
  for (int k = 0; k < G::PER; ++k) {
    const uint32_t l = (lv[k / 4] >> (8 * (k % 4))) & 255u, f = flags(k);
    if (f)
      list[atomicAdd(&lds.hist[l], 1u)] =
          (uint32_t)(G::local(tid) + k * G::kSlot) | f << 12 | l << 18;
  }
  __syncthreads();
  int steps = 0;
  if (tid < 64) {
    uint32_t pos = 0, ent = list[tid & 63];
    while (pos < total) {
      const uint32_t l0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(ent >> 18));
      const uint64_t other = ~__ballot((ent >> 18) == l0 && pos + (uint32_t)(tid & 63) < total);
      const uint32_t n = other ? (uint32_t)__builtin_ctzll(other) : 64u;
      pos += n;
      const uint32_t next = list[min(pos + (uint32_t)(tid & 63), (uint32_t)G::NPT - 1u)];
      const bool act = (uint32_t)(tid & 63) < n;
      const int li = act ? (int)(ent & 4095u) : G::local(0);
      const uint32_t f = (ent >> 12) & 0x3fu, wd = P[li];
      uint32_t q[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) q[j] = P[li + kOff[j][0] * HXY + kOff[j][1] * HX + kOff[j][2]];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const uint32_t on = (uint32_t)((int32_t)(f << (31 - j)) >> 31);
        q[j] = WIDE ? q[j] & on : and_word(q[j], on);
      }
      const uint32_t cur = WIDE ? wd : wd & 0xffffu;
      const uint32_t best = fold_cands<NJ>(q, f, cur);
      if (act && best > cur) P[li] = WIDE ? best : (wd + (best - cur)) | kRose;
      ent = next;
      ++steps;
    }
  }
  __syncthreads();
  return steps;
}

// End of a tile run: the neighbour tiles of the lanes' dirs (27-direction set),
// block-uniform; with `blockers` (queue mode), thread 0 stores there those of
// higher index in `ups`.
template <bool QM, int NPT>
__device__ __forceinline__ uint32_t end_run(EventLds<NPT>& E, uint32_t dirs, uint32_t ups,
                                            uint32_t* blockers, uint32_t t) {
  // queue mode: every wave's subbins have to be out before wave 0, past the
  // barriers below, lets the tile go (q_finish), as its next run, on whatever
  // XCD, starts from them; a barrier alone does not wait for stores.  They are
  // agent-scope stores, which write through, so waiting for them is enough: a
  // release fence would write the whole L2 back (queue alone, 128^3 float64
  // lognormal 35.9 -> 31.0 ms, 128^3 float32 turbulence 1.25 -> 1.02 ms)
  if (QM) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if (QM && blockers) {
    const uint64_t both = block_or64((uint64_t)ups << 32 | dirs);
    if (threadIdx.x == 0) blockers[t] = (uint32_t)(both >> 32) & ~0x3fffu;
    return (uint32_t)both;
  }
  if (__ballot(dirs != 0u)) {
    dirs = wave_reduce(dirs, OpOr{});
    if (lane() == 0) atomicOr(&E.dirs, dirs);
  }
  __syncthreads();
  return E.dirs;
}

// The rest of a tile run over all of its points instead of events (2D by
// levels, else by passes): after more events than that takes (the words in LDS
// as the events left them), or, `wide`, from the start with 32-bit subbins.
// Its loops are rolled up and start from the thread's place alone (opaque), so
// that inlined it leaves the sweeps the registers of their event runs (3D 49,
// 2D 56; unrolled and called 87 and 100, rolled up and called 74 and 87).
// Bound by the chain of its steps.  Against events and passes to the end: 1800
// x 3600 fronts at bound 1e-2 2,250 -> 715 us a call, at 1e-1 8,830 -> 2,025, at
// 1e0 19,050 -> 7,160; with 32-bit subbins a chain of 2^18 points in a row
// 1,578 -> 318 ms under host sweeps.
template <int TZ, int TY, int TX, bool QM>
__device__ __forceinline__ uint32_t whole_run(RunLds<TZ, TY, TX>& lds, Box box, Tiling tl,
                                           const uint16_t* __restrict__ mask,
                                           uint32_t* __restrict__ sub, uint32_t* counters,
                                           unsigned long long* itot, uint32_t t,
                                           uint32_t* blockers, bool wide) {
  using G = TileGeom<TZ, TY, TX>;
  using F = Faces<TZ, TY, TX>;
  constexpr int NJ = TZ == 1 ? 6 : 14, HXY = G::HY * G::HX;
  int tid = (int)threadIdx.x;
  asm volatile("" : "+v"(tid));
  __builtin_assume(tid >= 0 && tid < kThreads);
  uint32_t* const P = lds.P;
  const TileCoord c = tile_coord<TZ, TY, TX>(t, tl);
  const int w = __builtin_amdgcn_readfirstlane(wave());
  const int li0 = G::local(tid);
  const int64_t g00 = ((int64_t)c.z0 * box.ny + c.y0) * box.nx + c.x0;
  // slot k's offset from the tile's first point (that point's if outside)
  constexpr int kRows = TZ > 1 ? 1 : kThreads / TX;
  const int iy = tid / TX, ix = tid % TX;
  const bool in0 = c.x0 + ix < box.nx;
  auto in = [&](int k) {
    return in0 && (TZ > 1 ? c.y0 + iy < box.ny && c.z0 + k < box.nz
                          : c.y0 + iy + k * kRows < box.ny);
  };
  auto at = [&](int k) -> int64_t {
    const int64_t step = TZ > 1 ? (int64_t)box.ny * box.nx : (int64_t)kRows * box.nx;
    return in(k) ? g00 + (int64_t)iy * box.nx + ix + k * step : g00;
  };
  auto load = [&](int64_t g) {
    return QM ? __hip_atomic_load(sub + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : sub[g];
  };
  auto store = [&](int64_t g, uint32_t v) {
    if (QM) __hip_atomic_store(sub + g, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else sub[g] = v;
  };
  auto level = [&](int k) { return (uint32_t)mask[at(k)] >> kLevelShift; };
  auto flags = [&](int k) {
    const uint32_t m = flags_of<TZ>(mask[at(k)]);
    return in(k) ? m : 0u;
  };
  uint32_t dirs = 0, ups = 0;
  if (QM && blockers) {
#pragma unroll 1
    for (int k = 0; k < G::PER; ++k) {
      const int i = tid + k * kThreads;
      const uint32_t m = flags(k);
      if (m && G::on_edge(i)) ups |= out_dirs<TZ, TY, TX>(i, m);
    }
  }
  int steps = -1;
  if (!wide) {
    if constexpr (TZ == 1)
      steps = level_run<TZ, TY, TX, false>(
          lds, tid, [&](int k) { return (~P[li0 + k * G::kSlot] >> 16) & 0x3fu; }, level);
    if (steps < 0) steps = word_passes<TZ, TY, TX>(P, lds.E, counters);
    // the face points that an event raised or a risen point of the tile would
#pragma unroll 1
    for (int s = w; s < F::kSlots; s += kWaves) {
      const FaceSlot& f = kFaces<TZ, TY, TX>.s[s];
      const FacePoint p = face_point(f, tid & 63, c, box, g00);
      if (!p.in) continue;
      const uint32_t h = P[p.li], wt = 1u - f.weight;
      bool up = (h & kRose) != 0;
#pragma unroll
      for (int k = 0; k < F::ND; ++k) {
        // the flag through which the face point sees the tile's point is the
        // one the point sees it through, from the other end
        const uint32_t x = P[p.li + f.d[k]], seen = f.keep[k] & kNoFlags;
        up |= (x & (kHalo | kRose)) == kRose && !(h & (f.weight ? seen << 1 : seen >> 1)) &&
              (x & 0xffffu) + wt > (h & 0xffffu);
      }
      if (up) dirs |= cell_dir<TZ, TY, TX>(p.li);
    }
#pragma unroll 1
    for (int k = 0; k < G::PER; ++k) {
      const uint32_t v = P[li0 + k * G::kSlot];
      if (v & kRose) store(at(k), v & 0xffffu);
    }
  } else {
    __syncthreads();  // the words have been read
#pragma unroll 2
    for (int k = 0; k < G::PER; ++k) {
      const uint32_t v = load(at(k));
      P[li0 + k * G::kSlot] = in(k) ? v : 0u;
    }
#pragma unroll 1
    for (int s = w; s < F::kSlots; s += kWaves) {
      const FacePoint p = face_point(kFaces<TZ, TY, TX>.s[s], tid & 63, c, box, g00);
      if (p.li >= 0) P[p.li] = p.in ? load(p.g) : 0u;
    }
    __syncthreads();
    if constexpr (TZ == 1) steps = level_run<TZ, TY, TX, true>(lds, tid, flags, level);
    // the flags of the owned and the face points
    uint16_t* const M = &lds.E.list[0][0][0];
    static_assert(sizeof(lds.E.list) >= G::H * 2, "the flags fit the event lists");
#pragma unroll 2
    for (int k = 0; k < G::PER; ++k) M[li0 + k * G::kSlot] = (uint16_t)flags(k);
#pragma unroll 1
    for (int s = w; s < F::kSlots; s += kWaves) {
      const FacePoint p = face_point(kFaces<TZ, TY, TX>.s[s], tid & 63, c, box, g00);
      if (p.li >= 0) M[p.li] = p.in ? (uint16_t)flags_of<TZ>(mask[p.g]) : (uint16_t)0;
    }
    if (steps < 0) steps = relax_wide<TZ, TY, TX>(P, M, counters);
    else __syncthreads();  // M
#pragma unroll 1
    for (int k = 0; k < G::PER; ++k) {
      const int i = tid + k * kThreads, li = li0 + k * G::kSlot;
      const uint32_t v = P[li];
      const int64_t g = at(k);
      if (!in(k) || v == load(g)) continue;
      store(g, v);
      if (!G::on_edge(i)) continue;
      // halo neighbours whose flags name this point (offset j from here is
      // offset j ^ 1 from there)
      const int pz = i / (TY * TX), py = (i / TX) % TY, px = i % TX;
      uint32_t dep = 0;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int z = pz + kOff[j][0], y = py + kOff[j][1], x = px + kOff[j][2];
        if (z < 0 || z >= TZ || y < 0 || y >= TY || x < 0 || x >= TX)
          dep |= (uint32_t)((M[li + kOff[j][0] * HXY + kOff[j][1] * G::HX + kOff[j][2]] >>
                             (j ^ 1)) & 1u) << j;
      }
      if (dep) dirs |= out_dirs<TZ, TY, TX>(i, dep);
    }
  }
  if (threadIdx.x == 0) atomicAdd(&itot[t % 64], (unsigned long long)steps);
  return end_run<QM>(lds.E, dirs, ups, blockers, t);
}

// One sweep of tile t if it is marked for it: a run reloads the subbins and the
// flags of the tile and its halo, raises what follows and writes what rose.
// Returns (block-uniform) the neighbour tiles holding a point that would rise
// from what changed in this tile (0 if the tile did not run).
// A run pushes the halo points into the tile (what changed since the tile's
// last run can only have come from there), then each wave runs event rounds
// from the points it raised; with too many events, or subbins that do not fit
// an LDS word, it goes over the whole tile (whole_run).
// QM (queue mode): the tile was taken from the repair queue, and other
// workgroups change subbins while it runs, so subbins are read and written
// as relaxed atomics at agent scope (coherent across the XCDs' L2 caches).
// LOOP: the tile is known to be marked, and the kernel runs several in turn.
// With `blockers` given, thread 0 stores there the higher-index
// neighbour tiles holding a same-bin lower neighbour of one of the tile's
// points (the tiles its run depends on; bits 14..26 of the 27-direction set).
template <int TZ, int TY, int TX, bool QM = false, bool LOOP = false>
__device__ __forceinline__ uint32_t repair_body(RunLds<TZ, TY, TX>& lds, Box box, Tiling tl,
                            const uint16_t* __restrict__ mask, uint32_t* __restrict__ sub,
                            const uint32_t* stamp, uint32_t* counters,
                            unsigned long long* itot, uint32_t sweep, uint32_t t, TileCoord& c,
                            uint32_t* blockers = nullptr) {
  using G = TileGeom<TZ, TY, TX>;
  using F = Faces<TZ, TY, TX>;
  uint32_t* const P = lds.P;
  EventLds<G::NPT>& E = lds.E;
  // one read decides for the whole block (a neighbour may raise the stamp
  // concurrently)
  if (threadIdx.x == 0) {
    if (!LOOP) lds.go = QM || stamp[t] >= sweep;
    E.big = 0;
    E.over = 0;
    E.dirs = 0;
  }
  __syncthreads();
  if (!LOOP && !lds.go) return 0;
  c = tile_coord<TZ, TY, TX>(t, tl);
  // in a loop: opaque, so that what follows from the thread's place alone is
  // computed anew for each tile instead of held in registers across it
  int tid = (int)threadIdx.x;
  if (LOOP) asm volatile("" : "+v"(tid));
  __builtin_assume(tid >= 0 && tid < kThreads);
  // (the face slots are a multiple of the waves for the default shapes: no
  // branch then stands between their loads)
  const int w = __builtin_amdgcn_readfirstlane(wave());
  __builtin_assume(w >= 0 && w < kWaves);
  const int li0 = G::local(tid);
  const int64_t nyx = (int64_t)box.ny * box.nx;
  const int64_t g00 = ((int64_t)c.z0 * box.ny + c.y0) * box.nx + c.x0;  // the tile's first point
  uint32_t ov[G::PER], hv[F::kPer];
  uint16_t om[G::PER], hm[F::kPer];
  int hl[F::kPer];  // LDS index of the slot's point (-1: none)
  int64_t og[G::PER];
  bool wide;
  {
    // every load issued unconditionally (points outside the grid read the
    // tile's first point and are zeroed afterwards), so that all of them are
    // in flight together
    auto take = [&](int64_t g, bool in, uint32_t& v, uint16_t& m) {
      g = in ? g : g00;
      v = QM ? __hip_atomic_load(sub + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : sub[g];
      m = mask[g];
      v = in ? v : 0u;
      m = in ? (uint16_t)flags_of<TZ>(m) : (uint16_t)0;
    };
#pragma unroll
    for (int k = 0; k < G::PER; ++k) {
      const int i = tid + k * kThreads;
      const int iz = i / (TY * TX), iy = (i / TX) % TY, ix = i % TX;
      og[k] = g00 + iz * nyx + (int64_t)iy * box.nx + ix;
      take(og[k], c.z0 + iz < box.nz && c.y0 + iy < box.ny && c.x0 + ix < box.nx, ov[k], om[k]);
    }
#pragma unroll
    for (int q = 0; q < F::kPer; ++q) {
      hl[q] = -1;
      hv[q] = 0;
      hm[q] = 0;
      if (w + q * kWaves < F::kSlots) {
        const FacePoint f = face_point(kFaces<TZ, TY, TX>.s[w + q * kWaves], tid & 63, c, box, g00);
        take(f.g, f.in, hv[q], hm[q]);
        hl[q] = f.li;
      }
    }
    uint32_t top = 0;
#pragma unroll
    for (int k = 0; k < G::PER; ++k) {
      P[li0 + k * G::kSlot] = (ov[k] | (uint32_t)om[k] << 16) ^ kNoFlags;
      top = max(top, ov[k]);
    }
#pragma unroll
    for (int q = 0; q < F::kPer; ++q) {
      if (hl[q] >= 0) P[hl[q]] = (hv[q] | (uint32_t)hm[q] << 16) ^ (kNoFlags | kHalo);
      top = max(top, hv[q]);
    }
    for (int i = tid; i < Blind<TZ, TY, TX>::kCells; i += kThreads)
      P[Blind<TZ, TY, TX>::cell(i)] = kNoFlags | kHalo;
    if (__ballot(top > kPackMax) && lane() == 0) E.big = 1;
    __syncthreads();
    wide = E.big;
  }
  if (__builtin_expect(wide, 0)) return whole_run<TZ, TY, TX, QM>(lds, box, tl, mask, sub, counters, itot, t, blockers, true);
  // the face points push into the tile
  uint32_t n = 0;
#pragma unroll
  for (int q = 0; q < F::kPer; ++q) {
    if (w + q * kWaves >= F::kSlots) continue;
    const FaceSlot& f = kFaces<TZ, TY, TX>.s[w + q * kWaves];
    const uint32_t nv = hl[q] >= 0 ? hv[q] + f.weight : 0u;
    const int l = hl[q] >= 0 ? hl[q] : f.li;
    uint32_t x[F::ND], old[F::ND];
#pragma unroll
    for (int k = 0; k < F::ND; ++k) x[k] = P[l + f.d[k]];
#pragma unroll
    for (int k = 0; k < F::ND; ++k)
      old[k] = raise_word(&P[l + f.d[k]], (x[k] & f.keep[k]) < nv, x[k], nv);
#pragma unroll
    for (int k = 0; k < F::ND; ++k) list_risen(E, E.list[w][0], n, old[k], l + f.d[k], nv);
  }
  const int rounds = 1 + push_rounds<TZ, TY, TX>(P, E, n);
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(&itot[t % 64], (unsigned long long)rounds);
  if (__builtin_expect(E.over, 0))
    return whole_run<TZ, TY, TX, QM>(lds, box, tl, mask, sub, counters, itot, t, blockers, false);
  // the neighbour tiles whose halo points rose
  uint32_t dirs = 0, ups = 0;
#pragma unroll
  for (int q = 0; q < F::kPer; ++q) {
    if (hl[q] >= 0 && P[hl[q]] >= (kHalo | kRose)) dirs |= cell_dir<TZ, TY, TX>(hl[q]);
  }
#pragma unroll
  for (int k = 0; k < G::PER; ++k) {
    const uint32_t wd = P[li0 + k * G::kSlot];
    if (QM && blockers) {
      const int i = tid + k * kThreads;
      if (om[k] && G::on_edge(i)) ups |= out_dirs<TZ, TY, TX>(i, om[k]);
    }
    if (wd & kRose) {
      if (QM)
        __hip_atomic_store(sub + og[k], wd & 0xffffu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else sub[og[k]] = wd & 0xffffu;
    }
  }
  return end_run<QM>(E, dirs, ups, blockers, t);
}

// mark_neighbours for a sweep run colour by colour: a neighbour of the later
// colour runs later in this same sweep (it is marked for `sweep`), others in
// the next sweep (marked for sweep + 1; an edge neighbour has the same colour
// and may have read the halo already in this same launch); newly marked
// tiles are counted in counters[1 + s % 64] of their sweep s
__device__ void mark_neighbours_col(uint32_t dirs, const TileCoord& c, const Tiling& tl,
                                    uint32_t* stamp, uint32_t* counters, uint32_t sweep,
                                    uint32_t colour) {
  bool now = false, later = false;
  if (threadIdx.x < 27 && ((dirs >> threadIdx.x) & 1u)) {
    const int dz = (int)threadIdx.x / 9 - 1, dy = ((int)threadIdx.x / 3) % 3 - 1,
              dx = (int)threadIdx.x % 3 - 1;
    const int nz = c.tz + dz, ny = c.ty + dy, nx = c.tx + dx;
    if ((dz | dy | dx) != 0 && nz >= 0 && nz < tl.ntz && ny >= 0 && ny < tl.nty && nx >= 0 &&
        nx < tl.ntx) {
      const uint32_t u = ((uint32_t)nz * tl.nty + ny) * tl.ntx + nx;
      const uint32_t next = tile_colour(nz, ny, nx) > colour ? sweep : sweep + 1;
      const bool newly = atomicMax(&stamp[u], next) < next;
      now = newly && next == sweep;
      later = newly && next != sweep;
    }
  }
  if (threadIdx.x < 64) {
    const uint64_t a = __ballot(now), b = __ballot(later);
    if (threadIdx.x == 0 && a) atomicAdd(&counters[1 + (sweep & 63)], (uint32_t)__popcll(a));
    if (threadIdx.x == 0 && b)
      atomicAdd(&counters[1 + ((sweep + 1) & 63)], (uint32_t)__popcll(b));
  }
}

// One sweep (colour 2: every tile) or one colour of a sweep: the tiles of
// colour `colour` marked for this sweep run.  A coloured sweep runs colour
// 0, then colour 1, so a tile of colour 1 sees what its face and corner
// neighbours changed earlier in the same sweep.
template <int TZ, int TY, int TX>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(6, 8))) void k_repair(
    Box box, Tiling tl, const uint16_t* __restrict__ mask,
    uint32_t* __restrict__ sub, uint32_t* stamp, uint32_t* counters,
    uint32_t sweep, uint32_t colour) {
  const uint32_t b = xcd_tile(blockIdx.x, gridDim.x);
  const uint32_t t = colour < 2 ? colour_tile(b, colour, tl) : b;
  if (t >= tl.ntiles) return;
  TileCoord c;
  __shared__ RunLds<TZ, TY, TX> lds;
  const uint32_t dirs = repair_body<TZ, TY, TX>(lds, box, tl, mask, sub, stamp, counters,
                                                relax_total(counters), sweep, t, c);
  if (!dirs) return;
  if (colour < 2) mark_neighbours_col(dirs, c, tl, stamp, counters, sweep, colour);
  else mark_neighbours(dirs, c, tl, stamp, counters, sweep + 1);
}

// The same sweep where few tiles are marked: of the n tiles (of that colour) a
// workgroup looks at every gridDim.x-th from its own on, all marks in one read,
// and runs the marked ones in turn.  With a workgroup per tile a sweep takes the
// time to start them all and read their marks: 30 us for 65,536 tiles of a
// colour, whatever is marked.  Where many are marked that is the better: a
// workgroup starts as another ends, and its registers leave room for eight
// (512^3 float64 lognormal: all sweeps this way 12.35 ms a call, none 10.9).
template <int TZ, int TY, int TX>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(kFewWaves, 8))) void k_repair_few(
    Box box, Tiling tl, const uint16_t* __restrict__ mask,
    uint32_t* __restrict__ sub, uint32_t* stamp, uint32_t* counters,
    uint32_t sweep, uint32_t colour, uint32_t n) {
  __shared__ RunLds<TZ, TY, TX> lds;
  __shared__ uint64_t s_go;
  const uint32_t b0 = xcd_tile(blockIdx.x, gridDim.x);
  auto tile = [&](uint32_t b) { return colour < 2 ? colour_tile(b, colour, tl) : b; };
  // one read decides for the whole block (a neighbour may raise the stamp
  // concurrently); gridDim.x is at least n / 64
  if (threadIdx.x < 64) {
    const uint32_t b = b0 + (uint32_t)lane() * gridDim.x;
    bool go = false;
    if (b < n) {
      const uint32_t t = tile(b);
      go = t < tl.ntiles && stamp[t] >= sweep;
    }
    const uint64_t m = __ballot(go);
    if (threadIdx.x == 0) s_go = m;
  }
  __syncthreads();
  uint64_t go = s_go;
  go = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)go) |
       (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(go >> 32)) << 32;
  while (go) {
    const uint32_t t = tile(b0 + (uint32_t)__builtin_ctzll(go) * gridDim.x);
    go &= go - 1;
    TileCoord c;
    const uint32_t dirs = repair_body<TZ, TY, TX, false, true>(
        lds, box, tl, mask, sub, stamp, counters, relax_total(counters), sweep, t, c);
    if (dirs) {
      if (colour < 2) mark_neighbours_col(dirs, c, tl, stamp, counters, sweep, colour);
      else mark_neighbours(dirs, c, tl, stamp, counters, sweep + 1);
    }
    if (go) __syncthreads();  // the next tile's LDS
  }
}

// One sweep over a work list: a persistent grid takes the listed tiles
// through a cursor; each reloads its halo, relaxes, writes what changed and
// lists the neighbour tiles that depend on a changed boundary point for the
// next sweep.  An empty list costs one atomic per workgroup.  The run is out
// of line, like repair_run below: the kernel takes 103 registers (3D; 116 in
// 2D), inlined and held to 6 waves per SIMD 72 (80), which gains on the largest
// fields and loses more on others (512^3 float64 18.9 -> 17.8 ms a call, 128^3
// 0.62 -> 0.77).
template <int TZ, int TY, int TX>
__device__ __noinline__ uint32_t sweep_run(Box box, Tiling tl, const uint16_t* __restrict__ mask,
                                           uint32_t* __restrict__ sub, const uint32_t* stamp,
                                           uint32_t* counters, uint32_t sweep, uint32_t t) {
  __shared__ RunLds<TZ, TY, TX> lds;
  TileCoord c;
  return repair_body<TZ, TY, TX>(lds, box, tl, mask, sub, stamp, counters, relax_total(counters),
                                 sweep, t, c);
}

template <int TZ, int TY, int TX>
__global__ __launch_bounds__(kThreads) void k_sweep_list(
    Box box, Tiling tl, const uint16_t* __restrict__ mask, uint32_t* __restrict__ sub,
    uint32_t* stamp, uint32_t* counters, uint32_t* lists, uint32_t sweep) {
  __shared__ uint32_t s_it;
  const uint32_t n = counters[1 + (sweep & 63)];
  const uint32_t* in = lists + (sweep & 1) * tl.ntiles;
  for (;;) {
    if (threadIdx.x == 0) s_it = atomicAdd(&counters[kCursorWord + (sweep & 63)], 1u);
    __syncthreads();
    const uint32_t it = s_it;
    __syncthreads();
    if (it >= n) break;
    const uint32_t t = in[it];
    const uint32_t dirs = sweep_run<TZ, TY, TX>(box, tl, mask, sub, stamp, counters, sweep, t);
    if (dirs) mark_list1(dirs, tile_coord<TZ, TY, TX>(t, tl), tl, stamp, counters, lists,
                         sweep + 1);
  }
}

// ---------------------------------------------------------- point worklists
// The paper's schedule of the repair, for comparison [Sec. IV-D, the loop of
// Alg. 1]: worklists of single points instead of tiles.  Iteration `it`
// recomputes the points listed for it from their lower neighbours in global
// memory and lists, for iteration it + 1, the upper neighbours of those that
// rose, each at most once per iteration (a per-point stamp holds the last
// iteration the point was listed for).  The two lists alternate; the list
// lengths sit in a 64-slot ring of counters.  Subbins only rise and stay
// below the least fixed point, so concurrent reads of stale values are
// harmless: a point that reads a value before it rises is listed again.

// list every point with a same-bin lower neighbour for iteration 0
__global__ __launch_bounds__(kThreads) void k_point_seed(const uint16_t* __restrict__ mask,
                                                         uint32_t n, uint32_t* wl,
                                                         uint32_t* ring) {
  for (uint32_t base = blockIdx.x * kThreads; base < n; base += gridDim.x * kThreads) {
    const uint32_t i = base + threadIdx.x;
    const bool go = i < n && mask[i] != 0;
    const uint64_t b = __ballot(go);
    if (!b) continue;  // wave-uniform
    uint32_t pos = 0;
    if (lane() == 0) pos = atomicAdd(&ring[0], (uint32_t)__popcll(b));
    pos = (uint32_t)__builtin_amdgcn_readfirstlane((int)pos);
    if (go) wl[pos + lane_prefix(b)] = i;
  }
}

__global__ __launch_bounds__(kThreads) void k_point_iter(Box box, const uint16_t* __restrict__ mask,
                                                         uint32_t* sub, const uint32_t* win,
                                                         uint32_t* wout, uint32_t* ring,
                                                         uint32_t* pstamp, uint32_t it) {
  const uint32_t nin = ring[it & 63];
  const uint32_t nx = (uint32_t)box.nx, nxy = (uint32_t)box.nx * (uint32_t)box.ny;
  for (uint32_t base = blockIdx.x * kThreads; base < nin; base += gridDim.x * kThreads) {
    const uint32_t e = base + threadIdx.x;
    bool rose = false;
    uint32_t p = 0;
    int z = 0, y = 0, x = 0;
    if (e < nin) {
      p = win[e];
      z = (int)(p / nxy);
      y = (int)((p / nx) % (uint32_t)box.ny);
      x = (int)(p % nx);
      const uint32_t m = box.nz == 1 ? flags_of<1>(mask[p]) : mask[p];
      const uint32_t cur = sub[p];
      uint32_t best = cur;
#pragma unroll
      for (int j = 0; j < 14; ++j) {
        if ((m >> j) & 1u) {  // a flagged neighbour lies in the grid
          const uint32_t q = p + (uint32_t)(kOff[j][0] * (int)nxy + kOff[j][1] * (int)nx + kOff[j][2]);
          const uint32_t c = sub[q] + ((j & 1) ? 0u : 1u);
          best = c > best ? c : best;
        }
      }
      if (best > cur) {
        atomicMax(&sub[p], best);
        rose = true;
      }
    }
    // list the upper neighbours of the points that rose: q at offset j from
    // p whose flags name p (flag j ^ 1)
#pragma unroll
    for (int j = 0; j < 14; ++j) {
      bool app = false;
      uint32_t q = 0;
      if (rose) {
        const int zz = z + kOff[j][0], yy = y + kOff[j][1], xx = x + kOff[j][2];
        if (zz >= 0 && zz < box.nz && yy >= 0 && yy < box.ny && xx >= 0 && xx < box.nx) {
          q = ((uint32_t)zz * (uint32_t)box.ny + (uint32_t)yy) * nx + (uint32_t)xx;
          app = ((mask[q] >> (j ^ 1)) & 1u) && atomicMax(&pstamp[q], it + 1) < it + 1;
        }
      }
      const uint64_t b = __ballot(app);
      if (b) {
        const int leader = __builtin_ctzll(b);
        uint32_t pos = 0;
        if (lane() == leader) pos = atomicAdd(&ring[(it + 1) & 63], (uint32_t)__popcll(b));
        pos = (uint32_t)__builtin_amdgcn_readlane((int)pos, leader);
        if (app) wout[pos + lane_prefix(b)] = q;
      }
    }
  }
}

// The tiles listed for sweep `sweep` become the first items of the queue.
__global__ __launch_bounds__(kThreads) void k_seed_queue(const uint32_t* counters,
                                                         const uint32_t* lists, uint32_t ntiles,
                                                         uint32_t sweep, QueueRef Q) {
  const uint32_t n = counters[1 + (sweep & 63)];
  const uint32_t* in = lists + (sweep & 1) * ntiles;
  for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads)
    q_push(Q, in[i], sweep);
}

// Device-driven repair of a single field: a persistent grid takes tiles from
// the repair queue until nothing is listed or running.  A tile run reloads
// the halo, relaxes, writes what changed, waits until that is out and lists the
// neighbour tiles that depend on a changed boundary point; then the run
// stops counting as pending.  Subbins only rise and stay below the least
// fixed point, so the result does not depend on the order of the runs.

// One queued tile run, kept out of line, so that what the body derives from the
// thread's place is not hoisted out of the worker loop and held across it.  Its
// LDS arrays are its own, so their accesses still compile to ds_* instructions.
template <int TZ, int TY, int TX>
__device__ __noinline__ uint32_t repair_run(Box box, Tiling tl, const uint16_t* __restrict__ mask,
                                            uint32_t* __restrict__ sub, uint32_t* counters,
                                            uint32_t t, uint32_t* blockers) {
  __shared__ RunLds<TZ, TY, TX> lds;
  TileCoord c;
  return repair_body<TZ, TY, TX, true>(lds, box, tl, mask, sub, nullptr, counters,
                                       relax_total(counters), 0, t, c, blockers);
}

template <int TZ, int TY, int TX>
__global__ __launch_bounds__(kThreads) void k_repair_q(
    Box box, Tiling tl, const uint16_t* __restrict__ mask, uint32_t* __restrict__ sub,
    uint32_t* counters, QueueRef Q) {
  __shared__ uint32_t s_item, s_depth, s_first;
  unsigned long long runs = 0, parks = 0;
  uint32_t deepest = 0;
  // nothing listed (the usual end of the work-list sweeps): leave at once
  // without taking tickets
  if (__hip_atomic_load(&Q.q->pending, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) return;
  for (;;) {
    if (threadIdx.x == 0) {
      uint32_t it;
      bool first = false;
      for (;;) {
        it = q_pop(Q);
        if (it == kNoTile) break;
        const TileCoord c = tile_coord<TZ, TY, TX>(it, tl);
        if (q_claim(Q, it, c, tl, 0, parks, first)) break;
      }
      s_item = it;
      s_first = first;
      s_depth = it == kNoTile ? 0u
                              : __hip_atomic_load(&Q.depth[it], __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    const uint32_t t = s_item, d = s_depth;
    if (t == kNoTile) break;
    // ends with block barriers: s_item may be rewritten after it
    const uint32_t dirs = repair_run<TZ, TY, TX>(box, tl, mask, sub, counters, t,
                                                 s_first ? Q.blockers : nullptr);
    const TileCoord c = tile_coord<TZ, TY, TX>(t, tl);
    if (threadIdx.x < 64) {
      q_finish(dirs, t, c, tl, Q, 0, d + 1);
      if (threadIdx.x == 0) {
        ++runs;
        deepest = d > deepest ? d : deepest;
      }
    }
  }
  if (threadIdx.x == 0 && runs + parks) {
    atomicAdd(&Q.q->runs, runs);
    atomicAdd(&Q.q->parks, parks);
    atomicMax(&Q.q->max_depth, deepest);
  }
}

// ------------------------------------------------------------------ batches
// Persistent kernels: a fixed grid drains the batch-wide items of one phase.

// mark the neighbour tiles in `dirs` (27-bit set, see out_dirs) of a tile of
// a batch field for sweep `next` and append the newly marked ones (as
// batch-wide tile items) to that sweep's work list; each tile is listed at
// most once per sweep
__device__ void mark_list(uint32_t dirs, const TileCoord& c, const Tiling& tl, uint32_t* stamp,
                          uint32_t t0, uint32_t* lens, uint32_t* list, uint32_t next) {
  if (threadIdx.x >= 64) return;
  bool newly = false;
  uint32_t item = 0;
  if (threadIdx.x < 27 && ((dirs >> threadIdx.x) & 1u)) {
    int dz = (int)threadIdx.x / 9 - 1, dy = ((int)threadIdx.x / 3) % 3 - 1,
        dx = (int)threadIdx.x % 3 - 1;
    int nz = c.tz + dz, ny = c.ty + dy, nx = c.tx + dx;
    if ((dz | dy | dx) != 0 && nz >= 0 && nz < tl.ntz && ny >= 0 && ny < tl.nty &&
        nx >= 0 && nx < tl.ntx) {
      uint32_t u = ((uint32_t)nz * tl.nty + ny) * tl.ntx + nx;
      newly = atomicMax(&stamp[u], next) < next;
      item = t0 + u;
    }
  }
  const uint64_t m = __ballot(newly);
  if (!m) return;
  uint32_t pos = 0;
  if (threadIdx.x == 0) pos = atomicAdd(&lens[next % kRing], (uint32_t)__popcll(m));
  pos = __shfl(pos, 0, 64);
  if (newly) list[pos + lane_prefix(m)] = item;
}

__global__ __launch_bounds__(kThreads) void k_zero_p(const BatchDesc* bd) {
  const uint64_t n = bd->zero_words;
  uint32_t* base = bd->zero_base;
  for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * kThreads)
    base[i] = 0;
}

__global__ __launch_bounds__(kThreads) void k_zero_n(uint32_t* w, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * kThreads)
    w[i] = 0;
}

template <int K>
__global__ __launch_bounds__(kThreads) void k_minmax_p(const BatchDesc* bd, const Job* jobs) {
  constexpr int g0 = K == 4 ? 0 : 2;
  const uint32_t i1 = bd->item0[PH_MM][g0 + 2];
  const int j0 = (int)bd->job0[g0], j1 = (int)bd->job0[g0 + 2];
  for (uint32_t it = bd->item0[PH_MM][g0] + blockIdx.x; it < i1; it += gridDim.x) {
    const Job& J = jobs[find_job<&Job::mm0>(jobs, j0, j1, it)];
    __syncthreads();
    minmax_body<K>((const typename Traits<K>::Raw*)J.x, J.box.n, J.part, it - J.mm0,
                   (uint32_t)J.mm_blocks);
  }
}

template <int K>
__global__ __launch_bounds__(kThreads) void k_params_p(const BatchDesc* bd, const Job* jobs) {
  constexpr int g0 = K == 4 ? 0 : 2;
  const int j1 = (int)bd->job0[g0 + 2];
  for (int j = (int)bd->job0[g0] + (int)blockIdx.x; j < j1; j += (int)gridDim.x) {
    const Job& J = jobs[j];
    __syncthreads();
    params_body<K>(J.mode, J.eb, J.part, J.mm_blocks, J.prm, J.stream, J.cap, J.ndim,
                   J.dims[0], J.dims[1], J.ndim == 3 ? J.dims[2] : 1);
  }
}

template <int K, int TZ, int TY, int TX>
__global__ __launch_bounds__(kThreads) void k_tile0_p(const BatchDesc* bd, const Job* jobs,
                                                      int g) {
  BatchCounters* bc = bd->bc;
  uint32_t* list1 = bd->lists + bd->tiles;  // sweep 1: odd list
  const uint32_t i1 = bd->item0[PH_T][g + 1];
  const int j0 = (int)bd->job0[g], j1 = (int)bd->job0[g + 1];
  for (uint32_t it = bd->item0[PH_T][g] + blockIdx.x; it < i1; it += gridDim.x) {
    const Job& J = jobs[find_job<&Job::t0>(jobs, j0, j1, it)];
    __syncthreads();
    TileCoord c;
    const uint32_t dirs = tile0_body<K, TZ, TY, TX>(
        (const typename Traits<K>::Raw*)J.x, J.box, J.tl, J.prm,
        (typename Traits<K>::Bin*)J.bins, J.mask, J.sub, &bc->err, bc->relax_iters,
        it - J.t0, c);
    mark_list(dirs, c, J.tl, J.stamp, J.t0, bc->lens, list1, 1);
  }
}

// One run of batch tile `t` of job J: the batch's 2D shape S2 or 3D shape S3.
template <int S2, int S3, bool LOOP = false>
__device__ __forceinline__ uint32_t batch_repair_run(const Job& J, uint32_t* err,
                                                     unsigned long long* itot, uint32_t sweep,
                                                     uint32_t t, TileCoord& c) {
  using L2 = RunLds<1, kTile2[S2][1], kTile2[S2][2]>;
  using L3 = RunLds<kTile3[S3][0], kTile3[S3][1], kTile3[S3][2]>;
  __shared__ __attribute__((aligned(16)))
  uint8_t lds[sizeof(L2) > sizeof(L3) ? sizeof(L2) : sizeof(L3)];
  if (J.tl.tz == 1)
    return repair_body<1, kTile2[S2][1], kTile2[S2][2], false, LOOP>(*(L2*)lds, J.box, J.tl, J.mask, J.sub,
                                                        J.stamp, err, itot, sweep, t, c);
  return repair_body<kTile3[S3][0], kTile3[S3][1], kTile3[S3][2], false, LOOP>(
      *(L3*)lds, J.box, J.tl, J.mask, J.sub, J.stamp, err, itot, sweep, t, c);
}

// One sweep over the tiles listed for it, of fields of both tile shapes.
template <int S2, int S3>
__global__ __launch_bounds__(kThreads) void k_repair_p(const BatchDesc* bd, const Job* jobs,
                                                       uint32_t sweep) {
  __shared__ uint32_t s_it;
  BatchCounters* bc = bd->bc;
  const uint32_t* list_in = bd->lists + (sweep & 1) * bd->tiles;
  uint32_t* list_out = bd->lists + ((sweep + 1) & 1) * bd->tiles;
  const uint32_t n = bc->lens[sweep % kRing];
  const int nj = (int)bd->job0[kGroups];
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) s_it = atomicAdd(&bc->cursors[sweep % kRing], 1u);
    __syncthreads();
    const uint32_t it = s_it;
    if (it >= n) break;
    const uint32_t item = list_in[it];
    const Job& J = jobs[find_job<&Job::t0>(jobs, 0, nj, item)];
    TileCoord c;
    const uint32_t dirs = batch_repair_run<S2, S3>(J, &bc->err, bc->relax_iters, sweep,
                                                   item - J.t0, c);
    if (dirs) mark_list(dirs, c, J.tl, J.stamp, J.t0, bc->lens, list_out, sweep + 1);
  }
}

// Direct grids: one workgroup per item (the grid is the phase's item count
// of the batch), so each kernel keeps the register budget of its body.
template <int K>
__global__ __launch_bounds__(kThreads) void k_minmax_d(const BatchDesc* bd, const Job* jobs) {
  constexpr int g0 = K == 4 ? 0 : 2;
  const uint32_t it = bd->item0[PH_MM][g0] + blockIdx.x;
  const Job& J = jobs[find_job<&Job::mm0>(jobs, (int)bd->job0[g0], (int)bd->job0[g0 + 2], it)];
  minmax_body<K>((const typename Traits<K>::Raw*)J.x, J.box.n, J.part, it - J.mm0,
                 (uint32_t)J.mm_blocks);
}

template <int K>
__global__ __launch_bounds__(kThreads) void k_params_d(const BatchDesc* bd, const Job* jobs) {
  constexpr int g0 = K == 4 ? 0 : 2;
  const Job& J = jobs[bd->job0[g0] + blockIdx.x];
  params_body<K>(J.mode, J.eb, J.part, J.mm_blocks, J.prm, J.stream, J.cap, J.ndim,
                 J.dims[0], J.dims[1], J.ndim == 3 ? J.dims[2] : 1);
}

template <int K, int TZ, int TY, int TX>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(kTile0Waves<K, TZ, TY, TX>, 8))) void k_tile0_d(const BatchDesc* bd, const Job* jobs,
                                                      int g) {
  const uint32_t it = bd->item0[PH_T][g] + xcd_tile(blockIdx.x, gridDim.x);
  const Job& J = jobs[find_job<&Job::t0>(jobs, (int)bd->job0[g], (int)bd->job0[g + 1], it)];
  TileCoord c;
  const uint32_t dirs = tile0_body<K, TZ, TY, TX>(
      (const typename Traits<K>::Raw*)J.x, J.box, J.tl, J.prm, (typename Traits<K>::Bin*)J.bins,
      J.mask, J.sub, &bd->bc->err, bd->bc->relax_iters, it - J.t0, c);
  mark_list(dirs, c, J.tl, J.stamp, J.t0, bd->bc->lens, bd->lists + bd->tiles, 1);
}

// One sweep: workgroup b takes the entries b, b + gridDim.x, ... of the sweep's
// work list, with as many workgroups as stay resident (kRepairWaves per CU).
// 48 fields, 25,550 tiles, 32 captured sweeps of which 13 find an empty list:
// with a workgroup per tile such a sweep took 6.8 us to start and end them, and
// the call 1,575 us; so 1,345 us (1,439 with a quarter more workgroups
// than resident, 1,529 with half as many).
template <int S2, int S3>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(kRepairWaves, 8))) void k_repair_d(
    const BatchDesc* bd, const Job* jobs, uint32_t sweep) {
  BatchCounters* bc = bd->bc;
  const uint32_t n = bc->lens[sweep % kRing];
  uint32_t* list_out = bd->lists + ((sweep + 1) & 1) * bd->tiles;
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const uint32_t item = bd->lists[(sweep & 1) * bd->tiles + i];
    const Job& J = jobs[find_job<&Job::t0>(jobs, 0, (int)bd->job0[kGroups], item)];
    TileCoord c;
    const uint32_t dirs = batch_repair_run<S2, S3, true>(J, &bc->err, bc->relax_iters, sweep,
                                                         item - J.t0, c);
    if (dirs) mark_list(dirs, c, J.tl, J.stamp, J.t0, bc->lens, list_out, sweep + 1);
    if (i + gridDim.x < n) __syncthreads();  // the next tile's LDS
  }
}

}  // namespace

// ------------------------------------------------------------------ launchers
hipError_t launch_minmax(int dtype, const void* x, uint32_t n, double* part,
                         int nblocks, void* zero, size_t zero_bytes, hipStream_t s, Ev ev) {
  const uint32_t nz = (uint32_t)(zero_bytes / 16);
  if (dtype == 0)
    launch_ev(k_minmax<4>, dim3(nblocks), dim3(kThreads), s, ev,
                          (const uint32_t*)x, n, (int64_t*)part, (uint4*)zero, nz);
  else
    launch_ev(k_minmax<8>, dim3(nblocks), dim3(kThreads), s, ev,
                          (const uint64_t*)x, n, (int64_t*)part, (uint4*)zero, nz);
  return hipGetLastError();
}

hipError_t launch_params(int dtype, int mode, double eb, const double* part,
                         int nblocks, Params* prm, uint8_t* stream, size_t cap,
                         int ndim, const int64_t* dims, hipStream_t s, Ev ev) {
  int64_t d2 = ndim == 3 ? dims[2] : 1;
  if (dtype == 0)
    launch_ev(k_params<4>, dim3(1), dim3(kThreads), s, ev, mode, eb,
                          (const int64_t*)part, nblocks, prm, stream, (uint64_t)cap, ndim,
                          dims[0], dims[1], d2);
  else
    launch_ev(k_params<8>, dim3(1), dim3(kThreads), s, ev, mode, eb,
                          (const int64_t*)part, nblocks, prm, stream, (uint64_t)cap, ndim,
                          dims[0], dims[1], d2);
  return hipGetLastError();
}

hipError_t launch_tile0(int dtype, const void* x, Box box, Tiling t, Params* prm, void* bins,
                        uint16_t* mask, uint32_t* sub, uint32_t* stamp,
                        uint32_t* counters, uint32_t* lists, const QueueRef& Q, hipStream_t s,
                        Ev ev, bool coloured) {
  const int nl = coloured ? 2 : 1;
  const dim3 b(kThreads);
  const dim3 g(coloured ? (uint32_t)t.ntz * (uint32_t)t.nty * (uint32_t)((t.ntx + 1) / 2)
                        : t.ntiles);
  for (int l = 0; l < nl; ++l) {
    const Ev e{l == 0 ? ev.a : nullptr, l == nl - 1 ? ev.b : nullptr};
    const uint32_t col = coloured ? (uint32_t)l : 2u;
    LOPC_WITH_TILE(t, {
      if (dtype == 0)
        launch_ev(k_tile0<4, TZ, TY, TX>, g, b, s, e, (const uint32_t*)x, box, t, prm,
                  (int32_t*)bins, mask, sub, stamp, counters, lists, Q, col);
      else
        launch_ev(k_tile0<8, TZ, TY, TX>, g, b, s, e, (const uint64_t*)x, box, t, prm,
                  (int64_t*)bins, mask, sub, stamp, counters, lists, Q, col);
    });
  }
  return hipGetLastError();
}

namespace {
// the caller's result words of an enqueued compression: the stream size
// (also when the buffer was short) and the status code of the ST_* bits
// (precedence as in the synchronous calls)
__global__ void k_report(const Params* prm, const RepairQueue* q, uint64_t* d_size,
                         int32_t* d_status) {
  const uint32_t st = prm->status | (q && q->err ? ST_INTERNAL : 0u);
  const int32_t code = (st & ST_NONFINITE) ? -2 : (st & ST_BOUND) ? -3 : (st & ST_RANGE) ? -4
                       : (st & ST_FORMAT) ? -6 : (st & ST_INTERNAL) ? -9
                       : (st & ST_CAPACITY) ? -5 : 0;
  if (d_size) *d_size = (code == 0 || code == -5) ? prm->stream_size : 0ull;
  if (d_status) *d_status = code;
}
}  // namespace

hipError_t launch_report(const Params* prm, const RepairQueue* q, uint64_t* d_size,
                         int32_t* d_status, hipStream_t s) {
  k_report<<<1, 1, 0, s>>>(prm, q, d_size, d_status);
  return hipGetLastError();
}

hipError_t launch_sweep_list(Box box, Tiling t, const uint16_t* mask, uint32_t* sub,
                             uint32_t* stamp, uint32_t* counters, uint32_t* lists,
                             uint32_t sweep, int grid, hipStream_t s, Ev ev) {
  const dim3 g(grid), b(kThreads);
  LOPC_WITH_TILE(t, launch_ev(k_sweep_list<TZ, TY, TX>, g, b, s, ev, box, t, mask, sub, stamp,
                              counters, lists, sweep));
  return hipGetLastError();
}

int sweep_list_blocks_per_cu(int sid) {
  int b = 0;
  Tiling t{};
  t.sid = sid;
  hipError_t e = hipErrorInvalidValue;
  LOPC_WITH_TILE(t, e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
                        &b, k_sweep_list<TZ, TY, TX>, kThreads, 0));
  return e == hipSuccess && b > 0 ? b : 1;
}

hipError_t launch_seed_queue(const uint32_t* counters, const uint32_t* lists, uint32_t ntiles,
                             uint32_t sweep, const QueueRef& Q, hipStream_t s) {
  const uint32_t grid = std::max<uint32_t>(1, std::min<uint32_t>(256, (ntiles + kThreads - 1) / kThreads));
  k_seed_queue<<<grid, kThreads, 0, s>>>(counters, lists, ntiles, sweep, Q);
  return hipGetLastError();
}

hipError_t launch_repair_q(Box box, Tiling t, const uint16_t* mask, uint32_t* sub,
                           uint32_t* counters, const QueueRef& Q, int grid, hipStream_t s,
                           Ev ev) {
  const dim3 g(grid), b(kThreads);
  LOPC_WITH_TILE(t, launch_ev(k_repair_q<TZ, TY, TX>, g, b, s, ev, box, t, mask, sub, counters,
                              Q));
  return hipGetLastError();
}

// resident workgroups per CU of the single-field repair-queue kernel
int repair_q_blocks_per_cu(int sid) {
  int b = 0;
  Tiling t{};
  t.sid = sid;
  hipError_t e = hipErrorInvalidValue;
  LOPC_WITH_TILE(t, e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
                        &b, k_repair_q<TZ, TY, TX>, kThreads, 0));
  return e == hipSuccess && b > 0 ? b : 1;
}

hipError_t launch_repair(Box box, Tiling t, const uint16_t* mask, uint32_t* sub,
                         uint32_t* stamp, uint32_t* counters, uint32_t sweep, uint32_t few,
                         hipStream_t s, Ev ev) {
  // both colours, or every tile at once; the events bracket the sweep
  const bool col2 = t.coloured != 0;
  const uint32_t n =
      col2 ? (uint32_t)t.ntz * (uint32_t)t.nty * (uint32_t)((t.ntx + 1) / 2) : t.ntiles;
  const uint32_t nl = col2 ? 2 : 1;
  // tiles a workgroup looks at where few are marked, and the workgroups then;
  // below eight each starting one per tile costs less than two marked tiles in
  // a row (2D 1800 x 3600, 3,219 tiles, bound 1e-1: 1,860 against 2,000 us)
  const uint32_t per = few && n >= 8 * few ? std::min(64u, (n + few - 1) / few) : 1u;
  for (uint32_t l = 0; l < nl; ++l) {
    Ev e{l == 0 ? ev.a : nullptr, l == nl - 1 ? ev.b : nullptr};
    if (per > 1) {
      LOPC_WITH_TILE(t, launch_ev(k_repair_few<TZ, TY, TX>, dim3((n + per - 1) / per), dim3(kThreads),
                                  s, e, box, t, mask, sub, stamp, counters, sweep, col2 ? l : 2u, n));
      continue;
    }
    LOPC_WITH_TILE(t, launch_ev(k_repair<TZ, TY, TX>, dim3(n), dim3(kThreads), s, e, box, t,
                                mask, sub, stamp, counters, sweep, col2 ? l : 2u));
  }
  return hipGetLastError();
}

hipError_t launch_point_seed(const uint16_t* mask, uint32_t n, uint32_t* wl, uint32_t* ring,
                             int grid, hipStream_t s, Ev ev) {
  launch_ev(k_point_seed, dim3(grid), dim3(kThreads), s, ev, mask, n, wl, ring);
  return hipGetLastError();
}

hipError_t launch_point_iter(Box box, const uint16_t* mask, uint32_t* sub, const uint32_t* win,
                             uint32_t* wout, uint32_t* ring, uint32_t* pstamp, uint32_t it,
                             int grid, hipStream_t s, Ev ev) {
  launch_ev(k_point_iter, dim3(grid), dim3(kThreads), s, ev, box, mask, sub, win, wout, ring,
            pstamp, it);
  return hipGetLastError();
}

hipError_t launch_zero_p(const BatchDesc* bd, int grid, hipStream_t s) {
  k_zero_p<<<grid, kThreads, 0, s>>>(bd);
  return hipGetLastError();
}

hipError_t launch_zero_n(uint32_t* words, uint64_t nwords, hipStream_t s, Ev ev) {
  if (!nwords) return hipSuccess;
  const uint32_t grid = (uint32_t)std::min<uint64_t>(1024, (nwords + kThreads - 1) / kThreads);
  launch_ev(k_zero_n, dim3(grid), dim3(kThreads), s, ev, words, nwords);
  return hipGetLastError();
}

hipError_t launch_minmax_p(int dtype, const BatchDesc* bd, const Job* jobs, int grid,
                           hipStream_t s) {
  if (dtype == 0) k_minmax_p<4><<<grid, kThreads, 0, s>>>(bd, jobs);
  else k_minmax_p<8><<<grid, kThreads, 0, s>>>(bd, jobs);
  return hipGetLastError();
}

hipError_t launch_params_p(int dtype, const BatchDesc* bd, const Job* jobs, int grid,
                           hipStream_t s) {
  if (dtype == 0) k_params_p<4><<<grid, kThreads, 0, s>>>(bd, jobs);
  else k_params_p<8><<<grid, kThreads, 0, s>>>(bd, jobs);
  return hipGetLastError();
}

// the tile extents of a batch group (2D groups: shape t2, 3D groups: t3)
static Tiling group_tiling(int group, int t2, int t3) {
  Tiling t{};
  t.sid = (group & 1) ? kTiles2 + t3 : t2;
  return t;
}

hipError_t launch_tile0_p(int group, int t2, int t3, const BatchDesc* bd, const Job* jobs,
                          int grid, hipStream_t s) {
  const Tiling t = group_tiling(group, t2, t3);
  LOPC_WITH_TILE(t, {
    if (group < 2) k_tile0_p<4, TZ, TY, TX><<<grid, kThreads, 0, s>>>(bd, jobs, group);
    else k_tile0_p<8, TZ, TY, TX><<<grid, kThreads, 0, s>>>(bd, jobs, group);
  });
  return hipGetLastError();
}

// the repair kernels of the batch for shape pair (t2, t3)
#define LOPC_WITH_PAIR(t2, t3, ...)                                          \
  do {                                                                       \
    const int pair_ = (t2) * kTiles3 + (t3);                                 \
    switch (pair_) {                                                         \
      case 0: { constexpr int S2 = 0, S3 = 0; __VA_ARGS__; } break;          \
      case 1: { constexpr int S2 = 0, S3 = 1; __VA_ARGS__; } break;          \
      case 2: { constexpr int S2 = 0, S3 = 2; __VA_ARGS__; } break;          \
      case 3: { constexpr int S2 = 1, S3 = 0; __VA_ARGS__; } break;          \
      case 4: { constexpr int S2 = 1, S3 = 1; __VA_ARGS__; } break;          \
      default: { constexpr int S2 = 1, S3 = 2; __VA_ARGS__; } break;         \
    }                                                                        \
  } while (0)
static_assert(kTiles2 == 2 && kTiles3 == 3, "LOPC_WITH_PAIR lists every shape pair");

hipError_t launch_repair_p(int t2, int t3, const BatchDesc* bd, const Job* jobs, uint32_t sweep,
                           int grid, hipStream_t s) {
  LOPC_WITH_PAIR(t2, t3, (k_repair_p<S2, S3><<<grid, kThreads, 0, s>>>(bd, jobs, sweep)));
  return hipGetLastError();
}

hipError_t launch_minmax_d(int dtype, const BatchDesc* bd, const Job* jobs, uint32_t items,
                           hipStream_t s) {
  if (!items) return hipSuccess;
  if (dtype == 0) k_minmax_d<4><<<items, kThreads, 0, s>>>(bd, jobs);
  else k_minmax_d<8><<<items, kThreads, 0, s>>>(bd, jobs);
  return hipGetLastError();
}

hipError_t launch_params_d(int dtype, const BatchDesc* bd, const Job* jobs, uint32_t njobs,
                           hipStream_t s) {
  if (!njobs) return hipSuccess;
  if (dtype == 0) k_params_d<4><<<njobs, kThreads, 0, s>>>(bd, jobs);
  else k_params_d<8><<<njobs, kThreads, 0, s>>>(bd, jobs);
  return hipGetLastError();
}

hipError_t launch_tile0_d(int group, int t2, int t3, const BatchDesc* bd, const Job* jobs,
                          uint32_t items, hipStream_t s) {
  if (!items) return hipSuccess;
  const Tiling t = group_tiling(group, t2, t3);
  LOPC_WITH_TILE(t, {
    if (group < 2) k_tile0_d<4, TZ, TY, TX><<<items, kThreads, 0, s>>>(bd, jobs, group);
    else k_tile0_d<8, TZ, TY, TX><<<items, kThreads, 0, s>>>(bd, jobs, group);
  });
  return hipGetLastError();
}

hipError_t launch_repair_d(int t2, int t3, const BatchDesc* bd, const Job* jobs, uint32_t sweep,
                           uint32_t grid, hipStream_t s) {
  if (!grid) return hipSuccess;
  LOPC_WITH_PAIR(t2, t3, (k_repair_d<S2, S3><<<grid, kThreads, 0, s>>>(bd, jobs, sweep)));
  return hipGetLastError();
}

// resident blocks per CU of the persistent kernels of this file
int batch_blocks_per_cu(int kernel) {
  int b = 0;
  hipError_t e = hipErrorInvalidValue;
  switch (kernel) {
    case PK_ZERO: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_zero_p, kThreads, 0); break;
    case PK_MINMAX: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_minmax_p<8>, kThreads, 0); break;
    case PK_PARAMS: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_params_p<8>, kThreads, 0); break;
    case PK_TILE0: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_tile0_p<8, 8, 8, 32>, kThreads, 0); break;
    case PK_REPAIR: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_repair_p<0, 1>, kThreads, 0); break;
    default: break;
  }
  return e == hipSuccess && b > 0 ? b : 1;
}

}  // namespace lopc
