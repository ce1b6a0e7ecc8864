// lopc_codec.hip -- chunk encoder and decoder of liblopc.so (gfx950).
//
// Lossless stages of Sec. III-B / Sec. IV-C on 16 kB chunks: bins go through
// DIFFNB_K BIT_K RZE_1, subbins through BIT_K RZE_K RZE_1.  The BIT_K output
// of a chunk of m words is handled as 64-bit "units": unit u = j*G + g (G =
// m/64) holds bit j of the 64 words of group g.  A thread owns 8 (4)
// consecutive words and turns 8 x 8 bits at a time into plane bytes and back.
// Every RZE variant then works unit-parallel: a unit carries 8 (RZE_1), 2
// (RZE_4) or 1 (RZE_8) bitmap bits, so bitmaps, counts and payload offsets
// come from wave scans over units instead of per-byte work.
//
// Chunk offsets in the stream.  A single field: every workgroup parks its
// record in rows of the workspace that its own chunk has finished with, and a
// placement kernel copies the records into the stream (their offsets from a
// one-workgroup scan, or summed by each placing workgroup where the chunks are
// few), so no workgroup waits for another.  Batches: a decoupled look-back over a ticket-ordered chunk queue
// (a workgroup only waits for chunks that started before it).  A look-back
// word packs its state and size into 64 bits, so it carries no other data
// and relaxed device-scope atomics suffice: release or acquire at that scope
// would write back / invalidate the per-XCD L2 on every publication.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "lopc_device.h"

namespace lopc {
namespace {

constexpr int kCT = 512;        // threads of a codec workgroup
constexpr int kCW = kCT / 64;   // its waves
constexpr uint32_t kMaxUnits = kChunkBytes / 8;  // 2048
constexpr uint32_t kMaxRounds = kMaxUnits / 64;  // 32

// Scratch of the decoder's unit-parallel RZE stages.
struct Scratch {
  // (unused: 512^3 float64 takes 1,183 us to decompress without these bytes,
  // 1,174 with them, with any more than them 1,174)
  uint8_t gap[256] __attribute__((aligned(16)));
  // the bitmap levels from level 1 up (level 0 is expanded in registers)
  uint8_t lv1[256 + 16] __attribute__((aligned(16)));
  uint8_t lv2[32 + 16] __attribute__((aligned(16)));
  uint8_t lv3[16] __attribute__((aligned(16)));
  uint32_t rpre[kMaxRounds];  // items of each round
  uint32_t nkept[2];
  uint64_t planes;
};

__device__ __forceinline__ uint8_t* lvl(Scratch& sc, int l) {
  return l == 1 ? sc.lv1 : (l == 2 ? sc.lv2 : sc.lv3);
}
// Bitmap bytes of RZE level l for `items` items: ceil(items / 8^(l+1)) (each
// level is the bitmap of the one below; nested ceilings compose).  Computed
// rather than tabulated so that nothing lands in a private array.
__device__ __forceinline__ uint32_t lvl_size(uint32_t items, int l) {
  const uint32_t sh = 3u * (uint32_t)(l + 1);
  return (items + (1u << sh) - 1u) >> sh;
}
// the top level: the first whose bitmap has at most 8 bytes
__device__ __forceinline__ int rze_top(uint32_t items) {
  int top = 0;
  while (lvl_size(items, top) > 8) ++top;
  return top;
}

// bit b (0..7) of the result: byte b of v is nonzero
__device__ __forceinline__ uint32_t nonzero_bytes(uint64_t v) {
  const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  // 0x80 in the bytes that are not zero, then their places' sum
  const uint32_t l = (((lo & 0x7f7f7f7fu) + 0x7f7f7f7fu) | lo) & 0x80808080u;
  const uint32_t h = (((hi & 0x7f7f7f7fu) + 0x7f7f7f7fu) | hi) & 0x80808080u;
  return __builtin_amdgcn_udot4(h, 0x80402010u, __builtin_amdgcn_udot4(l, 0x08040201u, 0u, false),
                                false) >> 7;
}

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t c) { return wave_scan_u32(c); }

// Scratch of rze_encode.
struct EncScratch {
  // the lowest bitmap level kept in memory (RZE_1: level 1, RZE_K: level 0)
  // and the two above it
  uint8_t lva[512 + 16] __attribute__((aligned(16)));
  uint8_t lvb[64 + 16] __attribute__((aligned(16)));
  uint8_t lvc[16] __attribute__((aligned(16)));
  uint32_t rpre[kMaxRounds];  // per round: kept items, kept level-0 bytes << 16
  uint32_t scan[kCW];
  uint32_t pos0, out_len;     // offset of the kept level-0 bytes; the output's length
  uint64_t orv[kCW];
};

// One level of the bitmap recursion by one wave, for levels of at most 512
// bytes: lane l takes bytes 8l .. of cur[0, n), bit b of `bits`: its byte b
// differs from the byte before it (0 before the first).  The bits are the
// next level's byte l.
struct LevelStep {
  uint64_t v;
  uint32_t bits, excl, total;
  __device__ __forceinline__ void run(const uint8_t* cur, uint32_t n, uint8_t* nxt) {
    const uint32_t i0 = (uint32_t)lane() * 8;
    v = i0 < n ? ((const uint64_t*)cur)[lane()] : 0ull;
    const uint32_t prev = dpp_u32<0x138, 0xf, true>((uint32_t)(v >> 56));  // the lane below
    bits = nonzero_bytes(v ^ (v << 8 | prev));
    const uint32_t valid = i0 < n ? n - i0 : 0u;
    if (valid < 8) bits &= (1u << valid) - 1u;
    if (i0 < n) nxt[lane()] = (uint8_t)bits;
    const uint32_t c = (uint32_t)__popc(bits);
    excl = wave_incl_scan(c);
    total = (uint32_t)__builtin_amdgcn_readlane((int)excl, 63);
    excl -= c;
    __builtin_amdgcn_wave_barrier();
  }
  __device__ __forceinline__ void put(uint8_t* out) const {
    uint8_t* p = out + excl;
#pragma unroll
    for (int b = 0; b < 8; ++b)
      if ((bits >> b) & 1u) *p++ = (uint8_t)(v >> (8 * b));
  }
};

// RZE_W over the first `len` bytes of the unit array U, in place (the units
// are in registers before the first byte is written).  Units from `nua` on
// are known to be zero (bit planes above the highest set bit) and are not
// read.  Returns the output length; pt = 1 when the input is stored verbatim
// because the output would not be smaller.
//
// What bounds it is the chain of barriers, not the work between them: with a
// pass and a block-wide scan for every bitmap level a chunk's three RZE
// stages took about 45, and k_encode of a 1800x3600 binary32 field ran at 31%
// of the vector issue rate.  Three are left.  Each wave takes a run of the rounds of
// 64 units that may hold something, keeps its units in registers, and one
// ballot gives the round's 64 bits of level 1; a round's counts of kept items
// and kept level-0 bytes go out packed in one word.  Then every wave sums the
// rounds' counts for itself while the first one forms the levels above (at
// most 512 bytes, one lane per 8), and after the next barrier all write.
template <int W>
__device__ __forceinline__ uint32_t rze_encode(uint64_t* U, uint32_t len, uint32_t nua,
                                               EncScratch& sc, int& pt) {
  uint8_t* out = (uint8_t*)U;
  constexpr uint32_t kRPW = kMaxRounds / kCW;       // rounds per wave at most
  constexpr uint32_t kLB = W == 1 ? 8 : 64 / W;     // bytes of lva per round
  const uint32_t NU = (len + 7) / 8;
  const uint32_t items = len / W;
  const uint32_t rounds = (NU + 63) / 64;
  const uint32_t na = min(nua, NU);
  const uint32_t ra = (na + 63) / 64;  // rounds that may hold nonzero units
  // the first round without any may still differ from the byte before it
  const uint32_t rz = W == 1 ? min(rounds, ra + 1) : ra;
  const uint32_t rpw = (rz + kCW - 1) / kCW;
  const int top = rze_top(items);
  const uint32_t r0 = (uint32_t)__builtin_amdgcn_readfirstlane(wave()) * rpw;
  if (threadIdx.x < kMaxRounds * kLB / 4 && threadIdx.x >= rz * kLB / 4)
    ((uint32_t*)sc.lva)[threadIdx.x] = 0;  // the zero rounds
  uint64_t v[kRPW], dm[kRPW];
  uint32_t mi[kRPW], ex[kRPW];
  uint32_t prev = 0;  // the level-0 byte before the round
  if (W == 1 && r0 > 0 && r0 * 64 - 1 < na) prev = nonzero_bytes(U[r0 * 64 - 1]);
#pragma unroll
  for (uint32_t k = 0; k < kRPW; ++k) {
    const uint32_t r = r0 + k;
    v[k] = dm[k] = 0;
    mi[k] = ex[k] = 0;
    if (k >= rpw || r >= rz) continue;
    const uint32_t u = r * 64 + lane();
    v[k] = u < na ? U[u] : 0ull;
    uint32_t c, kept0 = 0;
    if (W == 1) {
      if ((len & 7u) && u == NU - 1) v[k] &= (1ull << (8 * (len & 7u))) - 1ull;
      mi[k] = nonzero_bytes(v[k]);
      c = __popc(mi[k]);
      if (top > 0) {
        const uint32_t p = (uint32_t)__builtin_amdgcn_update_dpp((int)prev, (int)mi[k], 0x138, 0xf,
                                                                 0xf, false);
        prev = (uint32_t)__builtin_amdgcn_readlane((int)mi[k], 63);
        dm[k] = __ballot(u < NU && mi[k] != p);
        kept0 = (uint32_t)__popcll(dm[k]);
        if (lane() == 0) ((uint64_t*)sc.lva)[r] = dm[k];
      } else if (u < NU) {
        sc.lva[u] = (uint8_t)mi[k];
      }
    } else if (W == 4) {
      mi[k] = ((uint32_t)v[k] != 0u) | ((uint32_t)((v[k] >> 32) != 0ull) << 1);
      c = __popc(mi[k]);
      // lanes 4q+1..4q+3 lie in the row of lane 4q: DPP row shifts left
      const uint32_t b = mi[k] | (dpp_u32<0x101, 0xf, true>(mi[k]) << 2) |
                         (dpp_u32<0x102, 0xf, true>(mi[k]) << 4) |
                         (dpp_u32<0x103, 0xf, true>(mi[k]) << 6);
      if ((lane() & 3) == 0) sc.lva[u / 4] = (uint8_t)b;
    } else {
      mi[k] = c = v[k] != 0ull;
      const uint64_t m = __ballot(mi[k]);
      if (lane() == 0) ((uint64_t*)sc.lva)[r] = m;
    }
    ex[k] = wave_incl_scan(c);
    if (lane() == 63) sc.rpre[r] = ex[k] | kept0 << 16;
    ex[k] -= c;
  }
  __syncthreads();
  const uint32_t cr = (uint32_t)lane() < rz ? sc.rpre[lane()] : 0u;
  const uint32_t ci = wave_incl_scan(cr);  // both counts fit 16 bits
  const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)ci, 63);
  const uint32_t before = ci - cr;
  const uint32_t kept0 = all >> 16;
  constexpr int kBase = W == 1 ? 1 : 0;  // the level in lva
  const int steps = top - kBase;         // at most 2
  LevelStep s0 = {}, s1 = {};
  const uint32_t sz_top = lvl_size(items, top);
  if (r0 == 0 && threadIdx.x < 64) {
    if (steps > 0) s0.run(sc.lva, lvl_size(items, kBase), sc.lvb);
    if (steps > 1) s1.run(sc.lvb, lvl_size(items, kBase + 1), sc.lvc);
    if (lane() == 0) {
      sc.pos0 = sz_top + s1.total + s0.total;
      sc.out_len = sc.pos0 + kept0 + (all & 0xffffu) * W;
    }
  }
  __syncthreads();
  const uint32_t out_len = (uint32_t)__builtin_amdgcn_readfirstlane((int)sc.out_len);
  if (out_len >= len) {
    for (uint32_t i = na + threadIdx.x; i < NU; i += kCT) U[i] = 0ull;
    pt = 1;
    __syncthreads();
    return len;
  }
  pt = 0;
  const uint32_t pos0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)sc.pos0);
  if (threadIdx.x < 64) {
    const uint8_t* tb = steps > 1 ? sc.lvc : (steps > 0 ? sc.lvb : sc.lva);
    if ((uint32_t)lane() < sz_top) out[lane()] = tb[lane()];
    if (steps > 1) s1.put(out + sz_top);
    if (steps > 0) s0.put(out + sz_top + s1.total);
  }
#pragma unroll
  for (uint32_t k = 0; k < kRPW; ++k) {
    const uint32_t r = r0 + k;
    if (k >= rpw || r >= rz) break;
    const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)before, (int)r);
    uint32_t d = pos0 + kept0 + W * ((b & 0xffffu) + ex[k]);
    if (W == 1) {
      const uint32_t lt = __builtin_amdgcn_mbcnt_hi((uint32_t)(dm[k] >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)dm[k], 0u));
      if ((dm[k] >> lane()) & 1ull) out[pos0 + (b >> 16) + lt] = (uint8_t)mi[k];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if ((mi[k] >> i) & 1u) out[d++] = (uint8_t)(v[k] >> (8 * i));
      }
    } else if (W == 4) {
      const uint32_t lo = (uint32_t)v[k], hi = (uint32_t)(v[k] >> 32);
      if (lo) {
        put_bytes(out + d, lo, 4);
        d += 4;
      }
      if (hi) put_bytes(out + d, hi, 4);
    } else {
      if (v[k]) put_bytes(out + d, v[k], 8);
    }
  }
  __syncthreads();
  return out_len;
}

// Item bits of unit u (of NU, `items` items in all) taken from its level-0
// bitmap byte b0.
template <int W>
__device__ __forceinline__ uint32_t unit_bits(uint32_t b0, uint32_t u, uint32_t items) {
  if (W == 1) {
    const uint32_t valid = items - u * 8;
    return valid < 8 ? b0 & ((1u << valid) - 1) : b0;
  } else if (W == 4) {
    return (b0 >> (2 * (u % 4))) & 3u;
  } else {
    return (b0 >> (u % 8)) & 1u;
  }
}

// One level of the bitmap recursion undone by one wave (no block barrier),
// for levels of at most 512 bytes (level 1 and above of a 16 kB input):
// child byte i = the last kept byte at or before i (0 if none), the kept
// bytes read from in[pos...); lane l handles parent byte l.  Returns false
// (wave-uniform) if the kept bytes run past in_len.  The 8 child bytes of a
// parent byte m (e kept bytes before it) come from one window of kept
// bytes, read as aligned words and joined by byte-align moves: it starts
// one byte before the first kept byte of m when m's bit 0 is clear (that
// byte fills the leading children), at it otherwise; the selector of child
// b is its inclusive count of set bits minus bit 0 of m, or 0x0c (zero)
// while no kept byte has been seen at all (e = 0).
__device__ bool level_decode_w(const uint8_t* par, uint32_t n, const uint8_t* in,
                               uint32_t& pos, uint32_t in_len, uint8_t* child) {
  const uint32_t np = (n + 7) / 8;  // <= 64
  const uint32_t idx = (uint32_t)lane();
  const uint32_t valid = n - idx * 8;
  uint32_t m = 0;
  if (idx < np) {
    m = par[idx];
    if (valid < 8) m &= (1u << valid) - 1;
  }
  const uint32_t cq = (uint32_t)__popc(m);
  const uint32_t incl = wave_incl_scan(cq);
  const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
  if (pos + tot > in_len) return false;
  const uint32_t e = incl - cq;
  if (idx < np) {
    const uint32_t b0 = m & 1u;
    // window: from kept byte e - 1 + b0 (in[pos - 1] when e = 0 and b0 = 0,
    // a byte of the levels above, selected by no child), cq + 1 - b0 bytes
    const uint8_t* p = in + pos + e + b0 - 1;
    const uint32_t mis = (uint32_t)(uintptr_t)p & 3u;
    const uint32_t* wq = (const uint32_t*)(p - mis);
    const uint32_t nd = (mis + cq + 1 - b0 + 3) / 4;  // 1..3 words
    const uint32_t w0 = wq[0];
    const uint32_t w1 = nd > 1 ? wq[1] : 0u;
    const uint32_t w2 = nd > 2 ? wq[2] : 0u;
    const uint32_t x0 = __builtin_amdgcn_alignbyte(w1, w0, mis);
    const uint32_t x1 = __builtin_amdgcn_alignbyte(w2, w1, mis);
    // inclusive counts of set bits per child byte (as in unit_payload)
    const uint32_t slo = ((m & 0xfu) * 0x00204081u) & 0x01010101u;
    const uint32_t shi = (((m >> 4) & 0xfu) * 0x00204081u) & 0x01010101u;
    const uint32_t ilo = slo * 0x01010101u;
    const uint32_t ihi = shi * 0x01010101u + (uint32_t)__popc(m & 0xfu) * 0x01010101u;
    uint32_t sel_lo = ilo - b0 * 0x01010101u, sel_hi = ihi - b0 * 0x01010101u;
    if (e == 0) {  // children before the first kept byte of the level are 0
      sel_lo |= ((~(ilo + 0x7f7f7f7fu) & 0x80808080u) >> 7) * 0x0cu;
      sel_hi |= ((~(ihi + 0x7f7f7f7fu) & 0x80808080u) >> 7) * 0x0cu;
    }
    uint64_t v = (uint64_t)__builtin_amdgcn_perm(x1, x0, sel_lo) |
                 (uint64_t)__builtin_amdgcn_perm(x1, x0, sel_hi) << 32;
    if (valid < 8) v &= (1ull << (8 * valid)) - 1ull;  // bytes past n are zero
    ((uint32_t*)child)[2 * idx] = (uint32_t)v;
    ((uint32_t*)child)[2 * idx + 1] = (uint32_t)(v >> 32);
  }
  pos += tot;
  __builtin_amdgcn_wave_barrier();
  return true;
}

// The payload of one unit: its c kept items at p (c * W bytes, any
// alignment) placed at the items of mask m, the others zero.  Reads the
// aligned words covering those bytes only (never past p + c * W rounded up
// to a word), joins them into the 8 bytes from p with byte-align moves, then
// for W = 1 spreads the bytes with one byte permute per half: the selector
// of output byte b is the number of mask bits below b when bit b is set,
// else 0x0c (the permute's zero byte).
template <int W>
__device__ __forceinline__ uint64_t unit_payload(const uint8_t* p, uint32_t m, uint32_t c) {
  if (!m) return 0;
  const uint32_t mis = (uint32_t)(uintptr_t)p & 3u;
  const uint32_t* q = (const uint32_t*)(p - mis);
  const uint32_t nd = (mis + c * W + 3) / 4;  // 1..3 words
  const uint32_t w0 = q[0];
  const uint32_t w1 = nd > 1 ? q[1] : 0u;
  const uint32_t w2 = nd > 2 ? q[2] : 0u;
  const uint32_t x0 = __builtin_amdgcn_alignbyte(w1, w0, mis);
  const uint32_t x1 = __builtin_amdgcn_alignbyte(w2, w1, mis);
  if (W == 8) return (uint64_t)x0 | (uint64_t)x1 << 32;
  if (W == 4) {
    const uint32_t lo = (m & 1) ? x0 : 0u;
    const uint32_t hi = (m & 2) ? ((m & 1) ? x1 : x0) : 0u;
    return (uint64_t)lo | (uint64_t)hi << 32;
  }
  // bit i of each nibble of m to bit 0 of byte i (the four shifted copies
  // do not overlap, so nothing carries)
  const uint32_t slo = ((m & 0xfu) * 0x00204081u) & 0x01010101u;
  const uint32_t shi = (((m >> 4) & 0xfu) * 0x00204081u) & 0x01010101u;
  // inclusive counts per byte, then exclusive: the selector of a set byte
  const uint32_t ilo = slo * 0x01010101u;
  const uint32_t ihi = shi * 0x01010101u + (uint32_t)__popc(m & 0xfu) * 0x01010101u;
  const uint32_t sel_lo = ((ilo - slo) & (slo * 0xffu)) | ((slo ^ 0x01010101u) * 0x0cu);
  const uint32_t sel_hi = ((ihi - shi) & (shi * 0xffu)) | ((shi ^ 0x01010101u) * 0x0cu);
  return (uint64_t)__builtin_amdgcn_perm(x1, x0, sel_lo) |
         (uint64_t)__builtin_amdgcn_perm(x1, x0, sel_hi) << 32;
}

// Upper levels of an RZE decode, on wave 0 alone: the top bitmap and every
// level down to level 1 (the bitmap of the level-0 bitmap) into sc.lv1, zero
// past its last byte.  Leaves sc.nkept[0] = ok and sc.nkept[1] = offset of
// the level-0 kept bytes (with a single level: of the payload).
__device__ void rze_decode_upper(const uint8_t* in, uint32_t in_len, uint32_t items,
                                 Scratch& sc) {
  const int top = rze_top(items);
  const uint32_t sz_top = lvl_size(items, top);
  bool ok = sz_top <= in_len;
  uint32_t pos = sz_top;
  if (ok && top == 1) {
    if (lane() < 16) sc.lv1[lane()] = (uint32_t)lane() < sz_top ? in[lane()] : (uint8_t)0;
  } else if (ok && top >= 2) {
    // the top level is read in place (its sz_top bytes are the parents)
    ok = level_decode_w(in, lvl_size(items, top - 1), in, pos, in_len, lvl(sc, top - 1));
    for (int l = top - 2; l >= 1 && ok; --l)
      ok = level_decode_w(lvl(sc, l + 1), lvl_size(items, l), in, pos, in_len, lvl(sc, l));
  }
  if (lane() == 0) {
    sc.nkept[0] = ok ? 1u : 0u;
    sc.nkept[1] = pos;
  }
}

// Inverse of rze_encode: in[0, in_len) -> the first `len` bytes of U (units
// rounded up; bytes past len are zero).  Returns false on malformed input;
// never reads outside [in, in + in_len).  If G > 0 the units are bit planes
// of G groups and sc.planes receives the mask of planes holding a nonzero
// unit.  Wave 0 decodes the levels above level 0 (small); then every wave
// expands the level-0 bitmap bytes of its own rounds of 64 units straight
// into registers (a byte's position among the kept bytes is a prefix count
// over level 1) and counts their items; after the per-round counts are
// exchanged, the same lanes fetch their units' payload.  Block barriers:
// after the upper levels, after the round counts, after the payload.  Units of
// planes left out of sc.planes hold anything.
template <int W>
__device__ __forceinline__ bool rze_decode(const uint8_t* in, uint32_t in_len, uint32_t len,
                           uint64_t* U, Scratch& sc, uint32_t G) {
  constexpr int kRPW = (int)(kMaxRounds / kCW);  // rounds per wave at most
  const uint32_t NU = (len + 7) / 8;
  const uint32_t items = len / W;
  const uint32_t rounds = (NU + 63) / 64;
  const int top = rze_top(items);
  const uint32_t n0 = lvl_size(items, 0);  // level-0 bitmap bytes
  if (wave() == 0) rze_decode_upper(in, in_len, items, sc);
  __syncthreads();
  if (!sc.nkept[0]) return false;
  const uint32_t pos1 = sc.nkept[1];
  // level 1 as 64-bit words (bit q: level-0 byte q differs from the one
  // before); bits from n0 on do not count
  const uint64_t* l1 = (const uint64_t*)sc.lv1;
  auto level1 = [&](uint32_t wi) -> uint64_t {
    const uint64_t wd = l1[wi];
    const uint32_t v = n0 - 64u * wi;
    return v < 64 ? wd & ((1ull << v) - 1ull) : wd;
  };
  uint32_t wexcl = 0, pos0 = pos1;
  uint64_t live = ~0ull;  // rounds that may hold items
  if (top >= 1) {
    const uint32_t nw = (n0 + 63) / 64;  // <= 32
    const uint64_t wd = (uint32_t)lane() < nw ? level1((uint32_t)lane()) : 0ull;
    const uint32_t c = (uint32_t)__popcll(wd);
    const uint32_t inc = wave_scan_u32(c);
    wexcl = inc - c;
    pos0 = pos1 + (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    if (pos0 > in_len) return false;
    // a round none of whose level-0 bytes differs from the one before it,
    // after a zero byte, holds no items (most rounds: the bit planes above the
    // highest set bit of the chunk); lane r looks at round r
    constexpr uint32_t kB = 64 / W;  // level-0 bytes of a round
    const uint32_t wi = (uint32_t)lane() / W, s0 = ((uint32_t)lane() % W) * kB;
    const uint64_t rw = W == 1 ? wd : (uint64_t)__shfl((unsigned long long)wd, (int)wi, 64);
    const uint32_t before =
        (W == 1 ? wexcl : (uint32_t)__shfl((int)wexcl, (int)wi, 64)) +
        (W == 1 ? 0u : (uint32_t)__popcll(rw & ((1ull << s0) - 1ull)));
    const bool same = (uint32_t)lane() < rounds &&
                      (W == 1 ? rw : (rw >> s0) & ((1ull << (kB & 63)) - 1ull)) == 0;
    const uint32_t byte = same && before ? in[pos1 + before - 1] : 0u;
    live = ~__ballot(same && byte == 0);
    if (wave() == 0 && (uint32_t)lane() < rounds && !((live >> lane()) & 1u)) sc.rpre[lane()] = 0;
  }
  if (threadIdx.x == 0) sc.planes = 0;
  uint32_t mi[kRPW], incl[kRPW];
  const uint32_t w0 = (uint32_t)__builtin_amdgcn_readfirstlane(wave());
#pragma unroll
  for (int k = 0; k < kRPW; ++k) {
    const uint32_t r = w0 + kCW * k;
    mi[k] = 0;
    incl[k] = 0;
    if (r >= rounds || !((live >> r) & 1u)) continue;
    const uint32_t u = r * 64 + lane();
    if (u < NU) {
      const uint32_t q = W == 1 ? u : (W == 4 ? u / 4 : u / 8);  // its level-0 byte
      uint32_t b0;
      if (top == 0) {
        b0 = in[q];  // the top level is level 0 (q < n0 = its size)
      } else {
        // the level-1 word holding the bits of this round's level-0 bytes
        // (r / W: one word per round of 8 / W items a unit) and the kept bytes
        // before it
        const uint64_t wd = level1(r / W);
        const uint32_t wb = (uint32_t)__builtin_amdgcn_readlane((int)wexcl, (int)(r / W));
        const uint32_t e = wb + (uint32_t)__popcll(wd & ((2ull << (q & 63)) - 1ull));
        b0 = e ? in[pos1 + e - 1] : 0u;
      }
      mi[k] = unit_bits<W>(b0, u, items);
    }
    incl[k] = wave_incl_scan((uint32_t)__popc(mi[k]));
    if (lane() == 63) sc.rpre[r] = incl[k];
  }
  __syncthreads();
  // payload offsets of the rounds; the payload must end the input exactly
  const uint32_t rc = (uint32_t)lane() < rounds ? sc.rpre[lane()] : 0u;
  const uint32_t rinc = wave_scan_u32(rc);
  const uint32_t npay = (uint32_t)__builtin_amdgcn_readlane((int)rinc, 63);
  if (pos0 + npay * W != in_len) return false;
  // a round without items needs no zeros where nobody reads a plane left out
  // of the mask: whole planes to a round
  const bool blank = !G || (64u % G) != 0;
  uint64_t pm = 0;
#pragma unroll
  for (int k = 0; k < kRPW; ++k) {
    const uint32_t r = w0 + kCW * k;
    if (r >= rounds) break;
    const uint32_t u = r * 64 + lane();
    if (!((live >> r) & 1u) || !__ballot(mi[k] != 0u)) {
      if (blank && u < NU) U[u] = 0;
      continue;
    }
    const uint32_t base = (uint32_t)__builtin_amdgcn_readlane((int)(rinc - rc), (int)r);
    const uint32_t m = mi[k];
    const uint32_t c = (uint32_t)__popc(m);
    uint64_t v = 0;
    if (u < NU) {
      v = unit_payload<W>(in + pos0 + W * (base + incl[k] - c), m, c);
      U[u] = v;
    }
    if (G == 64) {
      pm |= (uint64_t)(__ballot(v != 0) != 0) << r;
    } else if (G == 32) {
      const uint64_t b = __ballot(v != 0);
      pm |= (uint64_t)((uint32_t)b != 0) << (2 * r) | (uint64_t)((b >> 32) != 0) << (2 * r + 1);
    } else if (G && v) {
      pm |= 1ull << (u / G);
    }
  }
  if (G) {
    if (G != 64 && G != 32) pm = wave_reduce(pm, OpOr{});
    if (pm && lane() == 0) atomicOr((unsigned long long*)&sc.planes, (unsigned long long)pm);
  }
  __syncthreads();
  return true;
}

// bits of the four 4 x 4 blocks' rows (bytes) and columns exchanged, twice per
// byte: steps of an 8 x 8 bit transpose inside half a matrix
__device__ __forceinline__ uint32_t transpose4(uint32_t x) {
  uint32_t t = (x ^ (x >> 7)) & 0x00aa00aau;
  x ^= t ^ (t << 7);
  t = (x ^ (x >> 14)) & 0x0000ccccu;
  return x ^ t ^ (t << 14);
}

// planes 8C .. 8C + 7 of the thread's PER consecutive words (lo, hi: their
// halves) into the units at `planes`
template <int K, int C, int PER>
__device__ __forceinline__ void bytes_to_planes(const uint32_t (&lo)[PER],
                                                const uint32_t (&hi)[PER], uint32_t G,
                                                uint32_t np, uint8_t* planes) {
  if (np <= 8 * C) return;  // uniform
  const uint32_t(&w)[PER] = C < 4 ? lo : hi;
  // byte C of four words: rows of half a bit matrix
  constexpr uint32_t D = C & 3, kPair = D | (D + 4) << 8 | 0x0c0c0000u;
  auto four = [&](int i) {
    return __builtin_amdgcn_perm(w[i + 1], w[i], kPair) |
           __builtin_amdgcn_perm(w[i + 3], w[i + 2], kPair) << 16;
  };
  uint8_t* p = planes + (size_t)(8 * C) * G * 8;
  if constexpr (K == 4) {
    const uint32_t x = transpose4(four(0)), y = transpose4(four(4));
    // rows: planes, columns: the eight words
    const uint32_t l = (x & 0x0f0f0f0fu) | ((y << 4) & 0xf0f0f0f0u);
    const uint32_t h = ((x >> 4) & 0x0f0f0f0fu) | (y & 0xf0f0f0f0u);
    p += threadIdx.x;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      p[j * (G * 8)] = (uint8_t)(l >> (8 * j));
      p[(j + 4) * (G * 8)] = (uint8_t)(h >> (8 * j));
    }
  } else {
    // the four words are half of each plane byte: a pair of threads joins its
    // halves, the even one for planes 8C .. 8C + 3, the odd one for the others
    const uint32_t x = transpose4(four(0));
    const uint32_t y = dpp_u32<0xb1, 0xf, true>(x);  // the other thread of the pair
    const bool odd = threadIdx.x & 1u;
    const uint32_t a = odd ? y >> 4 : x, b = odd ? x : y << 4;
    const uint32_t l = (a & 0x0f0f0f0fu) | (b & 0xf0f0f0f0u);
    p += (odd ? 4 * (G * 8) : 0u) + (threadIdx.x >> 1);
#pragma unroll
    for (int j = 0; j < 4; ++j) p[j * (G * 8)] = (uint8_t)(l >> (8 * j));
  }
}
// BIT_K of a chunk: thread t holds its PER consecutive words t * PER ..; planes
// from np on are zero, and those from the next multiple of 8 on are not
// written.  The inverse of planes_to_words: about 45 (25) vector instructions
// for 8 x 8 (8 x 4) bits, where one ballot per plane and group took about 4
// per plane for a word.
template <int K, int PER>
__device__ __forceinline__ void words_to_planes(const typename Traits<K>::Word (&w)[PER],
                                                uint32_t G, uint32_t np, uint64_t* U) {
  uint32_t lo[PER], hi[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    lo[i] = (uint32_t)w[i];
    hi[i] = K == 8 ? (uint32_t)((uint64_t)w[i] >> 32) : 0u;
  }
  if (threadIdx.x >= (K == 4 ? G * 8 : G * 16)) return;
  uint8_t* p = (uint8_t*)U;
  bytes_to_planes<K, 0, PER>(lo, hi, G, np, p);
  bytes_to_planes<K, 1, PER>(lo, hi, G, np, p);
  bytes_to_planes<K, 2, PER>(lo, hi, G, np, p);
  bytes_to_planes<K, 3, PER>(lo, hi, G, np, p);
  if constexpr (K == 8) {
    bytes_to_planes<K, 4, PER>(lo, hi, G, np, p);
    bytes_to_planes<K, 5, PER>(lo, hi, G, np, p);
    bytes_to_planes<K, 6, PER>(lo, hi, G, np, p);
    bytes_to_planes<K, 7, PER>(lo, hi, G, np, p);
  }
}

// Planes holding a nonzero unit (bit j set: plane j not all zero).
template <int K>
__device__ uint64_t nonzero_planes(const uint64_t* U, uint32_t G, Scratch& sc) {
  uint64_t any = 0;
  if (threadIdx.x < 8 * K) {
    const uint64_t* p = U + threadIdx.x * G;
    for (uint32_t g = 0; g < G; ++g) any |= p[g];
  }
  if (threadIdx.x < 64) {
    uint64_t m = __ballot(any != 0ull);
    if (threadIdx.x == 0) sc.planes = m;
  }
  __syncthreads();
  return sc.planes;
}

constexpr uint64_t kLbAgg = 1ull << 62, kLbInc = 2ull << 62,
                   kLbVal = (1ull << 62) - 1;

// ------------------------------------------------------------------ encoder
// Word q of a chunk's record: 16-byte header, then the bins part (blen bytes at
// bp), the subbin part (slen at sp) and zero padding to a multiple of 4.  Reads
// at most one word past either part.
__device__ __forceinline__ uint32_t record_word(uint32_t q, const uint32_t* hdr,
                                                const uint32_t* bp, uint32_t blen,
                                                const uint32_t* sp, uint32_t slen) {
  if (q < kRecordHeaderBytes / 4) return hdr[q];
  const uint32_t r = 4 * q - kRecordHeaderBytes;
  if (r + 4 <= blen) return bp[r / 4];
  auto low = [](uint32_t v, uint32_t n) { return n < 4 ? v & ((1u << (8 * n)) - 1u) : v; };
  if (r < blen) {  // the bins part's last bytes, the subbin part's first
    const uint32_t k = blen - r;
    return low(bp[r / 4], k) | low(sp[0], slen) << (8 * k);
  }
  const uint32_t o = r - blen;
  if (o >= slen) return 0;
  return low(__builtin_amdgcn_alignbyte(sp[o / 4 + 1], sp[o / 4], o & 3), slen - o);
}

// Where the record of chunk c of a single field waits for its offset: the
// chunk's rows of the bins, subbins and order-flag arrays, in that order
// (free once the encoder has read the chunk; nothing reads them after it),
// and a separate place for the last chunk, whose rows may be short.  The
// rows hold W*sizeof(Bin) + 4W + 2W bytes: 40 KiB for binary32, 28 KiB for
// binary64.  A record is at most 16 + (bins part) + (subbin part) bytes with
// each part at most the bit-plane bytes of its stage input: 16 + 16 KiB +
// 16 KiB for binary32; for binary64 the subbins (below 2^32) fill at most 32
// of the 64 planes, so that part stays under 8 KiB plus its bitmaps, about
// 24.3 KiB in all.  The encoder still checks the room.
struct RecordSlots {
  uint8_t* seg[3];   // chunk 0's rows
  uint32_t len[3];   // bytes of one chunk's rows in each
  uint8_t* tail;     // the last chunk's place
  uint32_t tail_len;
};

__device__ __forceinline__ uint32_t* slot_word(const RecordSlots& S, uint32_t c, bool last,
                                               uint32_t q) {
  uint32_t r = 4 * q;
  if (last) return (uint32_t*)(S.tail + r);
  if (r < S.len[0]) return (uint32_t*)(S.seg[0] + (size_t)c * S.len[0] + r);
  r -= S.len[0];
  if (r < S.len[1]) return (uint32_t*)(S.seg[1] + (size_t)c * S.len[1] + r);
  r -= S.len[1];
  return (uint32_t*)(S.seg[2] + (size_t)c * S.len[2] + r);
}

__device__ __forceinline__ uint32_t record_size(uint32_t blen, uint32_t slen) {
  return (kRecordHeaderBytes + blen + slen + 3) & ~3u;
}

// Encodes chunk c of a field (Sec. III-B, IV-C).  kSlot: parks the record
// in its slot (single field; offsets and placement follow in their own
// kernels); else writes it into the stream after a decoupled look-back.
// Bound by vector issue (0.3 to 0.5 of its rate) and the barriers between the
// stages; a third of its time streams the bins and subbins.  With planes by
// byte transposes, three barriers per RZE stage and both parts in LDS:
// 256^3 binary32 109 -> 62 us, 1800 x 3600 57 -> 31 us, 512^3 binary64 1.25 ->
// 0.82 ms, 48-field batch (with the look-back) 333 -> 159 us.
template <int K, bool kSlot>
__device__ __forceinline__ void encode_body(uint32_t n, const typename Traits<K>::Bin* __restrict__ bins,
                            const uint32_t* __restrict__ sub, uint64_t* lookback,
                            uint32_t* parts, Params* prm, uint8_t* stream, uint64_t cap,
                            uint32_t nch, uint32_t c, const RecordSlots& S) {
  using Tr = Traits<K>;
  using Word = typename Tr::Word;
  constexpr uint32_t W = kChunkBytes / K;
  constexpr int PER = (int)(W / kCT);  // consecutive words of a thread
  // LDS: both parts from bit planes to the end, 34 KB, so that four workgroups
  // fill a CU's waves
  __shared__ uint64_t B[kMaxUnits + 1];  // bins (and a word read past them)
  __shared__ uint64_t U[kMaxUnits + 1];  // subbins
  __shared__ EncScratch sc;
  // the record header and the chunk's offset live in sc.orv, which is free
  // once the planes in use are known
  uint8_t* hdr = (uint8_t*)sc.orv;
  uint64_t& s_excl = sc.orv[2];

  const uint32_t p0 = c * W;
  const uint32_t nc = min(W, n - p0);
  const uint32_t m = (nc + 63) / 64 * 64;
  const uint32_t G = m / 64;
  const uint32_t L = m * K;
  const Word M = (Word)0xAAAAAAAAAAAAAAAAull;

  // The thread's bins and subbins, as 16-byte vectors (the rows of a chunk
  // start on one).  bins: DIFFNB_K (delta from the previous bin, 0 before the
  // chunk, then negabinary), zero words up to m.
  Word wv[PER], sv[PER];
  const uint32_t j0 = threadIdx.x * PER;
  const bool full = nc == W;
  {
    typename Tr::Bin bn[PER];
    uint32_t sb[PER];
    const typename Tr::Bin* bsrc = bins + p0 + j0;
    const uint32_t* ssrc = sub + p0 + j0;
    // the bin before the wave's first
    typename Tr::Bin before = 0;
    if (threadIdx.x >= 64 && lane() == 0 && j0 <= nc) before = bsrc[-1];
    if (full) {
#pragma unroll
      for (int q = 0; q < PER * K / 16; ++q) ((uint4*)bn)[q] = ((const uint4*)bsrc)[q];
#pragma unroll
      for (int q = 0; q < PER / 4; ++q) ((uint4*)sb)[q] = ((const uint4*)ssrc)[q];
    } else {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        bn[i] = j0 + i < nc ? bsrc[i] : 0;
        sb[i] = j0 + i < nc ? ssrc[i] : 0u;
      }
    }
    // from the lane below (wave_shr:1), its last bin; lane 0 keeps `before`
    typename Tr::Bin prev;
    const uint64_t lastb = (uint64_t)bn[PER - 1], bef = (uint64_t)before;
    uint64_t pv = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)bef, (int)(uint32_t)lastb,
                                                        0x138, 0xf, 0xf, false);
    if constexpr (K == 8)
      pv |= (uint64_t)(uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(bef >> 32),
                                                            (int)(uint32_t)(lastb >> 32), 0x138,
                                                            0xf, 0xf, false) << 32;
    prev = (typename Tr::Bin)pv;
    Word ob = 0, os = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const Word d = (Word)bn[i] - (Word)prev;
      prev = bn[i];
      wv[i] = full || j0 + i < nc ? (d + M) ^ M : (Word)0;
      sv[i] = (Word)sb[i];
      ob |= wv[i];
      os |= sv[i];
    }
    // the highest planes in use
    ob = wave_reduce(ob, OpOr{});
    const uint32_t os32 = wave_reduce((uint32_t)os, OpOr{});
    if (lane() == 0) {
      sc.orv[wave()] = (uint64_t)ob;
      sc.scan[wave()] = os32;
    }
  }
  __syncthreads();
  uint64_t orb = 0;
  uint32_t ors = 0;
#pragma unroll
  for (int w = 0; w < kCW; ++w) {
    orb |= sc.orv[w];
    ors |= sc.scan[w];
  }
  const uint32_t npb = (uint32_t)__builtin_amdgcn_readfirstlane(
      orb ? 64 - __builtin_clzll(orb) : 0);
  const uint32_t nps = (uint32_t)__builtin_amdgcn_readfirstlane(ors ? 32 - __builtin_clz(ors) : 0);
  words_to_planes<K, PER>(wv, G, npb, B);
  words_to_planes<K, PER>(sv, G, nps, U);
  __syncthreads();
  int pt_b = 0, pt_s1 = 0, pt_s2 = 0;
  const uint32_t blen = rze_encode<1>(B, L, npb * G, sc, pt_b);
  const uint32_t smid = rze_encode<K>(U, L, nps * G, sc, pt_s1);
  const uint32_t slen = rze_encode<1>(U, smid, (smid + 7) / 8, sc, pt_s2);

  const uint32_t size = record_size(blen, slen);
  if (threadIdx.x == 0) {
    hdr[0] = (uint8_t)pt_b;
    hdr[1] = (uint8_t)(pt_s1 | (pt_s2 << 1));
    hdr[2] = (uint8_t)nc;
    hdr[3] = (uint8_t)(nc >> 8);
    put_bytes(hdr + 4, blen, 4);
    put_bytes(hdr + 8, smid, 4);
    put_bytes(hdr + 12, slen, 4);
  }
  if constexpr (kSlot) {
    if (threadIdx.x == 0) {
      parts[2 * c] = blen;
      parts[2 * c + 1] = slen;
      if (kHeaderBytes + 4ull * c + 4 <= cap)
        *(uint32_t*)(stream + kHeaderBytes + 4ull * c) = size;
    }
    __syncthreads();  // hdr
    const bool last = c == nch - 1;
    if (size <= (last ? S.tail_len : S.len[0] + S.len[1] + S.len[2])) {
      for (uint32_t q = threadIdx.x; q < size / 4; q += kCT)
        *slot_word(S, c, last, q) = record_word(q, (const uint32_t*)hdr, (const uint32_t*)B, blen,
                                                (const uint32_t*)U, slen);
    } else if (threadIdx.x == 0) {
      set_status(prm, ST_INTERNAL);
    }
    return;
  }

  // decoupled look-back for this chunk's offset in the stream body: wave 0
  // reads 64 predecessors per round trip (lane l reads chunk c - 1 - l - 64r)
  // and adds the sizes up to the nearest inclusive prefix
  if (threadIdx.x < 64) {
    uint64_t excl = 0;
    if (threadIdx.x == 0)
      __hip_atomic_store(&lookback[c], (c == 0 ? kLbInc : kLbAgg) | size, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    if (c > 0) {
      int64_t j0 = (int64_t)c - 1;
      uint32_t spins = 0;
      for (;;) {
        const int64_t j = j0 - lane();
        uint64_t v = kLbInc;  // before the first chunk: an inclusive prefix of 0
        if (j >= 0)
          v = __hip_atomic_load(&lookback[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t st = v & ~kLbVal;
        const uint64_t inc = __ballot(st == kLbInc);
        const uint64_t open = __ballot(st == 0);
        // lanes up to and including the nearest inclusive one (all if none)
        const uint64_t need = inc ? ((inc & (0ull - inc)) << 1) - 1ull : ~0ull;
        if (open & need) {  // a needed predecessor has not published yet
          if (++spins > (1u << 24)) {  // never reached when every chunk runs
            if (threadIdx.x == 0) set_status(prm, ST_INTERNAL);
            break;
          }
          __builtin_amdgcn_s_sleep(1);
          continue;
        }
        uint64_t x = ((need >> lane()) & 1ull) ? (v & kLbVal) : 0ull;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) x += __shfl_xor(x, d, 64);
        excl += x;
        if (inc) break;
        j0 -= 64;
      }
      if (threadIdx.x == 0)
        __hip_atomic_store(&lookback[c], kLbInc | (excl + size), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    if (threadIdx.x == 0) {
      s_excl = excl;
      parts[2 * c] = blen;
      parts[2 * c + 1] = slen;
    }
  }
  __syncthreads();
  const uint64_t body = kHeaderBytes + 4ull * nch;
  const uint64_t dst = body + s_excl;
  if (threadIdx.x == 0) {
    if (kHeaderBytes + 4ull * c + 4 <= cap)
      *(uint32_t*)(stream + kHeaderBytes + 4ull * c) = size;
    if (c == nch - 1) prm->stream_size = dst + size;
  }
  if (dst + size <= cap) {
    for (uint32_t q = threadIdx.x; q < size / 4; q += kCT)
      ((uint32_t*)(stream + dst))[q] = record_word(q, (const uint32_t*)hdr, (const uint32_t*)B,
                                                   blen, (const uint32_t*)U, slen);
  } else if (threadIdx.x == 0) {
    set_status(prm, ST_CAPACITY);
  }
}

// Single field, one workgroup per chunk: encode and park the record.  This
// kernel and the two after it are skipped entirely when gate is given and
// *gate != 0 (the repair sweeps enqueued before them have not reached the
// fixed point; the host then sweeps on and encodes).
template <int K>
__global__ __launch_bounds__(kCT) void k_encode(
    uint32_t n, const typename Traits<K>::Bin* __restrict__ bins,
    const uint32_t* __restrict__ sub, uint32_t* parts, Params* prm, uint8_t* stream,
    uint64_t cap, uint32_t nch, RecordSlots S, const uint32_t* gate) {
  if (gate && *gate) return;
  encode_body<K, true>(n, bins, sub, nullptr, parts, prm, stream, cap, nch, blockIdx.x, S);
}

// Single field: exclusive offsets of the records in the stream body from
// their part sizes, 4096 chunks per pass (four per thread, read as two
// 16-byte vectors); the stream size.
constexpr int kOT = 1024;  // threads of the offset scan
__global__ __launch_bounds__(kOT) void k_record_offsets(const uint32_t* parts, uint32_t nch,
                                                        uint64_t* offs, Params* prm,
                                                        const uint32_t* gate) {
  if (gate && *gate) return;
  __shared__ uint64_t sh[kOT / 64 + 1];
  uint64_t carry = 0;
  for (uint32_t t0 = 0; t0 < nch; t0 += 4 * kOT) {
    const uint32_t i = t0 + 4 * threadIdx.x;
    uint32_t sz[4];
    if (i + 3 < nch) {
      const uint4 a = ((const uint4*)parts)[i / 2], b = ((const uint4*)parts)[i / 2 + 1];
      sz[0] = record_size(a.x, a.y);
      sz[1] = record_size(a.z, a.w);
      sz[2] = record_size(b.x, b.y);
      sz[3] = record_size(b.z, b.w);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        sz[k] = i + k < nch ? record_size(parts[2 * (i + k)], parts[2 * (i + k) + 1]) : 0u;
    }
    const uint64_t sum = (uint64_t)sz[0] + sz[1] + sz[2] + sz[3];
    uint64_t total;
    uint64_t off = carry + block_excl_scan<uint64_t, kOT / 64>(sum, sh, total);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i + k < nch) offs[i + k] = off;
      off += sz[k];
    }
    carry += total;
  }
  if (threadIdx.x == 0) prm->stream_size = kHeaderBytes + 4ull * nch + carry;
}

// Single field, one workgroup per chunk: copy the parked record to its
// offset (ST_CAPACITY when the stream buffer is too short for it).
__global__ __launch_bounds__(kThreads) void k_place(const uint32_t* parts, const uint64_t* offs,
                                                    uint32_t nch, RecordSlots S, Params* prm,
                                                    uint8_t* stream, uint64_t cap,
                                                    const uint32_t* gate) {
  if (gate && *gate) return;
  const uint32_t c = blockIdx.x;
  const uint32_t size = record_size(parts[2 * c], parts[2 * c + 1]);
  const uint64_t dst = kHeaderBytes + 4ull * nch + offs[c];
  const bool last = c == nch - 1;
  if (size > (last ? S.tail_len : S.len[0] + S.len[1] + S.len[2])) return;  // flagged already
  if (dst + size > cap) {
    if (threadIdx.x == 0) set_status(prm, ST_CAPACITY);
    return;
  }
  uint32_t* out = (uint32_t*)(stream + dst);
  const uint32_t nw = size / 4;
  for (uint32_t q0 = 0; q0 < nw; q0 += 4 * kThreads) {
    uint32_t v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t q = q0 + k * kThreads + threadIdx.x;
      v[k] = q < nw ? *slot_word(S, c, last, q) : 0u;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t q = q0 + k * kThreads + threadIdx.x;
      if (q < nw) out[q] = v[k];
    }
  }
}

// The same without the offsets, for at most kPlaceChunks chunks: a wave per
// record, and each workgroup sums the sizes of the records before its four
// (two chunks per 16-byte load).  Saves the one-workgroup scan; its reads grow
// with the square of the chunks, and beyond 16,384 they cost more than the scan.
// Encoder and placement, with / without the scan: 4,096 chunks 75.9 / 74.8 us,
// 8,192 140.0 / 137.1, 16,384 262.7 / 259.6, 32,768 523.0 / 528.4.
constexpr uint32_t kPlaceChunks = 16384;
__global__ __launch_bounds__(kThreads) void k_place_few(const uint32_t* parts, uint32_t nch,
                                                        RecordSlots S, Params* prm,
                                                        uint8_t* stream, uint64_t cap,
                                                        const uint32_t* gate) {
  if (gate && *gate) return;
  __shared__ uint32_t sh[kThreads / 64];
  constexpr uint32_t kWaves = kThreads / 64;
  const uint32_t c0 = blockIdx.x * kWaves, w = (uint32_t)__builtin_amdgcn_readfirstlane(wave());
  uint32_t sum = 0;  // at most kPlaceChunks records of at most 40 KiB: 32 bits
  static_assert((uint64_t)kPlaceChunks * (kRecordTailBytes + 8192) < (1ull << 32), "offsets in 32 bits");
  for (uint32_t i = threadIdx.x; i < c0 / 2; i += kThreads) {
    const uint4 a = ((const uint4*)parts)[i];
    sum += record_size(a.x, a.y) + record_size(a.z, a.w);
  }
  sum = wave_scan_u32(sum);
  if (lane() == 63) sh[w] = sum;
  __syncthreads();
  const uint32_t c = c0 + w;
  if (c >= nch) return;
  uint32_t off = 0;
  for (uint32_t k = 0; k < kWaves; ++k) {
    off += sh[k];
    if (k < w) off += record_size(parts[2 * (c0 + k)], parts[2 * (c0 + k) + 1]);
  }
  const uint32_t size = record_size(parts[2 * c], parts[2 * c + 1]);
  const uint64_t dst = kHeaderBytes + 4ull * nch + off;
  const bool last = c == nch - 1;
  if (last && lane() == 0) prm->stream_size = dst + size;
  if (size > (last ? S.tail_len : S.len[0] + S.len[1] + S.len[2])) return;  // flagged already
  if (dst + size > cap) {
    if (lane() == 0) set_status(prm, ST_CAPACITY);
    return;
  }
  uint32_t* out = (uint32_t*)(stream + dst);
  const uint32_t nw = size / 4;
  constexpr int kU = 8;
  for (uint32_t q0 = 0; q0 < nw; q0 += kU * 64) {
    uint32_t v[kU];
#pragma unroll
    for (int k = 0; k < kU; ++k) {
      const uint32_t q = q0 + k * 64 + lane();
      v[k] = q < nw ? *slot_word(S, c, last, q) : 0u;
    }
#pragma unroll
    for (int k = 0; k < kU; ++k) {
      const uint32_t q = q0 + k * 64 + lane();
      if (q < nw) out[q] = v[k];
    }
  }
}

// ------------------------------------------------------------------ decoder
// Exclusive offsets of the records from the size table; the sizes must add
// up to the stream body exactly.
__device__ __forceinline__ void offsets_body(const uint8_t* stream, uint32_t nch, uint64_t body_bytes,
                             uint64_t* offsets, Params* prm) {
  __shared__ uint64_t sh[kWaves + 1];
  const uint32_t per = (nch + kThreads - 1) / kThreads;
  const uint32_t b = threadIdx.x * per, e = min(nch, b + per);
  const uint32_t* tab = (const uint32_t*)(stream + kHeaderBytes);
  uint64_t sum = 0;
  for (uint32_t i = b; i < e; ++i) sum += tab[i];
  uint64_t total;
  uint64_t off = block_excl_scan<uint64_t>(sum, sh, total);
  for (uint32_t i = b; i < e; ++i) {
    offsets[i] = off;
    off += tab[i];
  }
  if (threadIdx.x == 0 && total != body_bytes) set_status(prm, ST_FORMAT);
}

// Single field, one 1024-thread block: the same scan, four sizes per thread
// per pass (one 16-byte read where the table allows; the table starts 4
// bytes past a 16-byte boundary of the stream only if the stream does), and
// the start of the decoder's status word (no separate clear).
constexpr int kOfT = 1024;
__global__ __launch_bounds__(kOfT) void k_offsets(
    const uint8_t* stream, uint32_t nch, uint64_t body_bytes,
    uint64_t* offsets, Params* prm) {
  __shared__ uint64_t sh[kOfT / 64 + 1];
  if (threadIdx.x == 0) prm->status = 0;
  const uint32_t* tab = (const uint32_t*)(stream + kHeaderBytes);
  const bool vec = ((uintptr_t)tab & 15u) == 0;
  uint64_t carry = 0;
  for (uint32_t t0 = 0; t0 < nch; t0 += 4 * kOfT) {
    const uint32_t i = t0 + 4 * threadIdx.x;
    uint32_t sz[4];
    if (vec && i + 3 < nch) {
      const uint4 a = *(const uint4*)(tab + i);
      sz[0] = a.x;
      sz[1] = a.y;
      sz[2] = a.z;
      sz[3] = a.w;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) sz[k] = i + k < nch ? tab[i + k] : 0u;
    }
    const uint64_t sum = (uint64_t)sz[0] + sz[1] + sz[2] + sz[3];
    uint64_t total;
    uint64_t off = carry + block_excl_scan<uint64_t, kOfT / 64>(sum, sh, total);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i + k < nch) offsets[i + k] = off;
      off += sz[k];
    }
    carry += total;
  }
  if (threadIdx.x == 0 && carry != body_bytes) set_status(prm, ST_FORMAT);
}

// Totals of the bins and subbin parts over all chunks (statistics only).
__global__ __launch_bounds__(kThreads) void k_sum_parts(const uint32_t* parts,
                                                        uint32_t nch, Params* prm) {
  __shared__ uint64_t sh[kWaves + 1];
  uint64_t b = 0, u = 0;
  for (uint32_t i = threadIdx.x; i < nch; i += kThreads) {
    b += parts[2 * i];
    u += parts[2 * i + 1];
  }
  uint64_t tb, tu;
  block_excl_scan<uint64_t>(b, sh, tb);
  block_excl_scan<uint64_t>(u, sh, tu);
  if (threadIdx.x == 0) {
    prm->bins_bytes = tb;
    prm->sub_bytes = tu;
  }
}

// Lower edge of bin b: the key of the lowest value whose bin is b or above (the
// bins are monotone in the value, so bin b holds the keys from its edge up to
// the edge of b + 1, none if they are equal); kNoKey if the search fails.
template <int K>
constexpr typename Traits<K>::Bin kNoKey =
    (typename Traits<K>::Bin)((uint64_t)1 << (8 * sizeof(typename Traits<K>::Bin) - 1));
// By steps: from next to the real edge (b - 1/2) / inv to the first value whose
// bin is b or above.
template <int K>
__device__ __noinline__ typename Traits<K>::Bin edge_walk(int64_t b, double inv, double c) {
  using Tr = Traits<K>;
  int64_t k;
  if (K == 4) {
    const uint32_t u = __float_as_uint((float)c);
    if (!finite32(u)) return kNoKey<K>;
    k = key32(u);
  } else {
    const uint64_t u = (uint64_t)__double_as_longlong(c);
    if (!finite64(u)) return kNoKey<K>;
    k = key64(u);
  }
  int steps = 0;
  while (k > -Tr::kMaxKey && Tr::q(Tr::to_double(Tr::unkey(k - 1)), inv) >= b) {
    --k;
    if (++steps > 8) return kNoKey<K>;
  }
  while (Tr::q(Tr::to_double(Tr::unkey(k)), inv) < b) {
    if (k >= Tr::kMaxKey || ++steps > 8) return kNoKey<K>;
    ++k;
  }
  return (typename Tr::Bin)k;
}
// Directly where rounding cannot blur it.  The real edge is at most 2^-51 |c|
// from c = RN((b - 1/2) winv).  float32: values are 2^-24 apart, so the value
// next to c on the far side of the edge is known unless c lies within 2^-50 of
// a value.  float64: a value x reaches the bin iff x inv > b - 1/2, the sign of
// one fma; the four values around c bracket the edge.  A tie or no bracket
// goes by steps.  About 15 (float32) and 40 (float64) vector instructions an
// edge; quantizing the candidates took 120 and 170, a quarter of the decoder's
// instructions on a 1800 x 3600 float32 field (316 of 1351 per wave).
template <int K>
__device__ __forceinline__ typename Traits<K>::Bin lower_edge(int64_t b, double inv,
                                                              double winv) {
  const double h = (double)b - 0.5;
  const double c = h * winv;
  if constexpr (K == 4) {
    const float f = (float)c;
    const uint32_t u = __float_as_uint(f);
    const double d = (double)f - c;
    if (finite32(u) && fabs(d) > fabs(c) * 8.8817841970012523e-16)  // 2^-50
      return (int32_t)key32(u) + (d < 0.0);
  } else {
    const uint64_t u = (uint64_t)__double_as_longlong(c);
    const uint64_t mag = u & 0x7fffffffffffffffull;
    if (mag >= 8 && mag < 0x7fe0000000000000ull && fabs(h) < 2251799813685248.0) {
      const int64_t step = (int64_t)u < 0 ? -1 : 1;
      uint32_t below = 0;
      bool tie = false;
#pragma unroll
      for (int i = -2; i < 2; ++i) {
        const double r = fma(__longlong_as_double((int64_t)u + i * step), inv, -h);
        below += r < 0.0;
        tie |= r == 0.0;
      }
      if (!tie && below - 1u < 3u) return key64(u) - 2 + (int64_t)below;
    }
  }
  return edge_walk<K>(b, inv, c);
}

// The value of subbin s above lower edge t of bin b, and whether it exists and
// lies in the bin (next: the edge of bin b + 1).
template <int K>
__device__ __forceinline__ bool point_ok(int64_t b, uint64_t s, typename Traits<K>::Bin t,
                                         typename Traits<K>::Bin next, double inv,
                                         typename Traits<K>::Raw& v) {
  using Tr = Traits<K>;
  v = 0;
  // the room above t can exceed the int64 range: unsigned difference
  if (b > Tr::kBinLimit || b < -Tr::kBinLimit || t == kNoKey<K> ||
      (int64_t)t > Tr::kMaxKey || s > (uint64_t)Tr::kMaxKey - (uint64_t)(int64_t)t)
    return false;
  v = Tr::unkey((int64_t)t + (int64_t)s);
  // inside bin b iff below the edge of bin b + 1
  if (next != kNoKey<K>) return s < (uint64_t)((int64_t)next - (int64_t)t);
  return Tr::q(Tr::to_double(v), inv) == b;
}

// copy n bytes from global src (4-byte aligned base) to LDS dst
__device__ __forceinline__ void stage(uint8_t* dst, const uint8_t* src, uint32_t n) {
  const uint32_t nw = (n + 3) / 4;
  const uint32_t* s = (const uint32_t*)src;
  uint32_t* d = (uint32_t*)dst;
  for (uint32_t i0 = 0; i0 < nw; i0 += 4 * kCT) {
    uint32_t v[4];  // four loads in flight per thread
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t i = i0 + k * kCT + threadIdx.x;
      v[k] = i < nw ? s[i] : 0u;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t i = i0 + k * kCT + threadIdx.x;
      if (i < nw) d[i] = v[k];
    }
  }
}

// Byte c of w from byte i of t (the other bytes of w stay).
template <int C, int I>
__device__ __forceinline__ void put_byte(uint32_t& w, uint32_t t) {
#define LOPC_PUT(c, i)                                                                     \
  if constexpr (C == c && I == i)                                                          \
    asm("v_mov_b32_sdwa %0, %1 dst_sel:BYTE_" #c " dst_unused:UNUSED_PRESERVE src0_sel:BYTE_" #i \
        : "+v"(w) : "v"(t))
#define LOPC_PUT4(c) LOPC_PUT(c, 0); LOPC_PUT(c, 1); LOPC_PUT(c, 2); LOPC_PUT(c, 3)
  LOPC_PUT4(0);
  LOPC_PUT4(1);
  LOPC_PUT4(2);
  LOPC_PUT4(3);
#undef LOPC_PUT4
#undef LOPC_PUT
}
// bit b (0..3) of m as byte b of all ones
__device__ __forceinline__ uint32_t byte_mask(uint32_t m) {
  const uint32_t y = ((m & 0xfu) * 0x00204081u) & 0x01010101u;
  return (y << 8) - y;
}
// byte C of the PER words w from planes 8C .. 8C + 7 (mask pm, the others
// zero) of G groups at `planes`
template <int K, int C, int PER>
__device__ __forceinline__ void plane_bytes(const uint8_t* planes, uint32_t G, uint64_t pm,
                                            uint32_t (&lo)[PER], uint32_t (&hi)[PER]) {
  const uint32_t bits = (uint32_t)(pm >> (8 * C)) & 0xffu;
  if (!bits) return;  // uniform
  const uint8_t* p = planes + (size_t)(8 * C) * G * 8 + (K == 4 ? threadIdx.x : threadIdx.x >> 1);
  uint32_t b[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) b[j] = p[j * (G * 8)];
  uint32_t x = b[0] | b[1] << 8 | b[2] << 16 | b[3] << 24;
  uint32_t y = b[4] | b[5] << 8 | b[6] << 16 | b[7] << 24;
  x &= byte_mask(bits);
  y &= byte_mask(bits >> 4);
  uint32_t(&w)[PER] = C < 4 ? lo : hi;
  constexpr int D = C & 3;
  if constexpr (K == 4) {
    // rows: planes, columns: the eight words
    x = transpose4(x);
    y = transpose4(y);
    const uint32_t l = (x & 0x0f0f0f0fu) | ((y << 4) & 0xf0f0f0f0u);
    const uint32_t h = ((x >> 4) & 0x0f0f0f0fu) | (y & 0xf0f0f0f0u);
    put_byte<D, 0>(w[0], l);
    put_byte<D, 1>(w[1], l);
    put_byte<D, 2>(w[2], l);
    put_byte<D, 3>(w[3], l);
    put_byte<D, 0>(w[4], h);
    put_byte<D, 1>(w[5], h);
    put_byte<D, 2>(w[6], h);
    put_byte<D, 3>(w[7], h);
  } else {
    // the four words are half of each plane byte
    const uint32_t sh = (threadIdx.x & 1u) * 4;
    x = ((x >> sh) & 0x0f0f0f0fu) | ((y >> sh) & 0x0f0f0f0fu) << 4;
    x = transpose4(x);
    put_byte<D, 0>(w[0], x);
    put_byte<D, 1>(w[1], x);
    put_byte<D, 2>(w[2], x);
    put_byte<D, 3>(w[3], x);
  }
}
// BIT_K inverse of a chunk: thread t gets its PER consecutive words t * PER ..
// (zero past the G groups).  Plane j holds bit j of word 64g + i as bit i of
// unit j * G + g, so a thread's words are a byte (K = 4) or half a byte (K = 8)
// of each plane: eight planes are read as eight bytes (neighbouring threads,
// neighbouring bytes) and transposed in registers, about 45 (25) vector
// instructions for 8 x 8 (8 x 4) bits instead of two per bit, and a chunk's
// prefix sum needs one wave scan instead of one per group.
template <int K, int PER>
__device__ __forceinline__ void planes_to_words(const uint64_t* planes, uint32_t G, uint64_t pm,
                                                typename Traits<K>::Word (&w)[PER]) {
  uint32_t lo[PER], hi[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) lo[i] = hi[i] = 0;
  pm = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)pm) |
       (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(pm >> 32)) << 32;
  if (threadIdx.x < (K == 4 ? G * 8 : G * 16)) {
    const uint8_t* p = (const uint8_t*)planes;
    plane_bytes<K, 0, PER>(p, G, pm, lo, hi);
    plane_bytes<K, 1, PER>(p, G, pm, lo, hi);
    plane_bytes<K, 2, PER>(p, G, pm, lo, hi);
    plane_bytes<K, 3, PER>(p, G, pm, lo, hi);
    if constexpr (K == 8) {
      plane_bytes<K, 4, PER>(p, G, pm, lo, hi);
      plane_bytes<K, 5, PER>(p, G, pm, lo, hi);
      plane_bytes<K, 6, PER>(p, G, pm, lo, hi);
      plane_bytes<K, 7, PER>(p, G, pm, lo, hi);
    }
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if constexpr (K == 4) w[i] = lo[i];
    else w[i] = (uint64_t)lo[i] | (uint64_t)hi[i] << 32;
  }
}

// Decodes chunk c of a field (Sec. IV-E); a malformed record sets FORMAT.
// Bound by vector issue (0.6 of the chip's rate) and the chunk's serial chain
// (record, bitmap levels, prefix, edges; four chunks of eight waves fill a
// CU).  Rounds without items are left out of the RZE stages, planes become
// words by byte transposes, edges come from one comparison: 256^3 float32
// 125 -> 100 us (vector instructions 1853 -> 1081 per wave), 512^3 float64 1422
// -> 1113 us (1396 -> 834).
template <int K>
__device__ __forceinline__ void decode_body(const uint8_t* __restrict__ stream, uint32_t n,
                            const uint64_t* __restrict__ offsets, Params* prm,
                            typename Traits<K>::Raw* __restrict__ out, uint32_t nch,
                            uint32_t c) {
  using Tr = Traits<K>;
  using Word = typename Tr::Word;
  constexpr uint32_t W = kChunkBytes / K;
  constexpr int PER = (int)(W / kCT);  // consecutive points of a thread
  __shared__ uint64_t U[kMaxUnits + 2];
  __shared__ uint64_t Mb[kMaxUnits + 2];
  __shared__ Scratch sc;
  __shared__ uint64_t wsum[kCW];     // per-wave sums of the bin deltas
  __shared__ uint64_t s_first;       // the chunk's first bin
  __shared__ uint32_t s_mm[2][kCW];  // per-wave least / greatest bin, from the first - 2^30
  __shared__ uint32_t s_far;         // some bin is 2^30 or more from the first
  __shared__ int s_bad;

  const uint32_t p0 = c * W, nc = min(W, n - p0);
  const uint32_t m = (nc + 63) / 64 * 64, G = m / 64, L = m * K;
  const uint64_t body = kHeaderBytes + 4ull * nch;
  // the record's size and offset are read together with the status;
  // offsets inconsistent (one read decides for the block: other chunks may
  // set the flag concurrently)
  const uint32_t rsize = ((const uint32_t*)(stream + kHeaderBytes))[c];
  const uint64_t roff = offsets[c];
  if (threadIdx.x == 0) {
    s_bad = 0;
    s_far = 0;
  }
  __shared__ uint32_t s_fail;
  if (threadIdx.x == 0) s_fail = prm->status & ST_FORMAT;
  __syncthreads();
  if (s_fail) return;
  const uint8_t* rec = stream + body + roff;
  if (rsize < kRecordHeaderBytes || (rsize & 3)) {
    if (threadIdx.x == 0) set_status(prm, ST_FORMAT);
    return;
  }
  // a record that fits in Mb (every record of a chunk that compresses at all)
  // comes in with one load per word, its parts are then read from LDS; the
  // header is read (scalar loads) while the words are in flight
  const bool whole = rsize <= 8 * (kMaxUnits + 2);
  if (whole) stage((uint8_t*)Mb, rec, rsize);
  const uint8_t* hd = rec;
  const double inv = __longlong_as_double(*(const long long*)(stream + 56));
  const double winv = 1.0 / inv;
  const uint32_t bfl = hd[0], sfl = hd[1];
  const uint32_t npts = hd[2] | (hd[3] << 8);
  const uint32_t blen = *(const uint32_t*)(hd + 4);
  const uint32_t smid = *(const uint32_t*)(hd + 8);
  const uint32_t slen = *(const uint32_t*)(hd + 12);
  bool ok = !(bfl & ~1u) && !(sfl & ~3u) && npts == nc && blen <= L &&
            smid <= L && slen <= L;
  const uint32_t used = kRecordHeaderBytes + blen + slen;
  ok = ok && ((used + 3) & ~3u) == rsize;
  if (ok && threadIdx.x < rsize - used && hd[used + threadIdx.x] != 0) s_bad = 1;
  __syncthreads();  // s_bad, and the staged record
  ok = ok && !s_bad;
  if (!ok) {
    if (threadIdx.x == 0) set_status(prm, ST_FORMAT);
    return;
  }

  // bins: RZE_1 -> BIT_K -> negabinary -> prefix sum (words kept in registers)
  const uint64_t* bsrc = Mb + (whole ? kRecordHeaderBytes / 8 : 0);
  if (!whole) {
    stage((uint8_t*)Mb, rec + kRecordHeaderBytes, blen);
    __syncthreads();
  }
  const uint64_t* planes;
  uint64_t pm0 = 0;
  if (bfl & 1) {
    ok = blen == L;
    planes = bsrc;
    if (ok) pm0 = nonzero_planes<K>(planes, G, sc);
  } else {
    ok = rze_decode<1>((const uint8_t*)bsrc, blen, L, U, sc, G);
    planes = U;
    pm0 = sc.planes;
  }
  if (!ok) {
    if (threadIdx.x == 0) set_status(prm, ST_FORMAT);
    return;
  }
  // bins of the thread's points, each wave's first relative to the wave
  Word wv[PER];
  const uint32_t j0 = threadIdx.x * PER;
  const bool full = nc == W;
  {
    planes_to_words<K, PER>(planes, G, pm0, wv);
    const Word Mk = (Word)0xAAAAAAAAAAAAAAAAull;
    Word run = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      // negabinary -> delta; inclusive prefix within the thread
      Word d = (Word)((wv[i] ^ Mk) - Mk);
      if (!full && j0 + i >= nc) d = 0;
      run += d;
      wv[i] = run;
    }
    const Word inc = wave_scan<Word>(run), exc = inc - run;
    if (lane() == 63) wsum[wave()] = (uint64_t)inc;
    if (threadIdx.x == 0) s_first = (uint64_t)wv[0];
    __syncthreads();
    Word base = exc;
    const int w0 = __builtin_amdgcn_readfirstlane(wave());
#pragma unroll
    for (int w = 0; w < kCW - 1; ++w)
      if (w0 > w) base += (Word)wsum[w];
    // the chunk's bin range (for the edge table below), as distances from its
    // first bin plus 2^30; the wave results are read after the next barrier
    const Word first = (Word)s_first - (Word)(1u << 30);
    uint32_t lo = 0xffffffffu, hi = 0;
    bool far = false;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      wv[i] += base;
      const Word off = wv[i] - first;
      const bool on = full || j0 + i < nc;
      if (K == 8) far |= on && (off >> 31) != 0;
      const uint32_t o = (uint32_t)off;
      lo = on && o < lo ? o : lo;
      hi = on && o > hi ? o : hi;
    }
    far |= (hi >> 31) != 0;
    lo = wave_reduce(lo, OpMin{});
    hi = wave_reduce(hi, OpMax{});
    if (lane() == 0) {
      s_mm[0][wave()] = lo;
      s_mm[1][wave()] = hi;
    }
    if (__ballot(far) && lane() == 0) s_far = 1;
  }

  // subbins: RZE_1 -> RZE_K -> BIT_K (the part goes to U, free now)
  const uint32_t soff = kRecordHeaderBytes + blen;
  const uint32_t shift = soff & 3u;
  if (whole) {
    const uint32_t* src = (const uint32_t*)((const uint8_t*)Mb + (soff - shift));
    for (uint32_t i = threadIdx.x; i < (slen + shift + 3) / 4; i += kCT) ((uint32_t*)U)[i] = src[i];
  } else {
    stage((uint8_t*)U, rec + (soff - shift), slen + shift);
  }
  __syncthreads();
  const uint8_t* sp = (const uint8_t*)U + shift;
  if (sfl & 2) {
    ok = slen == smid;
    if (ok) {
      uint8_t* mb = (uint8_t*)Mb;
      for (uint32_t i = threadIdx.x; i < smid; i += kCT) mb[i] = sp[i];
    }
    __syncthreads();
  } else {
    ok = rze_decode<1>(sp, slen, smid, Mb, sc, 0);
  }
  uint64_t* spare = Mb;  // the buffer not holding the subbin planes
  uint64_t spm = 0;
  if (ok) {
    if (sfl & 1) {
      ok = smid == L;
      planes = Mb;
      spare = U;
      if (ok) spm = nonzero_planes<K>(planes, G, sc);
    } else {
      ok = rze_decode<K>((const uint8_t*)Mb, smid, L, U, sc, G);
      planes = U;
      spm = sc.planes;
    }
  }
  if (!ok) {
    if (threadIdx.x == 0) set_status(prm, ST_FORMAT);
    return;
  }
  Word sv[PER];
  planes_to_words<K, PER>(planes, G, spm, sv);

  // reconstruct (Sec. IV-E).  The lower edges of the chunk's bin range and of
  // the bin above it go to a table in the spare buffer when the range is small
  // enough, so that each distinct bin's edge is found once.
  using Key = typename Tr::Bin;  // order keys fit the signed bin type
  using UKey = std::make_unsigned_t<Key>;
  constexpr uint32_t kTab = kChunkBytes / sizeof(Key);
  uint32_t olo = 0xffffffffu, ohi = 0;
#pragma unroll
  for (int w = 0; w < kCW; ++w) {
    olo = min(olo, s_mm[0][w]);
    ohi = max(ohi, s_mm[1][w]);
  }
  const Word first = (Word)s_first - (Word)(1u << 30) + (Word)olo;  // the chunk's lowest bin
  auto bin_of = [](Word v) -> int64_t {
    return K == 4 ? (int64_t)(int32_t)(uint32_t)v : (int64_t)(uint64_t)v;
  };
  const int64_t bmin = bin_of(first), bmax = bmin + (int64_t)(uint64_t)(ohi - olo);
  const bool table = !s_far && ohi - olo < kTab - 1 && bmin >= -Tr::kBinLimit &&
                     bmax <= Tr::kBinLimit;
  Key* T = (Key*)spare;
  if (table)
    for (uint32_t e = threadIdx.x; e < ohi - olo + 2; e += kCT)
      T[e] = lower_edge<K>(bmin + (int64_t)e, inv, winv);
  __syncthreads();
  bool bad = false, odd = !table;
  typename Tr::Raw v[PER];
  if (table) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const bool on = full || j0 + i < nc;
      const uint32_t e = on ? (uint32_t)(wv[i] - first) : 0u;
      const Key t = T[e], next = T[e + 1];
      odd |= on && (t == kNoKey<K> || next == kNoKey<K>);
      // inside bin b iff below the edge of bin b + 1
      bad |= on && sv[i] >= (Word)((UKey)next - (UKey)t);
      v[i] = Tr::unkey((int64_t)(Key)((UKey)t + (UKey)sv[i]));
    }
  }
  if (__ballot(odd)) {  // no table, or an edge is missing
    bad = false;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (!full && j0 + i >= nc) break;
      const int64_t b = bin_of(wv[i]);
      bad |= !point_ok<K>(b, (uint64_t)sv[i], lower_edge<K>(b, inv, winv),
                          lower_edge<K>(b + 1, inv, winv), inv, v[i]);
    }
  }
  // the thread's points are consecutive: 16-byte stores where the field
  // allows (it need only be aligned to its elements)
  typename Tr::Raw* dst = out + p0 + j0;
  if (full && ((uintptr_t)out & 15u) == 0) {
#pragma unroll
    for (int q = 0; q < PER * K / 16; ++q) ((uint4*)dst)[q] = ((const uint4*)v)[q];
  } else {
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (j0 + i < nc) dst[i] = v[i];
  }
  if (bad) set_status(prm, ST_FORMAT);
}

template <int K>
__global__ __launch_bounds__(kCT, 6) void k_decode(
    const uint8_t* __restrict__ stream, uint32_t n,
    const uint64_t* __restrict__ offsets, Params* prm,
    typename Traits<K>::Raw* __restrict__ out) {
  decode_body<K>(stream, n, offsets, prm, out, gridDim.x, blockIdx.x);
}

// ------------------------------------------------------------------ batches
// Encoder over the chunks of every field of one dtype, in ticket order: a
// chunk's look-back only waits for chunks of its field with earlier tickets,
// which workgroups already hold.  Skipped when *gate != 0 (the repair sweeps
// before it have not reached the fixed point: tiles are listed for sweep
// gate_sweep).
template <int K>
__global__ __launch_bounds__(kCT) void k_encode_p(const BatchDesc* bd, const Job* jobs,
                                                  int gate_sweep) {
  constexpr int g0 = K == 4 ? 0 : 2;
  __shared__ uint32_t s_t;
  BatchCounters* bc = bd->bc;
  if (gate_sweep > 0 && bc->lens[gate_sweep % kRing]) return;
  const uint32_t i0 = bd->item0[PH_C][g0], i1 = bd->item0[PH_C][g0 + 2];
  const int j0 = (int)bd->job0[g0], j1 = (int)bd->job0[g0 + 2];
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) s_t = i0 + atomicAdd(&bc->enc_cursor[K == 4 ? 0 : 1], 1u);
    __syncthreads();
    const uint32_t t = s_t;
    if (t >= i1) break;
    const Job& J = jobs[find_job<&Job::c0>(jobs, j0, j1, t)];
    encode_body<K, false>(J.box.n, (const typename Traits<K>::Bin*)J.bins, J.sub, J.lookback,
                          J.parts, J.prm, J.stream, J.cap, J.nch, t - J.c0, RecordSlots{});
  }
}

__device__ int status_of(uint32_t st) {
  if (st & ST_NONFINITE) return -2;
  if (st & ST_BOUND) return -3;
  if (st & ST_RANGE) return -4;
  if (st & ST_FORMAT) return -6;
  if (st & ST_INTERNAL) return -9;
  if (st & ST_CAPACITY) return -5;
  return 0;
}

// Per-field results of a compress batch: stream size and status.
__global__ __launch_bounds__(kThreads) void k_finalize_c(const BatchDesc* bd, const Job* jobs,
                                                         int gate_sweep) {
  if (gate_sweep > 0 && bd->bc->lens[gate_sweep % kRing]) return;
  BatchResult* res = bd->res;
  const uint32_t nj = bd->job0[kGroups];
  // a thread per word of a header (one thread's 64 dependent byte copies took
  // 18 us)
  constexpr uint32_t HW = kHeaderBytes / 4;
  static_assert(offsetof(Params, header) % 4 == 0 && offsetof(BatchResult, header) % 4 == 0,
                "headers are copied as words");
  for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < nj * HW; i += gridDim.x * kThreads) {
    const uint32_t j = i / HW, w = i % HW;
    const Job& J = jobs[j];
    ((uint32_t*)res[j].header)[w] = ((const uint32_t*)J.prm->header)[w];
    if (w) continue;
    const int st = status_of(J.prm->status);
    const uint64_t size = J.prm->stream_size;
    res[j].size = size;
    res[j].status = st;
    if (J.out_size) *J.out_size = size;
    if (J.out_status) *J.out_status = st;
  }
}

// Header check of a field to decode (the same rules as the host parser),
// then the record offsets from its size table.
__global__ __launch_bounds__(kThreads) void k_dhead_p(const BatchDesc* bd, const Job* jobs) {
  __shared__ int s_ok;
  const int nj = (int)bd->job0[kGroups];
  for (int j = blockIdx.x; j < nj; j += gridDim.x) {
    const Job& J = jobs[j];
    __syncthreads();
    if (threadIdx.x == 0) {
      const uint8_t* h = J.stream;
      auto u64 = [&](int o) {
        uint64_t v = 0;
        for (int b = 0; b < 8; ++b) v |= (uint64_t)h[o + b] << (8 * b);
        return v;
      };
      bool ok = (u64(0) & 0xFFFFFFFFFFFFull) == ((uint64_t)kMagic | ((uint64_t)kVersion << 32));
      ok = ok && h[6] == J.dtype && h[7] == J.ndim && h[32] <= 1 &&
           (uint32_t)u64(36) == kChunkBytes;
      for (int i = 0; i < 3; ++i)
        ok = ok && u64(8 + 8 * i) == (uint64_t)(i < J.ndim ? J.dims[i] : 1);
      const double e = __longlong_as_double((long long)u64(48));
      const double v = __longlong_as_double((long long)u64(56));
      ok = ok && finite64(u64(48)) && e > 0.0 && finite64(u64(56)) && v > 0.0;
      ok = ok && fma(v, e, -1.0) >= 0.0 &&
           fma(__longlong_as_double((long long)u64(56) - 1), e, -1.0) < 0.0;
      if (!ok) set_status(J.prm, ST_FORMAT);
      s_ok = ok;
    }
    __syncthreads();
    if (s_ok)
      offsets_body(J.stream, J.nch, J.stream_size - kHeaderBytes - 4ull * J.nch, J.offsets,
                   J.prm);
  }
}

template <int K>
__global__ __launch_bounds__(kCT, 6) void k_decode_p(const BatchDesc* bd, const Job* jobs) {
  constexpr int g0 = K == 4 ? 0 : 2;
  __shared__ uint32_t s_t;
  BatchCounters* bc = bd->bc;
  const uint32_t i0 = bd->item0[PH_C][g0], i1 = bd->item0[PH_C][g0 + 2];
  const int j0 = (int)bd->job0[g0], j1 = (int)bd->job0[g0 + 2];
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) s_t = i0 + atomicAdd(&bc->dec_cursor[K == 4 ? 0 : 1], 1u);
    __syncthreads();
    const uint32_t t = s_t;
    if (t >= i1) break;
    const Job& J = jobs[find_job<&Job::c0>(jobs, j0, j1, t)];
    decode_body<K>(J.stream, J.box.n, J.offsets, J.prm,
                   (typename Traits<K>::Raw*)J.y, J.nch, t - J.c0);
  }
}

// Per-field results of a decompress batch: field bytes and status.
__global__ __launch_bounds__(kThreads) void k_finalize_d(const BatchDesc* bd, const Job* jobs) {
  BatchResult* res = bd->res;
  const uint32_t nj = bd->job0[kGroups];
  for (uint32_t j = blockIdx.x * kThreads + threadIdx.x; j < nj; j += gridDim.x * kThreads) {
    const Job& J = jobs[j];
    const int st = status_of(J.prm->status);
    const uint64_t size = st ? 0 : (uint64_t)J.box.n * (J.dtype == 0 ? 4u : 8u);
    res[j].size = size;
    res[j].status = st;
    if (J.out_size) *J.out_size = size;
    if (J.out_status) *J.out_status = st;
  }
}

// Direct grids: one workgroup per chunk.  The encoder still takes its chunk
// from the ticket counter, so chunks start in field-major order.
template <int K>
__global__ __launch_bounds__(kCT) void k_encode_d(const BatchDesc* bd, const Job* jobs,
                                                  int gate_sweep) {
  constexpr int g0 = K == 4 ? 0 : 2;
  __shared__ uint32_t s_t;
  BatchCounters* bc = bd->bc;
  if (gate_sweep > 0 && bc->lens[gate_sweep % kRing]) return;
  if (threadIdx.x == 0) s_t = bd->item0[PH_C][g0] + atomicAdd(&bc->enc_cursor[K == 4 ? 0 : 1], 1u);
  __syncthreads();
  const uint32_t t = s_t;
  const Job& J = jobs[find_job<&Job::c0>(jobs, (int)bd->job0[g0], (int)bd->job0[g0 + 2], t)];
  encode_body<K, false>(J.box.n, (const typename Traits<K>::Bin*)J.bins, J.sub, J.lookback,
                        J.parts, J.prm, J.stream, J.cap, J.nch, t - J.c0, RecordSlots{});
}

template <int K>
__global__ __launch_bounds__(kCT, 6) void k_decode_d(const BatchDesc* bd, const Job* jobs) {
  constexpr int g0 = K == 4 ? 0 : 2;
  const uint32_t t = bd->item0[PH_C][g0] + blockIdx.x;
  const Job& J = jobs[find_job<&Job::c0>(jobs, (int)bd->job0[g0], (int)bd->job0[g0 + 2], t)];
  decode_body<K>(J.stream, J.box.n, J.offsets, J.prm, (typename Traits<K>::Raw*)J.y, J.nch,
                 t - J.c0);
}

}  // namespace

// ------------------------------------------------------------------ launchers
hipError_t launch_encode(int dtype, uint32_t n, const void* bins, uint32_t* sub,
                         uint16_t* mask, uint8_t* tail, uint64_t* offs, uint32_t* parts,
                         Params* prm, uint8_t* stream, size_t cap, const uint32_t* gate,
                         hipStream_t s, Ev ev) {
  const uint32_t K = dtype == 0 ? 4 : 8;
  const uint32_t W = kChunkBytes / K;
  const uint32_t nch = (n + W - 1) / W;
  RecordSlots S;
  S.seg[0] = (uint8_t*)bins;
  S.seg[1] = (uint8_t*)sub;
  S.seg[2] = (uint8_t*)mask;
  S.len[0] = W * K;
  S.len[1] = W * 4;
  S.len[2] = W * 2;
  S.tail = tail;
  S.tail_len = kRecordTailBytes;
  if (dtype == 0)
    launch_ev(k_encode<4>, dim3(nch), dim3(kCT), s, Ev{ev.a, nullptr}, n,
                          (const int32_t*)bins, (const uint32_t*)sub, parts, prm, stream,
                          (uint64_t)cap, nch, S, gate);
  else
    launch_ev(k_encode<8>, dim3(nch), dim3(kCT), s, Ev{ev.a, nullptr}, n,
                          (const int64_t*)bins, (const uint32_t*)sub, parts, prm, stream,
                          (uint64_t)cap, nch, S, gate);
  if (nch <= kPlaceChunks) {
    launch_ev(k_place_few, dim3((nch + kThreads / 64 - 1) / (kThreads / 64)), dim3(kThreads), s,
              Ev{nullptr, ev.b}, (const uint32_t*)parts, nch, S, prm, stream, (uint64_t)cap, gate);
    return hipGetLastError();
  }
  k_record_offsets<<<1, kOT, 0, s>>>(parts, nch, offs, prm, gate);
  launch_ev(k_place, dim3(nch), dim3(kThreads), s, Ev{nullptr, ev.b},
                        (const uint32_t*)parts, (const uint64_t*)offs, nch, S, prm, stream,
                        (uint64_t)cap, gate);
  return hipGetLastError();
}

hipError_t launch_sum_parts(const uint32_t* parts, uint32_t nch, Params* prm,
                            hipStream_t s) {
  k_sum_parts<<<1, kThreads, 0, s>>>(parts, nch, prm);
  return hipGetLastError();
}

hipError_t launch_offsets(const uint8_t* stream, uint32_t nch,
                          uint64_t body_bytes, uint64_t* offsets, Params* prm,
                          hipStream_t s, Ev ev) {
  launch_ev(k_offsets, dim3(1), dim3(kOfT), s, ev, stream, nch,
                        body_bytes, offsets, prm);
  return hipGetLastError();
}

hipError_t launch_decode(int dtype, const uint8_t* stream, uint32_t n,
                         const uint64_t* offsets, Params* prm, void* field,
                         hipStream_t s, Ev ev) {
  uint32_t W = kChunkBytes / (dtype == 0 ? 4 : 8);
  uint32_t nch = (n + W - 1) / W;
  if (dtype == 0)
    launch_ev(k_decode<4>, dim3(nch), dim3(kCT), s, ev, stream, n,
                          offsets, prm, (uint32_t*)field);
  else
    launch_ev(k_decode<8>, dim3(nch), dim3(kCT), s, ev, stream, n,
                          offsets, prm, (uint64_t*)field);
  return hipGetLastError();
}

hipError_t launch_encode_p(int dtype, const BatchDesc* bd, const Job* jobs, int gate_sweep,
                           int grid, hipStream_t s) {
  if (dtype == 0) k_encode_p<4><<<grid, kCT, 0, s>>>(bd, jobs, gate_sweep);
  else k_encode_p<8><<<grid, kCT, 0, s>>>(bd, jobs, gate_sweep);
  return hipGetLastError();
}

hipError_t launch_finalize_c(const BatchDesc* bd, const Job* jobs, int gate_sweep,
                             hipStream_t s) {
  k_finalize_c<<<4, kThreads, 0, s>>>(bd, jobs, gate_sweep);
  return hipGetLastError();
}

hipError_t launch_dhead_p(const BatchDesc* bd, const Job* jobs, int grid, hipStream_t s) {
  k_dhead_p<<<grid, kThreads, 0, s>>>(bd, jobs);
  return hipGetLastError();
}

hipError_t launch_decode_p(int dtype, const BatchDesc* bd, const Job* jobs, int grid,
                           hipStream_t s) {
  if (dtype == 0) k_decode_p<4><<<grid, kCT, 0, s>>>(bd, jobs);
  else k_decode_p<8><<<grid, kCT, 0, s>>>(bd, jobs);
  return hipGetLastError();
}

hipError_t launch_finalize_d(const BatchDesc* bd, const Job* jobs, hipStream_t s) {
  k_finalize_d<<<4, kThreads, 0, s>>>(bd, jobs);
  return hipGetLastError();
}

hipError_t launch_encode_d(int dtype, const BatchDesc* bd, const Job* jobs, int gate_sweep,
                           uint32_t items, hipStream_t s) {
  if (!items) return hipSuccess;
  if (dtype == 0) k_encode_d<4><<<items, kCT, 0, s>>>(bd, jobs, gate_sweep);
  else k_encode_d<8><<<items, kCT, 0, s>>>(bd, jobs, gate_sweep);
  return hipGetLastError();
}

hipError_t launch_decode_d(int dtype, const BatchDesc* bd, const Job* jobs, uint32_t items,
                           hipStream_t s) {
  if (!items) return hipSuccess;
  if (dtype == 0) k_decode_d<4><<<items, kCT, 0, s>>>(bd, jobs);
  else k_decode_d<8><<<items, kCT, 0, s>>>(bd, jobs);
  return hipGetLastError();
}

int codec_blocks_per_cu(int kernel) {
  int b = 0;
  hipError_t e = hipErrorInvalidValue;
  switch (kernel) {
    case PK_ENCODE: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_encode_p<8>, kCT, 0); break;
    case PK_DHEAD: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_dhead_p, kThreads, 0); break;
    case PK_DECODE: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_decode_p<8>, kCT, 0); break;
    default: break;
  }
  return e == hipSuccess && b > 0 ? b : 1;
}

}  // namespace lopc
