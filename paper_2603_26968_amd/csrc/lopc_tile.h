// Geometry of the repair's tiles: the LDS box of a tile and its one-point
// halo, and the halo points a run needs, face by face; and the bins and
// comparisons the first pass makes its order flags of.  Host+device so that a
// CPU harness can check the same source.
#pragma once

#include "lopc_device.h"

namespace lopc {

constexpr uint32_t kHalo = 1u << 31;  // LDS word of a point outside the tile

template <int TZ, int TY, int TX>
struct TileGeom {
  static constexpr int ZO = TZ == 1 ? 0 : 1;  // 2D tiles carry no z halo
  static constexpr int HZ = TZ + 2 * ZO, HY = TY + 2, HX = TX + 2;
  static constexpr int H = HZ * HY * HX;
  static constexpr int NPT = TZ * TY * TX;
  static constexpr int PER = NPT / kThreads;
  static_assert(NPT % kThreads == 0, "tile must be a multiple of the block");
  // owned point tid + k * kThreads (slot k of thread tid) lies kSlot LDS
  // words after slot 0: the block covers whole planes of a 3D tile, or whole
  // rows of a 2D one
  static_assert((TZ > 1 && TY * TX == kThreads) || (TZ == 1 && kThreads % TX == 0),
                "slots of a thread are evenly spaced in LDS");
  static constexpr int kSlot = TZ > 1 ? HY * HX : (kThreads / TX) * HX;
  // halo-local index of interior point i
  __host__ __device__ static int local(int i) {
    int iz = i / (TY * TX), iy = (i / TX) % TY, ix = i % TX;
    return ((iz + ZO) * HY + iy + 1) * HX + ix + 1;
  }
  __host__ __device__ static bool on_edge(int i) {
    int iz = i / (TY * TX), iy = (i / TX) % TY, ix = i % TX;
    return (TZ > 1 && (iz == 0 || iz == TZ - 1)) || iy == 0 || iy == TY - 1 ||
           ix == 0 || ix == TX - 1;
  }
};

// ------------------------------------------------------------------ faces
// The halo points a tile run needs are those with a stencil neighbour in the
// tile: 922 of the 1016 around a 4 x 8 x 32 tile.  They are taken face by face
// in slots of 64 lanes whose points lie on one face: lane r of a face is point
// (u, v) = (r / width, r % width) of it.  A point of a low face (z, y or x =
// -1) reaches the tile along +axis plus any of the two other positive unit
// steps, one of a high face along the negatives: four neighbours in 3D, two in
// 2D, at distances d from the point's LDS index that are the same for the
// whole slot.
struct FaceSlot {
  int32_t r0, cnt, width, magic;  // first lane's r, points of the face, r / width = r * magic >> 16
  int32_t z, y, x;                // tile coordinates of the face's point (0, 0)
  int32_t ua, va;                 // axis of u and v (0 x, 1 y, 2 z)
  int32_t li, lu, lv;             // LDS index of point (0, 0), steps along u and v
  int32_t d[4];                   // LDS distances to the neighbours in the tile
  uint32_t keep[4];               // subbin, kHalo and the flag through which each sees the point
  uint32_t weight;                // 1: the face's points have higher indices
};
template <int TZ, int TY, int TX>
struct Faces {
  using G = TileGeom<TZ, TY, TX>;
  static constexpr int NF = TZ == 1 ? 4 : 6, ND = TZ == 1 ? 2 : 4;
  // faces: x-, x+, y-, y+, z-, z+.  Edges belong to the z faces first, then to
  // the x faces.
  static constexpr int count(int f) {
    return f < 2 ? TZ * (TY + 1) : f < 4 ? TZ * TX : (TY + 1) * (TX + 1);
  }
  static constexpr int slots() {
    int n = 0;
    for (int f = 0; f < NF; ++f) n += (count(f) + 63) / 64;
    return n;
  }
  static constexpr int kSlots = slots(), kPer = (kSlots + kWaves - 1) / kWaves;
  FaceSlot s[kSlots] = {};
  constexpr Faces() {
    int i = 0;
    for (int f = 0; f < NF; ++f) {
      const int a = f / 2, high = f & 1;
      const int step[3] = {1, G::HX, G::HY * G::HX}, ext[3] = {TX, TY, TZ};
      const int va = a == 0 ? 1 : 0, ua = a == 2 ? 1 : 2;
      // along an axis whose edge points the face owns it starts one point
      // before the tile (low faces) or ends one after it
      const bool ve = a != 1, ue = a == 2;
      int c[3] = {0, 0, 0};
      c[a] = high ? ext[a] : -1;
      if (ve && !high) c[va] = -1;
      if (ue && !high) c[ua] = -1;
      const int width = ext[va] + (ve ? 1 : 0);
      const int ea = 1 << a, ev = 1 << va, eu = 1 << ua;
      for (int r0 = 0; r0 < count(f); r0 += 64, ++i) {
        FaceSlot& q = s[i];
        q.r0 = r0;
        q.cnt = count(f);
        q.width = width;
        q.magic = 65536 / width + 1;
        q.z = c[2];
        q.y = c[1];
        q.x = c[0];
        q.ua = ua;
        q.va = va;
        q.li = ((c[2] + G::ZO) * G::HY + c[1] + 1) * G::HX + c[0] + 1;
        q.lu = step[ua];
        q.lv = step[va];
        q.weight = (uint32_t)high;
        for (int k = 0; k < ND; ++k) {
          const int e = ea | (k & 1 ? ev : 0) | (k & 2 ? eu : 0);
          const int d = step[a] + (k & 1 ? step[va] : 0) + (k & 2 ? step[ua] : 0);
          q.d[k] = high ? -d : d;
          q.keep[k] = 0xffffu | kHalo | 1u << (16 + 2 * (e - 1) + (high ? 0 : 1));
        }
      }
    }
  }
};
// Halo cells of the LDS box that no owned point reaches (cell i of them, i <
// kBlindCells): a face point's step may land on one.
template <int TZ, int TY, int TX>
struct Blind {
  using G = TileGeom<TZ, TY, TX>;
  static constexpr int kZ = TZ > 1 ? G::HY + G::HX - 1 : 0;  // per z face
  static constexpr int kCells = 2 * kZ + 2 * TZ;
  __host__ __device__ static int cell(int i) {
    if (i < kZ)
      return i < G::HY ? i * G::HX + G::HX - 1 : (G::HY - 1) * G::HX + i - G::HY;
    i -= kZ;
    const int top = (G::HZ - 1) * G::HY * G::HX;
    if (i < kZ) return top + (i < G::HY ? i * G::HX : i - G::HY + 1);
    i -= kZ;
    const int z = i < TZ ? i : i - TZ;
    return (z + G::ZO) * G::HY * G::HX + (i < TZ ? G::HX - 1 : (G::HY - 1) * G::HX);
  }
};

// ------------------------------------------------------------------ flags
// The first pass compares the bins of neighbours in 32 bits.  A cell outside
// the grid holds kNoBin, a bin that no point has, so that no comparison needs
// a bounds check.
constexpr int32_t kNoBin = (int32_t)0x80000000;

// Bin of value y in the first pass (Sec. IV-A): q_bin / q_bin32 with the
// common case branch-free.  float32: the conversion saturates, so a product
// out of range gives a bin outside the limits, of which the lowest is raised
// by one to leave kNoBin free.  float64: below 2^51 the rounded product plus
// 1.5 * 2^52 holds the integer in its low bits.
template <int K>
LOPC_HD int64_t first_bin(double y, double inv, bool& bad) {
  const double p = y * inv;
  double q = rint(p);
  if (fabs(p - q) == 0.5) {
    const double r = fma(y, inv, -p);
    if (r != 0.0) q = r > 0.0 ? p + 0.5 : p - 0.5;
  }
  if constexpr (K == 4) {
    int32_t b;
#if defined(__HIP_DEVICE_COMPILE__)
    asm("v_cvt_i32_f64 %0, %1" : "=v"(b) : "v"(q));
#else
    b = q >= 2147483647.0    ? 0x7fffffff
        : q <= -2147483648.0 ? (int32_t)0x80000000
        : q == q             ? (int32_t)q
                             : 0;
#endif
    b = b < -0x7fffffff ? -0x7fffffff : b;
    bad |= (uint32_t)b + 0x7ffffffeu > 0xfffffffcu;  // |b| > 2^31 - 2
    return b;
  } else {
    int64_t b = (int64_t)__builtin_bit_cast(uint64_t, q + 6755399441055744.0) - 0x4338000000000000ll;
    if (!(fabs(p) < 2251799813685248.0)) {
      b = q_bin(y, inv);
      bad |= b > Traits<8>::kBinLimit || b < -Traits<8>::kBinLimit;
    }
    return b;
  }
}

// Of two neighbours in one bin, whether vq, at stencil offset j of vp, is the
// lower in (value, index) order: an odd j has the lower index.
template <typename Val>
LOPC_HD bool flag_lower(int j, Val vq, Val vp) {
  return (j & 1) ? vq <= vp : vq < vp;
}

}  // namespace lopc
