// Host harness for the order flags of the first pass (lopc_tile.h, compiled
// here for the CPU): a tile's cells as the kernel fills them, cells outside the
// grid holding kNoBin and the tile's first value, and every flag of every
// point by the kernel's two comparisons.  A flag may only name a neighbour
// inside the grid, whatever the values, and where both values are in range it
// is the definition's: same bin (q_bin / q_bin32) and lower in (value, index)
// order.  Exits with the number of mistakes.
#include <cmath>
#include <cstdio>
#include <limits>
#include <vector>

#include "../paper_2603_26968_amd/csrc/lopc_tile.h"

using namespace lopc;

static int bad_flags, bad_status, checked;

template <int K, int TZ, int TY, int TX, typename Val>
void check(int nz, int ny, int nx, const std::vector<Val>& field, double inv) {
  using G = TileGeom<TZ, TY, TX>;
  constexpr int NJ = TZ == 1 ? 6 : 14;
  auto at = [&](int z, int y, int x) { return field[(z * ny + y) * nx + x]; };
  bool bad = false, out = false;
  const int64_t bref = K == 8 ? first_bin<K>((double)field[0], inv, bad) : 0;
  std::vector<int32_t> B(G::H, kNoBin);
  std::vector<Val> X(G::H, field[0]);
  bool far = false;
  auto cell = [&](int z, int y, int x) { return ((z + G::ZO) * G::HY + y + 1) * G::HX + x + 1; };
  for (int z = 0; z < nz; ++z)
    for (int y = 0; y < ny; ++y)
      for (int x = 0; x < nx; ++x) {
        const double v = (double)at(z, y, x);
        const int64_t b = first_bin<K>(v, inv, bad), want = K == 4 ? q_bin32(v, inv) : q_bin(v, inv);
        const bool in = std::isfinite(v) && want <= Traits<K>::kBinLimit && want >= -Traits<K>::kBinLimit;
        out |= std::isfinite(v) && !in;
        if (in && b != want) ++bad_flags;
        far |= K == 8 && (uint64_t)b - (uint64_t)bref + (1ull << 30) >= (1ull << 31);
        B[cell(z, y, x)] = K == 4 ? (int32_t)b : (int32_t)((uint64_t)b - (uint64_t)bref);
        X[cell(z, y, x)] = at(z, y, x);
      }
  if (out && !bad) ++bad_status;
  if (far) return;  // the kernel quantizes again with bounds checks
  for (int z = 0; z < nz; ++z)
    for (int y = 0; y < ny; ++y)
      for (int x = 0; x < nx; ++x)
        for (int j = 0; j < NJ; ++j) {
          const int li = cell(z, y, x);
          const int ln = li + kOff[j][0] * G::HY * G::HX + kOff[j][1] * G::HX + kOff[j][2];
          const bool flag = B[ln] == B[li] && flag_lower(j, X[ln], X[li]);
          const int zz = z + kOff[j][0], yy = y + kOff[j][1], xx = x + kOff[j][2];
          const bool in = zz >= 0 && zz < nz && yy >= 0 && yy < ny && xx >= 0 && xx < nx;
          ++checked;
          if (!in) {
            if (flag) ++bad_flags;
            continue;
          }
          const double p = (double)at(z, y, x), q = (double)at(zz, yy, xx);
          const int64_t bp = K == 4 ? q_bin32(p, inv) : q_bin(p, inv),
                        bq = K == 4 ? q_bin32(q, inv) : q_bin(q, inv);
          const bool lower = q < p || (q == p && (j & 1));
          if (std::llabs(bp) <= Traits<K>::kBinLimit && std::llabs(bq) <= Traits<K>::kBinLimit &&
              flag != (bp == bq && lower))
            ++bad_flags;
        }
}

template <int K, typename Val>
void sweep(const std::vector<Val>& special) {
  const int shapes[][3] = {{1, 1, 1}, {1, 1, 5}, {1, 4, 1}, {1, 3, 4}, {2, 1, 1}, {2, 3, 4}, {3, 2, 2}};
  for (const auto& s : shapes) {
    const int n = s[0] * s[1] * s[2];
    for (double inv : {1.0, 0.5, 3.0})
      for (Val v : special)
        for (Val w : {(Val)0, (Val)0.25, v})
          for (int at = 0; at <= n; ++at) {  // at == n: everywhere
            std::vector<Val> f(n, w);
            for (int i = 0; i < n; ++i)
              if (i == at || at == n) f[i] = v;
            if (s[0] == 1) check<K, 1, 32, 64, Val>(s[0], s[1], s[2], f, inv);
            else check<K, 4, 8, 32, Val>(s[0], s[1], s[2], f, inv);
          }
  }
}

int main() {
  const float fi = std::numeric_limits<float>::infinity();
  const double di = std::numeric_limits<double>::infinity();
  sweep<4, float>({-fi, fi, std::nanf(""), -3e9f, 3e9f, -2147483648.0f, 2147483648.0f, -2147483520.0f,
                   2147483520.0f, -4294967296.0f, -715827904.0f, -3.4e38f, 1.0f, -0.0f});
  sweep<8, double>({-di, di, std::nan(""), -1e19, 1e19, -4611686018427387904.0, 4611686018427387904.0,
                    -2147483648.0, 2147483648.0, -1073741824.0, 1073741823.0, -1e300, 1.0, -0.0});
  std::printf("%d flags, %d wrong, %d wrong states\n", checked, bad_flags, bad_status);
  return bad_flags + bad_status != 0;
}
