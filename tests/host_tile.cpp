// Host harness for the geometry of the repair's tiles
// (paper_2603_26968_amd/csrc/lopc_tile.h, compiled here for the CPU): every
// cell of a tile's LDS box is an owned point, a face point or a blind cell,
// and every stencil pair of a halo point and an owned point is one face step,
// with the right flag and weight.  Prints one line per tile shape and exits
// with the number of mistakes.
#include <cstdio>
#include <map>
#include <utility>
#include <vector>

#include "../paper_2603_26968_amd/csrc/lopc_tile.h"

using namespace lopc;

template <int TZ, int TY, int TX>
int check() {
  using G = TileGeom<TZ, TY, TX>;
  using F = Faces<TZ, TY, TX>;
  static const F faces;
  constexpr int NJ = TZ == 1 ? 6 : 14, HXY = G::HY * G::HX;
  int bad = 0;
  enum { None, Owned, Face, Blank };
  std::vector<int> kind(G::H, None);
  for (int i = 0; i < G::NPT; ++i) kind[G::local(i)] = Owned;
  std::map<std::pair<int, int>, std::pair<int, unsigned>> steps;  // (halo, owned): flag, weight
  for (const FaceSlot& f : faces.s) {
    for (int lane = 0; lane < 64; ++lane) {
      const int r = f.r0 + lane, u = (r * f.magic) >> 16, v = r - u * f.width;
      const bool on = r < f.cnt;
      const int li = on ? f.li + u * f.lu + v * f.lv : f.li;
      if (on) {
        const int z = f.z + (f.ua == 2 ? u : 0), x = f.x + (f.va == 0 ? v : 0),
                  y = f.y + (f.ua == 1 ? u : 0) + (f.va == 1 ? v : 0);
        if (u != r / f.width || li < 0 || li >= G::H || kind[li] != None ||
            li != ((z + G::ZO) * G::HY + y + 1) * G::HX + x + 1) {
          ++bad;
          continue;
        }
        kind[li] = Face;
      }
      for (int k = 0; k < F::ND; ++k) {
        const int to = li + f.d[k];
        if (to < 0 || to >= G::H) {
          ++bad;
        } else if (on && kind[to] == Owned) {
          const unsigned flag = f.keep[k] & (0x3fffu << 16);
          if ((f.keep[k] ^ flag) != (0xffffu | kHalo) || (flag & (flag - 1)) ||
              !steps.emplace(std::make_pair(li, to),
                             std::make_pair(__builtin_ctz(flag) - 16, f.weight)).second)
            ++bad;
        }
      }
    }
  }
  for (int i = 0; i < Blind<TZ, TY, TX>::kCells; ++i) {
    const int c = Blind<TZ, TY, TX>::cell(i);
    if (c < 0 || c >= G::H || kind[c] != None) ++bad;
    else kind[c] = Blank;
  }
  for (int k : kind) bad += k == None;
  size_t pairs = 0;
  for (int i = 0; i < G::NPT; ++i) {
    const int li = G::local(i);
    for (int j = 0; j < NJ; ++j) {
      const int h = li + kOff[j][0] * HXY + kOff[j][1] * G::HX + kOff[j][2];
      if (kind[h] == Owned) continue;
      ++pairs;
      const auto it = steps.find({h, li});
      // a neighbour at an even offset has the higher index
      if (kind[h] != Face || it == steps.end() || it->second.first != j ||
          it->second.second != ((j & 1) ? 0u : 1u))
        ++bad;
    }
  }
  if (pairs != steps.size()) ++bad;
  std::printf("%dx%dx%d: %d slots, %zu pairs, %d mistakes\n", TZ, TY, TX, F::kSlots, pairs, bad);
  return bad;
}

int main() {
  return check<1, 32, 64>() + check<1, 16, 128>() + check<4, 8, 32>() + check<8, 8, 32>() +
         check<8, 16, 16>();
}
