// CPU check of the slabs in which the device converts a component between the
// host layout and the planes (hl_host_layout.hpp), built by
// tests/test_host_slabs.py: every slab fits the staging buffer and a launch
// (fewer than 2^32 work-items), a plane's bytes have 32-bit offsets, the slabs
// cover the component, and a component is left to the host only if a single j_1
// does not fit or the planes are too large.
#include <cstdio>

#include "hl_host_layout.hpp"

int main() {
  int bad = 0;
  const int64_t big = ((int64_t)1 << 24) - 1;  // 2^32 / 256 work-items, less one
  const int32_t Ks[][3] = {
      {2, 2, 2},         {1000, 777, 1},          {5, 7, 3},
      {1 << 28, 1, 1},   {(1 << 29) - 1, 1, 1},  {1 << 29, 1, 1},
      {600000000, 1, 1}, {32768, 16384, 1},      {1000, 900, 800},
      {2, (int32_t)big, 1}, {2, (int32_t)big + 1, 1},
      {33, 1 << 20, 1},  {40, (1 << 19) + 1, 1},  {2, 4096, 4096},
      {4, 4097, 4096},   {100, 2896, 2897},       {65, 1 << 20, 8},
      {2, 1 << 25, 1},   {2, 2100000, 1},         {400, 400, 400},
  };
  for (const auto& K : Ks)
    for (int d = 1; d <= 3; ++d)
      for (int m = 0; m <= (d == 1 ? 7 : d == 2 ? 5 : 3); ++m)
        for (int walls = 0; walls < 2; ++walls)
          for (int field = 0; field < 2; ++field)
            for (int word = 4; word <= 8; word += 4) {
              const hl_host::LayoutMap L = hl_host::field_layout(d, m, K, walls, field);
              const hl_host::Slabs q = hl_host::slabs_of(L, word);
              const int64_t rows = (d > 1 ? L.K[1] : 1) * (d > 2 ? L.K[2] : 1);
              const int64_t one = rows * L.nc * 8;  // bytes of one j_1
              bool ok = q.per == rows * L.nc && q.jn >= 0 && q.jn <= L.K[0];
              const bool wide = L.nodes * word > ((int64_t)1 << 32) - 1;
              if (q.jn > 0) {
                ok = ok && !wide;
                const int64_t groups = (q.jn + hl_host::kConvNodes - 1) / hl_host::kConvNodes * rows;
                ok = ok && one * q.jn <= (int64_t)256 << 20 && groups * 256 < (int64_t)1 << 32;
              } else {
                ok = ok && (wide || one > (int64_t)256 << 20 || rows * 256 >= (int64_t)1 << 32);
              }
              if (!ok) {
                std::printf("FAIL d=%d m=%d K=%d,%d,%d walls=%d field=%d word=%d: jn=%lld\n", d, m, K[0], K[1], K[2], walls,
                            field, word, (long long)q.jn);
                ++bad;
              }
            }
  if (bad) return 1;
  std::printf("ok\n");
  return 0;
}
