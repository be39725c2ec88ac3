// Host-only check of tile_end and clamp_step (tiles.hpp) against 64-bit sums:
// tiles of every size at both ends of short axes and of axes up to 2^31 - 1, steps
// from one before to well past the end, and the parts that a tile is split into.
#include "wave_tiles.hpp"
#include <cstdio>
using namespace pmsz;
int main() {
  long long bad = 0, tests = 0;
  auto expect = [&](long long got, long long want, long long at, long long k, long long n) {
    ++tests;
    if (got != want && ++bad < 10)
      printf("bad at=%lld k=%lld n=%lld: %lld, not %lld\n", at, k, n, got, want);
  };
  const int32_t sizes[] = {1, 2, 3, 4, 31, 32, 64, 256, 8192};
  for (int64_t n64 : {1ll, 2ll, 5ll, 63ll, 64ll, 65ll, 8191ll, 8192ll, 2147483647ll, 2147483646ll,
                      2147483647ll - 31, 2147483647ll - 255, 2147483647ll - 8191}) {
    const int32_t n = (int32_t)n64;
    for (int32_t size : sizes) {
      const int64_t tiles = (n64 + size - 1) / size;
      for (int64_t t = 0; t < tiles; t = t < 3 || t >= tiles - 3 ? t + 1 : tiles - 3) {
        const int32_t at = (int32_t)(t * size);
        const long long end = (long long)at + size < n64 ? (long long)at + size : n64;
        expect(tile_end(at, size, n), end, at, size, n);
        for (int32_t step = -1; step <= size + 3; step += step > 8 && step < size - 2 ? 7 : 1) {
          long long v = (long long)at + step;
          v = v < 0 ? 0 : v < n64 ? v : n64 - 1;
          expect(clamp_step(at, step, n), v, at, step, n);
        }
        for (int32_t parts : {1, 2, 4, 8}) {
          // the parts cover the tile, in order
          long long next = at;
          for (int32_t p = 0; p < parts; ++p) {
            const Span s = part_of(at, size, n, p, parts);
            if (s.a >= s.b) continue;
            expect(s.a, next, at, p, n);
            next = s.b;
          }
          expect(next, end, at, parts, n);
        }
      }
    }
  }
  printf("tests %lld bad %lld\n", tests, bad);
  return bad != 0;
}
