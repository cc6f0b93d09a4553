// Host-side driver for the input transform's aligned row segments (csrc/address_math.hpp), built by
// tests/test_host_aligned_segments.py with -fsanitize=address,undefined; touches no GPU.  The tensor lies at every distance from a
// multiple of four, inside a larger buffer whose other bytes must neither be loaded nor show.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <vector>

#include "address_math.hpp"

using namespace rnswino;

static uint64_t state = 88172645463325252ull;
static uint32_t rnd() {                                    // xorshift64*
  state ^= state >> 12; state ^= state << 25; state ^= state >> 27;
  return (uint32_t)((state * 2685821657736338717ull) >> 32);
}
static int between(int lo, int hi) { return lo + (int)(rnd() % (uint32_t)(hi - lo + 1)); }

int main() {
  long long bad = 0, checks = 0;
  const int tiles_m[] = {1, 2, 4, 6, 7, 8, 10};
  for (int layer = 0; layer < 3000; ++layer) {
    const int N = between(1, 3), C = between(1, layer % 8 ? 6 : 70), H = between(1, layer % 3 ? 6 : 30), W = between(1, layer % 3 ? 9 : 40);
    const int r = between(1, 3), pad = rnd() % 4 ? between(0, 3) : between(4, 24), m = tiles_m[rnd() % 7], t = m + r - 1;
    const int Ho = H + 2 * pad - r + 1, Wo = W + 2 * pad - r + 1, HW = H * W, mis = (int)(rnd() & 3);
    const long long total = (long long)N * C * HW;
    if (Ho <= 0 || Wo <= 0 || total < 16) continue;
    const int th = (Ho + m - 1) / m, tw = (Wo + m - 1) / m, last = (int)total - 16 + mis;
    std::vector<uint8_t> x((size_t)total);
    for (auto &b : x) b = (uint8_t)(rnd() | 1);            // no zeros: a byte that should have been masked shows
    for (int img = 0; img < N; ++img)
      for (int ty = 0; ty < th; ++ty)
        for (int tx = 0; tx < tw; ++tx)
          for (int c = 0; c < C; ++c)
            for (int a = 0; a < t; ++a) {
              const int y0 = ty * m - pad, x0 = tx * m - pad, gy = y0 + a;
              const bool in = gy >= 0 && gy < H;
              const unsigned long long m0 = byte_range(std::max(-x0, 0), std::min(t, W - x0), 0), m1 = byte_range(std::max(-x0, 0), std::min(t, W - x0), 8);
              uint8_t want[16] = {};
              for (int b = 0; b < t; ++b)
                if (in && x0 + b >= 0 && x0 + b < W) want[b] = x[(size_t)(((long long)img * C + c) * HW + (long long)gy * W + x0 + b)];
              // rows outside the image repeat its first or last row
              const int from = (img * C + c) * HW + x0 + mis + std::min(std::max(gy, 0), H - 1) * W, load = aligned_segment_at(from, mis, last);
              const int at = load - mis;                   // from the tensor's start
              // the kernel's short form shifts by the low bits of `from`
              const int moved = load == (from & ~3) ? from & 3 : from - load;
              ++checks;
              bool ok = at >= 0 && at + 16 <= total;
              if (ok) {
                unsigned long long w[2];
                std::memcpy(w, x.data() + at, 16);
                if (moved & ~3) move_segment(moved, w[0], w[1]);
                else if (moved) { w[0] = w[0] >> (8 * moved) | w[1] << (64 - 8 * moved); w[1] >>= 8 * moved; }
                w[0] &= in ? m0 : 0; w[1] &= in ? m1 : 0;
                ok = std::memcmp(w, want, 16) == 0;
                // away from the tensor's ends every load starts at a multiple of four
                if (at > 3 && at + 19 < total && ((at + mis) & 3)) ok = false;
              }
              if (!ok && ++bad <= 10)
                std::printf("mis %d N=%d C=%d H=%d W=%d r=%d m=%d pad=%d tile %d,%d,%d channel %d row %d: at %d\n", mis, N, C, H, W, r, m, pad,
                            img, ty, tx, c, a, at);
            }
  }
  std::printf("checks=%lld bad=%lld\n", checks, bad);
  return bad ? 1 : 0;
}
