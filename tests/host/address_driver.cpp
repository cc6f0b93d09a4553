// Host-side driver for the arithmetic that the kernels' addresses and residues rest on (csrc/address_math.hpp, plan_math.cpp).
// Built by tests/test_host_arithmetic.py with -fsanitize=address,undefined; touches no GPU.  Argument: which part to run.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "address_math.hpp"
#include "plan.hpp"

using namespace rnswino;

static long long bad = 0, checks = 0;
#define CHECK(cond, ...)                                   \
  do {                                                     \
    ++checks;                                              \
    if (!(cond) && ++bad <= 10) { std::printf(__VA_ARGS__); std::printf("\n"); } \
  } while (0)

static uint64_t state = 88172645463325252ull;
static uint32_t rnd() {                                    // xorshift64*
  state ^= state >> 12; state ^= state << 25; state ^= state >> 27;
  return (uint32_t)((state * 2685821657736338717ull) >> 32);
}
static int between(int lo, int hi) { return lo + (int)(rnd() % (uint32_t)(hi - lo + 1)); }

static void divisions() {
  auto one = [](uint32_t d) {
    const FastDiv f = make_fast_div(d);
    auto at = [&](uint64_t n) { if (n < (1ull << 31)) CHECK(fast_div((uint32_t)n, f) == n / d, "fast_div(%llu, %u)", (unsigned long long)n, d); };
    at(0); at((1ull << 31) - 1); at((1ull << 31) - 2);
    for (int e = 0; e < 40; ++e) {
      const uint64_t q = rnd() % ((1ull << 31) / d + 1);
      at(q * d); at(q * d + d - 1); at(rnd() >> 1);
      if (q) at(q * d - 1);
    }
    const uint64_t top = ((1ull << 31) - 1) / d;            // the largest quotient's first and last numerators
    at(top * d); at(top * d - 1);
  };
  for (uint32_t d = 1; d <= 5000; ++d) one(d);
  for (int k = 12; k < 31; ++k)
    for (int e = -3; e <= 3; ++e) one((1u << k) + e);
  one(0x7FFFFFFFu);
  for (int e = 0; e < 20000; ++e) { const uint32_t d = rnd() >> between(1, 20); if (d) one(d); }
}

// The gather of k_input_transform.hpp on a small tensor: every segment of every tile, as each of its three forms takes it.
static void segments() {
  const int tiles_m[] = {1, 2, 4, 6, 7, 8, 10, 12, 14};
  for (int layer = 0; layer < 4000; ++layer) {
    const int N = between(1, 3), C = between(1, layer % 8 ? 6 : 70), H = between(1, layer % 3 ? 6 : 30), W = between(1, layer % 3 ? 9 : 40);
    const int r = between(1, 5), pad = rnd() % 4 ? between(0, 3) : between(4, 24), m = tiles_m[rnd() % 9], t = m + r - 1;
    const int Ho = H + 2 * pad - r + 1, Wo = W + 2 * pad - r + 1;
    if (Ho <= 0 || Wo <= 0 || t > 16 || t < 2) continue;
    const int th = (Ho + m - 1) / m, tw = (Wo + m - 1) / m, HW = H * W;
    const long long total = (long long)N * C * HW;
    std::vector<uint8_t> x((size_t)total);
    for (auto &b : x) b = (uint8_t)(rnd() | 1);            // no zeros: a byte that should have been masked shows
    for (int img = 0; img < N; ++img)
      for (int ty = 0; ty < th; ++ty)
        for (int tx = 0; tx < tw; ++tx)
          for (int cb = 0; cb < (C + 63) / 64; ++cb) {
            const int y0 = ty * m - pad, x0 = tx * m - pad, cbase = cb * 64;
            const long long base = ((long long)img * C + cbase) * HW + (long long)y0 * W + x0;
            const SegmentRange range = segment_range(base, total), whole = {0, (int)total - 16};
            const bool columns = x0 < W && x0 + t > 0;
            const unsigned long long m0 = byte_range(std::max(-x0, 0), std::min(t, W - x0), 0), m1 = byte_range(std::max(-x0, 0), std::min(t, W - x0), 8);
            for (int c = 0; c < 64 && cbase + c < C; ++c)
              for (int a = 0; a < t; ++a) {
                const int gy = y0 + a;
                if (gy < 0 || gy >= H) continue;           // a row outside the image: nothing is loaded
                uint8_t want[16] = {};
                for (int b = 0; b < t; ++b)
                  if (x0 + b >= 0 && x0 + b < W) want[b] = x[(size_t)(((long long)img * C + cbase + c) * HW + (long long)gy * W + x0 + b)];
                const int from = c * HW + a * W;
                for (int form = 0; form < 3; ++form) {
                  if ((form == 0 && !columns) || (form == 2 && total < 16)) continue;
                  long long at, moved;
                  if (form == 0) {                         // one tile per block: relative to the tile's origin
                    const int off = segment_at(from, range);
                    at = base + off;
                    moved = total < 16 ? base + from : from - off;
                    if (total >= 16) CHECK(off >= -16, "offset %d below the loads' base", off);
                  } else if (form == 1) {                  // packed tiles: 64 bits
                    at = segment_at(base + from, total);
                    moved = base + from - at;
                  } else {                                 // sixteen tiles per block: 32 bits from the tensor's start
                    at = segment_at((int)(base + from), whole);
                    moved = base + from - at;
                  }
                  uint8_t got[16] = {};
                  if (total >= 16) {
                    CHECK(at >= 0 && at + 16 <= total, "form %d loads [%lld, %lld) of %lld bytes", form, at, at + 16, total);
                    if (at < 0 || at + 16 > total) continue;
                    std::memcpy(got, x.data() + at, 16);
                  } else {
                    std::memcpy(got, x.data(), (size_t)total);
                  }
                  unsigned long long w[2];
                  std::memcpy(w, got, 16);
                  if (moved != 0) move_segment((int)moved, w[0], w[1]);
                  w[0] &= m0; w[1] &= m1;
                  CHECK(std::memcmp(w, want, 16) == 0, "form %d N=%d C=%d H=%d W=%d r=%d m=%d pad=%d tile %d,%d,%d channel %d row %d", form, N, C, H, W, r, m,
                        pad, img, ty, tx, cbase + c, a);
                }
              }
          }
  }
  // tensors beyond 2 GiB, arithmetic only: origins at both ends and in the middle, rows up to 64 planes of 2^24 bytes on
  for (int e = 0; e < 200000; ++e) {
    const long long total = 16 + ((long long)rnd() << between(0, 8)), origin = between(0, 2) == 0 ? between(0, 40) : (long long)(((uint64_t)rnd() << 8) % (uint64_t)total);
    const long long base = between(0, 1) ? total - origin : origin - between(0, 40);
    const SegmentRange range = segment_range(base, total);
    const int from = between(0, 1) ? between(0, 64) : (int)(rnd() % ((1u << 30) + (1u << 28)));
    if (base + from >= total || base + from + 15 < 0) continue;                    // overlaps the tensor, as a row inside the image does
    const int off = segment_at(from, range);
    CHECK(base + off >= 0 && base + off + 16 <= total && off >= -16 && std::abs((long long)from - off) <= 15,
          "base %lld total %lld from %d: offset %d", base, total, from, off);
  }
}

// copy_share() and piece_at(): every byte is in some share's pieces, and no piece leaves the buffer
static void copies() {
  for (int e = 0; e < 4000; ++e) {
    const uint32_t step = 4096u << between(0, 2), n = 8 * (uint32_t)(e % 2 ? between(1, 31) : between(1, 400));
    const uint32_t bytes = (uint32_t)between(16, e % 3 ? 3000 : 4000000), share = share_of(bytes, n, step);
    CHECK(share % step == 0 && (uint64_t)share * n > bytes, "%u bytes, %u shares of %u", bytes, n, share);
    uint32_t covered = 0;                                  // [0, covered) is copied: the shares follow each other, and so do a share's pieces
    for (uint32_t block = 0; block < n; ++block) {
      const CopyShare s = copy_share(bytes, block, share);
      CHECK(s.first <= s.end && s.end <= bytes && s.end - s.first <= share, "%u bytes, share %u of %u: [%u, %u)", bytes, block, n, s.first, s.end);
      if (s.first >= s.end) continue;
      for (uint32_t at = s.first; at < s.first + 4 * share; at += 16) {        // (threads past the end of a share repeat its last piece)
        const uint32_t got = piece_at(at, s.end);
        CHECK(got <= covered && got + 16 <= bytes && got < s.end, "%u bytes, share %u of %u: piece at %u, %u covered", bytes, block, n, got, covered);
        if (got + 16 <= covered && at >= s.end) break;
        covered = std::max(covered, got + 16);
      }
    }
    CHECK(covered == bytes, "%u bytes in %u shares: %u covered", bytes, n, covered);
  }
  for (uint32_t n = 8; n < 1u << 21; n += n < 4096 ? 8 : 4096) {               // the largest input, and more workgroups than it has steps
    const uint32_t share = share_of(0x7FFFFFFFu, n, 16384);
    for (uint32_t block : {0u, 1u, n / 2, n - 2, n - 1}) {
      const CopyShare s = copy_share(0x7FFFFFFFu, block, share);
      const uint64_t first = std::min((uint64_t)block * share, (uint64_t)0x7FFFFFFF), end = std::min((uint64_t)(block + 1) * share, (uint64_t)0x7FFFFFFF);
      CHECK(s.first == first && s.end == end, "share %u of %u", block, n);
    }
  }
}

// patch_pixels() against the patches of every block of every shape, taken pixel by pixel
static void patches() {
  for (int e = 0; e < 6000; ++e) {
    const int r = between(1, 7), pad = between(0, 4), N = between(1, 5), H = between(1, e % 4 ? 12 : 90), W = between(1, e % 4 ? 15 : 130);
    const int Ho = H + 2 * pad - r + 1, Wo = W + 2 * pad - r + 1, Hp = H + 2 * pad, Wp = W + 2 * pad;
    if (Ho <= 0 || Wo <= 0) continue;
    const long long npix = (long long)N * Ho * Wo;
    auto origin = [&](long long pix) {
      const long long n = pix / (Ho * Wo), rem = pix % (Ho * Wo);
      return (n * Hp + rem / Wo) * Wp + rem % Wo;
    };
    for (int pixels : {64, 128, 256}) {
      const long long room = patch_pixels(pixels, N, Ho, Wo, Wp, r);
      for (long long first = 0; first < npix; first += pixels) {
        const long long last = std::min(first + pixels - 1, npix - 1);
        const long long len = origin(last) - origin(first) + (long long)(r - 1) * (Wp + 1) + 1;
        CHECK(len <= room, "r=%d pad=%d N=%d H=%d W=%d: %lld pixels in a patch of %lld", r, pad, N, H, W, len, room);
        CHECK(origin(last) + (long long)(r - 1) * (Wp + 1) < (long long)N * Hp * Wp, "r=%d pad=%d N=%d H=%d W=%d: past the end", r, pad, N, H, W);
      }
    }
  }
}

// biased_lowbyte() over the sums that the input transform and the GEMM admit, |sum| <= 2^22 - 2^15, for every odd modulus
static void residues() {
  for (int p = 3; p <= 253; p += 2) {
    const BiasedStart b = biased_start(p);
    const int a = b.acc_bias - 0x4B400000, limit = (1 << 22) - (1 << 15);
    CHECK(a % 256 == 0 && std::abs(a) < 1 << 15, "p=%d starts at %d", p, a);
    const float inv = 1.0f / (float)p;
    const int step = p == 3 || p == 251 || p == 253 ? 1 : 97;
    for (int x = -limit; x <= limit; x += step) {
      const int acc = b.acc_bias + x;
      float f;
      std::memcpy(&f, &acc, 4);
      f = std::fmaf(f, inv, b.quot_bias);
      int q;
      std::memcpy(&q, &f, 4);
      q = (int)((uint32_t)q << 8) >> 8;                    // the 24-bit multiply-add takes the low 24 bits, signed
      const int got = (int8_t)(uint8_t)((uint32_t)q * (uint32_t)-p + (uint32_t)acc);
      CHECK((got - x) % p == 0 && std::abs(got) <= 127, "p=%d sum %d gives %d", p, x, got);
    }
  }
}

int main(int argc, char **argv) {
  const std::string part = argc > 1 ? argv[1] : "";
  if (part == "divisions") divisions();
  else if (part == "segments") segments();
  else if (part == "copies") copies();
  else if (part == "patches") patches();
  else if (part == "residues") residues();
  else return 2;
  std::printf("%s checks=%lld bad=%lld\n", part.c_str(), checks, bad);
  return bad ? 1 : 0;
}
