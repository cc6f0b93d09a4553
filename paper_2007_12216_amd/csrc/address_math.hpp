// Integer arithmetic behind the kernels' addresses, shared with the host so that a CPU test can walk over it
// (tests/host/address_driver.cpp).  Nothing of HIP in here.
#pragma once
#include "layout.hpp"

namespace rnswino {

// Division of 0 <= n < 2^31 by a fixed d >= 1 as one high multiplication: mul = ceil(2^(31 + shift) / d), shift = ceil(log2 d),
// so mul d - 2^(31 + shift) < d <= 2^shift and the quotient of 2n mul / 2^(32 + shift) is off by less than 1/d.  (The division
// that the compiler writes is 25 dependent instructions, and a kernel's first load waits for up to five of them.)
struct FastDiv {
  uint32_t mul, shift;
};
inline FastDiv make_fast_div(uint32_t d) {
  FastDiv f;
  f.shift = 0;
  while ((1ull << f.shift) < d) ++f.shift;
  f.mul = (uint32_t)(((1ull << (31 + f.shift)) + d - 1) / d);
  return f;
}
RNSW_HD uint32_t fast_div(uint32_t n, FastDiv d) { return (uint32_t)(((uint64_t)(n << 1) * d.mul) >> 32) >> d.shift; }

// ---- 16-byte row segments (input transform) ----
// A segment that begins before the tensor or ends behind it is loaded from the nearest 16 bytes inside, `moved` = wanted - loaded
// bytes away, and put into place by move_segment().  What it holds of other rows, or of nothing, is masked afterwards.

RNSW_HD long long segment_at(long long from, long long total) {
  const long long at = from < total - 16 ? from : total - 16;
  return at > 0 ? at : 0;
}

// The same relative to an origin at tensor byte `base`: offsets [lo, hi] from it that a load may start at.  Saturating the bounds to
// 32 bits changes nothing, since offsets of rows inside the image are smaller.  An origin inside the last 16 bytes of the tensor makes hi
// negative, down to -16: the loads' base lies 16 bytes before the origin, so that their offsets are not.
struct SegmentRange {
  int lo, hi;
};
RNSW_HD SegmentRange segment_range(long long base, long long total) {
  const long long lo = base < 0 ? -base : 0, room = total - 16 - base, hi = room > -16 ? room : -16;
  return {(int)(lo < 0x7FFFFFFFll ? lo : 0x7FFFFFFFll), (int)(hi < 0x7FFFFFFFll ? hi : 0x7FFFFFFFll)};
}
RNSW_HD int segment_at(int from, SegmentRange r) {
  const int at = from > r.lo ? from : r.lo;
  return at < r.hi ? at : r.hi;
}

// Where the load of the segment at `want` begins that starts at a multiple of four if it can: offsets from the multiple of four at or
// before the tensor's start, `mis` bytes before it; loads of 16 bytes begin in [mis, last].  A wave's 16-byte loads from any byte take 59
// cycles of a compute unit's address unit (37 with several waves at it), from multiples of four 27 (21).
RNSW_HD int aligned_segment_at(int want, int mis, int last) {
  const int at = (want & ~3) > mis ? (want & ~3) : mis;
  return at < last ? at : last;
}

// byte b of the segment is byte b + moved of what was loaded (16 and more bytes apart: everything is masked)
RNSW_HD void move_segment(int moved, unsigned long long &w0, unsigned long long &w1) {
  const int dist = moved < 0 ? -moved : moved, s = dist < 15 ? dist : 15;
  if (moved > 0) {
    if (s >= 8) { w0 = w1; w1 = 0; }
    if (s & 7) { w0 = w0 >> (8 * (s & 7)) | w1 << (64 - 8 * (s & 7)); w1 >>= 8 * (s & 7); }
  } else {
    if (s >= 8) { w1 = w0; w0 = 0; }
    if (s & 7) { w1 = w1 << (8 * (s & 7)) | w0 >> (64 - 8 * (s & 7)); w0 <<= 8 * (s & 7); }
  }
}

// bytes [lo, hi) of an 8-byte word that starts at byte `at`: a mask
RNSW_HD unsigned long long byte_range(int lo, int hi, int at) {
  const int l = lo - at < 0 ? 0 : lo - at > 8 ? 8 : lo - at, h = hi - at < 0 ? 0 : hi - at > 8 ? 8 : hi - at;
  const unsigned long long below_h = h == 8 ? ~0ull : (1ull << (8 * h)) - 1, below_l = l == 8 ? ~0ull : (1ull << (8 * l)) - 1;
  return below_h & ~below_l;
}

// ---- a copy by several workgroups ----
// Bytes [first, end) of workgroup `block`, a share of whole steps but for the last one (the product in 64 bits: with many workgroups that have next to nothing
// to copy it leaves 32).  A load of 16 bytes that would end behind them ends with them; below 16 (a last share) with the first 16 of all.
struct CopyShare {
  uint32_t first, end;
};
inline uint32_t share_of(uint32_t bytes, uint32_t blocks, uint32_t step) { return (bytes / blocks / step + 1) * step; }
RNSW_HD CopyShare copy_share(uint32_t bytes, uint32_t block, uint32_t share) {
  const uint64_t first = (uint64_t)block * share;
  return {(uint32_t)(first < bytes ? first : bytes), (uint32_t)(first + share < bytes ? first + share : bytes)};
}
RNSW_HD uint32_t piece_at(uint32_t at, uint32_t end) {
  const uint32_t last = end > 16 ? end - 16 : 0;
  return at < last ? at : last;
}

// ---- staged patches (direct convolution) ----
// The longest run of padded pixels that `pixels` consecutive output pixels, beginning at a multiple of `pixels`, need for all r x r
// taps: every row boundary among them adds r - 1 pixels of border, every image boundary r - 1 rows more.
inline long long patch_pixels(long long pixels, int N, int Ho, int Wo, int Wp, int r) {
  const long long plane = (long long)Ho * Wo, images = N == 1 || plane % pixels == 0 ? 0 : (pixels - 2) / plane + 1;
  return pixels + ((pixels - 2) / Wo + 1) * (r - 1) + images * (r - 1) * Wp + (r - 1) * (Wp + 1LL);
}

}  // namespace rnswino
