// K1 and K2 in one kernel, for layers of one block of 64 channels (33 to 64, or, t <= 10, 16 tiles of up to four; 8-bit moduli): the input
// transform of 16 or 32 tiles and the residue GEMM over all their channels, V passing through LDS and never through device memory.
//
// Block = TH blocks of 16 tiles, 4 k12_quads() waves.  A wave gathers the pixels of 16 tiles in 16 channels once (the channels of one slice of V) and
// keeps them in registers as operand fragments (128 registers at t = 9, 10; with three and four contraction steps, t > 10, two waves share a slice's
// channels).  Then the block goes through its items: four groups of four
// transform points, the groups of all residues in a row (25 items of F(8,3) with four moduli; by 16 points of a residue there would be
// 28, four of them with four points).  Per item every wave transforms its slice of the 16 points (products and residues as in k1_input_transform_tiles)
// and writes 4 x 16 bytes a lane to LDS; behind the barrier wave (group, TH-th of the row blocks) multiplies the group's four points one after the
// other with fragments of U from L2, requested a set of row blocks ahead, and stores finished words of O (as k2_residue_gemm_lds does).  V has two buffers: one
// barrier an item.
//
// What bounds it: the vector unit (400 instructions a wave and item, of them 256 residues' multiply-adds and 48 matrix instructions: 53 % of
// the time on 64 -> 64 at 224 x 224, batch 8, matrix cores 22 %), 196 blocks on 256 compute units there, and the way of U.  V's way to memory
// and back was 320 MB of that layer: K1 43 + K2 61 us, so 83 (a layer 168 -> 131 us); 64 -> 128 at 112 x 112 68 -> 60, at batch 1 20.4 -> 18.9, 64 -> 64 at
// 224 x 224, batch 1, 32.4 -> 27.0.  On the way there (us of this kernel on the first two): 32 tiles a block 83 and 33, 16 tiles 93 and 36 (U crosses the L2
// twice as often); all blocks of a part through the items in the same order 100 and 42 (they wait for the same fragments from memory), U from a single resident
// fragment 64 and 26; multiply-adds right behind their quotients 103 and 40 (16 tiles); points of one residue an item 105 and 47 (16 tiles).
// 65 to 128 channels (eight waves, 16 tiles) lose: 128 -> 128 at 112 x 112, batch 8, 94 -> 110 us a layer.
//
// PACK: layers of up to four channels, 16 tiles a block.  A fragment of U then is four bytes in 16 places and zeros: made in registers from one byte quadruple
// per filter and point, where the GEMM fetched 1 KiB (and exchanged its results through LDS).  What bounds it are the words of O, 123 MB of 3 -> 64 at 224 x 224,
// batch 8, and the residues: K1 8.9 + K2 45.6 us, so 41 (a layer with cold operands 107.4 -> 87.6; with fragments from L2 143).  The filters may be split over workgroups, each
// transforming anew.
// Grid: one-dimensional, ceil(Tp / (16 TH)) x parts of the filters x parts of the items, rounded up to a multiple of 8 (kernels_common.hpp); in
// front of them the workgroups that only copy the input, also a multiple of 8, or none.
#pragma once
#include "k_input_transform.hpp"
#include "k_residue_gemm.hpp"

namespace rnswino {

// The residue of group g of Q: g / Q as a product with this, 16 bits shifted out; with eight moduli and t = 16 there are 512 groups, 64 a residue.
RNSW_HD constexpr uint32_t group_mul(uint32_t Q) { return (65535u + Q) / Q; }
constexpr bool group_division_is_exact() {
  for (uint32_t t = 2; t <= 16; ++t) {
    const uint32_t Q = (t * t + 3) / 4;
    for (uint32_t g = 0; g < 8 * Q; ++g)
      if (g * group_mul(Q) >> 16 != g / Q) return false;
  }
  return true;
}
static_assert(group_division_is_exact(), "");

struct K12Args {
  const ResidueParams *more;
  const int8_t *x;
  const int8_t *KB, *U;
  uint32_t *O;
  int per_xcd;                // the grid / 8
  int ntb, nkb;               // tile and row blocks of 16
  uint32_t tile_groups_mul, tw_mul, th_mul;          // FastDiv's, with the shifts below
  int C, H, W, pad, tw, th, T;
  int total;                  // N * C * H * W
  uint32_t Q_mul;             // group_mul(Q), Q = ceil(t*t / 4)
  uint32_t shifts;            // bytes: of the divisions by the tile blocks' groups, tw, th; packed layers: parts the filters are split into
  uint32_t sizes;             // bytes: m, t, n, items of a part
  uint32_t kept;              // the input's copy: where it lies in front of O, in 256 bytes; in the upper five bits its own workgroups / 8
  RNSW_HD FastDiv by_tile_groups() const { return {tile_groups_mul, shifts & 31u}; }
  RNSW_HD FastDiv by_tw() const { return {tw_mul, shifts >> 8 & 31u}; }
  RNSW_HD FastDiv by_th() const { return {th_mul, shifts >> 16 & 31u}; }
  RNSW_HD int row_parts() const { return (int)(shifts >> 24); }
  RNSW_HD int m() const { return (int)byte_of(sizes, 0); }
  RNSW_HD int t() const { return (int)byte_of(sizes, 1); }
  RNSW_HD int n() const { return (int)byte_of(sizes, 2); }
  RNSW_HD int part() const { return (int)(sizes >> 24); }
  RNSW_HD size_t kept_offset() const { return (size_t)(kept & 0x07FFFFFFu) * 256u; }
  RNSW_HD uint32_t copies() const { return kept >> 27 << 3; }
};
static_assert(sizeof(K12Args) <= 112, "kernels_common.hpp");

// biased_lowbyte() of four accumulators, constants of the lane's own; the multiply-adds stand behind all four quotients (right behind its own, each waits 8
// cycles, and two waves a SIMD do not hide them).
__device__ __forceinline__ void biased_lowbytes(uint32_t (&r)[4], int a0, int a1, int a2, int a3, float inv_p, float quot_bias, int neg_p) {
  r[0] = __float_as_uint(__builtin_fmaf(__int_as_float(a0), inv_p, quot_bias));
  r[1] = __float_as_uint(__builtin_fmaf(__int_as_float(a1), inv_p, quot_bias));
  r[2] = __float_as_uint(__builtin_fmaf(__int_as_float(a2), inv_p, quot_bias));
  r[3] = __float_as_uint(__builtin_fmaf(__int_as_float(a3), inv_p, quot_bias));
  asm("v_mad_i32_i24 %0, %0, %4, %5\n\tv_mad_i32_i24 %1, %1, %4, %6\n\tv_mad_i32_i24 %2, %2, %4, %7\n\tv_mad_i32_i24 %3, %3, %4, %8"
      : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]) : "v"(neg_p), "v"(a0), "v"(a1), "v"(a2), "v"(a3));
}

// A call leaves in the workspace what V can be had from again: not V itself but, in its place, the input (rnswino_debug_stage transforms it).  Workgroups
// copy it, each its share, four loads of 16 bytes a thread at a time: either ones of their own, on compute units that the others leave idle, or all of them,
// requested behind the gather and stored behind the wait in front of the items.  What it costs is the traffic: us a layer without a copy, with own
// workgroups and by all: 64 -> 64 at 224 x 224, batch 8 (56 of 256 compute units idle) 125.9, 130.7, 131.3; batch 1 (8 idle) 25.8, 25.6, 26.0; 64 -> 128 at
// 112 x 112, batch 8 (8) 59.7, 60.5, 61.3; where none is idle, 64 -> 51 at 188 x 48, three moduli, 27.1, 38.5, 27.6; 48 -> 9 at 124 x 142, F(14,3), 36.4, 51.4, 37.6.
template <int THREADS>
struct InputCopy {
  typedef int Bytes __attribute__((ext_vector_type(4), aligned(1), may_alias));
  static constexpr int AHEAD = 4;
  static constexpr uint32_t STEP = THREADS * 16;
  const int8_t *from;
  int8_t *to;
  uint32_t at, end;                                    // uniform: what is left of the share
  Bytes held[AHEAD];
  __device__ __forceinline__ InputCopy(const int8_t *x, int8_t *v, CopyShare own) : from(x), to(v), at(own.first), end(own.end) {}
  __device__ __forceinline__ uint32_t place(int j) const { return piece_at(at + threadIdx.x * 16u + j * STEP, end); }
  __device__ __forceinline__ void request() {
    if (at >= end) return;
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) held[j] = *(const Bytes *)(from + place(j));
  }
  __device__ __forceinline__ void store() {
    if (at >= end) return;
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) *(Bytes *)(to + place(j)) = held[j];
    at += AHEAD * STEP;
  }
  __device__ __forceinline__ void rest() {
    while (at < end) { request(); store(); }
  }
};
__global__ __launch_bounds__(256) void k_keep_input(const int8_t *x, int8_t *to, uint32_t bytes, uint32_t share) {
  InputCopy<256>(x, to, copy_share(bytes, blockIdx.x, share)).rest();
}

// Waves of a workgroup / 4: with three and four steps a wave takes half of a slice's channels, so that its pixels fit the same registers.
constexpr int k12_quads(int ks1, int th) { return ks1 > 2 ? 2 * th : th; }

template <int KS1, int TH, int RM, bool PACK>
__global__ __launch_bounds__(256 * k12_quads(KS1, TH), 2) void k12_transform_gemm(K12Args P) {
  Constant<ResidueParams> &R = constant(P.more);
  constexpr int QUADS = k12_quads(KS1, TH), NU = KS1 > 2 ? 2 : 4;      // channel groups of four a wave takes
  constexpr int ROWS = KS1 == 1 ? 8 : KS1 == 2 ? 10 : KS1 == 3 ? 12 : 16;
  constexpr int WPR = KS1 == 1 ? 2 : KS1 == 4 ? 4 : 3;                 // words of a row
  constexpr bool ALIGNED = KS1 < 4;                                    // a 16-byte load from a multiple of four holds a row
  constexpr int VBUF = 16 * TH * 1024;                                 // 16 points of V: [point][tile block][slice][tile][16 B]
  // gather: per wave [4 channels][step][slice h][tile][16 slots]; then two buffers of V
  __shared__ __attribute__((aligned(16))) uint8_t lds[16384 * QUADS * KS1 > 2 * VBUF ? 16384 * QUADS * KS1 : 2 * VBUF];
  asm volatile("" ::"s"(P.more), "s"(P.x), "s"(P.KB), "s"(P.U), "s"(P.O), "s"(P.per_xcd), "s"(P.ntb), "s"(P.nkb), "s"(P.tile_groups_mul),
               "s"(P.tw_mul), "s"(P.th_mul), "s"(P.C), "s"(P.H), "s"(P.W), "s"(P.pad), "s"(P.tw), "s"(P.th), "s"(P.T), "s"(P.total), "s"(P.Q_mul), "s"(P.shifts),
               "s"(P.sizes), "s"(P.kept));
  const int t = P.t(), P2 = t * t, CB1 = (P2 + 15) >> 4, Q = (P2 + 3) >> 2, HW = P.H * P.W;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, h = lane >> 4, col = lane & 15;
  const int slice = wave & 3, th = KS1 > 2 ? 0 : wave >> 2, u0 = KS1 > 2 ? NU * (wave >> 2) : 0;             // of V: what this wave transforms
  const uint32_t copies = P.copies(), id = blockIdx.x - copies;
  const int unit = (int)(id & 7) * P.per_xcd + (int)(id >> 3);
  auto share = [&](uint32_t block) { return InputCopy<256 * QUADS>(P.x, (int8_t *)P.O - P.kept_offset(), copy_share((uint32_t)P.total, block, R.kept_share)); };
  if (blockIdx.x < copies) return share(blockIdx.x).rest();
  const int tile_groups = (P.ntb + TH - 1) / TH, which = (int)fast_div((uint32_t)unit, P.by_tile_groups()), tb0 = (unit - which * tile_groups) * TH;
  const int part = PACK ? which / P.row_parts() : which;
  const int ngroups = P.n() * Q;
  const int first = part * P.part();
  if (4 * first >= ngroups) {                                           // the grid is padded to a multiple of 8
    if (!copies) share((uint32_t)unit).rest();
    return;
  }
  const int tau = min(tb0 + th, P.ntb - 1) * 16 + col;                 // past the last tile block: that one again
  // ---- gather: lane (channel h of four, tile) takes the t row segments of one channel after the other (see k1_input_transform_tiles) ----
  const int mis = (int)((uint32_t)(uintptr_t)P.x & 3u), last = P.total - 16 + mis;
  const int8_t *const xa = P.x - mis;
  struct Origin { int tile, y0, x0, img; };
  auto origin = [&](int tile) -> Origin {
    const int trow = (int)fast_div((uint32_t)tile, P.by_tw()), tx = tile - trow * P.tw;
    const int img = (int)fast_div((uint32_t)trow, P.by_th()), ty = trow - img * P.th;
    return {tile, ty * P.m() - P.pad, tx * P.m() - P.pad, img};
  };
  struct Segment { Origin o; int from; bool live; };
  const Origin own = PACK ? Origin() : origin(min(tau, P.T - 1));
  const int Tg = PACK ? (P.T + 15) >> 4 : P.T;
  auto segment = [&](int u) -> Segment {
    const int c64 = 16 * (u0 + u) + 4 * slice + h;                            // channel order of layout.hpp
    const int tile = PACK ? (4 * u + slice) * Tg + tau : tau, ch = PACK ? h : c64;
    Segment s;
    s.live = tau < Tg && tile < P.T && ch < P.C;
    s.o = PACK ? origin(s.live ? tile : 0) : own;
    s.from = (s.o.img * P.C + (s.live ? ch : 0)) * HW + s.o.x0 + mis;
    return s;
  };
  auto wanted = [&](const Segment &s, int a) { return s.from + min(max(s.o.y0 + a, 0), P.H - 1) * P.W; };
  auto load_at = [&](int want) { return ALIGNED ? aligned_segment_at(want, mis, last) : min(max(want, mis), last); };
  v4i pix[4 * NU][KS1];
  uint8_t *const staged = lds + wave * (4 * KS1 * 1024);
  auto request = [&](int u, v4i (&val)[ROWS], int &clamped) {
    const Segment s = segment(u);
    clamped = 0;
#pragma unroll
    for (int a = 0; a < ROWS; ++a) {
      const int want = wanted(s, a), at = load_at(want);
      clamped |= at ^ (ALIGNED ? want & ~3 : want);
      __builtin_memcpy(&val[a], xa + (uint32_t)at, 16);                // one 16-byte load
    }
  };
  auto settle = [&](int u, v4i (&val)[ROWS], int clamped) {
    const Segment s = segment(u);
    const unsigned long long m0 = byte_range(max(-s.o.x0, 0), min(t, P.W - s.o.x0), 0), m1 = byte_range(max(-s.o.x0, 0), min(t, P.W - s.o.x0), 8);
    const uint32_t mask[4] = {s.live ? (uint32_t)m0 : 0u, s.live ? (uint32_t)(m0 >> 32) : 0u, s.live ? (uint32_t)m1 : 0u, s.live ? (uint32_t)(m1 >> 32) : 0u};
    const int rows_in = min(t, P.H - s.o.y0);                          // row a is inside the image and the tile: -y0 <= a < rows_in
    uint32_t slots[16 * KS1];
#pragma unroll
    for (int d = 0; d < 16 * KS1; ++d) slots[d] = 0;
    if (__builtin_expect(__any(clamped != 0), 0)) {
#pragma unroll
      for (int a = 0; a < ROWS; ++a) {
        const int want = wanted(s, a), at = load_at(want);
        unsigned long long w0 = (uint32_t)val[a][0] | (unsigned long long)(uint32_t)val[a][1] << 32;
        unsigned long long w1 = (uint32_t)val[a][2] | (unsigned long long)(uint32_t)val[a][3] << 32;
        move_segment(want - at, w0, w1);
        slots[a * WPR] = (uint32_t)w0; slots[a * WPR + 1] = (uint32_t)(w0 >> 32);
        if (WPR > 2) slots[a * WPR + 2] = (uint32_t)w1;
        if (WPR > 3) slots[a * WPR + 3] = (uint32_t)(w1 >> 32);
      }
    } else {
#pragma unroll
      for (int a = 0; a < ROWS; ++a) {
        const uint32_t by = (uint32_t)wanted(s, a);                    // its low two bits count
#pragma unroll
        for (int d = 0; d < WPR; ++d) slots[a * WPR + d] = ALIGNED ? __builtin_amdgcn_alignbyte((uint32_t)val[a][ALIGNED ? d + 1 : d], (uint32_t)val[a][d], by) : (uint32_t)val[a][d];
      }
    }
#pragma unroll
    for (int a = 0; a < ROWS; ++a) {
      const bool in = a >= -s.o.y0 && a < rows_in;
#pragma unroll
      for (int d = 0; d < WPR; ++d) slots[a * WPR + d] &= in ? mask[d] : 0u;
    }
    if (KS1 == 1 && ((t + 3) & ~3) == 4) {                             // uniform: rows of one word
#pragma unroll
      for (int a = 0; a < ROWS; ++a) slots[a] = slots[2 * a];
    }
#pragma unroll
    for (int q = 0; q < 4 * KS1; ++q)
      *(v4i *)(staged + h * (KS1 * 1024) + q * 256 + col * 16) = (v4i){(int)slots[4 * q], (int)slots[4 * q + 1], (int)slots[4 * q + 2], (int)slots[4 * q + 3]};
    // (A wave reads only what it has written, and its LDS accesses stay in order; the compiler keeps them so, the addresses being one array's.)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int s1 = 0; s1 < KS1; ++s1) pix[4 * u + j][s1] = *(const v4i *)(staged + (j * KS1 + s1) * 1024 + lane * 16);
  };

  // ---- items: four groups of four points each, the groups of all residues in a row ----
  // The tile blocks of a part begin at different items and go round: side by side through the same ones, all would wait for the same
  // fragments of U on their way from memory.
  const int count = min(P.part(), ((ngroups + 3) >> 2) - first);
  int left = count, item = first + (int)((uint32_t)(unit - which * tile_groups) % (uint32_t)count);
  auto after = [&](int it) { return it + 1 == first + count ? first : it + 1; };
  struct Group { int i, q; };                                          // residue and points 4 q .. 4 q + 3; past the last group: that one again
  auto group = [&](int number) -> Group {
    const int g = min(number, ngroups - 1), i = (int)(((uint32_t)g * P.Q_mul) >> 16);
    return {i, g - i * Q};
  };
  const int wq = wave & 3, half = wave >> 2;                           // of O: what this wave multiplies: a group, every QUADS-th set of row blocks
  auto mine = [&](int it) -> Group {
    Group p = group(4 * it + wq);
    p.i = __builtin_amdgcn_readfirstlane(p.i);
    p.q = __builtin_amdgcn_readfirstlane(p.q);
    return p;
  };
  const uint32_t lane16 = (uint32_t)lane * 16u;
  v4i tab[KS1], uf[4][RM], consts;
  // Row 4 g + e of an item's table is point e of its group g, its constants those of that group's residue: lane l holds row l % 16 and results of group l / 16.
  auto load_table = [&](int it) {
    const Group p = group(4 * it + (col >> 2));
    const uint32_t pt = (uint32_t)(4 * p.q + (lane & 3));
    const uint32_t at = (((uint32_t)(p.i * CB1) + (pt >> 4)) * KS1) * 1024u + (pt & 15u) * 16u + (uint32_t)h * 256u;
#pragma unroll
    for (int s = 0; s < KS1; ++s) tab[s] = *(const v4i *)(P.KB + s * 1024 + at);
    consts = *(const v4i *)((const char *)P.more + (uint32_t)group(4 * it + h).i * (uint32_t)sizeof(Residue8));
  };
  const int sets = (P.nkb + RM * QUADS - 1) / (RM * QUADS);
  // Fragments of set `set` at the points of a group: uniform addresses plus the lane's.  (Were the lane's offset known to be the same for the whole
  // loop, the compiler would widen it in front of it and add 64-bit vectors for every load.)
  const uint32_t slab_bytes = (uint32_t)P.nkb * 1024u;
  struct Rows { const int8_t *first; uint32_t step; int last; };       // of U: first row block at the group's first point, to the next row block, last point's number
  auto rows_of = [&](const Group &p, int set) -> Rows {
    const int kb = min((set * QUADS + half) * RM, P.nkb - 1);             // past the last row block: that one again
    return {P.U + (size_t)(uint32_t)(p.i * P2 + 4 * p.q) * slab_bytes + (size_t)(uint32_t)kb * 1024u, kb + 1 < P.nkb ? 1024u : 0u, min(P2 - 1 - 4 * p.q, 3)};
  };
  auto load_u = [&](const Rows &rows, int e, uint32_t lane_at) {
    const int8_t *frag = rows.first + (size_t)((uint32_t)min(e, rows.last) * slab_bytes);
#pragma unroll
    for (int rm = 0; rm < RM; ++rm) {
      uf[e][rm] = *(const v4i *)(frag + lane_at);
      frag += rows.step;
    }
  };
  // Packed layers (16 tiles of four channels a block): row block kb holds filter kb in 16 slots, its fragment the same four bytes in the 16 places where a row's
  // slot is the channels'.  So lane l fetches those of filter k0 + l, and every fragment is made from a lane's word: row r has it in word r / 4 of
  // slice r % 4.
  const int filters = PACK ? (P.nkb + P.row_parts() - 1) / P.row_parts() : 0, k0 = PACK ? (which - part * P.row_parts()) * filters : 0;
  uint32_t words[4], diagonal[4];
  auto load_words = [&](const Group &p) {
    const int8_t *first = P.U + (size_t)(uint32_t)(p.i * P2 + 4 * p.q) * slab_bytes;
    const uint32_t lane_at = (uint32_t)min(k0 + lane, P.nkb - 1) * 1024u;
#pragma unroll
    for (int e = 0; e < 4; ++e) words[e] = *(const uint32_t *)(first + (size_t)((uint32_t)min(e, P2 - 1 - 4 * p.q) * slab_bytes) + lane_at);
  };
#pragma unroll
  for (int d = 0; d < 4; ++d) diagonal[d] = PACK && (col & 3) == h && (col >> 2) == d ? 0xFFFFFFFFu : 0u;
  Group at = mine(item);
  InputCopy<256 * QUADS> copy(nullptr, nullptr, {0, 0});
  {
    v4i va[ROWS], vb[ROWS];
    int ca, cb;
    request(0, va, ca);
    request(1, vb, cb);
    __builtin_amdgcn_sched_barrier(0);
    settle(0, va, ca);
    if constexpr (NU == 4) request(2, va, ca);
    __builtin_amdgcn_sched_barrier(0);
    settle(1, vb, cb);
    if constexpr (NU == 4) {
      request(3, vb, cb);
      __builtin_amdgcn_sched_barrier(0);
      settle(2, va, ca);
      __builtin_amdgcn_sched_barrier(0);
      settle(3, vb, cb);
    }
    copy = share((uint32_t)unit);
    if (copies) copy.end = 0;
    copy.request();
    __builtin_amdgcn_sched_barrier(0);                                 // (requested any earlier, these take more registers than there are: 0.5 us a call)
    load_table(item);
    if constexpr (PACK) load_words(at);
    else
#pragma unroll
      for (int e = 0; e < 4; ++e) load_u(rows_of(at, 0), e, lane16);
  }
  __syncthreads();                                                     // the staged pixels make room for V
  // Everything requested so far is awaited here: otherwise the compiler, merging this entry state with the loop's own, makes the loop's waits wait for its
  // stores.
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0), other counters untouched
  copy.store();
  copy.rest();

  const uint32_t krow = (uint32_t)(P.n() * Q) * (uint32_t)(P.ntb * 16) * 4u;             // bytes of a row of O, which is smaller than 4 GiB
  uint32_t lane_store[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) lane_store[j] = (uint32_t)(4 * h + j) * krow + (uint32_t)col * 4u;
  uint32_t buf = 0;
  for (; left > 0; --left) {
    {
      const float inv = __int_as_float(consts[0]), qb = __int_as_float(consts[1]);
      const int neg_p = consts[2];
      const v4i start = (v4i){consts[3], consts[3], consts[3], consts[3]};
      uint32_t out[4][NU];                                             // out[e]: the wave's 16 (or 8) channels of the point that table row 4 h + e is for
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        v4i acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          acc[j] = start;
#pragma unroll
          for (int s = 0; s < KS1; ++s) acc[j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(tab[s], pix[4 * u + j][s], acc[j], 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
        {
          uint32_t low[4];
          biased_lowbytes(low, acc[0][e], acc[1][e], acc[2][e], acc[3][e], inv, qb, neg_p);
          out[e][u] = pack_low_bytes(low[0], low[1], low[2], low[3]);
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint8_t *const to = lds + buf + ((4 * h + e) * TH + th) * 1024 + slice * 256 + col * 16 + u0 * 4;
        if constexpr (NU == 4) *(v4i *)to = (v4i){(int)out[e][0], (int)out[e][1], (int)out[e][NU - 2], (int)out[e][NU - 1]};
        else *(v2i *)to = (v2i){(int)out[e][0], (int)out[e][1]};
      }
    }
    const int following = after(item);
    load_table(following);                                             // (once more than there are items: fetched, not used)
    const Group next = mine(following);
    __syncthreads();
    const Residue8 r = residue(R.res[at.i]);
    const float inv = in_vgpr(r.inv), qb = in_vgpr(r.quot_bias);
    const v4i start = (v4i){r.acc_bias, r.acc_bias, r.acc_bias, r.acc_bias};
    const uint8_t *vfrag = lds + buf + (uint32_t)(4 * wq * TH * 1024) + lane16;
    if constexpr (PACK) {
      v4i vf[4][TH];
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int x = 0; x < TH; ++x) vf[e][x] = *(const v4i *)(vfrag + (e * TH + x) * 1024);
      uint32_t mine_now[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) mine_now[e] = words[e];
      load_words(next);
      const int kend = min(k0 + filters, P.nkb);
      char *row = (char *)P.O + (size_t)(uint32_t)((uint32_t)(at.i * Q + at.q) * (uint32_t)P.ntb * 64u) + (size_t)((uint32_t)((k0 + half) * 16) * krow);
      for (int k = k0 + half; k < kend; k += TH) {
        uint32_t word[TH][4], store_at[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          store_at[j] = lane_store[j];
          asm volatile("" : "+v"(store_at[j]));
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)mine_now[e], k - k0);
          const v4i frag = (v4i){(int)(w & diagonal[0]), (int)(w & diagonal[1]), (int)(w & diagonal[2]), (int)(w & diagonal[3])};
          const uint32_t sel = e == 1 ? 0x0c0c0400u : e == 2 ? 0x0c040100u : 0x04020100u;
#pragma unroll
          for (int x = 0; x < TH; ++x) {
            const v4i acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(frag, vf[e][x], start, 0, 0, 0);
            uint32_t low[4];
            biased_lowbytes(low, acc[0], acc[1], acc[2], acc[3], inv, qb, r.neg_p);
#pragma unroll
            for (int j = 0; j < 4; ++j) word[x][j] = e == 0 ? low[j] : __builtin_amdgcn_perm(low[j], word[x][j], sel);
          }
        }
#pragma unroll
        for (int x = 0; x < TH; ++x)
#pragma unroll
          for (int j = 0; j < 4; ++j) *(uint32_t *)(row + (uint32_t)min(tb0 + x, P.ntb - 1) * 64u + store_at[j]) = word[x][j];
        row += (size_t)(16 * TH * krow);
      }
    } else {
    int set = 0;
    do {
      const bool same = set + 1 < sets;
      const Rows rows = rows_of(same ? at : next, same ? set + 1 : 0);
      uint32_t lane_at = lane16, store_at[4];
      asm volatile("" : "+v"(lane_at));
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        store_at[j] = lane_store[j];
        asm volatile("" : "+v"(store_at[j]));
      }
      uint32_t word[RM][TH][4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v4i acc[RM][TH];
#pragma unroll
        for (int x = 0; x < TH; ++x) {
          const v4i v = *(const v4i *)(vfrag + (e * TH + x) * 1024);
#pragma unroll
          for (int rm = 0; rm < RM; ++rm) acc[rm][x] = __builtin_amdgcn_mfma_i32_16x16x64_i8(uf[e][rm], v, start, 0, 0, 0);
        }
        load_u(rows, e, lane_at);
        const uint32_t sel = e == 1 ? 0x0c0c0400u : e == 2 ? 0x0c040100u : 0x04020100u;
#pragma unroll
        for (int rm = 0; rm < RM; ++rm)
#pragma unroll
          for (int x = 0; x < TH; ++x) {
            uint32_t low[4];
            biased_lowbytes(low, acc[rm][x][0], acc[rm][x][1], acc[rm][x][2], acc[rm][x][3], inv, qb, r.neg_p);
#pragma unroll
            for (int j = 0; j < 4; ++j) word[rm][x][j] = e == 0 ? low[j] : __builtin_amdgcn_perm(low[j], word[rm][x][j], sel);
          }
      }
      const int kb = min((set * QUADS + half) * RM, P.nkb - 1);
      char *row = (char *)P.O + (size_t)(uint32_t)((uint32_t)(at.i * Q + at.q) * (uint32_t)P.ntb * 64u) + (size_t)((uint32_t)(kb * 16) * krow);
#pragma unroll
      for (int rm = 0; rm < RM; ++rm) {
#pragma unroll
        for (int x = 0; x < TH; ++x)
#pragma unroll
          for (int j = 0; j < 4; ++j) *(uint32_t *)(row + (uint32_t)min(tb0 + x, P.ntb - 1) * 64u + store_at[j]) = word[rm][x][j];
        row += kb + 1 < P.nkb ? (size_t)(16 * krow) : 0;
      }
    } while (++set < sets);
    }
    at = next;
    item = following;
    buf ^= VBUF;
  }
}

}  // namespace rnswino
