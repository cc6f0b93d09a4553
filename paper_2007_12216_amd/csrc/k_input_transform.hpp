// K1: input transform on the matrix cores.
//
// V[i][xi,nu][tau][c] = (B^T_p d B_p)[xi,nu] mod p_i for every tile tau and channel c (paper section 6: shared
// by all K filters).  B^T d B = (B^T kron B^T) vec(d): per residue one dense (t*t) x (t*t) matrix applied to the
// t*t pixels of a tile, i.e. a GEMM whose columns are the (tile, channel) pairs.  MFMA roles
// (v_mfma_i32_16x16x64_i8): A operand = pixels (rows = 16 channels of one tile), B operand = the Kronecker
// table (columns = 16 transform points), contraction index = pixel.  A tile row takes RP1 = 4 ceil(t/4)
// contraction slots (its t pixels, then zero weights), the tile t * RP1 slots in KS1 = ceil(t * RP1 / 64) steps of
// 64 (t = 10: 120 slots, two steps; rows of 16 slots would need three).  A row segment is one unaligned 16-byte
// load of an image row, masked where the tile hangs over the image border (zero padding and ragged last tiles),
// of which the first RP1 bytes go to LDS; a lane's 16 operand bytes are then 16 consecutive slots.
//
// Block = (tile, block of 64 channels, one residue or all of them): its 64 x t x RP1 pixel patch is gathered once into
// LDS (the gather of 16-byte row segments is what costs; sharing it between the four waves pays), then each wave
// walks over its steps (residue, group of K1_CPW column blocks: every fourth, every eighth where two blocks share them), the table fragments of the next
// step in flight while the current one is multiplied.  Accumulator rows are channels 4g+j, so the four channel
// groups u give one lane exactly the 16 bytes of V it has to store (channel order of layout.hpp).
// 16-bit moduli: the table has a high and a low byte plane, V = (256 * sum_h + sum_l) mod p, stored as two planes.
// Grid: x = T * Cp/64 rounded up to a multiple of 8 (see kernels_common.hpp), y = n (one residue per block) or 1 (the block
// walks over all residues with the same gathered patch), z = 1 or 2 (blocks that share a residue's column blocks); 256 threads; 64 * (4*KS1 + 1) * 16 bytes of LDS.
#pragma once
#include "kernels_common.hpp"

namespace rnswino {

constexpr int K1_CPW = 2;

// The kernels' arguments, fetched together at entry: scattered over the layer's full parameter block, they took three dependent fetches
// of the launch's argument memory (about 500 cycles each) before the first pixel was asked for, and the divisions as many
// again.  256 channels at 56 x 56 (800 blocks): 2000 cycles from entry to the last load, now 900; whole layer 23.4 -> 22.1 us,
// 5 x 5 128 channels at 28 x 28 18.8 -> 17.1, 100 channels at 57 x 43 20.0 -> 18.3, VGG16 stack at batch 1 397 -> 379.
struct K1Args {
  const ResidueParams *more;
  const int8_t *x;
  int8_t *V;
  const int8_t *KB;           // (B^T kron B^T) mod p, [n][CB1][KS1][planes][64 lanes][16]
  int units, per_xcd;         // T * Cp/64 (of the packed problem), and the grid's x extent / 8
  int ncb;                    // channel blocks of 64
  uint32_t ncb_mul, tw_mul, th_mul;          // FastDiv's, with the shifts below
  int C, H, W, pad, tw, th, T, Tg;
  long long total;            // N * C * H * W
  uint32_t shifts;            // bytes: of the divisions by ncb, tw, th; log2 of a tile's channel slots
  uint32_t sizes;             // bytes: m, t, n, split
  RNSW_HD FastDiv by_ncb() const { return {ncb_mul, shifts & 31u}; }
  RNSW_HD FastDiv by_tw() const { return {tw_mul, shifts >> 8 & 31u}; }
  RNSW_HD FastDiv by_th() const { return {th_mul, shifts >> 16 & 31u}; }
  RNSW_HD int cq_shift() const { return (int)(shifts >> 24); }
  RNSW_HD int m() const { return (int)byte_of(sizes, 0); }
  RNSW_HD int t() const { return (int)byte_of(sizes, 1); }
  RNSW_HD int n() const { return (int)byte_of(sizes, 2); }
  // 0: a block takes all residues; else it takes one (blockIdx.y), and `split` blocks share its column blocks (blockIdx.z)
  RNSW_HD int split() const { return (int)(sizes >> 24); }
};
static_assert(sizeof(K1Args) <= 112, "kernels_common.hpp");
#define RNSW_K1_FETCH_ARGUMENTS(P)                                                                                                       \
  asm volatile("" ::"s"(P.x), "s"(P.V), "s"(P.KB), "s"(P.units), "s"(P.per_xcd), "s"(P.ncb), "s"(P.ncb_mul), "s"(P.tw_mul), "s"(P.th_mul), "s"(P.C), \
               "s"(P.H), "s"(P.W), "s"(P.pad), "s"(P.tw), "s"(P.th), "s"(P.total), "s"(P.shifts), "s"(P.sizes))

// PACK: the layer packs TL tiles into one 64-channel block (plan.hpp): block channel c' holds channel c' % Cq of tile
// (c' / Cq) * Tg + tau, so every gathered row segment has its own tile origin; everything after the gather is the same.
template <int KS1, bool WIDE, bool PACK>
__global__ __launch_bounds__(256) void k1_input_transform(K1Args P) {
  Constant<ResidueParams> &R = constant(P.more);
  constexpr int ROWS = KS1 == 1 ? 8 : KS1 == 2 ? 10 : KS1 == 3 ? 12 : 16;   // largest t with this many steps
  constexpr int PL = WIDE ? 2 : 1;
  constexpr int CROW = (4 * KS1 + 1) * 16;   // bytes per channel in LDS: one 16-byte pad, so that the 16 channels a
                                             // fragment read touches fall into different banks
  __shared__ __attribute__((aligned(16))) uint8_t xs[64 * CROW];
  RNSW_K1_FETCH_ARGUMENTS(P);
  const int t = P.t(), P2 = t * t, CB1 = (P2 + 15) >> 4, HW = P.H * P.W;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: table addresses stay scalar
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int ncb = P.ncb;
  const int i0 = P.split() ? blockIdx.y : 0, i1 = P.split() ? i0 + 1 : P.n();   // residues of this block
  // neighbouring tiles (shared image lines) on one XCD, see kernels_common.hpp
  const int unit = (int)(blockIdx.x & 7) * P.per_xcd + (int)(blockIdx.x >> 3);
  if (unit >= P.units) return;
  const int tau = (int)fast_div((uint32_t)unit, P.by_ncb()), cb = unit - tau * ncb;   // tau: GEMM column (a group of TL tiles when PACK)
  // first image row and column of a tile and the byte index of (channel ch, that row, that column)
  struct Origin { long long base; int y0, x0; };
  auto tile_origin = [&](int tile, int ch) -> Origin {
    const int trow = (int)fast_div((uint32_t)tile, P.by_tw()), tx = tile - trow * P.tw;
    const int img = (int)fast_div((uint32_t)trow, P.by_th()), ty = trow - img * P.th;
    Origin o;
    o.y0 = ty * P.m() - P.pad;
    o.x0 = tx * P.m() - P.pad;
    o.base = ((long long)img * P.C + ch) * HW + (long long)o.y0 * P.W + o.x0;
    return o;
  };
  // A thread's NT row segments are requested together and only then masked and written to LDS (one after the
  // other, each load would be waited for in turn: three memory latencies instead of one).  A segment that sticks out of the
  // tensor is loaded from the nearest 16 bytes inside and moved into place (byte by byte, the few blocks it happens in took
  // half as long again as all others, and the next kernel waits for them).
  constexpr int NT = (64 * ROWS + 255) / 256;
  const bool tiny = P.total < 16;                    // the tensor itself is smaller than a load
  v4i val[NT];
  bool there[NT];
  int moved[NT];                                     // how far the load was moved, in bytes
  unsigned long long mask0[PACK ? NT : 1], mask1[PACK ? NT : 1];   // columns inside the image and inside the tile
  if constexpr (PACK) {
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const int task = threadIdx.x + 256 * k;
      const int cblk = task / ROWS, a = task - cblk * ROWS;
      const int ch = cblk & ((1 << P.cq_shift()) - 1), tile = (cblk >> P.cq_shift()) * P.Tg + tau;
      const Origin o = tile_origin(min(tile, P.T - 1), ch);
      const int gy = o.y0 + a;
      const long long from = o.base + (long long)a * P.W, at = segment_at(from, P.total);
      moved[k] = (int)(from - at);                   // rows inside the image: their segments overlap the tensor or are masked
      there[k] = task < 64 * ROWS && tile < P.T && ch < P.C && a < t && gy >= 0 && gy < P.H;
      val[k] = (v4i){0, 0, 0, 0};
      if (there[k] && !tiny) __builtin_memcpy(&val[k], P.x + at, 16);       // one unaligned 16-byte load
      mask0[k] = byte_range(max(-o.x0, 0), min(t, P.W - o.x0), 0);
      mask1[k] = byte_range(max(-o.x0, 0), min(t, P.W - o.x0), 8);
    }
  } else {
    const Origin o = tile_origin(tau, cb * 64);
    // offsets from the origin that a load may start at (rows outside the image are excluded separately)
    const SegmentRange inside = segment_range(o.base, P.total);
    const bool columns = o.x0 < P.W && o.x0 + t > 0;                                 // (wide padding: perhaps none)
    const int a_lo = max(-o.y0, 0), a_count = columns ? max(min(t, P.H - o.y0) - a_lo, 0) : 0;     // rows inside the image
    const int chans = P.C - cb * 64;
    const int8_t *xb = P.x + (o.base - 16);
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const int task = threadIdx.x + 256 * k;
      const int cblk = task / ROWS, a = task - cblk * ROWS;
      const int from = cblk * HW + a * P.W, at = segment_at(from, inside);   // 64 * H * W stays far below 2^31
      moved[k] = tiny ? (int)o.base + from : from - at;
      there[k] = (256 * (k + 1) <= 64 * ROWS || task < 64 * ROWS) && cblk < chans && (uint32_t)(a - a_lo) < (uint32_t)a_count;
      val[k] = (v4i){0, 0, 0, 0};
      if (there[k] && !tiny) __builtin_memcpy(&val[k], xb + (uint32_t)(at + 16), 16);   // one unaligned 16-byte load
    }
    mask0[0] = byte_range(max(-o.x0, 0), min(t, P.W - o.x0), 0);
    mask1[0] = byte_range(max(-o.x0, 0), min(t, P.W - o.x0), 8);
  }
  // This wave's work: steps (residue i, column-block group cg) with cg = first, first + stride, ...  The table fragments
  // of step k+1 are requested before step k is multiplied; those of step 0 behind the gather's own loads, so that their
  // latency overlaps the gather.  A step's position is kept as wave-uniform scalars and advanced incrementally
  // (no divisions, and only a few scalar operations per column block: every instruction counts here).
  const int ncg = (CB1 + K1_CPW - 1) / K1_CPW;
  const int part_shift = P.split() >> 1;                // log2 of the blocks that share a residue: one or two
  const int first = wave + 4 * (int)blockIdx.z, stride = 4 << part_shift;
  const int per_i = max(ncg - first + stride - 1, 0) >> (2 + part_shift);              // groups of this wave per residue
  const int nsteps = (i1 - i0) * per_i;
  struct Pos { int i, cg; };                          // residue and column-block group
  auto advance = [&](Pos &q) {
    q.cg += stride;
    if (q.cg >= ncg) { q.cg = first; ++q.i; }
  };
  constexpr uint32_t FRAG = KS1 * PL * 1024;          // table bytes per column block (all steps and planes)
  const int8_t *KBl = P.KB + lane * 16;
  auto load_table = [&](const Pos &q, v4i (&b)[K1_CPW][KS1][PL]) {
#pragma unroll
    for (int cc = 0; cc < K1_CPW; ++cc) {
      const int cbk = min(q.cg * K1_CPW + cc, CB1 - 1);
      const int8_t *frag = KBl + (uint32_t)(q.i * CB1 + cbk) * FRAG;   // the whole table is far below 4 GiB
#pragma unroll
      for (int s = 0; s < KS1; ++s)
#pragma unroll
        for (int pl = 0; pl < PL; ++pl) b[cc][s][pl] = *(const v4i *)(frag + (s * PL + pl) * 1024);
    }
  };
  // Where a column block's 16 transform points go in V: wave-uniform 64-bit part (tile block, residue, column block,
  // channel block, tile) + the lane's 32-bit part (its point within the column block, its four channels), so the
  // address costs the vector unit next to nothing.  stride_pt = bytes between consecutive transform points.
  const uint32_t stride_pt = (uint32_t)(ncb * PL * 1024);
  const uint32_t lane_store = (uint32_t)(lane & 15) * stride_pt + g * 16;   // 16 points * ncb KiB: far below 2^32
  int8_t *const Vtile = P.V + ((size_t)(tau >> 4) * (size_t)(P.n() * P2) * ncb + cb) * (PL * 1024) + (tau & 15) * 64;
  v4i bf[K1_CPW][KS1][PL], bn[K1_CPW][KS1][PL];
  Pos cur = {i0, first};
  if (nsteps > 0) load_table(cur, bf);
  __builtin_amdgcn_sched_barrier(0);
  Residue8 rf = residue(R.res[i0]), rn = rf;          // constants of the first step's residue: fetched behind the loads, not in front of them
  if (tiny) {
#pragma unroll
    for (int k = 0; k < NT; ++k)
      if (there[k]) {
        uint32_t wv[4] = {0, 0, 0, 0};
        for (int b = 0; b < (int)P.total; ++b) wv[b >> 2] |= (uint32_t)(uint8_t)P.x[b] << (8 * (b & 3));
        val[k] = (v4i){(int)wv[0], (int)wv[1], (int)wv[2], (int)wv[3]};
      }
  }
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    if (there[k] && moved[k] != 0) {
      unsigned long long w0 = (uint32_t)val[k][0] | (unsigned long long)(uint32_t)val[k][1] << 32;
      unsigned long long w1 = (uint32_t)val[k][2] | (unsigned long long)(uint32_t)val[k][3] << 32;
      move_segment(moved[k], w0, w1);
      val[k] = (v4i){(int)(uint32_t)w0, (int)(uint32_t)(w0 >> 32), (int)(uint32_t)w1, (int)(uint32_t)(w1 >> 32)};
    }
  }
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    const int task = threadIdx.x + 256 * k;
    const int cblk = task / ROWS, a = task - cblk * ROWS;
    const unsigned long long m0 = mask0[PACK ? k : 0], m1 = mask1[PACK ? k : 0];
    val[k][0] &= (int)(uint32_t)m0; val[k][1] &= (int)(uint32_t)(m0 >> 32);
    val[k][2] &= (int)(uint32_t)m1; val[k][3] &= (int)(uint32_t)(m1 >> 32);
    // the first RP1 bytes of the segment are the row's slots (the slots past t * RP1 are never written: their
    // table entries are zero, and any byte times zero is zero); RP1 is 4 or 8, 12, 12, 16 for KS1 = 1, 2, 3, 4
    if (task < 64 * ROWS && a < t) {
      const int rp = KS1 == 1 ? ((t + 3) & ~3) : KS1 == 4 ? 16 : 12;
      uint32_t *row = (uint32_t *)(xs + cblk * CROW + a * rp);
      row[0] = (uint32_t)val[k][0];
      if (rp > 4) row[1] = (uint32_t)val[k][1];
      if (rp > 8) row[2] = (uint32_t)val[k][2];
      if (rp > 12) row[3] = (uint32_t)val[k][3];
    }
  }
  __syncthreads();
  if (nsteps <= 0) return;
  // All loads issued so far are awaited here, explicitly: otherwise the compiler, merging this entry state with the
  // loop's own, makes every step wait for the fragments it has just requested for the next one.
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0), other counters untouched

  v4i af[4][KS1];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int s = 0; s < KS1; ++s) af[u][s] = *(const v4i *)(xs + (16 * u + (lane & 15)) * CROW + (4 * s + g) * 16);   // slots 64 s + 16 g ..

  // One step with the fragments in `b`, while those of the following step travel into `bnext`.  The loop below
  // alternates the two register sets instead of copying one into the other: a copy would have to wait for every
  // memory operation issued before it, the step's own stores included.
  auto do_step = [&](int step, v4i (&b)[K1_CPW][KS1][PL], v4i (&bnext)[K1_CPW][KS1][PL], const Residue8 &rc, Residue8 &rnext) {
    const int i = cur.i, cg = cur.cg;
    advance(cur);
    if (step + 1 < nsteps) { load_table(cur, bnext); rnext = residue(R.res[cur.i]); }
    const int p = -rc.neg_p;
    const float inv = in_vgpr(rc.inv), qb = in_vgpr(rc.quot_bias);
    const double invd = WIDE ? R.inv_pd[i] : 0.0;
    const int a0 = WIDE ? 0 : rc.acc_bias;           // see biased_lowbyte()
    const v4i start = (v4i){a0, a0, a0, a0};
#pragma unroll
    for (int cc = 0; cc < K1_CPW; ++cc) {
      const int cbk = cg * K1_CPW + cc;
      if (cbk >= CB1) break;
      v4i acc[PL][4];
#pragma unroll
      for (int pl = 0; pl < PL; ++pl)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[pl][u] = start;
#pragma unroll
      for (int s = 0; s < KS1; ++s)
#pragma unroll
        for (int pl = 0; pl < PL; ++pl)
#pragma unroll
          for (int u = 0; u < 4; ++u)
            acc[pl][u] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[u][s], b[cc][s][pl], acc[pl][u], 0, 0, 0);
      const int pt = 16 * cbk + (lane & 15);
      int8_t *dst = Vtile + (size_t)(uint32_t)(i * P2 + 16 * cbk) * stride_pt + lane_store;
      if (WIDE) {
        // per plane |acc| <= t*t * 128 * 128 = 2^22, so 256 * acc_h + acc_l fits 32 bits
        v4i out_h, out_l;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          uint32_t wh = 0, wl = 0;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int tot = acc[0][u][j] * 256 + acc[PL - 1][u][j];
            const int v = storable16(mod_near32(tot, invd, p), p);
            const int lo = (int)(int8_t)(v & 0xFF), hi = (v - lo) >> 8;
            wh |= ((uint32_t)hi & 0xFFu) << (8 * j);
            wl |= ((uint32_t)lo & 0xFFu) << (8 * j);
          }
          out_h[u] = (int)wh;
          out_l[u] = (int)wl;
        }
        if (pt < P2) {
          *(v4i *)dst = out_h;
          *(v4i *)(dst + 1024) = out_l;
        }
      } else {
        // |sum| <= t*t * (p - 1)/2 * 128 <= 256 * 125 * 128 (moduli above 251 exclude t > 13), and |a| < 2^15: below 2^22
        v4i out;
#pragma unroll
        for (int u = 0; u < 4; ++u)
          out[u] = (int)pack_low_bytes(biased_lowbyte(acc[0][u][0], inv, qb, -p), biased_lowbyte(acc[0][u][1], inv, qb, -p),
                                       biased_lowbyte(acc[0][u][2], inv, qb, -p), biased_lowbyte(acc[0][u][3], inv, qb, -p));
        if (pt < P2) *(v4i *)dst = out;
      }
    }
  };
  for (int step = 0; step < nsteps; step += 2) {
    do_step(step, bf, bn, rf, rn);
    if (step + 1 < nsteps) do_step(step + 1, bn, bf, rn, rf);
  }
}

// The same transform for layers with many tiles (8-bit moduli, t <= 10, a tensor below 2 GiB), with the roles exchanged: A operand
// = table (rows = 16 transform points), B operand = pixels (columns = 16 tiles at one channel).  Sixteen channels' accumulators
// give a lane 16 bytes of V for each of four points, and V lies in lane order ([slice g][tile % 16][16 B], Dims::vlane), so a
// wave stores 256-byte runs instead of 64-byte ones, and the sixteen neighbouring tiles' row segments, 8 bytes apart, are
// gathered by neighbouring lanes.  What bounds the kernel above on large layers is the memory pipeline's work per store and
// gather, not the bytes: 64 channels at 112 x 112, batch 8 (40 MB of V) took 20.3 us, 13.8 without its stores, 16.6 with every
// gather from one line, 20.2 without its matrix instructions.  This one: 17.0; at 224 x 224 85 -> 53 us (cold input).
// Block = (16 tiles, slice g of a 64-channel block: 16 channels), all residues or one; thread (channel, tile) gathers its t row
// segments into operand fragments, then the waves take the (residue, 16-point block) items in turn, every item's pixels from LDS in lane
// order, its table fragments requested one item ahead.  (With one padded row per thread instead of fragments, half of the LDS cycles
// were bank conflicts; a gather of unaligned loads, each with a branch of its own, took 4100 cycles of a block's 30000: 100 channels
// at 57 x 43, batch 3, 14.9 -> 14.2 us a layer.)
// Of 44.6 us on 64 -> 64 at 224 x 224, batch 8, there are left: without stores 38.1, residues 40.5, products 37.4, stores and gather 37.8, all but
// products and table 28.9, so nothing alone holds it.  Two items a step against the same pixels, half the LDS reads, take 160 registers: 16.7 against 17.1 us
// with 392 blocks, 48 against 44.6 with 1568.
// Grid: x = 4 * Tp/16 * Cp/64 rounded up to a multiple of 8 (kernels_common.hpp), y = n or 1.
template <int KS1, bool PACK>
__global__ __launch_bounds__(256, 4) void k1_input_transform_tiles(K1Args P) {
  Constant<ResidueParams> &R = constant(P.more);
  constexpr int ROWS = KS1 == 1 ? 8 : 10;
  __shared__ __attribute__((aligned(16))) uint8_t xs[16 * KS1 * 1024];     // fragments [channel][step][slice h][tile][16 slots]
  RNSW_K1_FETCH_ARGUMENTS(P);                      // (the residues' constants are fetched with their items)
  const int t = P.t(), P2 = t * t, CB1 = (P2 + 15) >> 4, HW = P.H * P.W;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, h = lane >> 4;
  const int unit = (int)(blockIdx.x & 7) * P.per_xcd + (int)(blockIdx.x >> 3);
  if (unit >= P.units) return;
  const int g = unit & 3, tb = (int)fast_div((uint32_t)unit >> 2, P.by_ncb()), cb = (unit >> 2) - tb * P.ncb;
  const int i0 = P.split() ? blockIdx.y : 0, nres = P.split() ? 1 : P.n();
  // gather: this thread's tile and channel
  const int col = threadIdx.x & 15, ch16 = threadIdx.x >> 4;
  const int cblk = 16 * (ch16 >> 2) + 4 * g + (ch16 & 3);              // channel order of layout.hpp
  const int tau = tb * 16 + col;
  const int tile = PACK ? (cblk >> P.cq_shift()) * P.Tg + tau : tau, ch = PACK ? (cblk & ((1 << P.cq_shift()) - 1)) : cb * 64 + cblk;
  const bool live = tau < P.Tg && tile < P.T && ch < P.C;
  const int tc = live ? tile : 0;
  const int trow = (int)fast_div((uint32_t)tc, P.by_tw()), tx = tc - trow * P.tw;
  const int img = (int)fast_div((uint32_t)trow, P.by_th()), ty = trow - img * P.th;
  const int y0 = ty * P.m() - P.pad, x0 = tx * P.m() - P.pad;
  const int plane = (img * P.C + (live ? ch : 0)) * HW;              // below 2^31, as the whole tensor
  // Row segments as offsets from the multiple of four at or before the tensor's start; rows outside the image repeat its first or last
  // row and are masked.  Only what the tensor holds is loaded: where clamping moves a load, the segment is put right below.
  const int mis = (int)((uint32_t)(uintptr_t)P.x & 3u), last = (int)P.total - 16 + mis;     // (the tensor has 16 bytes and more)
  const int8_t *const xa = P.x - mis;
  const int from = plane + x0 + mis;
  v4i val[ROWS];
  int clamped = 0;
  if (live) {
#pragma unroll
    for (int a = 0; a < ROWS; ++a) {
      const int want = from + min(max(y0 + a, 0), P.H - 1) * P.W, at = aligned_segment_at(want, mis, last);
      clamped |= at ^ (want & ~3);
      __builtin_memcpy(&val[a], xa + (uint32_t)at, 16);                // one 16-byte load
    }
  } else {
#pragma unroll
    for (int a = 0; a < ROWS; ++a) val[a] = (v4i){0, 0, 0, 0};
  }
  // Items of this wave, wave, wave + 4, ...: full 16-point blocks of all residues first (their stores need no test, so that the wait for
  // the next item's table does not become a wait for them), then the residues' last, partial blocks.  Item n is block n % nfull of residue
  // n / nfull, by a multiplication that is exact up to n = 4096.  The residue is wave-uniform for the compiler too: counted up in a loop, it took
  // it for a lane's own and fetched its constants by vector loads, which waited for the stores before them (64 -> 64 at 224 x 224,
  // batch 8: 44.6 us, so 42.9; 256 channels at 56 x 56, batch 8: 20.0 and 18.4; 64 -> 128 at 112 x 112, pooled, 66.5 and 64.2 a layer).  The rest is
  // not: the division here runs on the vector unit, in front of the first table load, and with it the number of items, the loop's condition and
  // the addresses of an item's table and output.
  const int nfull = P2 >> 4, nitems = nfull * nres;
  const uint32_t per_block = __builtin_amdgcn_readfirstlane(nfull > 0 ? (65535u + (uint32_t)nfull) / (uint32_t)nfull : 0);
  constexpr uint32_t FRAG = KS1 * 1024;
  const uint32_t lane16 = (uint32_t)lane * 16u;
  auto residue_of = [&](int n) { return (int)(((uint32_t)n * per_block) >> 16); };
  auto load_table = [&](int i, int cbk, v4i (&b)[KS1]) {
    const int8_t *frag = P.KB + (size_t)((uint32_t)(i * CB1 + cbk) * FRAG);
#pragma unroll
    for (int s = 0; s < KS1; ++s) b[s] = *(const v4i *)(frag + s * 1024 + lane16);
  };
  auto load_item = [&](int n, v4i (&b)[KS1]) {
    const int m = min(n, max(nitems - 1, 0)), k = residue_of(m);       // past the end: fetched, not used
    load_table(i0 + k, m - k * nfull, b);
  };
  v4i ta[KS1], tn[KS1];
  int item = wave;
  load_item(item, ta);
  const unsigned long long m0 = byte_range(max(-x0, 0), min(t, P.W - x0), 0), m1 = byte_range(max(-x0, 0), min(t, P.W - x0), 8);
  const uint32_t mask[3] = {live ? (uint32_t)m0 : 0u, live ? (uint32_t)(m0 >> 32) : 0u, live ? (uint32_t)m1 : 0u};
  const int rows_in = min(t, P.H - y0);                              // row a is inside the image and the tile: -y0 <= a < rows_in
  __builtin_amdgcn_sched_barrier(0);
  constexpr int WPR = KS1 == 1 ? 2 : 3;                                // words of a row
  uint32_t slots[16 * KS1];
#pragma unroll
  for (int d = 0; d < 16 * KS1; ++d) slots[d] = 0;
  if (__builtin_expect(__any(clamped != 0), 0)) {
#pragma unroll
    for (int a = 0; a < ROWS; ++a) {
      const int want = from + min(max(y0 + a, 0), P.H - 1) * P.W, at = aligned_segment_at(want, mis, last);
      unsigned long long w0 = (uint32_t)val[a][0] | (unsigned long long)(uint32_t)val[a][1] << 32;
      unsigned long long w1 = (uint32_t)val[a][2] | (unsigned long long)(uint32_t)val[a][3] << 32;
      move_segment(want - at, w0, w1);
      slots[a * WPR] = (uint32_t)w0; slots[a * WPR + 1] = (uint32_t)(w0 >> 32);
      if (WPR > 2) slots[a * WPR + 2] = (uint32_t)w1;
    }
  } else {
#pragma unroll
    for (int a = 0; a < ROWS; ++a) {
      const uint32_t by = (uint32_t)(from + min(max(y0 + a, 0), P.H - 1) * P.W);           // its low two bits count
#pragma unroll
      for (int d = 0; d < WPR; ++d) slots[a * WPR + d] = __builtin_amdgcn_alignbyte((uint32_t)val[a][d + 1], (uint32_t)val[a][d], by);
    }
  }
#pragma unroll
  for (int a = 0; a < ROWS; ++a) {
    const bool in = a >= -y0 && a < rows_in;
#pragma unroll
    for (int d = 0; d < WPR; ++d) slots[a * WPR + d] &= in ? mask[d] : 0u;
  }
  if (KS1 == 1 && ((t + 3) & ~3) == 4) {                                        // uniform: rows of one word
#pragma unroll
    for (int a = 0; a < ROWS; ++a) slots[a] = slots[2 * a];
  }
  uint8_t *const mine = xs + ch16 * (KS1 * 1024) + col * 16;
#pragma unroll
  for (int q = 0; q < 4 * KS1; ++q)
    *(v4i *)(mine + q * 256) = (v4i){(int)slots[4 * q], (int)slots[4 * q + 1], (int)slots[4 * q + 2], (int)slots[4 * q + 3]};
  __syncthreads();

  const uint8_t *px = xs + lane * 16;
  int8_t *const Vb = P.V + ((size_t)tb * (size_t)(P.n() * P2) * P.ncb + cb) * 1024 + g * 256;
  const uint32_t stride_pt = (uint32_t)P.ncb * 1024u;
  const uint32_t lane_store = (uint32_t)(4 * h) * stride_pt + (uint32_t)(lane & 15) * 16u;
  // out[e]: 16 channels of point 16 cbk + 4 h + e
  auto compute = [&](const v4i (&tab)[KS1], const Residue8 &r, v4i (&out)[4]) {
    const float inv = in_vgpr(r.inv), qb = in_vgpr(r.quot_bias);
    const v4i start = (v4i){r.acc_bias, r.acc_bias, r.acc_bias, r.acc_bias};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      v4i acc[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        acc[j] = start;
#pragma unroll
        for (int s = 0; s < KS1; ++s)
          acc[j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(tab[s], *(const v4i *)(px + ((4 * u + j) * KS1 + s) * 1024), acc[j], 0, 0, 0);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        out[e][u] = (int)pack_low_bytes(biased_lowbyte(acc[0][e], inv, qb, r.neg_p), biased_lowbyte(acc[1][e], inv, qb, r.neg_p),
                                        biased_lowbyte(acc[2][e], inv, qb, r.neg_p), biased_lowbyte(acc[3][e], inv, qb, r.neg_p));
    }
  };
  auto full_item = [&](v4i (&tab)[KS1], v4i (&next)[KS1]) {
    const int k = __builtin_amdgcn_readfirstlane(residue_of(item));
    const Residue8 r = residue(R.res[i0 + k]);
    int8_t *dst = Vb + (size_t)(uint32_t)((i0 + k) * P2 + 16 * (item - k * nfull)) * stride_pt + lane_store;
    item += 4;
    load_item(item, next);
    v4i out[4];
    compute(tab, r, out);
#pragma unroll
    for (int e = 0; e < 4; ++e) *(v4i *)(dst + (uint32_t)e * stride_pt) = out[e];
  };
  // The first table is awaited here: otherwise the compiler, merging this entry state with the loop's own, makes every other item wait
  // for the stores of the one before.
  __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0), other counters untouched
  while (item < nitems) {
    full_item(ta, tn);
    if (item >= nitems) break;
    full_item(tn, ta);
  }
  if (P2 & 15) {
    for (int pi = i0 + wave; pi < i0 + nres; pi += 4) {
      v4i tab[KS1], out[4];
      load_table(pi, nfull, tab);
      const Residue8 r = residue(R.res[pi]);
      compute(tab, r, out);
      int8_t *dst = Vb + (size_t)(uint32_t)(pi * P2 + 16 * nfull) * stride_pt + lane_store;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (16 * nfull + 4 * h + e < P2) *(v4i *)(dst + (uint32_t)e * stride_pt) = out[e];
    }
  }
}

}  // namespace rnswino
