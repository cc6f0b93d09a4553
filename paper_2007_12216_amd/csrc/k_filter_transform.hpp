// K0: offline filter transform  U[i][xi,nu][k][c] = (G_p g G_p^T)[xi,nu] mod p_i   (paper section 6: the
// filter transform depends on the weights only and is computed ahead of time).
//
// G g G^T = (G kron G) vec(g): per residue one (t*t) x (r*r) matrix applied to the filters, on the matrix cores
// (v_mfma_i32_16x16x64_i8): A operand = the Kronecker table (rows = 16 transform points), B operand = filters (columns =
// 16 rows k of the padded GEMM grid at one channel), contraction = filter tap (r*r <= 49 of 64 slots; the products wasted
// on the empty slots cost a tenth of the stores' time).  Sixteen channels' accumulators give a lane 16 bytes of U for each
// of its four points, so a wave stores 256-byte runs.
// |sum| <= 49 * 126 * 128 < 2^20 (per byte plane < 2^20 with 16-bit moduli): the quotient estimate is off by less than
// 1/(2p), so the residue is the symmetric one, always.
//
// Block = (16 rows k, 64 channels, a run of (residue, 16-point block) items): its 1024 filters are gathered into LDS once
// (16-byte pieces, slot k ^ (c % 16) of channel c against bank conflicts), wave g computes slice g of the fragments.
// Padding rows and channels, and in packed layers the entries off the diagonal, are zeros: that is what lets the GEMM
// ignore them.  512 x 512, t = 10, four residues (105 MB): 26.5 us, 4.0 TB/s (31.7 with the filters read from LDS for every item and the sums
// converted to binary32; one thread per (residue, k, c) with 64-bit divisions and byte stores: 437).  What bounds it: the blocks are all
// resident at once, so that its parts follow each other: into eight buffers in turn (28.3 us) 18.6 without the stores, 24 without the residues, 27
// without the products, and 10 without residues and stores, launch, gather, table and products.  Two, three, five
// to fourteen blocks per compute unit instead of four take 35 to 40.
#pragma once
#include "kernels_common.hpp"

namespace rnswino {

template <bool WIDE, int PP>
__global__ __launch_bounds__(256, WIDE ? 2 : PP == 1 ? 4 : 3) void k0_filter_transform(KParams P, const int8_t *__restrict__ w, int8_t *__restrict__ U) {
  constexpr int PL = WIDE ? 2 : 1;
  extern __shared__ __attribute__((aligned(16))) v4i filt[];      // [16-tap piece][channel][16 rows]
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, h = lane >> 4, kcol = lane & 15;
  const int nkb = P.Kp >> 4, ncb = P.Cp >> 6;
  const int kb = blockIdx.x / ncb, cb = blockIdx.x - kb * ncb;
  const int rr = P.r * P.r, pieces = (rr + 15) >> 4;
  {
    const long long total = (long long)P.K * P.C * rr;
    for (int q = 0; q < pieces; ++q) {
      const int have = min(16, rr - 16 * q);
      // a thread's four pieces are requested together and only then masked and written
      v4i val[4];
      long long at[4];
      int state[4];                                               // 0: zeros, 1: plain 16-byte load, 2: end of the tensor
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int pair = threadIdx.x + 256 * e, cc = pair & 63, kk = pair >> 6;
        // GEMM row kg and channel cg; for packed layers (TL > 1) kg = k * TL + tl and cg = tl' * Cq + c, and the entry is
        // the filter's where the tile slots agree (tl = tl') and zero elsewhere
        const int kg = kb * 16 + kk, cg = cb * 64 + cc;
        const int k = P.TL > 1 ? kg / P.TL : kg, c = P.TL > 1 ? cg % P.Cq : cg;
        const bool live = k < P.K && c < P.C && (P.TL == 1 || (kg % P.TL) == (cg / P.Cq));
        at[e] = ((long long)k * P.C + c) * rr + 16 * q;
        state[e] = !live ? 0 : at[e] + 16 <= total ? 1 : 2;
        val[e] = (v4i){0, 0, 0, 0};
        if (state[e] == 1) __builtin_memcpy(&val[e], w + at[e], 16);          // one unaligned 16-byte load
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (state[e] == 2) {
          uint32_t wv[4] = {0, 0, 0, 0};
          for (int b = 0; b < have; ++b) wv[b >> 2] |= (uint32_t)(uint8_t)w[at[e] + b] << (8 * (b & 3));
          val[e] = (v4i){(int)wv[0], (int)wv[1], (int)wv[2], (int)wv[3]};
        }
      }
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const int keep = min(max(have - 4 * d, 0), 4);            // taps of this word; what follows is the next filter's
        const uint32_t mask = keep == 4 ? 0xFFFFFFFFu : (1u << (8 * keep)) - 1u;
#pragma unroll
        for (int e = 0; e < 4; ++e) val[e][d] &= mask;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int pair = threadIdx.x + 256 * e, cc = pair & 63, kk = pair >> 6;
        filt[q * 1024 + cc * 16 + (kk ^ (cc & 15))] = val[e];
      }
    }
  }
  __syncthreads();

  const int nitems = P.n * P.CB1;
  const int it0 = (int)((long long)nitems * blockIdx.y / gridDim.y), it1 = (int)((long long)nitems * (blockIdx.y + 1) / gridDim.y);
  const uint32_t lane_store = (uint32_t)((kcol + 16 * wave) * 16);
  // A filter fills PP = 1, 2 or 4 of the contraction's four 16-tap slices, so a fragment holds 4 / PP channels, slice h those of channel
  // h / PP, and the products of channel `sub` take the table in its slices and zeros in the others.  The filters are the same for
  // every item: the wave keeps its sixteen channels' fragments in registers.  (One channel a fragment, 172 registers: 28.1 us on 512 x 512
  // filters of four residues where this takes 26.5.)
  constexpr int CPF = 4 / PP;
  v4i kept[16 / CPF];
#pragma unroll
  for (int f = 0; f < 16 / CPF; ++f) {
    const int c = f * CPF + h / PP, piece = h % PP;
    const int cc = 16 * (c >> 2) + 4 * wave + (c & 3);            // channel order of layout.hpp
    kept[f] = (v4i){0, 0, 0, 0};
    if (piece < pieces) kept[f] = filt[piece * 1024 + cc * 16 + (kcol ^ (cc & 15))];
  }
  // An item's table fragment and its residue's constants are requested one item ahead.
  struct Item { int i, pb, p; float inv; double invd; v4i tab[PL]; };
  const uint32_t table_lane = (uint32_t)((lane & 15) + 16 * (h % PP)) * 16u;
  auto fetch = [&](int i, int pb) {
    Item q;
    q.i = i; q.pb = pb; q.p = P.p[i]; q.inv = P.inv_p[i]; q.invd = WIDE ? P.inv_pd[i] : 0.0;
#pragma unroll
    for (int pl = 0; pl < PL; ++pl) q.tab[pl] = *(const v4i *)(P.KG + ((size_t)(i * P.CB1 + pb) * PL + pl) * 1024 + table_lane);
    return q;
  };
  const float magic = in_vgpr(12582912.0f);
  Item next = fetch(it0 / P.CB1, it0 % P.CB1);
  for (int it = it0; it < it1; ++it) {
    const Item q = next;
    if (it + 1 < it1) next = q.pb + 1 < P.CB1 ? fetch(q.i, q.pb + 1) : fetch(q.i + 1, 0);
    const int p = q.p;
    const float inv = in_vgpr(q.inv);
    const int a0 = WIDE ? 0 : 0x4B400000;                         // 8-bit moduli: centred_lowbyte()
    const v4i start = (v4i){a0, a0, a0, a0};
    v4i tab[PL][CPF];
#pragma unroll
    for (int pl = 0; pl < PL; ++pl)
#pragma unroll
      for (int sub = 0; sub < CPF; ++sub)
#pragma unroll
        for (int d = 0; d < 4; ++d) tab[pl][sub][d] = h / PP == sub ? q.tab[pl][d] : 0;
    v4i out[PL][4];                                               // [plane][point]: 16 channels of slice `wave`
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      v4i acc[PL][4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int pl = 0; pl < PL; ++pl)
          acc[pl][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(tab[pl][(4 * u + j) % CPF], kept[(4 * u + j) / CPF], start, 0, 0, 0);
#pragma unroll
      for (int e = 0; e < 4; ++e) {                               // point 16 pb + 4 h + e
        if constexpr (WIDE) {
          uint32_t wh = 0, wl = 0;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int tot = acc[0][j][e] * 256 + acc[PL - 1][j][e];           // |tot| <= 49 * 128 * 32896 < 2^28
            const int v = storable16(mod_near32(tot, q.invd, p), p);
            const int lo = (int)(int8_t)(v & 0xFF), hi = (v - lo) >> 8;
            wh |= ((uint32_t)hi & 0xFFu) << (8 * j);
            wl |= ((uint32_t)lo & 0xFFu) << (8 * j);
          }
          out[0][e][u] = (int)wh;
          out[PL - 1][e][u] = (int)wl;
        } else {
          out[0][e][u] = (int)pack_low_bytes(centred_lowbyte(acc[0][0][e], magic, inv, -p), centred_lowbyte(acc[0][1][e], magic, inv, -p),
                                             centred_lowbyte(acc[0][2][e], magic, inv, -p), centred_lowbyte(acc[0][3][e], magic, inv, -p));
        }
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int pt = 16 * q.pb + 4 * h + e;
      if (pt < P.P2) {
        int8_t *dst = U + (((size_t)(q.i * P.P2 + pt) * nkb + kb) * ncb + cb) * (PL * 1024) + lane_store;
#pragma unroll
        for (int pl = 0; pl < PL; ++pl) __builtin_memcpy(dst + pl * 1024, &out[pl][e], 16);      // U may have any alignment here
      }
    }
  }
}

}  // namespace rnswino
