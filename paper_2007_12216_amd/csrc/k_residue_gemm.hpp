// K2: the residue-domain GEMM  O[i][xi,nu][k][tau] = (sum_c U[i][xi,nu][k][c] V[i][xi,nu][tau][c]) mod p_i,
// one GEMM per transform point and residue, the modulo taken after the sum over C (paper section 6, eq. "gemm").
// int8 operands on v_mfma_i32_16x16x64_i8, int32 accumulation.
//
// Block = 4 waves = the 4 transform points of one group q (they end up as the 4 bytes of one O word); every
// wave computes a 16*RM (k) x 16*NTB (tile) block of its point over the whole of C (RM = 2, or 4 on layers large
// enough to fill the chip with the bigger blocks: each V fragment then feeds four MFMAs instead of two).  Operand fragments are read
// straight from global memory in 1 KiB runs (layout.hpp); KS contraction steps are loaded before any is
// consumed.  The four results of a group are exchanged through LDS so that O is written as whole words,
// 16 bytes per thread.
//
// 16-bit moduli: both operands are two byte planes, U = 256 Uh + Ul, V = 256 Vh + Vl, and
//   sum U V = 65536 sum(Uh Vh) + 256 sum(Uh Vl + Ul Vh) + sum(Ul Vl):
// four int8 MFMAs into three accumulators, combined in 64 bits and reduced once at the end.
//
// Grid: one-dimensional, 8 * (ceil(n*Q / 8) rounded up to a multiple of xgroup) * ceil(Kp / (16*RM)) * ceil(Tp / (16*NTB)).
#pragma once
#include <type_traits>

#include "kernels_common.hpp"

namespace rnswino {

// The GEMM kernels' arguments, fetched together at entry, see K1Args.
struct K2Args {
  const ResidueParams *more;
  const int8_t *U, *V;
  uint32_t *O;
  int xgroup, gy, gz;         // grid order: values of x per group, row blocks, tile blocks
  uint32_t xgroup_mul, gy_mul, gz_mul, Q_mul;          // FastDiv's, with the shifts below
  int nkb, ntb, ncb;          // row and tile blocks of 16, channel blocks of 64
  int xs, slabs;              // n * Q, n * P2
  int P2;                     // points
  uint32_t shifts;            // bytes: of the divisions by xgroup, gy, gz, Q
  uint32_t sizes;             // bytes: Q (point groups), 1 if fragments of V are in lane order (layout.hpp)
  RNSW_HD FastDiv by_xgroup() const { return {xgroup_mul, shifts & 31u}; }
  RNSW_HD FastDiv by_gy() const { return {gy_mul, shifts >> 8 & 31u}; }
  RNSW_HD FastDiv by_gz() const { return {gz_mul, shifts >> 16 & 31u}; }
  RNSW_HD FastDiv by_Q() const { return {Q_mul, shifts >> 24 & 31u}; }
  RNSW_HD int Q() const { return (int)byte_of(sizes, 0); }
  // byte of tile l % 16 and slice l / 16 in a fragment of V
  RNSW_HD int v_offset(int lane) const { return sizes >> 8 ? lane * 16 : (lane & 15) * 64 + (lane >> 4) * 16; }
};
static_assert(sizeof(K2Args) <= 112, "kernels_common.hpp");

// Work item (x = residue and point group, y = row block, z = tile block) from the linear workgroup id.  Workgroups
// are handed to the 8 XCDs round-robin by id, so x = 8 * (...) + id % 8 keeps one x on one XCD.  Within an XCD the
// ids run over `xgroup` values of x first, then y, then z, then the groups of x: the workgroups that share a slice
// of U (same x and y, along z) or of V (same x and z, along y) follow each other closely enough to find it in the
// XCD's L2, while `xgroup` different x at a time spread the accesses over the L2's channels.
struct K2Item { int x, i, q, y, z; };
__device__ __forceinline__ K2Item k2_item(const K2Args &P, uint32_t id) {
  K2Item w;
  const uint32_t r0 = id >> 3, r1 = fast_div(r0, P.by_xgroup()), r2 = fast_div(r1, P.by_gy()), r3 = fast_div(r2, P.by_gz());
  w.y = (int)(r1 - r2 * (uint32_t)P.gy);
  w.z = (int)(r2 - r3 * (uint32_t)P.gz);
  w.x = (int)((r3 * (uint32_t)P.xgroup + (r0 - r1 * (uint32_t)P.xgroup)) * 8 + (id & 7));
  w.i = (int)fast_div((uint32_t)w.x, P.by_Q());
  w.q = w.x - w.i * P.Q();
  return w;
}
#define RNSW_K2_FETCH_ARGUMENTS(P)                                                                                                       \
  asm volatile("" ::"s"(P.U), "s"(P.V), "s"(P.O), "s"(P.xgroup), "s"(P.gy), "s"(P.gz), "s"(P.xgroup_mul), "s"(P.gy_mul), "s"(P.gz_mul),  \
               "s"(P.Q_mul), "s"(P.nkb), "s"(P.ntb), "s"(P.ncb), "s"(P.xs), "s"(P.slabs), "s"(P.P2), "s"(P.shifts), "s"(P.sizes))

template <int KS, int NTB, int RM, bool WIDE>
__global__ __launch_bounds__(256) void k2_residue_gemm(K2Args P) {
  Constant<ResidueParams> &R = constant(P.more);
  constexpr int PL = WIDE ? 2 : 1;
  constexpr int NACC = WIDE ? 3 : 1;
  constexpr int COLS = 16 * NTB;
  constexpr int ROWS = 16 * RM;          // k rows per wave and per block
  constexpr int ROWW = COLS * PL;        // words per tile row
  constexpr int PITCH = ROWW + 4;        // LDS row pitch: the four row groups of a byte store fall into different banks
  __shared__ __attribute__((aligned(16))) uint32_t tile[ROWS * PITCH];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: slab addresses stay scalar
  const int lane = threadIdx.x & 63;
  RNSW_K2_FETCH_ARGUMENTS(P);
  const int nkb = P.nkb, ntb = P.ntb, ncb = P.ncb;
  const K2Item item = k2_item(P, blockIdx.x);
  if (item.x >= P.xs) return;                      // x is padded to a multiple of 8
  const int i = item.i, q = item.q;
  const int pt = 4 * q + wave;
  const int kb0 = item.y * RM, tb0 = item.z * NTB;
  // Up to four steps |sum| <= 256 * 126 * 127 < 2^22 - 2^15: the accumulators may start at acc_bias and skip a conversion
  // per result (biased_lowbyte()).  The constants are fetched behind the first step's operands.
  const bool biased = !WIDE && ncb <= 4;

  v4i acc[NACC][RM][NTB];
  if (pt < P.P2) {
    const int slab = i * P.P2 + pt;
    // Row blocks and tile blocks past the end are clamped to the last one: what they compute is never stored, and
    // the loads need neither a branch nor a zero fill.
    const int8_t *Ur[RM], *Vt[NTB];
#pragma unroll
    for (int rm = 0; rm < RM; ++rm)
      Ur[rm] = P.U + ((size_t)slab * nkb + min(kb0 + rm, nkb - 1)) * ncb * (1024 * PL) + lane * 16;
#pragma unroll
    for (int tb = 0; tb < NTB; ++tb)
      Vt[tb] = P.V + ((size_t)min(tb0 + tb, ntb - 1) * P.slabs + slab) * ncb * (1024 * PL) + P.v_offset(lane);

    // KS contraction steps from s0 on; the very first step starts the accumulators (no zero fill)
    auto steps = [&](int s0, auto first_tag) {
      constexpr bool FIRST = decltype(first_tag)::value;
      v4i a[KS][RM][PL], b[KS][NTB][PL];
#pragma unroll
      for (int s = 0; s < KS; ++s) {
#pragma unroll
        for (int rm = 0; rm < RM; ++rm)
#pragma unroll
          for (int pl = 0; pl < PL; ++pl) a[s][rm][pl] = *(const v4i *)(Ur[rm] + (size_t)((s0 + s) * PL + pl) * 1024);
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
          for (int pl = 0; pl < PL; ++pl) b[s][tb][pl] = *(const v4i *)(Vt[tb] + (size_t)((s0 + s) * PL + pl) * 1024);
      }
      // every load of the step is issued before its first product (left alone, the scheduler sinks the loads
      // between the products to save registers, and the wave then waits for them one at a time)
      __builtin_amdgcn_sched_barrier(0);
      const int a0 = FIRST && biased ? R.res[i].acc_bias : 0;
      const v4i acc0 = (v4i){a0, a0, a0, a0};
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int rm = 0; rm < RM; ++rm)
#pragma unroll
          for (int tb = 0; tb < NTB; ++tb) {
            const bool start = FIRST && s == 0;
            if constexpr (WIDE) {
              acc[0][rm][tb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[s][rm][0], b[s][tb][0], start ? acc0 : acc[0][rm][tb], 0, 0, 0);
              acc[1][rm][tb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[s][rm][0], b[s][tb][PL - 1], start ? acc0 : acc[1][rm][tb], 0, 0, 0);
              acc[1][rm][tb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[s][rm][PL - 1], b[s][tb][0], acc[1][rm][tb], 0, 0, 0);
              acc[NACC - 1][rm][tb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[s][rm][PL - 1], b[s][tb][PL - 1], start ? acc0 : acc[NACC - 1][rm][tb], 0, 0, 0);
            } else {
              acc[0][rm][tb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[s][rm][0], b[s][tb][0], start ? acc0 : acc[0][rm][tb], 0, 0, 0);
            }
          }
      // 8-bit residues, |U|,|V| <= 127: 512 channels add at most 8.3e6, so reducing every 8 steps keeps
      // |acc| < 2^24.  (Byte planes need nothing here: a step adds at most 2^21 to the middle sum and the plan
      // admits 16-bit moduli only with fewer than 1024 steps.)
      if (!WIDE && (((s0 + KS) & 7) == 0) && (s0 + KS < ncb)) {
#pragma unroll
        for (int rm = 0; rm < RM; ++rm)
#pragma unroll
          for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[0][rm][tb][j] = mod_near(acc[0][rm][tb][j], R.res[i].inv, -R.res[i].neg_p);
      }
    };
    steps(0, std::true_type{});
    for (int s0 = KS; s0 < ncb; s0 += KS) steps(s0, std::false_type{});
  } else {
    // a point group's unused byte lanes (t*t not a multiple of 4) are written as zeros
#pragma unroll
    for (int a = 0; a < NACC; ++a)
#pragma unroll
      for (int rm = 0; rm < RM; ++rm)
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) acc[a][rm][tb] = (v4i){0, 0, 0, 0};
  }

  // the four results of a point group become the four bytes of one word, through LDS.  The lane's part of the
  // address is computed once and hidden from the optimiser, so that each byte store carries its (compile-time)
  // row and column as the instruction's immediate offset instead of recomputing the address.
  uint32_t lane_byte = (uint32_t)((4 * (lane >> 4)) * PITCH + (lane & 15) * PL) * 4 + wave;
  asm volatile("" : "+v"(lane_byte));
  uint8_t *tile8 = (uint8_t *)tile + lane_byte;
  const Residue8 rc = residue(R.res[i]);
  const int p = -rc.neg_p;
  const float inv = in_vgpr(rc.inv), qb = in_vgpr(rc.quot_bias);
  auto exchange = [&](auto biased_tag) {
    constexpr bool BIASED = decltype(biased_tag)::value;
#pragma unroll
    for (int rm = 0; rm < RM; ++rm)
#pragma unroll
      for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int at = ((rm * 16 + j) * PITCH + tb * 16 * PL) * 4;   // row rm*16 + 4*(lane>>4) + j, column tb*16 + lane%16
          if constexpr (WIDE) {
            const int v = storable16((int)mod_near64(acc[0][rm][tb][j], acc[1][rm][tb][j], acc[NACC - 1][rm][tb][j], R.inv_pd[i], (double)p), p);
            const int lo = (int)(int8_t)(v & 0xFF), hi = (v - lo) >> 8;
            tile8[at] = (uint8_t)hi;
            tile8[at + (PL - 1) * 4] = (uint8_t)lo;
          } else {
            tile8[at] = (uint8_t)(BIASED ? biased_lowbyte(acc[0][rm][tb][j], inv, qb, -p) : mod_lowbyte(acc[0][rm][tb][j], inv, -p));
          }
        }
  };
  if (biased) exchange(std::true_type{});
  else exchange(std::false_type{});
  __syncthreads();
  // O is [Kp][n][Q][Tp] words (x PL) and smaller than 4 GiB: 32-bit word offsets.  16 bytes per thread; whole tile
  // rows are written, padding tiles included (nothing depends on what they hold); only rows >= Kp and tile blocks
  // beyond Tp are left out.
  constexpr int VPR = ROWW / 4;           // 16-byte vectors per tile row
  constexpr int RP = 256 / VPR;           // rows per pass of the block
  const int Tp = P.ntb * 16;
  const uint32_t krow = (uint32_t)(P.xs * Tp) * PL;
  const int r0 = threadIdx.x / VPR, c4 = threadIdx.x % VPR;
  const int valid_rows = min(ROWS, P.nkb * 16 - kb0 * 16);
  const bool vec_ok = tb0 * 16 * PL + 4 * c4 < Tp * PL;
  uint32_t off = (uint32_t)(kb0 * 16 + r0) * krow + (uint32_t)((i * P.Q() + q) * Tp + tb0 * 16) * PL + 4 * c4;
#pragma unroll
  for (int ps = 0; ps < (ROWS + RP - 1) / RP; ++ps) {
    const int row = ps * RP + r0;
    if (vec_ok && row < valid_rows) *(v4i *)(P.O + off) = *(const v4i *)(tile + row * PITCH + 4 * c4);
    off += RP * krow;
  }
}

}  // namespace rnswino
