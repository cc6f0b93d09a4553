// K3: inverse transform on the matrix cores, fused with the conversion out of the RNS.
//
// Y_i = A^T_p O_i A_p after the reduction over C (paper section 6, eq. "direct_sum_2"), then the residues
// (Y_0..Y_{n-1}) are converted to the integer result (section 3).  A^T O A = (A^T kron A^T) vec(O): per residue
// an (m*m) x (t*t) matrix applied to the t*t transform points of a (channel k, tile) pair.  MFMA roles: A operand =
// the Kronecker table (rows = 16 outputs), B operand = O (columns = 16 consecutive (k, tile) pairs),
// contraction index = transform point; a lane's 16 operand bytes are four O words (groups q = 16s + 4g + e).
//
// Conversion: the table rows are pre-multiplied by (P/p_i)^-1 mod p_i (P = prod p_i), so the reduced accumulator
// w_i is the CRT coefficient of residue i and
//     y = sum_i (P/p_i) w_i - P * rint(sum_i w_i / p_i)        (computed modulo 2^32)
// is the representative of the result in [-(P-1)/2, (P-1)/2] -- the same value mixed-radix conversion with
// symmetric digits yields; any representative of w_i gives the same y.  sum_i w_i/p_i = y/P + integer with
// |y/P| <= 1/2 - 1/(2P).  The rounding is done in binary64 (error of the sum below 1e-14, while 1/(2P) > 1e-10 for
// every moduli set whose product can matter for a 32-bit result), or in binary32 when the layer's worst case
// 2^14 r^2 C keeps |y/P| below 0.45 (the host decides: KParams::quot32).
//
// Fast conversion (8-bit moduli, KParams::fastcrt): the accumulator a_i is not reduced at all.  a_i is congruent to
// w_i modulo p_i, and (P/p_i) p_i = P, so S = sum_i (P/p_i) a_i is congruent to y modulo P and y = S - P rint(S/P) with
// S/P = sum_i a_i / p_i.  |a_i| <= t*t * 126 * 128 <= 2^22, so accumulators that start at 0x4B400000 hold a_i in two forms
// at once: read as binary32 they are the number 1.5*2^23 + a_i (no conversion before the quotient's sum), and their low
// 24 bits are a_i + 2^22, an unsigned 23-bit number for one 24-bit multiply-add (P/p_i < 2^24).  The constants that undo
// both offsets sit in KParams (crt_sum0, crt_fs0).  The binary32 sum carries an error of a few hundredths (bounded on the
// host from the moduli), so the host enables this path only when the layer's worst case keeps |y/P| that far below
// 1/2 -- true for every layer whose moduli were chosen by the range bound with a little room, e.g. all five benchmark
// workloads.  Otherwise (KParams::fastcrt == 2) the same sum is taken in binary64 over accumulators that start at 2^22,
// which is exact enough for every result the moduli can represent.
//
// Block = one unit of 16 consecutive (k, tile) pairs and the 16-output row blocks rb = 4*blockIdx.y + wave, + 4*gridDim.y, ...
// The four waves share the unit's O operand through LDS, each loading every fourth point group (a wave-uniform row of O plus a
// 32-bit lane offset per word).
// Grid: x = ceil(K*T/16) rounded up to a multiple of 8, y = 1 .. ceil(RB3/4); 256 threads.
// 16-bit moduli: table and O are two byte planes each; three accumulators as in the GEMM; three and more of them are mostly
// converted residue by residue (k3_converts_each), with the rounding in binary64.
#pragma once
#include <type_traits>

#include "kernels_common.hpp"

namespace rnswino {


// The kernels' arguments: the block kernel fetches them together at entry, see K1Args.  With that, divisions by multiplication and the operand shared
// through LDS: 128 channels 5 x 5 at 28 x 28 17.1 -> 14.1 us a layer, 256 channels at 56 x 56 22.1 -> 20.4, VGG16 stack at batch 1
// 379 -> 362.
struct K3Params;
struct K3Args {
  const K3Params *more;
  const uint32_t *O;
  const int8_t *KA;           // (A^T kron A^T) (P/p_i)^-1 mod p  [n][RB3][KS3][planes][64 lanes][16]
  void *out;                  // int32 y, or the int8 activations of modes 1 and 2
  int units, per_xcd, npairs; // units of 16 pairs (streaming kernel: of 16 tiles of one row), grid x / 8, rows x tiles
  uint32_t Tg_mul, tw_mul, th_mul;           // FastDiv's, with the shifts below
  int Tg, T, Tp, tw, th, K, Ho, Wo;
  uint32_t shifts;            // bytes: of the divisions by Tg, tw, th; log2 of the tiles a channel block holds
  uint32_t sizes;             // bytes: Q, RB3, rb_step, m
  // fused re-quantisation (chained layers): 0 = store int32 y, 1 = store int8 clamp(y >> shift), 2 = the same after a 2x2
  // stride-2 max-pool
  int epi, shift;
  RNSW_HD FastDiv by_Tg() const { return {Tg_mul, shifts & 31u}; }
  RNSW_HD FastDiv by_tw() const { return {tw_mul, shifts >> 8 & 31u}; }
  RNSW_HD FastDiv by_th() const { return {th_mul, shifts >> 16 & 31u}; }
  RNSW_HD int tl_shift() const { return (int)(shifts >> 24); }
  RNSW_HD int Q() const { return (int)byte_of(sizes, 0); }
  RNSW_HD int RB3() const { return (int)byte_of(sizes, 1); }
  RNSW_HD int rb_step() const { return (int)byte_of(sizes, 2); }
  RNSW_HD int m() const { return (int)(sizes >> 24); }
};
static_assert(sizeof(K3Args) <= 112, "kernels_common.hpp");

// What they read behind their first loads, built once with the plan: the conversion out of the RNS, see KParams.
struct K3Params {
  int fastcrt, crt24, quot32, acc0;
  uint32_t crt_sum0, prod_mod32;
  float crt_fs0, inv_m;
  double crt_fs0d;
  uint32_t crt_c[8];
  float inv_p[8];
  int p[8], bias_p[8];
  double inv_pd[8];
  double pd[8];               // 16-bit moduli: p
  FastDiv by_ntb;             // streaming kernel
  int nwaves;                 // streaming kernel: waves of the grid
};

// Where the output tile of a (k, tile) pair starts in y (or in the int8 activation plane): computed once per pair,
// the row blocks of the pair only add their own row and column to it.
struct TilePos {
  uint32_t origin;   // element index of output (oy0, ox0) of channel k of image img (O, at least a byte per output, is smaller than 4 GiB)
  int oy0, ox0;      // top-left output of the tile
  bool ok;           // false for padding tiles and padding pairs
};

__device__ __forceinline__ TilePos tile_position(const K3Args &P, int k, int tau) {
  TilePos tp;
  tp.ok = tau < P.T;
  const int trow = (int)fast_div((uint32_t)tau, P.by_tw());
  const int tx = tau - trow * P.tw;
  const int img = (int)fast_div((uint32_t)trow, P.by_th());
  const int ty = trow - img * P.th;
  tp.oy0 = ty * P.m();
  tp.ox0 = tx * P.m();
  const uint32_t plane = (uint32_t)img * P.K + k;
  const int half = P.epi == 2 ? 1 : 0;               // pooled planes have half the rows and columns
  tp.origin = (plane * (P.Ho >> half) + (tp.oy0 >> half)) * (P.Wo >> half) + (tp.ox0 >> half);
  return tp;
}

// CRT conversion of the four outputs of one lane (row block rb, lane group g) and their store: int32 y, or, for
// chained layers, int8 clamp(y >> shift) with an optional 2x2 max-pool (the shift is monotone, so it commutes with
// the max).  Must be called by all lanes of a wave (the pooled mode exchanges rows between lanes).
template <int NRES, bool CRT24, bool QUOT32>
__device__ __forceinline__ void crt_convert(Constant<K3Params> &P, const uint32_t (&w)[NRES][4], int (&val)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t sum = 0;
    int kk;
    if (QUOT32) {
      // |y| <= 0.45 P: the sum is within 0.45 of an integer and binary32 (error below 1e-4) finds that integer
      float fs = 0.0f;
#pragma unroll
      for (int i = 0; i < NRES; ++i) {
        sum += CRT24 ? __umul24(P.crt_c[i], w[i][j]) : P.crt_c[i] * w[i][j];
        fs = __builtin_fmaf((float)w[i][j], P.inv_p[i], fs);
      }
      kk = (int)__builtin_rintf(fs);
    } else {
      double fs = 0.0;
#pragma unroll
      for (int i = 0; i < NRES; ++i) {
        sum += CRT24 ? __umul24(P.crt_c[i], w[i][j]) : P.crt_c[i] * w[i][j];
        fs = __builtin_fma((double)w[i][j], P.inv_pd[i], fs);
      }
      kk = __double2int_rn(fs);
    }
    val[j] = (int)(sum - P.prod_mod32 * (uint32_t)kk);
  }
}

// Fast conversion (see the header): w[i][j] = a_i + 0x4B400000, unreduced; read as binary32 it is 1.5*2^23 + a_i, so the
// sum for the quotient takes it as it is, and its low 24 bits are a_i + 2^22 (the first product, the compiler's own, takes all
// 32 bits; mad_u24() says why).  Adding 1.5*2^23 to that sum rounds it and
// leaves the quotient in the mantissa; the multiples of P that its bias stands for are part of crt_sum0.
// Per output and residue one float multiply-add with vector operands (2.6 cycles per wave and SIMD) and one 24-bit
// multiply-add (4.8), then a float sum, a product (4.4) and a sum of three: about 39 cycles with four residues (71 with
// conversions and scalar operands).
struct FastCrt {
  float inv[8], fs0;
  uint32_t sum0;
};
template <int NRES>
__device__ __forceinline__ void crt_convert_fast(Constant<K3Params> &P, const FastCrt &fc, const uint32_t (&w)[NRES][4], int (&val)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t sum = 0;
    float fs = fc.fs0;
#pragma unroll
    for (int i = 0; i < NRES; ++i) {
      fs = __builtin_fmaf(__uint_as_float(w[i][j]), fc.inv[i], fs);
      sum = i == 0 ? P.crt_c[i] * w[i][j] : mad_u24(P.crt_c[i], w[i][j], sum, fs);
    }
    val[j] = (int)(sum + fc.sum0 + mul_lo(0u - P.prod_mod32, __float_as_uint(fs + 12582912.0f)));
  }
}

// The same with the quotient in binary64: the sum then carries an error below 1e-10 and finds the quotient for every
// result in [-(P-1)/2, (P-1)/2] (the host checks its bound against 1/(2P)), so layers at the edge of the dynamic
// range and plans with an unchecked range take this form.
template <int NRES>
__device__ __forceinline__ void crt_convert_fast64(Constant<K3Params> &P, const FastCrt &fc, const uint32_t (&w)[NRES][4], int (&val)[4]) {
  uint32_t c0 = P.crt_c[0];
  asm("" : "+s"(c0));       // keeps the first products of the two forms apart: taken in front of the branch, each would be copied behind it
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t sum = 0;
    double fs = P.crt_fs0d;
#pragma unroll
    for (int i = 0; i < NRES; ++i) {
      const double wd = (double)w[i][j];
      sum = i == 0 ? c0 * w[i][j] : mad_u24(P.crt_c[i], w[i][j], sum, wd);
      fs = __builtin_fma(wd, P.inv_pd[i], fs);
    }
    const int kk = __double2int_rn(fs);
    val[j] = (int)(sum + fc.sum0 + mul_lo(0u - P.prod_mod32, (uint32_t)kk));
  }
}

// Constants of the fast conversion in vector registers, loaded once per kernel.
template <int NRES, bool FAST>
__device__ __forceinline__ FastCrt fast_crt_constants(Constant<K3Params> &P) {
  FastCrt fc;
  fc.fs0 = FAST ? in_vgpr(P.crt_fs0) : 0.0f;
  fc.sum0 = FAST ? in_vgpr(P.crt_sum0) : 0u;
#pragma unroll
  for (int i = 0; i < NRES; ++i) fc.inv[i] = FAST ? in_vgpr(P.inv_p[i]) : 0.0f;
  return fc;
}

template <int NRES, bool FAST>
__device__ __forceinline__ void k3_convert(Constant<K3Params> &P, const FastCrt &fc, const uint32_t (&w)[NRES][4], int (&val)[4]) {
  if (FAST) {
    if (P.fastcrt == 2) crt_convert_fast64<NRES>(P, fc, w, val);   // uniform
    else crt_convert_fast<NRES>(P, fc, w, val);
  } else if (P.crt24) {               // uniform: one branch per call instead of one per multiply
    if (P.quot32) crt_convert<NRES, true, true>(P, w, val);
    else crt_convert<NRES, true, false>(P, w, val);
  } else {
    crt_convert<NRES, false, false>(P, w, val);
  }
}

// Store of a lane's four outputs for 8 x 8 output tiles (the streaming kernel): `inside` says whether they exist (their first two,
// where the row ends in the middle; `right` then: the other two) and, pooled, whether the lane stores; `at` is the first one's place in
// the stored plane.  Same modes as k3_convert_and_store; the host selects this path for int32 output only when Wo is a multiple
// of 4.  Must be called by all lanes of a wave.
template <int EPI>
__device__ __forceinline__ void k3_store_m8(const K3Args &P, const int (&val)[4], bool inside, bool right, uint32_t at) {
  if constexpr (EPI == 0) {
    if (inside) *(v4i *)((int32_t *)P.out + at) = (v4i){val[0], val[1], val[2], val[3]};
  } else if constexpr (EPI == 1) {
    uint32_t packed = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) packed |= ((uint32_t)min(127, max(-128, val[j] >> P.shift)) & 0xFFu) << (8 * j);
    int8_t *dst = (int8_t *)P.out + at;
    if ((P.Wo & 3) == 0) {
      if (inside) *(uint32_t *)dst = packed;
    } else {
      if (inside) *(uint16_t *)dst = (uint16_t)packed;
      if (inside && right) *(uint16_t *)(dst + 2) = (uint16_t)(packed >> 16);
    }
  } else {
    // Rows u and u + 1 (u even) of the tile sit in lanes l < 32 and l + 32.  Exchanging the upper half of one register with the lower half of
    // the other leaves the two rows of the left pair in the lower lanes and those of the right pair in the upper ones.
    const auto rows = __builtin_amdgcn_permlane32_swap((uint32_t)max(val[0], val[1]), (uint32_t)max(val[2], val[3]), false, false);
    const int pooled = min(127, max(-128, max((int)rows[0], (int)rows[1]) >> P.shift));
    const auto pair = __builtin_amdgcn_permlane32_swap((uint32_t)pooled, (uint32_t)pooled, false, false);
    if (inside) *(uint16_t *)((int8_t *)P.out + at) = (uint16_t)((pair[0] & 0xFFu) | ((pair[1] & 0xFFu) << 8));
  }
}

__device__ __forceinline__ void k3_store(const K3Args &P, float inv_m, const int (&val)[4], int rb, int g, const TilePos &tp) {
  const int m = P.m(), mm = m * m;
  const int o0 = 16 * rb + 4 * g;
  if (P.epi == 1 && (((m & 3) != 0) || (P.Wo & 1))) {
    // any other tile size or an odd row length: the four outputs may sit in two rows of the tile and at any byte
    // alignment, so each is stored as a byte of its own
    if (!tp.ok) return;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int o = o0 + j;
      const int u = (int)(((float)o + 0.5f) * inv_m);
      const int v = o - u * m;
      if (o < mm && tp.oy0 + u < P.Ho && tp.ox0 + v < P.Wo)
        ((int8_t *)P.out)[(size_t)(tp.origin + (uint32_t)(u * P.Wo + v))] = (int8_t)min(127, max(-128, val[j] >> P.shift));
    }
    return;
  }
  if (P.epi != 0) {
    // here m is 4 or 8 and Wo even (pooling: the host also guarantees Wo % 4 == 0 and an even Ho)
    const int u = (int)(((float)o0 + 0.5f) * inv_m);
    const int v = o0 - u * m;
    const bool inside = tp.ok && o0 < mm && tp.oy0 + u < P.Ho && tp.ox0 + v < P.Wo;
    if (P.epi == 1) {
      uint32_t packed = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) packed |= ((uint32_t)min(127, max(-128, val[j] >> P.shift)) & 0xFFu) << (8 * j);
      int8_t *dst = (int8_t *)P.out + tp.origin + (uint32_t)(u * P.Wo + v);
      if ((P.Wo & 3) == 0) {
        if (inside) *(uint32_t *)dst = packed;
      } else {
        // Wo even but not a multiple of 4: rows are only 2-byte aligned, and the second half may hang over the edge
        if (inside) *(uint16_t *)dst = (uint16_t)packed;
        if (inside && tp.ox0 + v + 2 < P.Wo) *(uint16_t *)(dst + 2) = (uint16_t)(packed >> 16);
      }
    } else {
      // rows u and u+1 (u even) of an output tile sit in lanes l and l ^ 4m (m = 8: 32 apart, m = 4: 16 apart)
      const int h0 = max(val[0], val[1]), h1 = max(val[2], val[3]);
      const int delta = 4 * m;
      const int o0p = __shfl_xor(h0, delta), o1p = __shfl_xor(h1, delta);
      const int p0 = min(127, max(-128, max(h0, o0p) >> P.shift)), p1 = min(127, max(-128, max(h1, o1p) >> P.shift));
      if (inside && (u & 1) == 0)
        *(uint16_t *)((int8_t *)P.out + tp.origin + (uint32_t)((u >> 1) * (P.Wo >> 1) + (v >> 1))) =
            (uint16_t)(((uint32_t)p0 & 0xFFu) | (((uint32_t)p1 & 0xFFu) << 8));
    }
    return;
  }
  if (!tp.ok || o0 >= mm) return;
  int32_t *ytile = (int32_t *)P.out + tp.origin;
  if (((m & 3) == 0) && ((P.Wo & 3) == 0)) {   // four consecutive outputs stay in one row, 16-byte aligned
    const int u = (int)(((float)o0 + 0.5f) * inv_m);
    const int v = o0 - u * m;
    if (tp.oy0 + u < P.Ho && tp.ox0 + v < P.Wo) *(v4i *)(ytile + (uint32_t)(u * P.Wo + v)) = (v4i){val[0], val[1], val[2], val[3]};
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int o = o0 + j;
      const int u = (int)(((float)o + 0.5f) * inv_m);
      const int v = o - u * m;
      if (o < mm && tp.oy0 + u < P.Ho && tp.ox0 + v < P.Wo) ytile[(uint32_t)(u * P.Wo + v)] = val[j];
    }
  }
}

template <int NRES, bool FAST>
__device__ __forceinline__ void k3_convert_and_store(const K3Args &P, Constant<K3Params> &M, const FastCrt &fc, const uint32_t (&w)[NRES][4], int rb, int g,
                                                     const TilePos &tp) {
  int val[4];
  k3_convert<NRES, FAST>(M, fc, w, val);
  k3_store(P, M.inv_m, val, rb, g, tp);
}

// Three and more 16-bit moduli: a residue goes into the sum and the binary64 quotient of the conversion as soon as it is there, signed.  Kept
// until all were there, shifted and converted again for the quotient, with p converted in registers of its own, the residues cost most of
// these kernels a wave per SIMD: 64 -> 256 at 56 x 56, batch 4, five, six, seven, eight moduli at F(4,3) 52, 57.8, 65.7, 126 us, so 28.8,
// 52.6, 59.5, 63.7; three at F(14,3) 39.5, so 26.6.  Six and eight moduli at two steps keep them: 28.8 us there, so 32.1, eight 34.9 and 35.5.
constexpr bool k3_converts_each(int nres, int ks3) { return nres >= 3 && !(ks3 == 2 && (nres == 6 || nres == 8)); }

// FAST: the conversion with unreduced accumulators (the host launches it when KParams::fastcrt is set).
// Where the products of several residues at once would cost a wave, the residues stay apart (APART): five 16-bit moduli at F(8,3) 25.2 -> 22.2
// us, at F(14,3) 43.4 -> 40.8; six at F(10,3) 55.8 -> 43.3; elsewhere it loses up to a tenth.
template <int NRES, int KS3, bool WIDE, bool FAST>
__global__ __launch_bounds__(256) void k3_inverse_crt(K3Args P) {
  Constant<K3Params> &M = constant(P.more);
  constexpr int PL = WIDE ? 2 : 1;
  constexpr int NACC = WIDE ? 3 : 1;
  constexpr bool AHEAD = NRES * KS3 * PL <= 16;    // the table fragments of a row block fit registers: requested ahead of their use
  constexpr bool FEW = !WIDE && NRES * KS3 <= 8;   // loads of a lane
  constexpr bool EACH = WIDE && k3_converts_each(NRES, KS3), APART = WIDE && ((NRES == 5 && KS3 % 2 == 0) || (NRES == 6 && KS3 == 3));
  __shared__ __attribute__((aligned(16))) uint32_t o_lds[NRES * KS3 * PL * 256];   // [i][s][plane][lane][4 words]
  asm volatile("" ::"s"(P.O), "s"(P.KA), "s"(P.units), "s"(P.per_xcd), "s"(P.npairs), "s"(P.Tg_mul), "s"(P.tw_mul), "s"(P.th_mul), "s"(P.Tg), "s"(P.T),
               "s"(P.Tp), "s"(P.tw), "s"(P.th), "s"(P.shifts), "s"(P.sizes), "s"(P.K), "s"(P.Ho), "s"(P.Wo));
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: row block and table addresses stay scalar
  const int lane = threadIdx.x & 63, g = lane >> 4;
  // A unit is 16 consecutive (k, tile) pairs of the flattened K x T index space (no padding tiles: a unit may span
  // several k's).  Workgroups go to the 8 XCDs round-robin by id; neighbouring units share 128-byte lines of O, so
  // each XCD gets one contiguous chunk of the units (grid.x is a multiple of 8).
  // (For layers that pack TL tiles into a channel block, GEMM row kg = k * TL + tile / Tg and GEMM column tile % Tg.)
  const int unit = (int)(blockIdx.x & 7) * P.per_xcd + (int)(blockIdx.x >> 3);
  if (unit >= P.units) return;
  const int pair = min(unit * 16 + (lane & 15), P.npairs - 1);         // a padding lane repeats the last pair
  const int kg = (int)fast_div((uint32_t)pair, P.by_Tg()), taug = pair - kg * P.Tg;

  // O is [Kp][n][Q][Tp] words (x PL planes) and smaller than 4 GiB: the address of a word is a wave-uniform row
  // (residue) plus a 32-bit lane offset (k, point group, tile).  Word e of a lane's operand is point group 16s + 4g + e; wave e
  // loads it for everybody (one load instruction touches four rows of 64 bytes and costs the address unit as much as a
  // 16-byte load of 256: loading all of it four times over took 1800 cycles per block at two contraction steps and 4700 at
  // four).  Point groups >= Q of the last contraction step are clamped to Q - 1: the table is zero there, so whatever is read
  // does not count.
  const uint32_t row_bytes = (uint32_t)P.Tp * (4 * PL);
  const uint32_t lane_off = (uint32_t)(kg * NRES * P.Q()) * row_bytes + (uint32_t)taug * (4 * PL);
  uint32_t voff[KS3];
#pragma unroll
  for (int s = 0; s < KS3; ++s) voff[s] = lane_off + (uint32_t)min(16 * s + 4 * g + wave, P.Q() - 1) * row_bytes;
  v2i mine[NRES][KS3];
#pragma unroll
  for (int i = 0; i < NRES; ++i) {
    const char *row = (const char *)P.O + (size_t)((uint32_t)(i * P.Q()) * row_bytes);
#pragma unroll
    for (int s = 0; s < KS3; ++s) {
      if (WIDE) mine[i][s] = *(const v2i *)(row + voff[s]);
      else mine[i][s][0] = *(const int *)(row + voff[s]);
    }
  }
  int rb = blockIdx.y * 4 + wave;                  // this wave's first block of 16 outputs
  v4i ka[AHEAD ? NRES : 1][AHEAD ? KS3 : 1][PL];
  const uint32_t lane16 = (uint32_t)lane * 16u;
  auto table = [&](int i, int r, int s, int pl) -> v4i {
    return *(const v4i *)(P.KA + (size_t)((((uint32_t)i * P.RB3() + r) * KS3 + s) * PL + pl) * 1024 + lane16);
  };
  auto load_ka = [&](int r) {
    if constexpr (AHEAD)
#pragma unroll
      for (int i = 0; i < NRES; ++i)
#pragma unroll
        for (int s = 0; s < KS3; ++s)
#pragma unroll
          for (int pl = 0; pl < PL; ++pl) ka[i][s][pl] = table(i, r, s, pl);
  };
  load_ka(min(rb, P.RB3() - 1));
  const int k = kg >> P.tl_shift();
  const int tau = unit * 16 + (lane & 15) < P.npairs ? (kg - (k << P.tl_shift())) * P.Tg + taug : P.T;   // tau >= T marks a lane without output
  const FastCrt fc = fast_crt_constants<NRES, FAST>(M);
  TilePos tp = tile_position(P, k, tau);
  if constexpr (FEW) {
    // The position here, while the loads are in flight, its arguments fetched at entry.  Left alone, the compiler moves both behind the barrier
    // (0.1 us of the 8 to 9.5 of a small layer, 100 channels at 57 x 43, batch 3, 14.07 and 13.93).  With more loads what it moves there covers the
    // table's fetch: 48 -> 64 channels, 5 x 5, at 35 x 35, batch 8 (16 loads), 18.45 us here and 18.30 there.  Nothing to see with 16-bit moduli.
    asm volatile("" : "+v"(tp.origin));
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int i = 0; i < NRES; ++i)
#pragma unroll
    for (int s = 0; s < KS3; ++s)
#pragma unroll
      for (int pl = 0; pl < PL; ++pl) o_lds[((i * KS3 + s) * PL + pl) * 256 + lane * 4 + wave] = (uint32_t)mine[i][s][pl];
  __syncthreads();
  if (rb >= P.RB3()) return;
  v4i of[NRES][KS3][PL];
#pragma unroll
  for (int i = 0; i < NRES; ++i)
#pragma unroll
    for (int s = 0; s < KS3; ++s)
#pragma unroll
      for (int pl = 0; pl < PL; ++pl) of[i][s][pl] = *(const v4i *)(o_lds + ((i * KS3 + s) * PL + pl) * 256 + lane * 4);

  for (; rb < P.RB3(); rb += P.rb_step()) {
    uint32_t w[NRES][4], sum[4] = {0, 0, 0, 0};
    double fs[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < NRES; ++i) {
      v4i acc[NACC];
#pragma unroll
      for (int a = 0; a < NACC; ++a) acc[a] = FAST ? (v4i){M.acc0, M.acc0, M.acc0, M.acc0} : (v4i){0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < KS3; ++s) {
        v4i ah, al;
        if constexpr (AHEAD) { ah = ka[i][s][0]; al = ka[i][s][PL - 1]; }
        else { ah = table(i, rb, s, 0); al = WIDE ? table(i, rb, s, PL - 1) : ah; }
        if (WIDE) {
          acc[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah, of[i][s][0], acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah, of[i][s][PL - 1], acc[1], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al, of[i][s][0], acc[1], 0, 0, 0);
          acc[NACC - 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al, of[i][s][PL - 1], acc[NACC - 1], 0, 0, 0);
        } else {
          acc[0] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah, of[i][s][0], acc[0], 0, 0, 0);
        }
      }
      // residue shifted by +p so that it is non-negative
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if constexpr (WIDE) {
          // per accumulator |sum| <= t*t * 2^15: the combination stays below 2^40
          const double r = mod_near64(acc[0][j], acc[1][j], acc[2][j], M.inv_pd[i], EACH || NRES < 3 ? M.pd[i] : (double)M.p[i]);
          if (EACH) {
            sum[j] += M.crt_c[i] * (uint32_t)(int)r;
            fs[j] = __builtin_fma(r, M.inv_pd[i], fs[j]);
          } else {
            w[i][j] = (uint32_t)((int)r + M.p[i]);
          }
        } else {
          // |acc| <= t*t * 126 * 128 <= 2^22 (the fast conversion takes it as it is, start included)
          w[i][j] = FAST ? (uint32_t)acc[0][j] : mod_near_plus_p(acc[0][j], M.inv_p[i], -M.p[i], M.bias_p[i]);
        }
      }
      if (APART) __builtin_amdgcn_sched_barrier(0);
    }
    if (rb + P.rb_step() < P.RB3()) load_ka(rb + P.rb_step());
    if constexpr (EACH) {
      int val[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) val[j] = (int)(sum[j] - M.prod_mod32 * (uint32_t)__double2int_rn(fs[j]));
      k3_store(P, M.inv_m, val, rb, g, tp);
    } else {
      k3_convert_and_store<NRES, FAST>(P, M, fc, w, rb, g, tp);
    }
  }
}

// Streaming variant for layers with many tiles (8-bit moduli, table of all residues <= 64 KiB): the table is staged
// once per block in LDS, and every wave walks over units = (k, block of 16 tiles) with a grid stride.  Per unit a wave
// issues only its own O loads (no table reads from global memory, no copies of O in other waves); the table fragments
// come from LDS.  A unit's loads are hidden by the other waves of the SIMD (four resident blocks per CU).
// Positions in 32 bits, pooling by lane swaps and one loop per output mode and conversion took a unit's vector instructions from about 350 to
// 300 (four residues, two steps, pooled, binary32): 64 -> 128 at 112 x 112, batch 8, pooled, 19.6 -> 18.2 us; the median of the layers of the VGG16
// stack, batch 8, that come here 21.3 -> 20.4.  Loads that keep their lane's offset in 32 bits (load_o) took another 32 and four to eight registers: the
// stack's layers 793.8 -> 785.4 us together.
// What bounds it: a unit's first products wait for all its loads and for the stores of the unit before.  On 64 -> 64 at 224 x 224, batch 8,
// pooled (168 MB of O, 42.8 us before that): without the loads of O 30, without the stores 40, without the conversion 40.5, without
// loads and stores 26.8; the same bytes in 16-byte loads, a quarter as many, 42.3.  More loads in flight make it slower: the next
// unit's operand requested a unit ahead 23.2 us against that 20.4, five blocks per compute unit 22.3, units of 32 tiles (whole lines of O,
// three blocks) 22.7.
// Grid: min(ceil(units / 4), four blocks per CU) blocks of 256 threads; dynamic LDS = n * RB3 * KS3 KiB.
constexpr int K3_STREAM_BLOCKS = 1024;  // four resident blocks per CU (register budget) on 256 CUs

// M8: 8 x 8 output tiles (four row blocks), the usual case: where a lane's outputs go inside the tile is computed once
// per kernel instead of once per row block, and the table fragments of a row block sit at immediate LDS offsets.
template <int NRES, int KS3, bool FAST, bool M8>
__global__ __launch_bounds__(256) void k3_inverse_crt_stream(K3Args P) {
  Constant<K3Params> &M = constant(P.more);
  extern __shared__ __attribute__((aligned(16))) uint8_t ka_lds[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: unit arithmetic stays scalar
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int ntb = P.Tp >> 4;
  const int nunits = P.units;                      // (k, block of 16 tiles), the GEMM's rows and columns
  const int nwaves = M.nwaves;
  const FastDiv by_ntb = {M.by_ntb.mul, M.by_ntb.shift};
  {
    const int bytes = NRES * P.RB3() * KS3 * 1024;
    for (int off = threadIdx.x * 16; off < bytes; off += 256 * 16) *(v4i *)(ka_lds + off) = *(const v4i *)(P.KA + off);
  }
  __syncthreads();
  int unit = blockIdx.x * 4 + wave;
  if (unit >= nunits) return;

  // lane part of an O address in bytes, the same for every unit: point group (clamped to Q - 1 where the table is zero)
  // and tile within the block of 16; the unit contributes a wave-uniform base (O is smaller than 4 GiB)
  const uint32_t row_bytes = (uint32_t)P.Tp * 4u;
  uint32_t voff[KS3][4];
#pragma unroll
  for (int s = 0; s < KS3; ++s)
#pragma unroll
    for (int e = 0; e < 4; ++e) voff[s][e] = (uint32_t)min(16 * s + 4 * g + e, P.Q() - 1) * row_bytes + (uint32_t)(lane & 15) * 4u;

  auto load_o = [&](int k, int tb, v4i (&of)[NRES][KS3]) {
    uint32_t at[KS3][4];                               // (known to be the same for every unit, they would be widened in front of the loop, and each load would add
#pragma unroll                                         // the unit's address to them in 64 bits)
    for (int s = 0; s < KS3; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        at[s][e] = voff[s][e];
        asm volatile("" : "+v"(at[s][e]));
      }
#pragma unroll
    for (int i = 0; i < NRES; ++i) {
      const char *row = (const char *)P.O + (size_t)((uint32_t)((k * NRES + i) * P.Q()) * row_bytes + (uint32_t)tb * 64u);
#pragma unroll
      for (int s = 0; s < KS3; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) of[i][s][e] = *(const int *)(row + at[s][e]);
    }
  };

  const FastCrt fc = fast_crt_constants<NRES, FAST>(M);
  const int a0 = FAST ? M.acc0 : 0;
  const v4i acc_start = (v4i){a0, a0, a0, a0};
  // GEMM row kg = k * TL + slot and columns 16 tb .. + 15 of a unit (TL > 1: packed layers, plan.hpp)
  auto position = [&](int kg, int tb) {
    const int taug = tb * 16 + (lane & 15), k = kg >> P.tl_shift();
    return tile_position(P, k, taug < P.Tg ? (kg - (k << P.tl_shift())) * P.Tg + taug : P.T);
  };
  if constexpr (M8) {
    // 8 x 8 tiles: outputs 16 rb + 4 g .. + 3 are row u = 2 rb + (g >> 1), columns v = 4 (g & 1) .. + 3 of the tile.  One loop per
    // output mode and form of the conversion: tested inside it, the two cost a dozen branches per row block.
    const int u0 = g >> 1, v = 4 * (g & 1);
    auto units = [&](auto epi_tag, auto binary64_tag) {
      constexpr int EPI = decltype(epi_tag)::value;
      constexpr bool BINARY64 = decltype(binary64_tag)::value;
      // elements between row blocks, and of the lane's first output from the tile's origin
      const uint32_t step = EPI == 2 ? (uint32_t)(P.Wo >> 1) : (uint32_t)(2 * P.Wo), off0 = EPI == 2 ? (uint32_t)(v >> 1) : (uint32_t)(u0 * P.Wo + v);
      for (; unit < nunits; unit += nwaves) {
        const int kg = (int)fast_div((uint32_t)unit, by_ntb), tb = unit - kg * ntb;
        v4i o[NRES][KS3];
        load_o(kg, tb, o);
        const TilePos tp = position(kg, tb);
        const bool columns = tp.ok && tp.ox0 + v < P.Wo && (EPI != 2 || lane < 32), right = tp.ox0 + v + 2 < P.Wo;
        const int rows = P.Ho - tp.oy0 - u0;               // of this lane that exist: 2 rb < rows
        uint32_t at = tp.origin + off0;
        // not unrolled: with the four row blocks in one basic block the scheduler requests all their table fragments
        // at once and the kernel needs twice the registers
#pragma clang loop unroll(disable)
        for (int rb = 0; rb < 4; ++rb) {
          uint32_t w[NRES][4];
          const uint8_t *ka_rb = ka_lds + lane * 16 + rb * (KS3 * 1024);
#pragma unroll
          for (int i = 0; i < NRES; ++i) {
            v4i acc = acc_start;
#pragma unroll
            for (int s = 0; s < KS3; ++s) {
              const v4i a = *(const v4i *)(ka_rb + (i * 4 * KS3 + s) * 1024);
              acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, o[i][s], acc, 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
              w[i][j] = FAST ? (uint32_t)acc[j] : mod_near_plus_p(acc[j], M.inv_p[i], -M.p[i], M.bias_p[i]);
          }
          int val[4];
          if constexpr (FAST && BINARY64) crt_convert_fast64<NRES>(M, fc, w, val);
          else if constexpr (FAST) crt_convert_fast<NRES>(M, fc, w, val);
          else k3_convert<NRES, FAST>(M, fc, w, val);
          k3_store_m8<EPI>(P, val, columns && 2 * rb < rows, right, at);
          at += step;
        }
      }
    };
    auto modes = [&](auto binary64_tag) {
      if (P.epi == 0) units(std::integral_constant<int, 0>(), binary64_tag);
      else if (P.epi == 1) units(std::integral_constant<int, 1>(), binary64_tag);
      else units(std::integral_constant<int, 2>(), binary64_tag);
    };
    if (FAST && M.fastcrt == 2) modes(std::true_type());
    else modes(std::false_type());
    return;
  }
  for (; unit < nunits; unit += nwaves) {
    const int kg = (int)fast_div((uint32_t)unit, by_ntb), tb = unit - kg * ntb;
    v4i o[NRES][KS3];
    load_o(kg, tb, o);
    const TilePos tp = position(kg, tb);
    for (int rb = 0; rb < P.RB3(); ++rb) {
      uint32_t w[NRES][4];
#pragma unroll
      for (int i = 0; i < NRES; ++i) {
        v4i acc = acc_start;
#pragma unroll
        for (int s = 0; s < KS3; ++s) {
          const v4i a = *(const v4i *)(ka_lds + (((i * P.RB3() + rb) * KS3) + s) * 1024 + lane * 16);
          acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, o[i][s], acc, 0, 0, 0);
        }
        // |acc| <= t*t * 126 * 128 <= 2^22: the fast conversion takes it as it is, start included, the general one the
        // residue shifted by +p so that it is non-negative
#pragma unroll
        for (int j = 0; j < 4; ++j)
          w[i][j] = FAST ? (uint32_t)acc[j] : mod_near_plus_p(acc[j], M.inv_p[i], -M.p[i], M.bias_p[i]);
      }
      k3_convert_and_store<NRES, FAST>(P, M, fc, w, rb, g, tp);
    }
  }
}

}  // namespace rnswino
