// Shared device-side definitions of the rnswino kernels (gfx950).
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

#include "address_math.hpp"

namespace rnswino {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));

// Constants of one 8-bit modulus for biased_lowbyte() and mod_near(): one 16-byte scalar load.
struct Residue8 {
  float inv, quot_bias;
  int neg_p, acc_bias;
};

// A launch carries a kernel's addresses and what it reads in front of its first loads, at most 112 bytes; the rest lies in device memory, written once
// with the plan, and is fetched while those loads are in flight.  All of it by value (300 to 500 bytes) is copied anew for every launch: in a
// row of launches that takes the host 3.5 to 3.9 us each from 120 bytes on, 2.8 up to 112: 16 channels
// at 16 x 16, whose three launches are more for the host than for the GPU, 12.4 -> 9.7 us a layer (medians of three
// comparisons of four, 11.1 -> 10.7 in the other; runs of one side differ by 14 to 39 %); the layers that the GPU bounds +-0.5 %.
// (All of it in device memory puts a fetch in front of the first loads: 256 channels at 56 x 56 19.75 -> 20.45 us a layer, 19.9 with the pointer to it in
// scalar registers when a wave starts.)
// Read through this address space the fields come by scalar loads wherever they are used.
template <typename T>
using Constant = const T __attribute__((address_space(4)));
template <typename T>
__device__ __forceinline__ Constant<T> &constant(const T *p) { return *(Constant<T> *)p; }
__device__ __forceinline__ Residue8 residue(Constant<Residue8> &r) { return {r.inv, r.quot_bias, r.neg_p, r.acc_bias}; }

// Small fields of a kernel's arguments share words: byte e of one, a scalar instruction each.
RNSW_HD uint32_t byte_of(uint32_t word, int e) { return (word >> (8 * e)) & 255u; }
inline uint32_t pack_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d) { return a | b << 8 | c << 16 | d << 24; }

// What the input transform and the GEMM read behind their first loads.
struct ResidueParams {
  alignas(16) Residue8 res[8];
  double inv_pd[8];           // 16-bit moduli
  uint32_t kept_share;        // k_transform_gemm.hpp: bytes of the input that a workgroup copies
};

// Everything the filter transform needs to know about the layer, passed by value, and what the other kernels' parameters are made of.
struct KParams {
  int N, C, K, H, W, r, m, t, pad;
  int Ho, Wo, th, tw, T, n;
  int TL, Cq, Kg, Tg;         // tile packing of layers with few channels (plan.hpp); TL = 1: none
  int Cp, Kp, Tp, P2, Q;      // GEMM extents (of the packed problem when TL > 1)
  int p[8];
  float inv_p[8];
  double inv_pd[8];           // 1 / p_i
  // transforms on the matrix cores: Kronecker tables in operand-fragment order (see plan_math.cpp)
  int CB1, KS1, RP1, RB3, KS3;
  const int8_t *KG;           // (G kron G) mod p              [n][CB1][planes][64 lanes][16]
  const int8_t *KB;           // (B^T kron B^T) mod p          [n][CB1][KS1][planes][64 lanes][16]
  const int8_t *KA;           // (A^T kron A^T) crt_inv mod p  [n][RB3][KS3][planes][64 lanes][16]
  uint32_t crt_c[8];          // prod_{l != i} p_l mod 2^32
  uint32_t prod_mod32;        // prod p_i mod 2^32
  int crt24;                  // every prod_{l != i} p_l is below 2^24: 24-bit multiplies suffice
  int quot32;                 // the layer's worst-case |y| is at most 0.45 prod p_i: binary32 finds the CRT quotient
  int bias_p[8];              // p_i * 2^22 + p_i (8-bit moduli), see mod_near_plus_p()
  int acc_bias[8];            // 8-bit moduli: what an accumulator starts at for biased_lowbyte()
  float quot_bias[8];         // and the constant that puts its quotient into the mantissa
  // fast conversion out of the RNS (k_inverse_crt.hpp): unreduced accumulators that start at acc0
  int fastcrt, acc0;          // fastcrt: 0 = off, 1 = binary32 quotient, 2 = binary64 quotient
  uint32_t crt_sum0;          // undoes, modulo 2^32, the accumulators' start and the bias of the quotient
  float crt_fs0;              // minus the start's share of the quotient
  double crt_fs0d;            // the same in binary64
};

// Workgroups are handed to the 8 XCDs (each with its own L2) round-robin by linear workgroup id.  A grid whose x extent is a
// multiple of 8 takes item (x % 8) * (gx / 8) + x / 8 in block x, so that each XCD gets one contiguous chunk of the items:
// neighbours (which share input lines) then share an L2.  Items past the count are padding.

// Instructions written as inline assembly.  The compiler keeps the wait states a matrix instruction's registers need (8 from a result
// to its reader or overwriter, 3 from a C operand to its overwriter, on this chip) only for instructions it selects itself.  So each
// of these overwrites one of its own inputs, never a register the allocator finds free, and reads a matrix result only behind a
// compiler's instruction that has read it: through its other inputs, or through the operand `after`, which the text leaves out.
// (Without the two, streaming inverse transforms of two and three moduli read results 5 and 7 states after their instruction, and
// others overwrote a result or an operand still in use.)

// ---- residues of 8-bit moduli -------------------------------------------------------------------

// Residue of x modulo p for |x| < 2^24 and p <= 253, without division: q = rint(x/p) from one fused
// multiply-add against 1.5*2^23 (whose mantissa then holds q), r = x - q p.  1/p carries a relative error
// of 2^-24, so |x/p - q| <= 1/2 + |x| 2^-24 / p and |r| <= p/2 + 1: a valid representative that fits int8
// (|r| <= 127), not always the canonical one.
__device__ __forceinline__ int mod_near(int x, float inv_p, int p) {
  const float f = __builtin_fmaf((float)x, inv_p, 12582912.0f);
  const int q = __float_as_int(f) - 0x4B400000;
  return x - __mul24(q, p);
}

// Low byte of that residue: the constant term 2^22 * p of the mantissa trick is a multiple of 256 and drops out.
// (Written as the full-rate 24-bit multiply-add itself: since only the low byte is kept, the compiler would
// otherwise swap it for a quarter-rate 64-bit multiply-add.)
__device__ __forceinline__ uint32_t mod_lowbyte(int x, float inv_p, int neg_p) {
  const float f = __builtin_fmaf((float)x, inv_p, 12582912.0f);
  int r = __float_as_int(f);
  asm("v_mad_i32_i24 %0, %0, %1, %2" : "+v"(r) : "v"(neg_p), "v"(x));
  return (uint32_t)r;
}

// The same from an accumulator that started at KParams::acc_bias = 0x4B400000 + a instead of zero.  Read as binary32
// such an accumulator is the number 1.5*2^23 + a + x (|a + x| < 2^22: the sum stays in one binade, whose unit is 1), so
// the sum needs no conversion.  a is a multiple of 256 with 1.5*2^23 + a = s p: then f/p + (1.5*2^23 - s) = 1.5*2^23 + x/p,
// one multiply-add whose mantissa holds q = rint(x/p), and x - q p has its low byte in acc - q p.
// 1/p carries a relative error of 2^-24 and f < 2^24, so x/p is off by less than 1/p and |x - q p| <= p/2 + 1.
// Cost of the arithmetic on this chip, cycles per wave and SIMD: the float multiply-add with all operands in vector
// registers 2.6 (with a scalar operand 4.8), v_mad_i32_i24 4.8, the conversion this saves 4.2.  The caller keeps inv_p
// and quot_bias in vector registers (in_vgpr()).
__device__ __forceinline__ uint32_t biased_lowbyte(int acc, float inv_p, float quot_bias, int neg_p) {
  const float f = __builtin_fmaf(__int_as_float(acc), inv_p, quot_bias);
  int r = __float_as_int(f);
  asm("v_mad_i32_i24 %0, %0, %1, %2" : "+v"(r) : "s"(neg_p), "v"(acc));
  return (uint32_t)r;
}

// The same low byte as mod_lowbyte(x), to the bit, from an accumulator 0x4B400000 + x: read as binary32 it is 1.5*2^23 + x, and one
// subtraction (2.6 cycles) gives the x that mod_lowbyte() converts (4.2).  The caller keeps magic = 1.5*2^23 and inv_p in vector registers.
__device__ __forceinline__ uint32_t centred_lowbyte(int acc, float magic, float inv_p, int neg_p) {
  const float f = __builtin_fmaf(__int_as_float(acc) - magic, inv_p, magic);
  int r = __float_as_int(f);
  asm("v_mad_i32_i24 %0, %0, %1, %2" : "+v"(r) : "s"(neg_p), "v"(acc));
  return (uint32_t)r;
}

// A wave-uniform value in a vector register, hidden from the optimiser (which would put it back into a scalar one).
template <typename T>
__device__ __forceinline__ T in_vgpr(T v) {
  asm("" : "+v"(v));
  return v;
}

// c * (low 24 bits of w) + acc modulo 2^32, c < 2^24 wave-uniform: one instruction (the compiler, left to choose, splits
// the products from their sums or takes 64-bit multiply-adds, each of which costs more than the 4.8 cycles of this).
// `after`: what a compiler's instruction made of w.
template <typename T>
__device__ __forceinline__ uint32_t mad_u24(uint32_t c, uint32_t w, uint32_t acc, T after) {
  asm("v_mad_u32_u24 %0, %1, %2, %0" : "+v"(acc) : "s"(c), "v"(w), "v"(after));
  return acc;
}

// Low 32 bits of c * v, c wave-uniform (4.4 cycles, full rate on this chip).
__device__ __forceinline__ uint32_t mul_lo(uint32_t c, uint32_t v) {
  asm("v_mul_lo_u32 %0, %1, %0" : "+v"(v) : "s"(c));
  return v;
}

// That residue plus p (so that it is positive), 8-bit p: the low 24 bits of the biased float are 2^22 + q, the
// 24-bit multiply-add gives x - q p - 2^22 p + bias with bias = 2^22 p + p.  Four full-rate instructions.
__device__ __forceinline__ uint32_t mod_near_plus_p(int x, float inv_p, int neg_p, int bias) {
  const float f = __builtin_fmaf((float)x, inv_p, 12582912.0f);
  int r = __float_as_int(f);
  asm("v_mad_i32_i24 %0, %0, %1, %2" : "+v"(r) : "v"(neg_p), "v"(x + bias));
  return (uint32_t)r;
}

// byte 0 of a, b, c, d -> one word (the selectors sit in scalar registers: 4.4 cycles each)
__device__ __forceinline__ uint32_t pack_low_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  const uint32_t ab = __builtin_amdgcn_perm(b, a, 0x0c0c0400u);
  const uint32_t cd = __builtin_amdgcn_perm(d, c, 0x0c0c0400u);
  return __builtin_amdgcn_perm(cd, ab, 0x05040100u);
}

// ---- residues of 16-bit moduli ------------------------------------------------------------------
// A residue is stored as two signed bytes, value = 256*h + l, which covers [-32896, 32639]; every class
// modulo p <= 65521 has a representative there.

// Representative of x = 65536 hh + 256 hl + ll modulo p with |r| <= p/2 + 1, |x| < 2^52: the sum, the quotient estimate and the
// remainder in binary64 (the sum and the remainder exact): nine instructions, about thirty with the sum, the quotient and its
// product as 64-bit integers.  64 -> 64 channels, 16-bit moduli, at 112 x 112, batch 8: GEMM 31.6 -> 21.9 us, inverse transform 23.2 -> 19.1,
// input transform (mod_near32()) 26.2 -> 24.4.
__device__ __forceinline__ double mod_near64(int hh, int hl, int ll, double inv_pd, double p) {
  const double x = __builtin_fma((double)hh, 65536.0, __builtin_fma((double)hl, 256.0, (double)ll));
  return __builtin_fma(-__builtin_rint(x * inv_pd), p, x);
}

// The same of a 32-bit x.
__device__ __forceinline__ int mod_near32(int x, double inv_pd, int p) { return x - __double2int_rn((double)x * inv_pd) * p; }

// move a representative with |r| <= 32761 into the storable range
__device__ __forceinline__ int storable16(int r, int p) { return r > 32639 ? r - p : r; }

}  // namespace rnswino
