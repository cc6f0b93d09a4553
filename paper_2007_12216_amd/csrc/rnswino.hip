// rnswino: C ABI entry points (host side) and kernel dispatch for gfx950.
//
// Pipeline of one layer (paper section 6):
//   K0  filter transform   U = G g G^T mod p                 (offline, once per weight set)   k_filter_transform.hpp
//   K1  input transform    V = B^T d B mod p                 (int8 MFMA, Kronecker form)      k_input_transform.hpp
//   K2  residue GEMM       O = sum_c U V mod p               (int8 MFMA)                      k_residue_gemm.hpp
//   K3  inverse transform  Y = A^T O A mod p, then CRT to int32 (int8 MFMA, Kronecker form)   k_inverse_crt.hpp
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "k_direct_conv.hpp"
#include "k_filter_transform.hpp"
#include "k_glue.hpp"
#include "k_input_transform.hpp"
#include "k_inverse_crt.hpp"
#include "k_residue_gemm.hpp"
#include "k_residue_gemm_lds.hpp"
#include "k_transform_gemm.hpp"
#include "layout.hpp"
#include "plan.hpp"
#include "rnswino.h"

using namespace rnswino;

// Workspace of rnswino_conv2d_static(): device memory that is part of the loaded code object, so the entry point needs
// no allocation.  Every GPU holds its own copy at its own address; in host code the name below is only a handle for
// hipGetSymbolAddress(), never an address to hand to a kernel.
static __device__ __align__(256) unsigned char scratch[RNSWINO_STATIC_WORKSPACE_BYTES];

namespace {

// Address of `scratch` on each device, looked up once per device (with that device current) when the first plan is
// made there; rnswino_conv2d_static() only reads it.
constexpr int MAX_DEVICES = 64;
std::mutex scratch_mutex;
void *scratch_ptr[MAX_DEVICES] = {};

int resolve_scratch(int dev) {          // called with device `dev` current
  if (dev < 0 || dev >= MAX_DEVICES) return RNSWINO_E_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (scratch_ptr[dev]) return RNSWINO_OK;
  void *ptr = nullptr;
  if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) { (void)hipGetLastError(); return RNSWINO_E_HIP; }
  scratch_ptr[dev] = ptr;
  return RNSWINO_OK;
}

// The largest |y| the plan has to represent: the worst case 2^14 r^2 C of int8 operands (sections 3, 5, 8), or the
// caller's tighter bound for the layer's actual weights (rnswino_desc_t::output_bound), whichever is smaller.
unsigned __int128 output_bound(const rnswino_desc_t &desc, const Dims &d) {
  const unsigned __int128 worst = (unsigned __int128)16384u * (unsigned)d.r * (unsigned)d.r * (unsigned)d.C;
  return desc.output_bound != 0 && (unsigned __int128)desc.output_bound < worst ? (unsigned __int128)desc.output_bound : worst;
}

KParams make_params(const rnswino_plan_t *pl) {
  KParams P;
  std::memset(&P, 0, sizeof(P));
  const Dims &d = pl->dims;
  P.N = d.N; P.C = d.C; P.K = d.K; P.H = d.H; P.W = d.W; P.r = d.r; P.m = d.m; P.t = d.t; P.pad = d.pad;
  P.Ho = d.Ho; P.Wo = d.Wo; P.th = d.th; P.tw = d.tw; P.T = d.T; P.n = d.n;
  P.TL = d.TL; P.Cq = d.Cq; P.Kg = d.Kg; P.Tg = d.Tg;
  P.Cp = d.Cp; P.Kp = d.Kp; P.Tp = d.Tp; P.P2 = d.P2; P.Q = d.Q;
  P.CB1 = d.CB1; P.KS1 = d.KS1; P.RP1 = d.RP1; P.RB3 = d.RB3; P.KS3 = d.KS3;
  P.crt24 = 1;
  for (int i = 0; i < d.n; ++i) {
    P.p[i] = (int)pl->desc.moduli[i];
    P.inv_p[i] = 1.0f / (float)pl->desc.moduli[i];
    P.inv_pd[i] = 1.0 / (double)pl->desc.moduli[i];
    P.crt_c[i] = pl->crt_c[i];
    if (!pl->crt_c_exact_small[i]) P.crt24 = 0;
    P.bias_p[i] = d.wide ? 0 : (int)(pl->desc.moduli[i] * 4194304u + pl->desc.moduli[i]);
    if (!d.wide) {
      const BiasedStart start = biased_start(P.p[i]);
      P.acc_bias[i] = start.acc_bias;
      P.quot_bias[i] = start.quot_bias;
    }
  }
  {
    // binary32 is enough for the CRT quotient when 2 * (worst-case |y|) <= 0.9 * prod p_i
    unsigned __int128 prod = 1;
    const unsigned __int128 cap = ((unsigned __int128)1 << 100);
    for (int i = 0; i < d.n; ++i) { prod *= pl->desc.moduli[i]; if (prod > cap) prod = cap; }
    const unsigned __int128 worst = output_bound(pl->desc, d);
    P.quot32 = (worst * 20 <= prod * 9) ? 1 : 0;
    // Fast conversion, binary32 quotient: the accumulators, read as binary32, are M + a_i with M = 1.5 * 2^23 and
    // |a_i| <= 2^22.  The sum starts at -M sum_i v_i (v_i: 1/p_i as rounded, so the rounding of 1/p_i counts for a_i
    // alone) and takes one multiply-add per residue; before residue i it lies within M sum_{l >= i} v_l +
    // 2^22 sum_{l < i} v_l of zero, and every step rounds by at most half an ulp of that: 0.021 for three moduli near 240,
    // 0.035 for four.  Enabled when the layer's worst case leaves twice the error below 0.49 - |y|/P, with the error taken
    // as no less than n + 1 roundings at 2B and 2B 2^-23, B = 2^22 sum_i 1/p_i (0.028 and 0.056): that keeps a reserve, and
    // layers beyond it take the binary64 quotient, whose cost they hardly see (1.3 times the instructions of a small stage).
    if (!d.wide && P.crt24 && prod < cap) {
      const double M = 12582912.0, A = 4194304.0;
      auto half_ulp = [](double bound, int mantissa) { int e = 0; std::frexp(bound, &e); return std::ldexp(1.0, e - mantissa - 1); };
      long double Bl = 0.0L;             // extended precision: the one rounding to binary64 is counted below
      double start = 0.0, done = 0.0, err = 0.0;
      uint32_t c32 = 0;
      for (int i = 0; i < d.n; ++i) {
        Bl += (long double)A / (long double)pl->desc.moduli[i];
        c32 += pl->crt_c[i];
        start += M * (double)P.inv_p[i];
      }
      double left = start;
      err += half_ulp(left, 24);                                 // the start itself
      for (int i = 0; i < d.n; ++i) {
        left -= M * (double)P.inv_p[i];
        done += A * (double)P.inv_p[i];
        err += half_ulp(std::fabs(left) + done, 24) + A * std::fabs((double)P.inv_p[i] - 1.0 / (double)pl->desc.moduli[i]);
      }
      const double B = (double)Bl;
      // The same sum over a_i + 2^22 in binary64 must find the quotient for every |y| <= (P - 1)/2, i.e. stay within
      // 1/(2P) of the true value: it takes n + 1 roundings of at most half an ulp of B = 2^22 sum_i 1/p_i, and the rounded
      // 1/p_i add at most 2B 2^-52 in all; twice that has to fit.
      const double err64 = (d.n + 1) * half_ulp(B, 53) + 2.0 * B * std::ldexp(1.0, -52);
      const double reserve = (d.n + 1) * half_ulp(2.0 * B, 24) + 2.0 * B * std::ldexp(1.0, -23);
      if ((double)worst / (double)prod + 2.0 * std::fmax(err, reserve) <= 0.49) P.fastcrt = 1;
      else if (2.0 * err64 <= 0.5 / (double)prod) P.fastcrt = 2;
      if (P.fastcrt == 1) {
        P.acc0 = 0x4B400000;             // the bits of M; its low 24 bits are 2^22
        // (the first residue's product takes all 32 bits of its accumulator)
        P.crt_sum0 = 0u - 4194304u * c32 - 0x4B000000u * pl->crt_c[0] + pl->prod_mod32 * 0x4B400000u;
        P.crt_fs0 = (float)(-start);
      } else if (P.fastcrt == 2) {
        P.acc0 = 4194304;
        P.crt_sum0 = 0u - 4194304u * c32;
        P.crt_fs0d = -B;
      }
    }
  }
  P.prod_mod32 = pl->prod_mod32;
  if (pl->d_tables) {                   // host-only plans are never executed: their table pointers stay null
    const char *base = (const char *)pl->d_tables;
    P.KG = (const int8_t *)(base + pl->off_KG);
    P.KB = (const int8_t *)(base + pl->off_KB);
    P.KA = (const int8_t *)(base + pl->off_KA);
  }
  return P;
}

// ---- the kernels' arguments (what changes from call to call is filled in there) and what they read from device memory ----
struct DeviceParams {
  ResidueParams residues;
  K3Params k3;
};
static_assert(sizeof(DeviceParams) <= PARAMS_BYTES, "build_tables() leaves them that much");
// The input transform and the GEMM in one kernel (k_transform_gemm.hpp).  TH: tile blocks of 16 a workgroup takes; RM: row blocks a wave multiplies at once;
// part: items of a workgroup, parts: what that splits the items of its tiles into; row_parts: packed layers, what the filters are split into; copies:
// workgroups that only copy the input into V's place (0: every other one copies a share).
struct K12Choice { bool fused, pack; int KS1, TH, RM, part; unsigned parts, row_parts, blocks, copies; };
struct LayerParams {
  KParams k;
  K1Args k1;
  K2Args k2;
  K12Args k12;
  K12Choice k12_choice;
  K3Args k3[3];               // per output mode
};

inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }
inline size_t elem_bytes(const Dims &d) { return d.wide ? 2 : 1; }
inline size_t v_bytes(const Dims &d) { return (size_t)d.n * d.P2 * d.Tp * d.Cp * elem_bytes(d); }
inline size_t o_bytes(const Dims &d) { return (size_t)d.n * d.Q * d.Kp * d.Tp * 4 * elem_bytes(d); }
inline size_t u_bytes(const Dims &d) { return (size_t)d.n * d.P2 * d.Kp * d.Cp * elem_bytes(d); }

// The plan's tables live on the device that was current when it was made: executing it from another device would hand
// the kernels pointers of the wrong GPU.
inline bool on_plan_device(const rnswino_plan_t *plan) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return false; }
  return dev == plan->device;
}

inline int launch_status() { return hipGetLastError() == hipSuccess ? RNSWINO_OK : RNSWINO_E_HIP; }

inline unsigned blocks_for(long long total, int bs) { return (unsigned)((total + bs - 1) / bs); }

// Optional pair of events that receive the kernel's own start and stop timestamps.
struct Timing {
  hipEvent_t start = nullptr, stop = nullptr;
};

template <typename Kern, typename... Args>
inline void launch(Kern kern, dim3 grid, size_t lds, hipStream_t st, Timing tm, Args... args) {
  if (tm.start || tm.stop)
    hipExtLaunchKernelGGL(kern, grid, dim3(256), lds, st, tm.start, tm.stop, 0, args...);
  else
    hipLaunchKernelGGL(kern, grid, dim3(256), lds, st, args...);
}

// =============================================================================================
// Kernel selection.  Which instantiation of each kernel a layer runs, and its grid, is decided here from the plan's
// sizes alone (no GPU needed), so that rnswino_plan_describe() can report it and the launches below cannot disagree
// with the report.
// =============================================================================================

struct K1Choice { int KS1; bool wide, pack, tiles; long long units; unsigned gx, gy, gz; };

K1Choice choose_k1(const Dims &d, int n_cus) {
  K1Choice c;
  c.KS1 = d.KS1 < 4 ? d.KS1 : 4;
  c.wide = d.wide != 0;
  c.pack = d.TL > 1;
  c.tiles = d.vlane != 0;
  const long long units = c.tiles ? 4LL * (d.Tp / 16) * (d.Cp / 64) : (long long)d.Tg * (d.Cp / 64);
  c.units = units;
  // x: multiple of 8 (see kernels_common.hpp); y: one block per residue, or one block for all residues when there are
  // enough units to fill the chip (the pixel gather is then done once instead of n times; measured on the VGG16
  // stack, two blocks per CU are already enough for that to win; of the 16-tile blocks, which gather sixteen times as much, three
  // for every four CUs: 128 -> 128 at 56 x 56, batch 8, 200 units 36.0 us a layer split, 34.5 not, and at 112 x 112, batch 1, 104
  // units 26.4 and 28.3; with 200 units only layers of t <= 8 and planes of one tile still take them)
  c.gx = (unsigned)((units + 7) / 8 * 8);
  c.gy = (unsigned)(units >= (c.tiles ? 192 : 512) ? 1 : d.n);
  // Where that leaves half of the CUs without a block and a wave more than one group of column blocks (t >= 12), two blocks share them,
  // each gathering anew.  345 layers (two to six 8-bit moduli, two and three 16-bit ones; 3 to 512 channels at 14 x 14 to 80 x 80, batch 1 to 8; us per
  // layer replayed from a graph): up to 128 blocks of 256 CUs two take 0.97 of one's time with 8-bit and 0.955 with 16-bit moduli at t = 12, where the
  // second has work for one wave, 0.945 and 0.91 at t = 13 to 16 (F(14,3), 128 -> 64 at 24 x 24, batch 3, four 8-bit 11.7 and 11.0, 128 -> 128 at 20 x 20, two
  // 16-bit 15.5 and 13.9); with 129 to 160 blocks 0.985 (256 -> 64 at 40 x 40, four 8-bit 14.6 and 14.6), to 256 0.99, above 1.00.
  const int cus = n_cus > 0 ? n_cus : 256;
  c.gz = !c.tiles && c.gy > 1 && 2 * units * d.n <= cus && d.CB1 > 4 * K1_CPW ? 2 : 1;
  return c;
}

// the device block: residues' constants, and what the inverse transform converts with (the same in every output mode)
ResidueParams make_residues(const Dims &d, const KParams &P) {
  ResidueParams q;
  std::memset(&q, 0, sizeof(q));
  for (int i = 0; i < d.n; ++i) {
    q.res[i] = {P.inv_p[i], P.quot_bias[i], -P.p[i], P.acc_bias[i]};
    q.inv_pd[i] = P.inv_pd[i];
  }
  return q;
}

// the multiplier of a division into an argument of its own; returns the shift
inline uint32_t store_div(uint32_t d, uint32_t &mul) {
  const FastDiv f = make_fast_div(d);
  mul = f.mul;
  return f.shift;
}

K1Args make_k1(const Dims &d, const KParams &P, const DeviceParams *dev, int n_cus) {
  const K1Choice c = choose_k1(d, n_cus);
  K1Args q;
  std::memset(&q, 0, sizeof(q));
  q.more = dev ? &dev->residues : nullptr;
  q.KB = P.KB;
  q.units = (int)c.units;
  q.per_xcd = (int)(c.gx / 8);
  q.ncb = d.Cp / 64;
  uint32_t cq_shift = 0;
  while ((1 << cq_shift) < d.Cq) ++cq_shift;
  const uint32_t s_ncb = store_div((uint32_t)q.ncb, q.ncb_mul), s_tw = store_div((uint32_t)d.tw, q.tw_mul), s_th = store_div((uint32_t)d.th, q.th_mul);
  q.shifts = pack_bytes(s_ncb, s_tw, s_th, cq_shift);
  q.sizes = pack_bytes((uint32_t)d.m, (uint32_t)d.t, (uint32_t)d.n, c.gy > 1 ? c.gz : 0);
  q.C = d.C; q.H = d.H; q.W = d.W; q.pad = d.pad; q.tw = d.tw; q.th = d.th; q.T = d.T; q.Tg = d.Tg;
  q.total = (long long)d.N * d.C * d.H * d.W;
  return q;
}

// NTB = 16-tile column blocks per wave (1, 2 or 4, the smallest that covers Tp up to 64); KS = contraction steps
// in flight, limited by the register budget of the variant; RM = 16-row blocks per wave.
// lds: the LDS-tiled kernel (8-bit moduli): WM x WN waves of RM x NTB fragments each, S steps in flight.
struct K2Choice { int KS, NTB, RM; bool wide; int xgroup; unsigned blocks; bool lds; int WM, WN, S; };

// L2-aware grouping of the x index (see the kernels): brf / btf = row / tile fragments per workgroup
void k2_grid(const Dims &d, int brf, int btf, K2Choice &c) {
  const int ntb = d.Tp / 16;
  const long long pl = c.wide ? 2 : 1;
  const long long nxh = (d.n * d.Q + 7) / 8, gy = (d.Kp / 16 + brf - 1) / brf, gz = (ntb + btf - 1) / btf;
  const long long u_x = 4LL * d.Kp * d.Cp * pl, v_slice = 4LL * 16 * btf * d.Cp * pl;
  long long xgroup = gz == 1 ? 1 : (3LL << 20) / (u_x + 2 * v_slice);
  xgroup = xgroup < 1 ? 1 : (xgroup > nxh ? nxh : xgroup);
  if (xgroup > 1 && xgroup < nxh && (xgroup & 1) == 0) --xgroup;
  c.xgroup = (int)xgroup;
  c.blocks = (unsigned)(8 * ((nxh + xgroup - 1) / xgroup * xgroup) * gy * gz);
}

K2Choice choose_k2(const Dims &d, uint32_t flags) {
  K2Choice c;
  c.wide = d.wide != 0;
  c.lds = false; c.WM = c.WN = c.S = 0;
  const int ntb = d.Tp / 16, ncb = d.Cp / 64;
  c.NTB = ntb == 1 ? 1 : ntb == 2 ? 2 : 4;
  if (!c.wide && (flags & RNSWINO_FLAG_GEMM_BLOCK_64X16)) {
    // measurement only: the GEMM on the block a fused GEMM + inverse transform could hold on chip
    c.lds = true; c.KS = 0; c.NTB = 1; c.WM = 4; c.WN = 1; c.RM = 1; c.S = 4;
    k2_grid(d, 4, 1, c);
    return c;
  }
  if (!c.wide && d.Kp >= 128) {
    // LDS-tiled kernel where it measured faster than the register-direct one (VGG16 stack at batch 8, the 256-channel
    // layer at batch 1): 128 x 64 blocks for 33..64 tiles; 128 x 128 blocks for many tiles and a contraction of two or
    // more steps (with a single step the pipeline over the four points never fills), unless the last tile block would be
    // mostly padding (more than a tenth of the tile blocks wasted)
    const int tb128 = (ntb + 7) / 8;
    const bool few = ntb == 3 || ntb == 4;
    const bool many = ntb >= 5 && ncb >= 2 && tb128 * 80 <= ntb * 11;
    if (few || many) {
      c.lds = true; c.KS = 0; c.NTB = 4;
      if (few) { c.WM = 4; c.WN = 1; c.RM = 2; c.S = 4; }
      else { c.WM = 2; c.WN = 2; c.RM = 4; c.S = 3; }
      k2_grid(d, c.WM * c.RM, c.WN * c.NTB, c);
      return c;
    }
  }
  // 64 rows per wave when K is large (V re-reads dominate), the contraction has more than one step and that still
  // leaves >= 4 blocks per CU; measured on the VGG16 stack this wins for K >= 256 and loses for K <= 128 (8-bit
  // moduli, full-width tiles only: the register budget of the other variants is spent on their extra accumulators)
  const long long big_blocks = (long long)((d.n * d.Q + 7) / 8 * 8) * ((d.Kp + 63) / 64) * ((ntb + c.NTB - 1) / c.NTB);
  if (!c.wide && c.NTB == 4 && d.Kp >= 256 && ncb >= 2 && big_blocks >= 1024) {
    c.RM = 4;
    c.KS = ncb % 2 == 0 ? 2 : 1;
  } else {
    const int ksmax = c.wide ? (c.NTB == 1 ? 4 : c.NTB == 2 ? 2 : 1) : 4;
    c.RM = 2;
    c.KS = (ksmax >= 4 && ncb % 4 == 0) ? 4 : (ksmax >= 2 && ncb % 2 == 0) ? 2 : 1;
  }
  // One-dimensional grid: the kernel derives (x, row block, tile block) from the id in an order that suits the L2s.
  // A slice of U is used again after xgroup * gy workgroups of its XCD, which meanwhile touch xgroup * (U of one x +
  // about two tile-block slices of V): xgroup is the largest count for which that stays within 3 of the L2's 4 MiB.
  // With a single tile block nothing of U is used twice: one x at a time, so that the workgroups in flight on an XCD
  // read neighbouring row blocks of one U slab (measured: 3-7 % faster than walking over all x at once).  Even group
  // sizes measured slower (they run into each other in the L2 channels).
  k2_grid(d, c.RM, c.NTB, c);
  return c;
}

K2Args make_k2(const Dims &d, const DeviceParams *dev, uint32_t flags) {
  const K2Choice c = choose_k2(d, flags);
  const int brf = c.lds ? c.WM * c.RM : c.RM, btf = c.lds ? c.WN * c.NTB : c.NTB;
  K2Args q;
  std::memset(&q, 0, sizeof(q));
  q.more = dev ? &dev->residues : nullptr;
  q.nkb = d.Kp / 16; q.ntb = d.Tp / 16; q.ncb = d.Cp / 64;
  q.xgroup = c.xgroup; q.gy = (q.nkb + brf - 1) / brf; q.gz = (q.ntb + btf - 1) / btf;
  const uint32_t s_x = store_div((uint32_t)c.xgroup, q.xgroup_mul), s_y = store_div((uint32_t)q.gy, q.gy_mul), s_z = store_div((uint32_t)q.gz, q.gz_mul);
  q.shifts = pack_bytes(s_x, s_y, s_z, store_div((uint32_t)d.Q, q.Q_mul));
  q.sizes = pack_bytes((uint32_t)d.Q, d.vlane ? 1 : 0, 0, 0);
  q.xs = d.n * d.Q; q.P2 = d.P2; q.slabs = d.n * d.P2;
  return q;
}

K12Choice choose_k12(const Dims &d, uint32_t flags, int n_cus) {
  K12Choice c{};
  const long long elements = (long long)d.N * d.C * d.H * d.W;
  const int nkb = d.Kp / 16, ntb = d.Tp / 16, cus = n_cus > 0 ? n_cus : 256, items = (d.n * d.Q + 3) / 4;
  // 8-bit moduli, one channel block, row segments with 32-bit offsets (as for k1_input_transform_tiles), and where it is faster.
  // The lines lie where random layers (4340 in profiles/transform_gemm_dispatch.csv: us as one kernel and as two, the input's copy included) stop gaining:
  // inside them 3695 take 0.875 of the time of two kernels in the mean, 91 of them (2.5 %) over 1.02 (up to 1.14); outside 645 take 1.004, 240 of them over 1.02.
  // - Filters: fragments of U cross the L2 once per 32 (t > 10: 16) tiles.  Over 160 filters at t <= 10 the mean is 0.97 (t <= 8; 1.03 at t = 9, 10), over
  //   128 at t > 10 1.00 to 1.03 (42 -> 281 at 79 x 77, F(9,3), six moduli, batch 9, 147.8 -> 172.0).
  // - (Tile block, item) pairs: with few, the few workgroups' latencies decide.  t <= 8 from 150 on 0.86 (40 -> 10 at 182 x 144, F(4,5), batch 9, 186.8 -> 88.2),
  //   t = 9, 10 from 300 on 0.90 (150 to 300: 0.96, up to 1.04), t = 11, 12 from 400 on 0.87, t > 12, whose rows take unaligned loads, from 2400 on 0.86 (1400
  //   to 2400: 0.97, up to 1.16).
  // - Packed layers of up to four channels: a workgroup gathers for one item, which pays for itself where (item, filter) pairs are 800 and more, or (tile
  //   block, item, filter) triples 37 500: 0.90.  With fewer 1.03 (1 -> 13 at 221 x 240, F(4,4), batch 6, 41.6 -> 57.5); below 12 500 triples the GPU is not full.
  if (d.wide || d.Cp != 64 || (flags & (RNSWINO_FLAG_GEMM_BLOCK_64X16 | RNSWINO_FLAG_SEPARATE_KERNELS)) || elements < 16 ||
      elements + d.W + 2LL * d.pad + 16 >= (1LL << 31))
    return c;
  c.pack = d.TL == 16 && d.KS1 <= 2;
  const long long pairs = (long long)ntb * items;
  if (c.pack) c.fused = d.K <= 8192 && pairs * d.K >= ((long long)items * d.K >= 800 ? 12500 : 37500);
  else c.fused = d.TL == 1 && nkb <= (d.KS1 <= 2 ? 10 : 8) && pairs >= (d.KS1 == 1 ? 150 : d.KS1 == 2 ? 300 : d.KS1 == 3 ? 400 : 2400);
  if (!c.fused) return c;
  c.KS1 = d.KS1;
  // The split.  A workgroup takes 5 us to gather (3 on packed layers) and 0.8 us an item plus 0.4 per 32 rows and 16 tiles (0.08 per filter); two on a compute
  // unit take 1.7 (1.5) times the work of one, and so does one of 32 tiles.  Over 43 layers the choice takes 0.2 % longer than the best split (6 % at
  // worst), over 21 packed ones 0.2 % (3 %).  Packed layers take one item a workgroup, and up to three parts of the filters more than the 64 that fit a wave's lanes
  // ask for (two items: 3 -> 64 at 224 x 224, batch 8, 110.9 us a layer).
  const bool wide_tile = d.KS1 > 2;                    // one workgroup of 16 tiles a compute unit: 6 us to gather, 1 us an item plus 0.2 per 16 rows of a wave
  const double gather = c.pack ? 3.0 : wide_tile ? 6.0 : 5.0, factor = c.pack ? 1.5 : 1.7;
  const int row_parts0 = c.pack ? (d.K + 63) / 64 : 1, row_parts1 = c.pack ? row_parts0 + 3 : 1, most = c.pack ? 1 : items;
  double best = 0.0;
  for (int TH = 1; TH <= (wide_tile ? 1 : 2); ++TH) {
    const int quads = k12_quads(c.KS1, TH), RM = !c.pack && nkb > quads ? 2 : 1, sets = (nkb + RM * quads - 1) / (RM * quads), groups = (ntb + TH - 1) / TH;
    for (int row_parts = row_parts0; row_parts <= row_parts1; ++row_parts) {
      const double item = wide_tile ? 1.0 + 0.2 * sets * RM : 0.8 + (c.pack ? 0.08 * ((d.K + row_parts - 1) / row_parts) : 0.2 * sets * RM * TH);
      for (int part = 1; part <= most; ++part) {
        const long long rounds = ((long long)groups * row_parts * ((items + part - 1) / part) + cus - 1) / cus;
        const double alone = gather + part * item, together = gather + factor * part * item;
        const double cost = wide_tile ? rounds * alone : TH == 2 ? rounds * together : rounds / 2 * 1.1 * together + rounds % 2 * alone;
        if (c.TH == 0 || cost < best) { best = cost; c.TH = TH; c.RM = RM; c.part = part; c.row_parts = (unsigned)row_parts; }
      }
    }
  }
  c.parts = (unsigned)((items + c.part - 1) / c.part);
  c.blocks = (unsigned)(((long long)((ntb + c.TH - 1) / c.TH) * c.parts * c.row_parts + 7) / 8 * 8);
  // The input's copy (V, whose place it takes, is never smaller: a tile of t x t pixels for m x m outputs, 64 channels): by workgroups of its own on the compute
  // units that the others leave idle, if those have time for it at 32 KB a us each (measured 36), else by all (figures: InputCopy).
  const unsigned idle = std::min(((unsigned)cus - 1 - (c.blocks - 1) % (unsigned)cus) / 8 * 8, 248u);
  if ((double)elements <= 32e3 * idle * best) c.copies = idle;
  return c;
}

K12Args make_k12(const Dims &d, const KParams &P, const DeviceParams *dev, const K12Choice &c) {
  K12Args q;
  std::memset(&q, 0, sizeof(q));
  if (!c.fused) return q;
  q.more = dev ? &dev->residues : nullptr;
  q.KB = P.KB;
  q.ntb = d.Tp / 16; q.nkb = d.Kp / 16;
  q.per_xcd = (int)(c.blocks / 8);
  const uint32_t s_groups = store_div((uint32_t)((q.ntb + c.TH - 1) / c.TH), q.tile_groups_mul), s_tw = store_div((uint32_t)d.tw, q.tw_mul), s_th = store_div((uint32_t)d.th, q.th_mul);
  q.shifts = pack_bytes(s_groups, s_tw, s_th, c.row_parts);
  q.sizes = pack_bytes((uint32_t)d.m, (uint32_t)d.t, (uint32_t)d.n, (uint32_t)c.part);
  q.Q_mul = group_mul((uint32_t)d.Q);
  q.C = d.C; q.H = d.H; q.W = d.W; q.pad = d.pad; q.tw = d.tw; q.th = d.th; q.T = d.T;
  q.total = (int)((long long)d.N * d.C * d.H * d.W);
  q.kept = (uint32_t)(align256(v_bytes(d)) / 256) | c.copies / 8 << 27;          // (V has at most four times the bytes of O, below 16 GiB)
  return q;
}

// stream: the streaming variant (8-bit moduli, table of all residues at most 64 KiB, n * KS3 <= 8: O operand in
// registers) for layers with 5000 and more units (us per layer, streaming / block form: 3136 units 33.7 / 32.0, 3200 35.0 / 33.5,
// 4096 37.0 / 36.5, 6400 60.1 / 60.1, 12544 63.9 / 66.6, 25088 160 / 184; four resident blocks per CU already take 4096);
// fast: conversion out of the RNS from unreduced accumulators; m8: the 8 x 8 store path of the streaming variant
// (int32 output: only with rows that keep four outputs 16-byte aligned; int8 output: only with an even row length).
struct K3Choice { bool stream, wide, fast, m8; int NRES, KS3; unsigned gx, gy; size_t lds; };

K3Choice choose_k3(const Dims &d, const KParams &P, int n_cus, int epi) {
  K3Choice c;
  c.wide = d.wide != 0;
  c.NRES = d.n;
  c.KS3 = d.KS3 < 4 ? d.KS3 : 4;
  c.fast = !c.wide && P.fastcrt != 0;
  c.stream = !c.wide && d.n * d.KS3 <= 8 && d.n <= 4 && d.KS3 <= 2 && (size_t)d.n * d.RB3 * d.KS3 * 1024 <= 65536 &&
             (long long)d.Kg * (d.Tp / 16) >= 5000;
  c.m8 = false;
  c.lds = 0;
  if (c.stream) {
    const long long blocks = ((long long)d.Kg * (d.Tp / 16) + 3) / 4;
    const long long max_blocks = n_cus > 0 ? 4LL * n_cus : K3_STREAM_BLOCKS;
    c.gx = (unsigned)(blocks < max_blocks ? blocks : max_blocks);
    c.gy = 1;
    c.lds = (size_t)d.n * d.RB3 * d.KS3 * 1024;
    c.m8 = c.fast && d.m == 8 && (epi == 0 ? (d.Wo & 3) == 0 : (d.Wo & 1) == 0);
  } else {
    const long long units = ((long long)d.Kg * d.Tg + 15) / 16;
    c.gx = (unsigned)((units + 7) / 8 * 8);       // x multiple of 8: see kernels_common.hpp
    // y: the blocks of a unit each load its operand, so no more of them than it takes to have two blocks per compute unit
    // (28 x 28, m = 14: 512 units 47.9 us a layer with one block each, 48.9 with four; 128 units 61.0 and 57.5)
    const long long most = (d.RB3 + 3) / 4, want = (512 + c.gx - 1) / c.gx;
    c.gy = (unsigned)(want < most ? want : most);
  }
  return c;
}

K3Args make_k3(const Dims &d, const KParams &P, const DeviceParams *dev, int n_cus, int epi) {
  const K3Choice c = choose_k3(d, P, n_cus, epi);
  K3Args q;
  std::memset(&q, 0, sizeof(q));
  q.more = dev ? &dev->k3 : nullptr;
  q.KA = P.KA;
  q.npairs = d.Kg * d.Tg;                          // below 2^31 (checked when the plan is made)
  q.units = c.stream ? d.Kg * (d.Tp / 16) : (q.npairs + 15) / 16;
  q.per_xcd = (int)(c.gx / 8);
  uint32_t tl_shift = 0;
  while ((1 << tl_shift) < d.TL) ++tl_shift;
  const uint32_t s_Tg = store_div((uint32_t)d.Tg, q.Tg_mul), s_tw = store_div((uint32_t)d.tw, q.tw_mul), s_th = store_div((uint32_t)d.th, q.th_mul);
  q.shifts = pack_bytes(s_Tg, s_tw, s_th, tl_shift);
  q.sizes = pack_bytes((uint32_t)d.Q, (uint32_t)d.RB3, 4 * c.gy, (uint32_t)d.m);
  q.Tg = d.Tg; q.T = d.T; q.Tp = d.Tp; q.tw = d.tw; q.th = d.th; q.K = d.K; q.Ho = d.Ho; q.Wo = d.Wo; q.epi = epi;
  return q;
}

K3Params make_conversion(const Dims &d, const KParams &P, int n_cus) {
  K3Params q;
  std::memset(&q, 0, sizeof(q));
  q.fastcrt = P.fastcrt; q.crt24 = P.crt24; q.quot32 = P.quot32; q.acc0 = P.acc0; q.crt_sum0 = P.crt_sum0; q.prod_mod32 = P.prod_mod32;
  q.crt_fs0 = P.crt_fs0; q.crt_fs0d = P.crt_fs0d; q.inv_m = 1.0f / (float)d.m;
  q.by_ntb = make_fast_div((uint32_t)(d.Tp / 16));
  q.nwaves = 4 * (int)choose_k3(d, P, n_cus, 0).gx;    // (of a streaming grid: the same in every output mode)
  for (int i = 0; i < d.n; ++i) {
    q.crt_c[i] = P.crt_c[i]; q.inv_p[i] = P.inv_p[i]; q.p[i] = P.p[i]; q.bias_p[i] = P.bias_p[i]; q.inv_pd[i] = P.inv_pd[i]; q.pd[i] = (double)P.p[i];
  }
  return q;
}

// The instantiations that exist, as tables: the launches below and rnswino_kernel_variants() both expand them.
// Inverse transform: 16-bit moduli take the general conversion (any moduli count); with 8-bit moduli the conversion from
// unreduced accumulators needs every P/p_i below 2^24, i.e. at most four moduli, and sets of fewer than four moduli
// always qualify for it (their product leaves the binary64 quotient ample room), so the reduced form exists from four
// moduli on (with exactly four, only up to t = 13: a product large enough to rule the unreduced form out needs 253,
// which 14 or more interpolation points exclude).  The streaming kernel's 8 x 8 store path exists for the unreduced
// form only.  A launch function returns false when the choice has no instantiation; rnswino_plan() refuses such a plan.
#define RNSW_K1_TABLE(X) \
  X(1, false, false) X(1, false, true) X(1, true, false) X(1, true, true) X(2, false, false) X(2, false, true) X(2, true, false) X(2, true, true) \
  X(3, false, false) X(3, false, true) X(3, true, false) X(3, true, true) X(4, false, false) X(4, false, true) X(4, true, false) X(4, true, true)
#define RNSW_K1T_TABLE(X) X(1, false) X(1, true) X(2, false) X(2, true)
#define RNSW_K2_TABLE(X) \
  X(1, 1, 2, false) X(2, 1, 2, false) X(4, 1, 2, false) X(1, 2, 2, false) X(2, 2, 2, false) X(4, 2, 2, false) \
  X(1, 4, 2, false) X(2, 4, 2, false) X(4, 4, 2, false) X(1, 4, 4, false) X(2, 4, 4, false) \
  X(1, 1, 2, true) X(2, 1, 2, true) X(4, 1, 2, true) X(1, 2, 2, true) X(2, 2, 2, true) X(1, 4, 2, true)
#define RNSW_K2L_TABLE(X) X(2, 2, 4, 4, 3) X(4, 1, 2, 4, 4) X(4, 1, 1, 1, 4)
#define RNSW_K12_TABLE(X) \
  X(1, 1, 1, false) X(1, 1, 2, false) X(1, 2, 1, false) X(1, 2, 2, false) X(2, 1, 1, false) X(2, 1, 2, false) X(2, 2, 1, false) X(2, 2, 2, false) \
  X(3, 1, 1, false) X(3, 1, 2, false) X(4, 1, 1, false) X(4, 1, 2, false) \
  X(1, 1, 1, true) X(1, 2, 1, true) X(2, 1, 1, true) X(2, 2, 1, true)
#define RNSW_K3_NK(X, nres, wd, fs) X(nres, 1, wd, fs) X(nres, 2, wd, fs) X(nres, 3, wd, fs) X(nres, 4, wd, fs)
#define RNSW_K3_TABLE(X) \
  RNSW_K3_NK(X, 1, true, false) RNSW_K3_NK(X, 2, true, false) RNSW_K3_NK(X, 3, true, false) RNSW_K3_NK(X, 4, true, false) \
  RNSW_K3_NK(X, 5, true, false) RNSW_K3_NK(X, 6, true, false) RNSW_K3_NK(X, 7, true, false) RNSW_K3_NK(X, 8, true, false) \
  RNSW_K3_NK(X, 1, false, true) RNSW_K3_NK(X, 2, false, true) RNSW_K3_NK(X, 3, false, true) RNSW_K3_NK(X, 4, false, true) \
  X(4, 1, false, false) X(4, 2, false, false) X(4, 3, false, false) RNSW_K3_NK(X, 5, false, false) RNSW_K3_NK(X, 6, false, false) RNSW_K3_NK(X, 7, false, false) \
  RNSW_K3_NK(X, 8, false, false)
#define RNSW_K3S_M8(X, nres, ks3, fs) X(nres, ks3, fs, true) X(nres, ks3, fs, false)
#define RNSW_K3S_TABLE(X) \
  RNSW_K3S_M8(X, 1, 1, true) RNSW_K3S_M8(X, 1, 2, true) RNSW_K3S_M8(X, 2, 1, true) RNSW_K3S_M8(X, 2, 2, true) \
  RNSW_K3S_M8(X, 3, 1, true) RNSW_K3S_M8(X, 3, 2, true) RNSW_K3S_M8(X, 4, 1, true) RNSW_K3S_M8(X, 4, 2, true) \
  X(4, 1, false, false) X(4, 2, false, false)

// ---- K1 ----  (dry: only report whether the instantiation exists)
bool launch_k1(const Dims &d, int n_cus, const K1Args &L, const int8_t *x, int8_t *V, hipStream_t st, Timing tm, bool dry = false) {
  const K1Choice c = choose_k1(d, n_cus);
  const dim3 grid(c.gx, c.gy, c.gz);
  K1Args P = L;
  P.x = x; P.V = V;
#define RNSW_X(ks, pk) \
  if (c.tiles && c.KS1 == ks && c.pack == pk) { if (!dry) launch(k1_input_transform_tiles<ks, pk>, grid, 0, st, tm, P); return true; }
  RNSW_K1T_TABLE(RNSW_X)
#undef RNSW_X
#define RNSW_X(ks, wd, pk) \
  if (!c.tiles && c.KS1 == ks && c.wide == wd && c.pack == pk) { if (!dry) launch(k1_input_transform<ks, wd, pk>, grid, 0, st, tm, P); return true; }
  RNSW_K1_TABLE(RNSW_X)
#undef RNSW_X
  return false;
}

// ---- K2 ----
bool launch_k2(const Dims &d, uint32_t flags, const K2Args &L, const int8_t *U, const int8_t *V, uint32_t *O, hipStream_t st, Timing tm, bool dry = false) {
  const K2Choice c = choose_k2(d, flags);
  const dim3 grid(c.blocks);
  K2Args P = L;
  P.U = U; P.V = V; P.O = O;
  if (c.lds) {
#define RNSW_X(wm_, wn_, rm, ntb, s_) \
    if (c.WM == wm_ && c.WN == wn_ && c.RM == rm && c.NTB == ntb && c.S == s_) { \
      if (!dry) launch(k2_residue_gemm_lds<wm_, wn_, rm, ntb, s_>, grid, 0, st, tm, P); return true; }
    RNSW_K2L_TABLE(RNSW_X)
#undef RNSW_X
    return false;
  }
#define RNSW_X(ks, ntb, rm, wd) \
  if (c.KS == ks && c.NTB == ntb && c.RM == rm && c.wide == wd) { if (!dry) launch(k2_residue_gemm<ks, ntb, rm, wd>, grid, 0, st, tm, P); return true; }
  RNSW_K2_TABLE(RNSW_X)
#undef RNSW_X
  return false;
}

// ---- K1 and K2 in one ----
bool launch_k12(const K12Choice &c, const K12Args &L, const int8_t *x, const int8_t *U, uint32_t *O, hipStream_t st, bool dry = false) {
  const dim3 grid(c.copies + c.blocks);
  K12Args P = L;
  P.x = x; P.U = U; P.O = O;
#define RNSW_X(ks, groups, rm, pk) \
  if (c.KS1 == ks && c.TH == groups && c.RM == rm && c.pack == pk) { \
    if (!dry) hipLaunchKernelGGL((k12_transform_gemm<ks, groups, rm, pk>), grid, dim3(256 * k12_quads(ks, groups)), 0, st, P); return true; }
  RNSW_K12_TABLE(RNSW_X)
#undef RNSW_X
  return false;
}

// ---- K3 ----
bool launch_k3(const Dims &d, const LayerParams &L, int n_cus, int epi, int shift, const uint32_t *O, void *out, hipStream_t st,
               Timing tm, bool dry = false) {
  const K3Choice c = choose_k3(d, L.k, n_cus, epi);
  const dim3 grid(c.gx, c.gy);
  K3Args P = L.k3[epi];
  P.O = O; P.out = out; P.shift = shift;
  if (c.stream) {
#define RNSW_X(nres, ks3, fs, e8) \
    if (c.NRES == nres && c.KS3 == ks3 && c.fast == fs && c.m8 == e8) { \
      if (!dry) launch(k3_inverse_crt_stream<nres, ks3, fs, e8>, grid, c.lds, st, tm, P); return true; }
    RNSW_K3S_TABLE(RNSW_X)
#undef RNSW_X
    return false;
  }
#define RNSW_X(nres, ks3, wd, fs) \
  if (c.NRES == nres && c.KS3 == ks3 && c.wide == wd && c.fast == fs) { \
    if (!dry) launch(k3_inverse_crt<nres, ks3, wd, fs>, grid, 0, st, tm, P); return true; }
  RNSW_K3_TABLE(RNSW_X)
#undef RNSW_X
  return false;
}

// Every name of the tables above, one per line, as a profiler prints them.
std::string all_kernel_variants() {
  std::string out;
#define RNSW_X(ks, wd, pk) out += "k1_input_transform<" #ks ", " #wd ", " #pk ">\n";
  RNSW_K1_TABLE(RNSW_X)
#undef RNSW_X
#define RNSW_X(ks, pk) out += "k1_input_transform_tiles<" #ks ", " #pk ">\n";
  RNSW_K1T_TABLE(RNSW_X)
#undef RNSW_X
#define RNSW_X(ks, ntb, rm, wd) out += "k2_residue_gemm<" #ks ", " #ntb ", " #rm ", " #wd ">\n";
  RNSW_K2_TABLE(RNSW_X)
#undef RNSW_X
#define RNSW_X(wm_, wn_, rm, ntb, s_) out += "k2_residue_gemm_lds<" #wm_ ", " #wn_ ", " #rm ", " #ntb ", " #s_ ">\n";
  RNSW_K2L_TABLE(RNSW_X)
#undef RNSW_X
#define RNSW_X(ks, groups, rm, pk) out += "k12_transform_gemm<" #ks ", " #groups ", " #rm ", " #pk ">\n";
  RNSW_K12_TABLE(RNSW_X)
#undef RNSW_X
#define RNSW_X(nres, ks3, wd, fs) out += "k3_inverse_crt<" #nres ", " #ks3 ", " #wd ", " #fs ">\n";
  RNSW_K3_TABLE(RNSW_X)
#undef RNSW_X
#define RNSW_X(nres, ks3, fs, m8) out += "k3_inverse_crt_stream<" #nres ", " #ks3 ", " #fs ", " #m8 ">\n";
  RNSW_K3S_TABLE(RNSW_X)
#undef RNSW_X
  return out;
}

// epi: 0 = int32 y_dev; 1 / 2 = int8 act_dev after shift/clamp (/ and 2x2 max-pool)
int conv2d_impl(const rnswino_plan_t *plan, const int8_t *x_dev, const void *U_dev, int32_t *y_dev,
                void *workspace_dev, void *stream, void *const *events, int epi = 0, int shift = 0,
                int8_t *act_dev = nullptr) {
  if (!plan || !x_dev || !U_dev || !workspace_dev) return RNSWINO_E_INVALID;
  if (epi == 0 ? !y_dev : !act_dev) return RNSWINO_E_INVALID;
  if (plan->device < 0) return RNSWINO_E_NO_DEVICE;
  if (!on_plan_device(plan)) return RNSWINO_E_INVALID;
  if (((uintptr_t)U_dev | (uintptr_t)workspace_dev | (uintptr_t)y_dev) & 15) return RNSWINO_E_INVALID;
  if ((uintptr_t)act_dev & 3) return RNSWINO_E_INVALID;
  const Dims &d = plan->dims;
  const LayerParams &L = *(const LayerParams *)plan->kparams;
  hipStream_t st = (hipStream_t)stream;
  int8_t *Vp = (int8_t *)workspace_dev;
  uint32_t *Op = (uint32_t *)((char *)workspace_dev + align256(v_bytes(d)));
  Timing t1, t2, t3;
  if (events) {
    t1.start = (hipEvent_t)events[0]; t1.stop = (hipEvent_t)events[1];
    t2.start = (hipEvent_t)events[2]; t2.stop = (hipEvent_t)events[3];
    t3.start = (hipEvent_t)events[4]; t3.stop = (hipEvent_t)events[5];
  }
  // (rnswino_plan() has checked that all instantiations exist)
  if (L.k12_choice.fused && !events) {
    if (!launch_k12(L.k12_choice, L.k12, x_dev, (const int8_t *)U_dev, Op, st) ||
        !launch_k3(d, L, plan->n_cus, epi, shift, Op, epi == 0 ? (void *)y_dev : (void *)act_dev, st, t3))
      return RNSWINO_E_UNSUPPORTED;
    return launch_status();
  }
  if (!launch_k1(d, plan->n_cus, L.k1, x_dev, Vp, st, t1) || !launch_k2(d, plan->desc.flags, L.k2, (const int8_t *)U_dev, Vp, Op, st, t2) ||
      !launch_k3(d, L, plan->n_cus, epi, shift, Op, epi == 0 ? (void *)y_dev : (void *)act_dev, st, t3))
    return RNSWINO_E_UNSUPPORTED;
  // in the workspace is then what the one kernel leaves there
  if (L.k12_choice.fused) hipLaunchKernelGGL(k_keep_input, dim3(256), dim3(256), 0, st, x_dev, Vp, (uint32_t)L.k12.total,
                                                share_of((uint32_t)L.k12.total, 256, 4096));
  return launch_status();
}

}  // namespace

// =============================================================================================
// C ABI
// =============================================================================================

extern "C" {

int rnswino_plan(rnswino_plan_t **out, const rnswino_desc_t *desc) {
  if (out) *out = nullptr;
  if (!out || !desc) return RNSWINO_E_INVALID;
  rnswino_plan_t *pl = new (std::nothrow) rnswino_plan_t();
  if (!pl) return RNSWINO_E_INVALID;
  pl->desc = *desc;
  pl->device = -1;
  pl->n_cus = 0;
  pl->d_tables = nullptr;
  pl->d_tables_bytes = 0;
  pl->kparams = nullptr;
  int rc = validate_desc(*desc, pl->dims);
  if (rc != RNSWINO_OK) { delete pl; return rc; }
  const Dims &d = pl->dims;
  pl->tf.resize(d.n);
  for (int i = 0; i < d.n; ++i) {
    rc = build_transforms(d.m, d.r, desc->moduli[i], pl->tf[i]);
    if (rc != RNSWINO_OK) { delete pl; return rc; }
  }
  // dynamic range (prod - 1)/2, saturated, against the worst case 2^14 r^2 C (sections 3, 5, 8)
  unsigned __int128 prod = 1;
  const unsigned __int128 cap = ((unsigned __int128)1 << 100);
  for (int i = 0; i < d.n; ++i) { prod *= desc->moduli[i]; if (prod > cap) prod = cap; }
  const unsigned __int128 half = (prod - 1) / 2;
  pl->dyn_range = half > (unsigned __int128)INT64_MAX ? INT64_MAX : (int64_t)half;
  const unsigned __int128 worst = output_bound(*desc, d);
  if (!(desc->flags & RNSWINO_FLAG_ALLOW_UNCHECKED_RANGE) && worst > half) { delete pl; return RNSWINO_E_RANGE; }
  std::memset(pl->mrc_inv, 0, sizeof(pl->mrc_inv));
  for (int l = 0; l < d.n; ++l)
    for (int j = l + 1; j < d.n; ++j) pl->mrc_inv[l][j] = (uint32_t)mod_inverse(desc->moduli[l], desc->moduli[j]);

  std::vector<char> &blob = pl->h_tables;
  build_tables(*pl, blob);
  // (the new plan owns what follows, and its destruction gives it back)
  auto fail = [&](int code) { (void)hipGetLastError(); (void)rnswino_plan_destroy(pl); return code; };
  const bool on_device = !(desc->flags & RNSWINO_FLAG_HOST_ONLY);
  if (on_device) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return fail(RNSWINO_E_NO_DEVICE);
    if (hipMalloc(&pl->d_tables, pl->d_tables_bytes) != hipSuccess) { pl->d_tables = nullptr; return fail(RNSWINO_E_HIP); }
    pl->device = dev;
    rc = resolve_scratch(dev);
    if (rc != RNSWINO_OK) return fail(rc);
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess) pl->n_cus = cus;
    else (void)hipGetLastError();
  }
  LayerParams *params = new (std::nothrow) LayerParams;
  pl->kparams = params;
  if (!params) return fail(RNSWINO_E_INVALID);
  params->k = make_params(pl);
  const DeviceParams *dev_params = on_device ? (const DeviceParams *)((char *)pl->d_tables + pl->off_params) : nullptr;   // (host-only plans are never executed)
  params->k1 = make_k1(d, params->k, dev_params, pl->n_cus);
  params->k2 = make_k2(d, dev_params, pl->desc.flags);
  params->k12_choice = choose_k12(d, pl->desc.flags, pl->n_cus);
  params->k12 = make_k12(d, params->k, dev_params, params->k12_choice);
  for (int epi = 0; epi < 3; ++epi) params->k3[epi] = make_k3(d, params->k, dev_params, pl->n_cus, epi);
  if (on_device) {
    // tables and parameters in one copy
    DeviceParams dp;
    dp.residues = make_residues(d, params->k);
    if (params->k12_choice.fused)
      dp.residues.kept_share = share_of((uint32_t)params->k12.total, params->k12_choice.copies ? params->k12_choice.copies : params->k12_choice.blocks,
                                        16u * 256u * (uint32_t)k12_quads(params->k12_choice.KS1, params->k12_choice.TH));
    dp.k3 = make_conversion(d, params->k, pl->n_cus);
    std::memcpy(blob.data() + pl->off_params, &dp, sizeof(dp));
    if (hipMemcpy(pl->d_tables, blob.data(), blob.size(), hipMemcpyHostToDevice) != hipSuccess) return fail(RNSWINO_E_HIP);
  }
  {
    // every kernel the layer would launch, in each output mode, must be an instantiation that exists
    bool ok = launch_k1(d, pl->n_cus, params->k1, nullptr, nullptr, nullptr, Timing(), true) && launch_k2(d, pl->desc.flags, params->k2, nullptr, nullptr, nullptr, nullptr, Timing(), true);
    ok = ok && (!params->k12_choice.fused || launch_k12(params->k12_choice, params->k12, nullptr, nullptr, nullptr, nullptr, true));
    for (int epi = 0; epi < 3 && ok; ++epi) ok = launch_k3(d, *params, pl->n_cus, epi, 0, nullptr, nullptr, nullptr, Timing(), true);
    if (!ok) return fail(RNSWINO_E_UNSUPPORTED);
  }
  *out = pl;
  return RNSWINO_OK;
}

int rnswino_plan_destroy(rnswino_plan_t *plan) {
  if (!plan) return RNSWINO_E_INVALID;
  int rc = RNSWINO_OK;
  if (plan->d_tables && hipFree(plan->d_tables) != hipSuccess) { (void)hipGetLastError(); rc = RNSWINO_E_HIP; }
  delete (LayerParams *)plan->kparams;
  delete plan;
  return rc;
}

int rnswino_output_dims(const rnswino_plan_t *plan, int32_t *Ho, int32_t *Wo) {
  if (!plan || !Ho || !Wo) return RNSWINO_E_INVALID;
  *Ho = plan->dims.Ho; *Wo = plan->dims.Wo;
  return RNSWINO_OK;
}

size_t rnswino_filter_bytes(const rnswino_plan_t *plan) { return plan ? align256(u_bytes(plan->dims)) : 0; }

size_t rnswino_workspace_bytes(const rnswino_plan_t *plan) {
  return plan ? align256(v_bytes(plan->dims)) + align256(o_bytes(plan->dims)) : 0;
}

int rnswino_filter_transform(const rnswino_plan_t *plan, const int8_t *w_dev, void *U_dev, void *stream) {
  if (!plan || !w_dev || !U_dev) return RNSWINO_E_INVALID;
  if (plan->device < 0) return RNSWINO_E_NO_DEVICE;
  if (!on_plan_device(plan)) return RNSWINO_E_INVALID;
  const Dims &d = plan->dims;
  const KParams P = ((const LayerParams *)plan->kparams)->k;
  hipStream_t st = (hipStream_t)stream;
  // one block per 16 rows x 64 channels, its (residue, 16-point block) items split over y until there are about four
  // blocks per compute unit (512 x 512, t = 10: 46 us with one block per compute unit, 35.5 with two, 32 with four, 33 with
  // seven, 36.5 with fourteen -- each block gathers its filters anew)
  const long long gx = (long long)(d.Kp / 16) * (d.Cp / 64), items = (long long)d.n * d.CB1, want = (1024 + gx - 1) / gx;
  const dim3 grid((unsigned)gx, (unsigned)(want < items ? want : items));
  const size_t lds = (size_t)((d.r * d.r + 15) / 16) * 16384;
  const int pieces = (d.r * d.r + 15) / 16;               // a filter's 16-tap slices: 1, 2, 3 or 4
#define RNSW_K0(wd, pp) hipLaunchKernelGGL((k0_filter_transform<wd, pp>), grid, dim3(256), lds, st, P, w_dev, (int8_t *)U_dev)
  if (d.wide) { if (pieces == 1) RNSW_K0(true, 1); else if (pieces == 2) RNSW_K0(true, 2); else RNSW_K0(true, 4); }
  else { if (pieces == 1) RNSW_K0(false, 1); else if (pieces == 2) RNSW_K0(false, 2); else RNSW_K0(false, 4); }
#undef RNSW_K0
  return launch_status();
}

int rnswino_conv2d(const rnswino_plan_t *plan, const int8_t *x_dev, const void *U_dev, int32_t *y_dev,
                   void *workspace_dev, void *stream) {
  return conv2d_impl(plan, x_dev, U_dev, y_dev, workspace_dev, stream, nullptr);
}

int rnswino_conv2d_requant(const rnswino_plan_t *plan, const int8_t *x_dev, const void *U_dev, int8_t *a_dev,
                           int32_t shift, int32_t pool, void *workspace_dev, void *stream) {
  if (!plan || shift < 0 || shift > 31) return RNSWINO_E_INVALID;
  const Dims &d = plan->dims;
  // pooling inside the kernel pairs rows and columns of one output tile: tiles of 4 or 8, whole pooling windows per row
  if (pool && ((d.m != 4 && d.m != 8) || (d.Wo & 3) || (d.Ho & 1))) return RNSWINO_E_UNSUPPORTED;
  return conv2d_impl(plan, x_dev, U_dev, nullptr, workspace_dev, stream, nullptr, pool ? 2 : 1, shift, a_dev);
}

int rnswino_conv2d_events(const rnswino_plan_t *plan, const int8_t *x_dev, const void *U_dev, int32_t *y_dev,
                          void *workspace_dev, void *stream, void *const events[6]) {
  if (!events) return RNSWINO_E_INVALID;
  return conv2d_impl(plan, x_dev, U_dev, y_dev, workspace_dev, stream, events);
}

int rnswino_debug_empty_launch(uint32_t grid_x, uint32_t grid_y, void *stream, void *start_event, void *stop_event) {
  if (grid_x == 0 || grid_y == 0 || grid_y > 65535u) return RNSWINO_E_INVALID;
  Timing tm;
  tm.start = (hipEvent_t)start_event;
  tm.stop = (hipEvent_t)stop_event;
  launch(k_empty, dim3(grid_x, grid_y), 0, (hipStream_t)stream, tm, 0);
  return launch_status();
}

int64_t rnswino_kernel_variants(char *host_out, size_t capacity) {
  const std::string all = all_kernel_variants();
  if (host_out && capacity > all.size()) std::memcpy(host_out, all.c_str(), all.size() + 1);
  return (int64_t)all.size() + 1;
}

int rnswino_conv2d_static(const rnswino_plan_t *plan, const int8_t *x_dev, const void *U_dev, int32_t *y_dev, void *stream) {
  if (!plan) return RNSWINO_E_INVALID;
  if (plan->device < 0) return RNSWINO_E_NO_DEVICE;
  if (rnswino_workspace_bytes(plan) > (size_t)RNSWINO_STATIC_WORKSPACE_BYTES) return RNSWINO_E_WORKSPACE;
  void *ws = plan->device < MAX_DEVICES ? scratch_ptr[plan->device] : nullptr;   // set when the plan was made
  if (!ws) return RNSWINO_E_HIP;
  return conv2d_impl(plan, x_dev, U_dev, y_dev, ws, stream, nullptr);
}

int64_t rnswino_plan_describe(const rnswino_plan_t *plan, int32_t output_mode, char *host_out, size_t capacity) {
  if (!plan || output_mode < 0 || output_mode > 2) return RNSWINO_E_INVALID;
  const Dims &d = plan->dims;
  const KParams &P = ((const LayerParams *)plan->kparams)->k;
  const K1Choice c1 = choose_k1(d, plan->n_cus);
  const K2Choice c2 = choose_k2(d, plan->desc.flags);
  const K3Choice c3 = choose_k3(d, P, plan->n_cus, output_mode);
  auto tf = [](bool b) { return b ? "true" : "false"; };
  char buf[1024];
  int len = c1.tiles ? std::snprintf(buf, sizeof(buf), "k1_input_transform_tiles<%d, %s> grid=%ux%u", c1.KS1, tf(c1.pack), c1.gx, c1.gy)
                     : std::snprintf(buf, sizeof(buf), "k1_input_transform<%d, %s, %s> grid=%ux%u", c1.KS1, tf(c1.wide), tf(c1.pack), c1.gx, c1.gy);
  if (c1.gz > 1) len += std::snprintf(buf + len, sizeof(buf) - len, "x%u", c1.gz);
  len += std::snprintf(buf + len, sizeof(buf) - len, "\n");
  if (c2.lds)
    len += std::snprintf(buf + len, sizeof(buf) - len, "k2_residue_gemm_lds<%d, %d, %d, %d, %d> grid=%u xgroup=%d\n", c2.WM, c2.WN, c2.RM,
                         c2.NTB, c2.S, c2.blocks, c2.xgroup);
  else
    len += std::snprintf(buf + len, sizeof(buf) - len, "k2_residue_gemm<%d, %d, %d, %s> grid=%u xgroup=%d\n", c2.KS, c2.NTB, c2.RM,
                         tf(c2.wide), c2.blocks, c2.xgroup);
  if (c3.stream)
    len += std::snprintf(buf + len, sizeof(buf) - len, "k3_inverse_crt_stream<%d, %d, %s, %s> grid=%ux%u lds=%zu\n", c3.NRES, c3.KS3,
                         tf(c3.fast), tf(c3.m8), c3.gx, c3.gy, c3.lds);
  else
    len += std::snprintf(buf + len, sizeof(buf) - len, "k3_inverse_crt<%d, %d, %s, %s> grid=%ux%u\n", c3.NRES, c3.KS3, tf(c3.wide),
                         tf(c3.fast), c3.gx, c3.gy);
  const char *conv = P.fastcrt == 1 ? "unreduced-binary32"
                     : P.fastcrt == 2 ? "unreduced-binary64"
                     : !P.crt24 || (d.wide && k3_converts_each(d.n, c3.KS3)) ? "reduced-binary64-mul32"
                     : P.quot32 ? "reduced-binary32" : "reduced-binary64";
  len += std::snprintf(buf + len, sizeof(buf) - len, "conversion=%s\n", conv);
  const K12Choice &c12 = ((const LayerParams *)plan->kparams)->k12_choice;
  if (c12.fused)
    len += std::snprintf(buf + len, sizeof(buf) - len, "fused=k12_transform_gemm<%d, %d, %d, %s> grid=%u copies=%u part=%d\n", c12.KS1, c12.TH, c12.RM, tf(c12.pack), c12.blocks,
                         c12.copies, c12.part);
  if (host_out && capacity > (size_t)len) std::memcpy(host_out, buf, (size_t)len + 1);
  return (int64_t)len + 1;
}

// ---- direct convolution (the comparison baseline of section 8) ----
static int direct_params(int32_t N, int32_t C, int32_t K, int32_t H, int32_t W, int32_t r, int32_t pad, DirectParams &P) {
  if (N <= 0 || C <= 0 || K <= 0 || H <= 0 || W <= 0 || r <= 0 || pad < 0) return RNSWINO_E_INVALID;
  const long long Ho = (long long)H + 2LL * pad - r + 1, Wo = (long long)W + 2LL * pad - r + 1;
  if (Ho <= 0 || Wo <= 0) return RNSWINO_E_INVALID;
  if (r > 16) return RNSWINO_E_UNSUPPORTED;
  if ((unsigned __int128)16384u * (unsigned)r * (unsigned)r * (unsigned)C > 2147483647u) return RNSWINO_E_UNSUPPORTED;   // int32 sums
  P.N = N; P.C = C; P.K = K; P.H = H; P.W = W; P.r = r; P.pad = pad;
  P.Ho = (int)Ho; P.Wo = (int)Wo; P.Hp = H + 2 * pad; P.Wp = W + 2 * pad;
  P.Cp = (C + 63) / 64 * 64; P.Kp = (K + 15) / 16 * 16;
  const long long npix = (long long)N * Ho * Wo, xt = (long long)N * P.Hp * P.Wp * P.Cp;
  if (npix >= (1LL << 28) || xt >= (1LL << 31) || (long long)r * r * P.Kp * P.Cp >= (1LL << 31)) return RNSWINO_E_UNSUPPORTED;   // 32-bit offsets
  P.npix = (int)npix;
  P.by_plane = make_fast_div((uint32_t)(Ho * Wo)); P.by_Wo = make_fast_div((uint32_t)Wo);
  P.by_groups = make_fast_div((uint32_t)((P.Wp + 15) / 16)); P.by_Hp = make_fast_div((uint32_t)P.Hp); P.by_ncb = make_fast_div((uint32_t)(P.Cp / 64));
  return RNSWINO_OK;
}

#define RNSW_DIRECT_PATCH_TABLE(X) X(1, 4, 2, 4, 4) X(1, 4, 4, 4, 4) X(2, 2, 2, 4, 4) X(2, 2, 1, 2, 8)
#define RNSW_DIRECT_TABLE(X) X(1, 4, 4, 4, 3) X(2, 2, 4, 4, 3) X(4, 1, 2, 4, 4) X(4, 1, 1, 4, 4)

// patch: pixels of the staged patch, 0 for k_direct_conv; depth: the kernel's D or S.
struct DirectChoice {
  int patch, WM, WN, RM, NT, depth;
  unsigned blocks;
  size_t lds;
  bool is(int wm, int wn, int rm, int nt, int d) const { return WM == wm && WN == wn && RM == rm && NT == nt && depth == d; }
};

static DirectChoice choose_direct(const DirectParams &P) {
  const long long nkb = P.Kp / 16, ntb = (P.npix + 15) / 16;
  auto blocks = [&](int brf, int btf) { return ((nkb + brf - 1) / brf) * (((ntb + btf - 1) / btf + 7) / 8 * 8); };
  // Patch kernel (k_direct_conv_patch) where its LDS leaves two workgroups per compute unit, unless there is too little to do with a
  // patch (us per call, patch / k_direct_conv; steps of a block: taps x 64-channel blocks):
  // - a single tap: a barrier per step, for which it has fetched one step ahead instead of three (2048 -> 256 at 7 x 7 17.3 / 13.4,
  //   1024 -> 1024 at 14 x 14 12.7 / 11.3);
  // - up to 18 steps and many blocks, where the stores of y decide and 128 x 128 blocks take them better (3 x 3, batch 8: 3 -> 512 at
  //   112 x 112 63.1 / 55.1, 64 -> 256 42.2 / 39.5; with 832 blocks, 64 -> 256 at 56 x 56, 16.4 / 18.6);
  // - 2 x 2 filters, up to 8 steps, from 800 of the smallest blocks on (batch 8, 64 -> 256 at 28 x 28 10.6 / 9.7, 64 -> 1024 19.4 / 16.8;
  //   below, 64 -> 64, 8.1 / 8.5; from 1536 of the largest on, 64 -> 1024 at 56 x 56, 41.0 / 43.4).
  const int steps = P.r * P.r * (P.Cp / 64);
  const bool many = blocks(4, 16) >= 1536;
  const bool patches = P.r > 2 ? !(steps <= 18 && P.Kp > 64 && many) : P.r == 2 ? !(steps <= 8 && blocks(2, 4) >= 800 && !many) : false;
  auto patch_pixels = [&](long long pixels) { return rnswino::patch_pixels(pixels, P.N, P.Ho, P.Wo, P.Wp, P.r); };
  auto patch_lds = [&](int btf) { return (patch_pixels(16 * btf) + 15) / 16 * 1024 * (P.Cp > 64 ? 2 : 1); };
  auto fits = [&](int btf) { return patches && patch_lds(btf) <= 81920; };
  auto patch = [&](int wm, int wn, int rm, int nt, int depth) {
    return DirectChoice{(int)patch_pixels(16 * wn * nt), wm, wn, rm, nt, depth, (unsigned)blocks(wm * rm, wn * nt), (size_t)patch_lds(wn * nt)};
  };
  auto plain = [&](int wm, int wn, int rm, int nt, int depth) {
    return DirectChoice{0, wm, wn, rm, nt, depth, (unsigned)blocks(wm * rm, wn * nt), 0};
  };
  // The largest block that still gives three workgroups per two compute units, 32 x 64 for the smallest layers (us per call,
  // batch 8 unless noted, 64 x 256 / 64 x 128 / 32 x 256 / 32 x 64 / k_direct_conv: 256 -> 256 at 56 x 56 28.2 / 33.0 / 31.6 /
  // 39.6 / 44.0; 512 -> 512 at 28 x 28 29.2 / 26.6 / 27.1 / 36.6 / 49.6; 64 -> 64 at 112 x 112 20.2 / 20.3 / 19.3 / 24.0 / 24.5;
  // 512 -> 512 at 14 x 14 26.9 / 21.2 / 22.0 / 19.3 / 26.4; 256 -> 256 at 56 x 56, batch 1 18.3 / 15.0 / 15.0 / 13.4 / 16.6).
  if (P.Kp <= 64 && P.Kp > 16 && blocks(2, 16) >= 384 && fits(16)) return patch(1, 4, 2, 4, 4);
  if (P.Kp > 64 && blocks(4, 16) >= 384 && fits(16)) return patch(1, 4, 4, 4, 4);
  if (P.Kp > 16 && blocks(4, 8) >= 384 && fits(8)) return patch(2, 2, 2, 4, 4);
  if ((P.Kp <= 16 || blocks(4, 8) < 384) && fits(4)) return patch(2, 2, 1, 2, 8);
  // The others -- planes so wide that a patch outgrows LDS, and the cases above -- fetch every tap's pixels anew.  Block shape: 128 x 128 when that
  // still gives the chip two workgroups per compute unit, else 128 x 64, else 64 x 64; layers with at most 64 filters 64 x 256
  if (P.Kp <= 64 && blocks(4, 16) >= 512) return plain(1, 4, 4, 4, 3);
  if (P.Kp > 64 && blocks(8, 8) >= 512) return plain(2, 2, 4, 4, 3);
  if (P.Kp > 64 && blocks(8, 4) >= 512) return plain(4, 1, 2, 4, 4);
  return plain(4, 1, 1, 4, 4);
}

size_t rnswino_direct_filter_bytes(int32_t C, int32_t K, int32_t r) {
  DirectParams P;
  if (direct_params(1, C, K, r, r, r, 0, P) != RNSWINO_OK) return 0;
  return align256((size_t)r * r * P.Kp * P.Cp);
}

size_t rnswino_direct_workspace_bytes(int32_t N, int32_t C, int32_t H, int32_t W, int32_t pad) {
  DirectParams P;
  if (direct_params(N, C, 1, H, W, 1, pad, P) != RNSWINO_OK) return 0;
  return align256((size_t)N * P.Hp * P.Wp * P.Cp);
}

int rnswino_direct_filter_pack(const int8_t *w_dev, void *wt_dev, int32_t C, int32_t K, int32_t r, void *stream) {
  if (!w_dev || !wt_dev) return RNSWINO_E_INVALID;
  if ((uintptr_t)wt_dev & 15) return RNSWINO_E_INVALID;
  DirectParams P;
  const int rc = direct_params(1, C, K, r, r, r, 0, P);
  if (rc != RNSWINO_OK) return rc;
  const long long total = (long long)r * r * P.Kp * (P.Cp / 16);
  hipLaunchKernelGGL(k_direct_pack_filter, dim3(blocks_for(total, 256)), dim3(256), 0, (hipStream_t)stream, P, w_dev, (int8_t *)wt_dev);
  return launch_status();
}

int rnswino_direct_conv2d(const int8_t *x_dev, const void *wt_dev, int32_t *y_dev, int32_t N, int32_t C, int32_t K, int32_t H,
                          int32_t W, int32_t r, int32_t pad, void *workspace_dev, void *stream) {
  if (!x_dev || !wt_dev || !y_dev || !workspace_dev) return RNSWINO_E_INVALID;
  if (((uintptr_t)wt_dev | (uintptr_t)workspace_dev) & 15) return RNSWINO_E_INVALID;
  DirectParams P;
  const int rc = direct_params(N, C, K, H, W, r, pad, P);
  if (rc != RNSWINO_OK) return rc;
  hipStream_t st = (hipStream_t)stream;
  int8_t *xt = (int8_t *)workspace_dev;
  const long long tblocks = ((long long)N * P.Hp * ((P.Wp + 15) / 16) + 15) / 16 * (P.Cp / 64);
  hipLaunchKernelGGL(k_direct_to_nhwc, dim3((unsigned)tblocks), dim3(256), 0, st, P, x_dev, xt);
  const DirectChoice c = choose_direct(P);
  if (c.patch > 0 && r < 2) return RNSWINO_E_UNSUPPORTED;   // k_direct_conv_patch counts on three steps and more per channel block, whatever the timings say
  P.gy = (P.Kp / 16 + c.WM * c.RM - 1) / (c.WM * c.RM);
  P.by_gy = make_fast_div((uint32_t)P.gy);
#define RNSW_X(wm_, wn_, rm, nt, d_) \
  if (c.patch > 0 && c.is(wm_, wn_, rm, nt, d_)) { \
    hipLaunchKernelGGL((k_direct_conv_patch<wm_, wn_, rm, nt, d_>), dim3(c.blocks), dim3(256), c.lds, st, P, c.patch, xt, (const int8_t *)wt_dev, y_dev); \
    return launch_status(); }
  RNSW_DIRECT_PATCH_TABLE(RNSW_X)
#undef RNSW_X
#define RNSW_X(wm_, wn_, rm, nt, s_) \
  if (c.patch == 0 && c.is(wm_, wn_, rm, nt, s_)) { \
    hipLaunchKernelGGL((k_direct_conv<wm_, wn_, rm, nt, s_>), dim3(c.blocks), dim3(256), 0, st, P, xt, (const int8_t *)wt_dev, y_dev); \
    return launch_status(); }
  RNSW_DIRECT_TABLE(RNSW_X)
#undef RNSW_X
  return RNSWINO_E_UNSUPPORTED;
}

int64_t rnswino_direct_describe(int32_t N, int32_t C, int32_t K, int32_t H, int32_t W, int32_t r, int32_t pad, char *host_out, size_t capacity) {
  DirectParams P;
  const int rc = direct_params(N, C, K, H, W, r, pad, P);
  if (rc != RNSWINO_OK) return rc;
  const DirectChoice c = choose_direct(P);
  char buf[256];
  const int len = c.patch > 0 ? std::snprintf(buf, sizeof(buf), "k_direct_conv_patch<%d, %d, %d, %d, %d> grid=%u lds=%zu patch=%d\n", c.WM, c.WN, c.RM,
                                              c.NT, c.depth, c.blocks, c.lds, c.patch)
                              : std::snprintf(buf, sizeof(buf), "k_direct_conv<%d, %d, %d, %d, %d> grid=%u\n", c.WM, c.WN, c.RM, c.NT, c.depth, c.blocks);
  if (host_out && capacity > (size_t)len) std::memcpy(host_out, buf, (size_t)len + 1);
  return (int64_t)len + 1;
}

int64_t rnswino_direct_variants(char *host_out, size_t capacity) {
  std::string all;
#define RNSW_X(wm_, wn_, rm, nt, d_) all += "k_direct_conv_patch<" #wm_ ", " #wn_ ", " #rm ", " #nt ", " #d_ ">\n";
  RNSW_DIRECT_PATCH_TABLE(RNSW_X)
#undef RNSW_X
#define RNSW_X(wm_, wn_, rm, nt, s_) all += "k_direct_conv<" #wm_ ", " #wn_ ", " #rm ", " #nt ", " #s_ ">\n";
  RNSW_DIRECT_TABLE(RNSW_X)
#undef RNSW_X
  if (host_out && capacity > all.size()) std::memcpy(host_out, all.c_str(), all.size() + 1);
  return (int64_t)all.size() + 1;
}

int rnswino_requant_pool(const int32_t *y_dev, int8_t *a_dev, int64_t planes, int32_t H, int32_t W, int32_t shift,
                         int32_t pool, void *stream) {
  if (!y_dev || !a_dev || planes <= 0 || H <= 0 || W <= 0 || shift < 0 || shift > 31) return RNSWINO_E_INVALID;
  if (pool && ((H | W) & 1)) return RNSWINO_E_INVALID;
  const long long total = (long long)planes * (pool ? H / 2 : H) * (pool ? W / 2 : W);
  unsigned blocks = blocks_for(total, 256);
  if (blocks > 65536u * 4u) blocks = 65536u * 4u;
  hipLaunchKernelGGL(k_requant_pool, dim3(blocks), dim3(256), 0, (hipStream_t)stream, y_dev, a_dev, (long long)planes, H, W,
                     shift, pool);
  return launch_status();
}

int rnswino_plan_get_matrix(const rnswino_plan_t *plan, int which, int modulus_idx, int32_t *host_out) {
  if (!plan || !host_out || modulus_idx < 0 || modulus_idx >= plan->dims.n) return RNSWINO_E_INVALID;
  const Transforms &tf = plan->tf[modulus_idx];
  const std::vector<int32_t> *src = which == RNSWINO_MATRIX_AT ? &tf.AT : which == RNSWINO_MATRIX_G ? &tf.G
                                    : which == RNSWINO_MATRIX_BT ? &tf.BT : nullptr;
  if (!src) return RNSWINO_E_INVALID;
  std::memcpy(host_out, src->data(), src->size() * sizeof(int32_t));
  return RNSWINO_OK;
}

int64_t rnswino_plan_get_table(const rnswino_plan_t *plan, int which, int modulus_idx, int8_t *host_out, size_t capacity) {
  if (!plan || modulus_idx < 0 || modulus_idx >= plan->dims.n) return RNSWINO_E_INVALID;
  const Dims &d = plan->dims;
  const size_t planes = d.wide ? 2 : 1;
  size_t per, off;
  if (which == RNSWINO_TABLE_INPUT) { per = (size_t)d.CB1 * d.KS1 * planes * 1024; off = plan->off_KB; }
  else if (which == RNSWINO_TABLE_INVERSE) { per = (size_t)d.RB3 * d.KS3 * planes * 1024; off = plan->off_KA; }
  else return RNSWINO_E_INVALID;
  off += per * (size_t)modulus_idx;
  if (off + per > plan->h_tables.size()) return RNSWINO_E_INVALID;
  if (host_out && capacity >= per) std::memcpy(host_out, plan->h_tables.data() + off, per);
  return (int64_t)per;
}

int rnswino_plan_get_mrc_inverse(const rnswino_plan_t *plan, int l, int j, uint32_t *host_out) {
  if (!plan || !host_out || l < 0 || j <= l || j >= plan->dims.n) return RNSWINO_E_INVALID;
  *host_out = plan->mrc_inv[l][j];
  return RNSWINO_OK;
}

int64_t rnswino_plan_dynamic_range(const rnswino_plan_t *plan) { return plan ? plan->dyn_range : 0; }

int rnswino_debug_stage(const rnswino_plan_t *plan, int stage, const void *src_dev, int32_t *host_out) {
  if (!plan || !src_dev || !host_out) return RNSWINO_E_INVALID;
  if (plan->device < 0) return RNSWINO_E_NO_DEVICE;
  const Dims &d = plan->dims;
  const LayerParams &L = *(const LayerParams *)plan->kparams;
  size_t bytes, skip = 0;
  if (stage == RNSWINO_STAGE_U) bytes = u_bytes(d);
  else if (stage == RNSWINO_STAGE_V) bytes = v_bytes(d);
  else if (stage == RNSWINO_STAGE_O) { bytes = o_bytes(d); skip = align256(v_bytes(d)); }
  else return RNSWINO_E_INVALID;
  std::vector<int8_t> raw(bytes);
  const char *from = (const char *)src_dev + skip;
  void *v = nullptr;
  bool ok = hipDeviceSynchronize() == hipSuccess;
  if (ok && stage == RNSWINO_STAGE_V && L.k12_choice.fused) {
    // the workspace holds the input in V's place: transformed here, on the plan's device
    int current = plan->device;
    ok = hipGetDevice(&current) == hipSuccess && hipSetDevice(plan->device) == hipSuccess && hipDeviceSynchronize() == hipSuccess;
    if (ok && hipMalloc(&v, bytes) != hipSuccess) { v = nullptr; ok = false; }
    ok = ok && launch_k1(d, plan->n_cus, L.k1, (const int8_t *)src_dev, (int8_t *)v, nullptr, Timing()) && hipGetLastError() == hipSuccess &&
         hipDeviceSynchronize() == hipSuccess;
    ok = hipSetDevice(current) == hipSuccess && ok;
    from = (const char *)v;
  }
  ok = ok && hipMemcpy(raw.data(), from, bytes, hipMemcpyDeviceToHost) == hipSuccess;
  if (v) ok = hipFree(v) == hipSuccess && ok;
  if (!ok) {
    (void)hipGetLastError();
    return RNSWINO_E_HIP;
  }
  for (int i = 0; i < d.n; ++i) {
    const int64_t p = plan->desc.moduli[i];
    for (int pt = 0; pt < d.P2; ++pt) {
      const int slab = i * d.P2 + pt;
      auto value = [&](size_t narrow, size_t hi, size_t lo) -> int32_t {
        return d.wide ? sym_residue(256 * (int64_t)raw[hi] + (int64_t)raw[lo], p) : sym_residue((int64_t)raw[narrow], p);
      };
      if (stage == RNSWINO_STAGE_U) {
        // packed layers: the filter sits in every diagonal block (k * TL + tl, tl * Cq + c); block tl = 0 is read
        for (int k = 0; k < d.K; ++k)
          for (int c = 0; c < d.C; ++c) {
            const int kg = k * d.TL;
            host_out[((size_t)slab * d.K + k) * d.C + c] =
                d.wide ? value(0, u_offset_wide(slab, kg, c, d.Kp, d.Cp, 0), u_offset_wide(slab, kg, c, d.Kp, d.Cp, 1))
                       : value(u_offset(slab, kg, c, d.Kp, d.Cp), 0, 0);
          }
      } else if (stage == RNSWINO_STAGE_V) {
        for (int tau = 0; tau < d.T; ++tau)
          for (int c = 0; c < d.C; ++c) {
            const int tg = tau % d.Tg, cg = (tau / d.Tg) * d.Cq + c;       // GEMM column and channel (cg = c when TL = 1)
            host_out[((size_t)slab * d.T + tau) * d.C + c] =
                d.wide ? value(0, v_offset_wide(slab, d.n * d.P2, tg, cg, d.Cp, 0), v_offset_wide(slab, d.n * d.P2, tg, cg, d.Cp, 1))
                       : value(v_offset(slab, d.n * d.P2, tg, cg, d.Cp, d.vlane), 0, 0);
          }
      } else {
        for (int k = 0; k < d.K; ++k)
          for (int tau = 0; tau < d.T; ++tau) {
            const int kg = k * d.TL + tau / d.Tg, tg = tau % d.Tg;          // GEMM row and column
            host_out[((size_t)slab * d.K + k) * d.T + tau] =
                d.wide ? value(0, o_offset_wide(i, pt, kg, tg, d.n, d.Q, d.Kp, d.Tp, 0), o_offset_wide(i, pt, kg, tg, d.n, d.Q, d.Kp, d.Tp, 1))
                       : value(o_offset(i, pt, kg, tg, d.n, d.Q, d.Kp, d.Tp), 0, 0);
          }
      }
    }
  }
  return RNSWINO_OK;
}

const char *rnswino_strerror(int code) {
  switch (code) {
    case RNSWINO_OK: return "ok";
    case RNSWINO_E_INVALID: return "invalid argument";
    case RNSWINO_E_UNSUPPORTED: return "unsupported configuration";
    case RNSWINO_E_NOT_COPRIME: return "moduli are not pairwise coprime";
    case RNSWINO_E_POINT_NOT_INVERTIBLE: return "a modulus shares a factor with an interpolation-point difference";
    case RNSWINO_E_RANGE: return "dynamic range of the moduli set is below the output bound (worst case 2^14 r^2 C unless the caller gave a tighter one)";
    case RNSWINO_E_HIP: return "HIP runtime error";
    case RNSWINO_E_NO_DEVICE: return "plan is host-only or no GPU is available";
    case RNSWINO_E_WORKSPACE: return "the layer needs more workspace than the library's static buffer holds";
    default: return "unknown error";
  }
}

}  // extern "C"
