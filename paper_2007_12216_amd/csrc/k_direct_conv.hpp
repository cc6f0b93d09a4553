// Direct int8 convolution as an implicit GEMM on the matrix cores: the baseline the paper measures its method against
// (section 8, Tables 4 and 5: Im2col + INT8 GEMM), written for the same chip so that the two can be timed side by side.
//
//   y[n][k][oy][ox] = sum_{c,i,j} xpad[n][c][oy+i-pad][ox+j-pad] w[k][c][i][j]            (int32, stride 1)
// is a GEMM with rows k, columns = output pixels and contraction index (i, j, c).  No im2col matrix is ever
// written: a column block's operand fragment for filter tap (i, j) and 64 channels is gathered straight from the
// activations, 16 bytes (16 channels of one pixel) per lane.  For that the activations are first copied once into a
// channel-innermost, zero-bordered layout (one pass over x; part of the timed call):
//   xt [Cp/64][N][H + 2 pad][W + 2 pad][64]      Cp = C rounded up to 64, padding channels and the border are zero
// and the weights are packed ahead of time into matrix-core fragments (they are constants of the layer):
//   wt [Cp/64][r*r taps][Kp/16][lane = k%16 + 16 g][16 B]     byte b of slice g = channel 64 cb + 16 g + b.
// The GEMM kernel has the structure of the LDS-tiled residue GEMM (k_residue_gemm_lds.hpp): WM x WN waves of
// RM x NT fragments each, operand fragments loaded from global memory straight into LDS S steps deep and shared by
// the waves; a step is one (tap, 64-channel block).  The int32 sums are stored as they are (no modulus anywhere).
#pragma once
#include "k_residue_gemm_lds.hpp"

namespace rnswino {

struct DirectParams {
  int N, C, K, H, W, r, pad;
  int Ho, Wo, Hp, Wp, Cp, Kp;
  int npix;                     // N * Ho * Wo
  FastDiv by_plane, by_Wo;      // by Ho * Wo, Wo
  FastDiv by_groups, by_Hp, by_ncb;   // k_direct_to_nhwc: by the 16-pixel groups of a padded row, Hp, Cp / 64
  FastDiv by_gy;                // GEMM kernels: by the row blocks, gy of them
  int gy;
};

// x [N][C][H][W] -> xt [Cp/64][N][Hp][Wp][64], zero border and zero padding channels.  A block takes 64 channels of 16 units
// (a unit: 16 consecutive padded pixels of one row): every thread loads four 16-byte row segments (unaligned, masked to the
// image), and after a transpose in LDS stores four pixels x 16 channels.  Bound by its two passes over the tensor; 256
// channels at 56 x 56, batch 8 (6.4 MB read, 6.9 MB written): 6.5 us (one byte per load: 15.9).
__global__ __launch_bounds__(256) void k_direct_to_nhwc(DirectParams P, const int8_t *__restrict__ x, int8_t *__restrict__ xt) {
  // row segment of (unit, channel) at dword 272 unit + 68 (channel / 16) + 4 (channel % 16): both the 16-byte writes and the
  // column reads below spread over all banks
  __shared__ __attribute__((aligned(16))) uint32_t tile[16 * 272];
  const int groups = (P.Wp + 15) >> 4, ncb = P.Cp >> 6;
  const int nunits = P.N * P.Hp * groups;               // below 2^31: xt is
  const int ub = (int)fast_div(blockIdx.x, P.by_ncb), cb = (int)blockIdx.x - ub * ncb;
  {
    const long long total = (long long)P.N * P.C * P.H * P.W;
    const int unit = ub * 16 + (threadIdx.x & 15), c0 = threadIdx.x >> 4;
    const int row = (int)fast_div((uint32_t)unit, P.by_groups), grp = unit - row * groups, n = (int)fast_div((uint32_t)row, P.by_Hp);
    const int iy = row - n * P.Hp - P.pad, ix = grp * 16 - P.pad;      // image row and column of the segment's first pixel
    const bool row_ok = unit < nunits && iy >= 0 && iy < P.H;
    v4i val[4];
    int state[4];                                       // 0: zeros, 1: plain 16-byte load, 2: ends of the tensor
    long long at[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int ch = cb * 64 + c0 + 16 * e;
      at[e] = (((long long)n * P.C + ch) * P.H + iy) * P.W + ix;
      state[e] = !(row_ok && ch < P.C) ? 0 : at[e] >= 0 && at[e] + 16 <= total ? 1 : 2;
      val[e] = (v4i){0, 0, 0, 0};
      if (state[e] == 1) __builtin_memcpy(&val[e], x + at[e], 16);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (state[e] == 2) {
        uint32_t wv[4] = {0, 0, 0, 0};
        for (int b = 0; b < 16; ++b)
          if (at[e] + b >= 0 && at[e] + b < total) wv[b >> 2] |= (uint32_t)(uint8_t)x[at[e] + b] << (8 * (b & 3));
        val[e] = (v4i){(int)wv[0], (int)wv[1], (int)wv[2], (int)wv[3]};
      }
    // columns [lo, hi) of the segment lie inside the image
    const int lo = min(max(-ix, 0), 16), hi = min(max(P.W - ix, 0), 16);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      uint32_t mask = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) mask |= (4 * d + e >= lo && 4 * d + e < hi) ? 0xFFu << (8 * e) : 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) val[e][d] &= mask;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) *(v4i *)(tile + (threadIdx.x & 15) * 272 + e * 68 + c0 * 4) = val[e];
  }
  __syncthreads();
  {
    const int g = threadIdx.x & 3, pq = (threadIdx.x >> 2) & 3, u = threadIdx.x >> 4, unit = ub * 16 + u;
    if (unit >= nunits) return;
    uint32_t in[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) in[e] = tile[u * 272 + g * 68 + e * 4 + pq];
    v4i out[4];                                         // pixel 4 pq + k: channels 16 g .. 16 g + 15
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const uint32_t t0 = __builtin_amdgcn_perm(in[4 * d + 1], in[4 * d], 0x05010400u), t1 = __builtin_amdgcn_perm(in[4 * d + 1], in[4 * d], 0x07030602u);
      const uint32_t t2 = __builtin_amdgcn_perm(in[4 * d + 3], in[4 * d + 2], 0x05010400u), t3 = __builtin_amdgcn_perm(in[4 * d + 3], in[4 * d + 2], 0x07030602u);
      out[0][d] = (int)__builtin_amdgcn_perm(t2, t0, 0x05040100u);
      out[1][d] = (int)__builtin_amdgcn_perm(t2, t0, 0x07060302u);
      out[2][d] = (int)__builtin_amdgcn_perm(t3, t1, 0x05040100u);
      out[3][d] = (int)__builtin_amdgcn_perm(t3, t1, 0x07060302u);
    }
    const int row = (int)fast_div((uint32_t)unit, P.by_groups), xp = (unit - row * groups) * 16 + 4 * pq;
    int8_t *dst = xt + (((size_t)cb * P.N * P.Hp + row) * P.Wp + xp) * 64 + 16 * g;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (xp + k < P.Wp) *(v4i *)(dst + k * 64) = out[k];
  }
}

// w [K][C][r][r] -> wt fragments (offline).  One thread per (tap, k, 16-channel slice).
__global__ __launch_bounds__(256) void k_direct_pack_filter(DirectParams P, const int8_t *__restrict__ w, int8_t *__restrict__ wt) {
  const long long total = (long long)P.r * P.r * P.Kp * (P.Cp / 16);
  const long long id = (long long)blockIdx.x * 256 + threadIdx.x;
  if (id >= total) return;
  const int sl = (int)(id % (P.Cp / 16));               // 16-channel slice
  long long rest = id / (P.Cp / 16);
  const int k = (int)(rest % P.Kp);
  const int tap = (int)(rest / P.Kp);
  const int cb = sl >> 2, g = sl & 3;
  uint32_t wv[4] = {0, 0, 0, 0};
  for (int e = 0; e < 16; ++e) {
    const int c = sl * 16 + e;
    if (k < P.K && c < P.C) wv[e >> 2] |= (uint32_t)(uint8_t)w[((size_t)k * P.C + c) * P.r * P.r + tap] << (8 * (e & 3));
  }
  const size_t frag = ((size_t)cb * P.r * P.r + tap) * (P.Kp / 16) + (k >> 4);
  *(v4i *)(wt + frag * 1024 + ((k & 15) + 16 * g) * 16) = (v4i){(int)wv[0], (int)wv[1], (int)wv[2], (int)wv[3]};
}

// Grid: one-dimensional, 8 * ceil(pixel blocks / 8) * row blocks.  Workgroups go to the 8 XCDs round-robin by id: pixel
// block = 8 * (id / 8 / row blocks) + id % 8, row block = (id / 8) % row blocks, so the workgroups that share a pixel
// block's activations follow each other on one XCD (one L2).  256 threads.
template <int WM, int WN, int RM, int NT, int S>
__global__ __launch_bounds__(256) void k_direct_conv(DirectParams P, const int8_t *__restrict__ xt, const int8_t *__restrict__ wt,
                                                      int32_t *__restrict__ y) {
  static_assert(WM * WN == 4, "four waves per workgroup");
  constexpr int BRF = WM * RM, BTF = WN * NT;
  constexpr int NF = BRF + BTF;
  constexpr int LPW = (NF + 3) / 4;
  constexpr int SLOTS = 4 * LPW;
  __shared__ __attribute__((aligned(16))) uint8_t stage[S * SLOTS * 1024];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int wm = wave / WN, wn = wave % WN;
  const int nkb = P.Kp >> 4, ntb = (P.npix + 15) >> 4, ncb = P.Cp >> 6;
  const int gy = P.gy, gz = (ntb + BTF - 1) / BTF;
  const int pb8 = (int)fast_div(blockIdx.x >> 3, P.by_gy), pb = pb8 * 8 + (int)(blockIdx.x & 7);
  if (pb >= gz) return;                            // block-uniform: the grid is padded to a multiple of 8 pixel blocks
  const int kb0 = ((int)(blockIdx.x >> 3) - pb8 * gy) * BRF, tb0 = pb * BTF;
  const int taps = P.r * P.r;
  const int total = taps * ncb;

  // where output pixel `pix` (clamped to the last one) starts in xt: the patch origin (oy, ox) of image n
  auto pixel_origin = [&](int pix) -> uint32_t {
    pix = min(pix, P.npix - 1);
    const int n = (int)fast_div((uint32_t)pix, P.by_plane), rem = pix - n * (P.Ho * P.Wo);
    const int oy = (int)fast_div((uint32_t)rem, P.by_Wo), ox = rem - oy * P.Wo;
    return (uint32_t)(((n * P.Hp + oy) * P.Wp + ox) * 64);          // xt is smaller than 4 GiB (checked on the host)
  };
  // this wave's loads of a step: fragment f = wave + 4 j: a weight fragment (contiguous) or a pixel-block fragment
  // (lane = pixel l % 16, channels 16 (l / 16) .. + 15); per step only the wave-uniform part of the address changes
  const int8_t *base[LPW];
  uint32_t lane_off[LPW];
  bool is_w[LPW];
#pragma unroll
  for (int j = 0; j < LPW; ++j) {
    const int f = min(wave + 4 * j, NF - 1);
    is_w[j] = f < BRF;
    if (is_w[j]) {
      base[j] = wt + (size_t)min(kb0 + f, nkb - 1) * 1024;
      lane_off[j] = (uint32_t)lane * 16u;
    } else {
      base[j] = xt;
      lane_off[j] = pixel_origin((min(tb0 + f - BRF, ntb - 1)) * 16 + (lane & 15)) + (uint32_t)(lane >> 4) * 16u;
    }
  }
  const uint32_t stage_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t *)stage;
  // the step's offsets in wt and xt (both below 2 GiB), carried along: worked out anew for every step they cost 64-bit scalar
  // multiplications per load, an eighth of the time of a long contraction (2048 -> 256, 1 x 1, at 7 x 7 15.1 us a call, 13.3 so)
  uint32_t w_off = 0, x_off = 0;
  const uint32_t w_step = (uint32_t)nkb * 1024u, x_block = (uint32_t)(P.N * P.Hp * P.Wp) * 64u;
  auto issue = [&](int slot) {
#pragma unroll
    for (int j = 0; j < LPW; ++j)
      load_to_lds16(base[j] + (is_w[j] ? w_off : x_off), lane_off[j], stage_lds + (uint32_t)((slot * SLOTS + wave + 4 * j) * 1024));
  };
  int ptap = 0, ptj = 0, pcb = 0;
  uint32_t w_tap = 0, x_tap = 0;                   // the offsets of the tap's first channel block
  auto advance = [&]() {
    if (++pcb == ncb) {
      pcb = 0;
      ++ptap;
      w_off = w_tap += w_step;
      x_tap += 64u;
      if (++ptj == P.r) { ptj = 0; x_tap += (uint32_t)(P.Wp - P.r) * 64u; }
      x_off = x_tap;
    } else {
      w_off += (uint32_t)taps * w_step;
      x_off += x_block;
    }
  };
#pragma unroll
  for (int s = 0; s < S - 1; ++s)
    if (ptap < taps) { issue(s); advance(); }

  v4i acc[RM][NT];
#pragma unroll
  for (int rm = 0; rm < RM; ++rm)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[rm][nt] = (v4i){0, 0, 0, 0};
  const uint8_t *lds_a = stage + (wm * RM) * 1024 + lane * 16;
  const uint8_t *lds_b = stage + (BRF + wn * NT) * 1024 + lane * 16;
  int slot = 0, fill = S - 1;
  for (int it = 0; it < total; ++it) {
    const int rem = total - 1 - it;
    if (rem >= S - 2) wait_vmcnt<LPW * (S - 2)>();
    else if (S >= 4 && rem == 1) wait_vmcnt<LPW>();
    else wait_vmcnt<0>();
    __syncthreads();
    if (ptap < taps) { issue(fill); advance(); }
    v4i a[RM];
#pragma unroll
    for (int rm = 0; rm < RM; ++rm) a[rm] = *(const v4i *)(lds_a + (slot * SLOTS + rm) * 1024);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const v4i b = *(const v4i *)(lds_b + (slot * SLOTS + nt) * 1024);
#pragma unroll
      for (int rm = 0; rm < RM; ++rm) acc[rm][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[rm], b, acc[rm][nt], 0, 0, 0);
    }
    if (++slot == S) slot = 0;
    if (++fill == S) fill = 0;
  }

  // a lane holds rows 16 kb + 4 (lane / 16) + j of pixel 16 tb + lane % 16
  const size_t plane = (size_t)P.Ho * P.Wo;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int pix = (tb0 + wn * NT + nt) * 16 + (lane & 15);
    if (pix >= P.npix) continue;
    const int n = (int)fast_div((uint32_t)pix, P.by_plane), rem = pix - n * (P.Ho * P.Wo);
    int32_t *ypix = y + (size_t)n * P.K * plane + rem;
#pragma unroll
    for (int rm = 0; rm < RM; ++rm)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = (kb0 + wm * RM + rm) * 16 + 4 * (lane >> 4) + j;
        if (k < P.K) ypix[(size_t)k * plane] = acc[rm][nt][j];
      }
  }
}

// Every access to LDS of this wave, and every scalar load, is done.
__device__ __forceinline__ void wait_lds() {
  __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0), other counters untouched
}

// The same product with the pixels of all taps staged once.  In xt the pixels of one 64-channel block are consecutive, so the
// patch that 16 * WN * NT consecutive output pixels need for all r*r taps is ONE run of `patch` pixels (64 bytes each); it is
// copied to LDS once per channel block (two buffers: the next block's patch arrives while this one is used) and every tap
// reads its operand at another offset, instead of fetching it from L2 again for every tap.  The weights lie in memory in the
// order of the steps and go from L2 straight into registers, D taps ahead.  A workgroup thus meets one barrier per channel
// block instead of one per tap.
// 256 -> 256 at 56 x 56, batch 8, 64 x 256 blocks: of a block's 35000 cycles 2200 went before its first load (the compiler's
// divisions), 3000 for its first patch, 23000 for 36 steps -- 640 each, of which 256 multiply: a step read its pixels and waited for them,
// and at each channel block for all weights in flight -- and 6600 for storing y.  With the pixels read a step ahead, counted waits and
// divisions by multiplication 26.4 -> 24.6 us a call; 512 -> 512 at 28 x 28 25.9 -> 22.3, at 14 x 14 18.8 -> 14.2, batch 1 16.5 -> 12.1.
// (Of the last two 0.5 and 0.7 come with the loop's entry: without its wait, and with the weights in the compiler's order, every D-th step
// waited for everything in flight.)
// What is left: the blocks are 1.5 per compute unit, and all store at the end.
// Dynamic LDS: (ncb > 1 ? 2 : 1) * ceil(patch / 16) KiB.  Grid as k_direct_conv.
template <int WM, int WN, int RM, int NT, int D>
__global__ __launch_bounds__(256, 2) void k_direct_conv_patch(DirectParams P, int patch, const int8_t *__restrict__ xt,
                                                              const int8_t *__restrict__ wt, int32_t *__restrict__ y) {
  static_assert(WM * WN == 4, "four waves per workgroup");
  constexpr int BRF = WM * RM, BTF = WN * NT;
  extern __shared__ __attribute__((aligned(16))) uint8_t patch_lds[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int wm = wave / WN, wn = wave % WN;
  const int nkb = P.Kp >> 4, ntb = (P.npix + 15) >> 4, ncb = P.Cp >> 6;
  const int gy = P.gy, gz = (ntb + BTF - 1) / BTF;
  const int pb8 = (int)fast_div(blockIdx.x >> 3, P.by_gy), pb = pb8 * 8 + (int)(blockIdx.x & 7);
  if (pb >= gz) return;                            // block-uniform: the grid is padded to a multiple of 8 pixel blocks
  // the last row blocks are shifted to end with the tensor (rows computed twice are stored twice, the same values); the host
  // takes RM <= nkb
  const int kb0 = min(((int)(blockIdx.x >> 3) - pb8 * gy) * BRF + wm * RM, nkb - RM), tb0 = pb * BTF;
  const int taps = P.r * P.r, total = taps * ncb;

  // where output pixel `pix` (clamped to the last one) starts in a channel block of xt, in pixels
  auto pixel_origin = [&](int pix) -> int {
    pix = min(pix, P.npix - 1);
    const int n = (int)fast_div((uint32_t)pix, P.by_plane), rem = pix - n * (P.Ho * P.Wo);
    const int oy = (int)fast_div((uint32_t)rem, P.by_Wo), ox = rem - oy * P.Wo;
    return (n * P.Hp + oy) * P.Wp + ox;
  };
  // the patch: from the first pixel's origin to the last tap of the last pixel (at most `patch` pixels: patch_pixels())
  // (the divisions run on the vector unit; the results are the same in all lanes)
  const int o0 = __builtin_amdgcn_readfirstlane(pixel_origin(tb0 * 16));
  const int len = __builtin_amdgcn_readfirstlane(min(pixel_origin(tb0 * 16 + 16 * BTF - 1) - o0 + (P.r - 1) * (P.Wp + 1) + 1, patch));
  const int pieces = (len + 15) >> 4;              // KiB
  const uint32_t buffer = (uint32_t)((patch + 15) >> 4) * 1024u;
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t *)patch_lds;
  const size_t block_bytes = (size_t)P.N * P.Hp * P.Wp * 64;
  auto fetch_patch = [&](int cb) {                 // this wave's share; lanes past the end repeat the last 16 bytes
    const int8_t *src = xt + (size_t)cb * block_bytes + (size_t)o0 * 64;
    for (int piece = wave; piece < pieces; piece += 4)
      load_to_lds16(src, min((uint32_t)(piece * 1024 + lane * 16), (uint32_t)(len * 64 - 16)),
                    __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(cb & 1) * buffer + (uint32_t)piece * 1024u));
  };

  uint32_t b_at[NT];                               // LDS offset of this lane's pixel and channel slice at tap (0, 0)
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
    b_at[nt] = (uint32_t)(pixel_origin((tb0 + wn * NT + nt) * 16 + (lane & 15)) - o0) * 64u + (uint32_t)(lane >> 4) * 16u;

  // weights: consecutive in memory in the order of the steps; D register sets, the one a step has used is refilled for the
  // step D later (past the last step the last one's weights are fetched again and not used)
  const int8_t *a_next = wt + (size_t)kb0 * 1024;
  const uint32_t a_step = (uint32_t)nkb * 1024u, a_lane = (uint32_t)lane * 16u;
  int a_left = total - 1;
  auto load_a = [&](v4i (&a)[RM]) {
#pragma unroll
    for (int rm = 0; rm < RM; ++rm) a[rm] = *(const v4i *)(a_next + rm * 1024 + a_lane);
    a_next += a_left > 0 ? a_step : 0u;
    --a_left;
  };

  // The waits below count these loads; a plain load of constant memory is ordered against them by nothing but the scheduling barriers.
  fetch_patch(0);
  __builtin_amdgcn_sched_barrier(0);
  v4i a[D][RM];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    load_a(a[d]);
    __builtin_amdgcn_sched_barrier(0);
  }

  v4i acc[RM][NT];
#pragma unroll
  for (int rm = 0; rm < RM; ++rm)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[rm][nt] = (v4i){0, 0, 0, 0};

  // A step's pixels are read from LDS while the step before it multiplies.
  int tap = 0, tj = 0, cb = 0;                     // of the step whose pixels are read next
  uint32_t tap_off = 0;                            // LDS offset of that tap, its block's buffer included
  const uint32_t row_skip = (uint32_t)(P.Wp - P.r + 1) * 64u;
  v4i b[2][NT];
  auto read_next = [&](v4i (&into)[NT]) {
    if (tap == taps) {
      // a new channel block: everybody's share of its patch has landed (the weights' loads behind the patch's, RM for each of at least
      // three steps, need not have: hence r >= 2, which the host checks), and everybody has read the last of the block before, whose buffer
      // is refilled (waited for here: of a barrier's own wait the compiler keeps only what it finds in flight at the loop's entry)
      tap = tj = 0;
      tap_off = 0;                                 // (behind the last step: read, not used)
      if (++cb < ncb) {
        wait_vmcnt<RM * (D < 3 ? D : 3)>();
        wait_lds();
        __syncthreads();
        if (cb + 1 < ncb) fetch_patch(cb + 1);
        tap_off = (uint32_t)(cb & 1) * buffer;
      }
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) into[nt] = *(const v4i *)(patch_lds + (b_at[nt] + tap_off));
    ++tap;
    tap_off += 64;
    if (++tj == P.r) { tj = 0; tap_off += row_skip - 64u; }
  };
  auto step = [&](v4i (&aset)[RM], v4i (&use)[NT], v4i (&next)[NT]) {
    read_next(next);
    __builtin_amdgcn_sched_barrier(0);             // (left alone, the scheduler moves the reads behind the products)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int rm = 0; rm < RM; ++rm) acc[rm][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(aset[rm], use[nt], acc[rm][nt], 0, 0, 0);
    load_a(aset);
  };
  static_assert(D % 2 == 0, "the two sets of pixels alternate");
  wait_vmcnt<RM * D>();
  __syncthreads();
  if (ncb > 1) fetch_patch(1);
  read_next(b[0]);
  // Awaited here, with the pointer of y that the compiler fetches above: scalar and LDS loads share a counter and return in any order, and
  // with it pending at the loop's entry the first step of every D would wait for the pixels it has just requested.
  wait_lds();
  int it = 0;
  for (; it + D <= total; it += D)
#pragma unroll
    for (int d = 0; d < D; ++d) step(a[d], b[d & 1], b[1 - (d & 1)]);
#pragma unroll
  for (int d = 0; d < D - 1; ++d)
    if (it + d < total) step(a[d], b[d & 1], b[1 - (d & 1)]);

  // a lane holds rows 16 kb + 4 (lane / 16) + j of pixel 16 tb + lane % 16
  const size_t plane = (size_t)P.Ho * P.Wo;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int pix = (tb0 + wn * NT + nt) * 16 + (lane & 15);
    if (pix >= P.npix) continue;
    const int n = (int)fast_div((uint32_t)pix, P.by_plane), rem = pix - n * (P.Ho * P.Wo);
    int32_t *ypix = y + (size_t)n * P.K * plane + rem;
#pragma unroll
    for (int rm = 0; rm < RM; ++rm)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = (kb0 + rm) * 16 + 4 * (lane >> 4) + j;
        if (k < P.K) ypix[(size_t)k * plane] = acc[rm][nt][j];
      }
  }
}

}  // namespace rnswino
