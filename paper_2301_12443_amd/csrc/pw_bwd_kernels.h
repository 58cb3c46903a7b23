// The backward pass of an expand layer (dense 1 x 1, stride 1, few inputs, at most 192 outputs, batch norm behind it) in one kernel.
//
// What bounds it: memory.  The output side (dz, the gradient of the normalised output, and y, the convolution output) is the largest tensor
// of an inverted residual, up to twelve times the input side.  Separate passes move it five times: the batch norm's last stage reads both
// and writes dy, the weight gradient and backward-data read dy.  Here each element of dz and y is read once, dy is formed between load and
// LDS and both products take it from there:
//   dx[m][ci]  = sum_c dy[m][c] w[c][ci]       reduction over the channels, 32 at a time, in order
//   dw[c][ci]  = sum_m dy[m][c] x[m][ci]       reduction over the pixels, accumulators of all channels kept in registers
// A wave works alone on tiles of 32 pixels: its chunk of 32 pixels x 32 channels passes through LDS rows of its own, so that the loop has
// no barrier and eight waves a compute unit drift apart and keep the loads flowing.  Chunks are requested `D` ahead (up to a whole tile), 4 KB
// a wave each.  One workgroup a compute unit walks the pixels; its waves' weight gradients meet in LDS at the end.
//
// Measured: 4.6 TB/s of what it has to move in MobileNetV2's step at batch 128, 4.2 in the supernet's at batch 64.  Same machine, alternating
// with the separate passes: supernet step 32.67 -> 30.94 ms, search step 17.92 -> 17.33, MobileNetV2 23.47 -> 22.50 ms for four batches, 1.839 ->
// 1.789 at batch 33.
#pragma once
#include "dw_mfma_kernels.h"

namespace pbd {

constexpr int kPwThreads = 512, kPwWaves = kPwThreads / 64;
constexpr int kPwMaxIn = 32, kPwMaxOut = 192;         // one 32-wide tile of inputs; 96 registers of accumulators beside the chunks in flight
constexpr int kPwPix = 32;                            // pixels a wave takes at a time
constexpr int kPwPitch = 40;                          // LDS row of 32 bf16: 80 bytes, no conflicts by rows or transposed

struct PwBwdArgs {
  int M, C, cin;            // pixels, output channels (a multiple of 8), input channels in memory (8, 16, 24 or 32)
  int tiles;                // of kPwPix pixels
  int accumulate;           // dx already holds a gradient
  unsigned y_bytes, x_bytes, dx_bytes;   // dx_bytes 0: no dx (the layer reads the block's input)
};
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
// Between a wave's accesses to LDS rows of its own that its lanes exchange data through.  The hardware carries out a wave's LDS accesses in
// order; the fence keeps the compiler from changing that order and costs no instruction.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// NC: chunks of 32 output channels.  WGRAD false: the architecture round.
// (No branch in the loop: loads and stores that a launch or a lane has no use for go out of range, which keeps the number of loads in flight
// known; a wait for a conditional one would be a wait for all that were requested ahead.)
template <int NC, bool WGRAD>
__global__ __launch_bounds__(kPwThreads, 2) void pw_bwd_kernel(const bf16_t* __restrict__ dz, const bf16_t* __restrict__ y,
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ w, bf16_t* __restrict__ dx, float* __restrict__ part, PwBwdArgs g, BnBwd f) {
  constexpr int D = NC > 4 ? 3 : NC;                 // chunks in flight (divides NC: a chunk's registers are known at compile time)
  constexpr int CP = NC * 32, WP = CP + 8;            // row of the transposed filter in LDS: no conflicts
  __shared__ __attribute__((aligned(16))) bf16_t wt[32 * WP];
  __shared__ __attribute__((aligned(16))) float cf[5 * CP];                         // mu, a, b, p, q of bn_bwd_terms
  __shared__ __attribute__((aligned(16))) bf16_t tile_s[kPwWaves * 2 * kPwPix * kPwPitch];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  bf16_t* const ds = tile_s + wave * 2 * kPwPix * kPwPitch;                         // dy: 32 pixels x 32 channels
  bf16_t* const xs = ds + kPwPix * kPwPitch;                                        // x: 32 pixels x 32 channels
  static_assert(kPwWaves * 2 * kPwPix * kPwPitch * 2 >= kPwWaves * 1024 * 4, "the waves' 32 x 32 sums fit where the tiles were");

  for (int i = tid; i < CP; i += kPwThreads) {
    const BnBwdTerms t = i < g.C ? bn_bwd_terms(f, i) : BnBwdTerms{};
    cf[i] = t.mu; cf[CP + i] = t.a; cf[2 * CP + i] = t.b; cf[3 * CP + i] = t.p; cf[4 * CP + i] = t.q;
  }
  for (int i = tid; i < 4 * CP; i += kPwThreads) {    // 8 inputs of an output channel at a time
    const int c = i >> 2, ci = (i & 3) * 8;
    uint4 q = make_uint4(0, 0, 0, 0);
    if (c < g.C && ci < g.cin) q = *reinterpret_cast<const uint4*>(w + (size_t)c * g.cin + ci);
    const bf16_t* e = reinterpret_cast<const bf16_t*>(&q);
#pragma unroll
    for (int k = 0; k < 8; ++k) wt[(ci + k) * WP + c] = e[k];
  }
  __syncthreads();

  const __amdgpu_buffer_rsrc_t zr = tensor_rsrc(dz, g.y_bytes), yr = tensor_rsrc(y, g.y_bytes), xr = tensor_rsrc(x, g.x_bytes);
  const unsigned limit = dw_pass_limit(f.act);
  const int lrow = lane >> 2, lcol = (lane & 3) * 8;  // a thread's rows lrow, lrow + 16 and its 8 channels of a chunk
  const int stride = (int)gridDim.x * kPwWaves;
  const __amdgpu_buffer_rsrc_t dr = tensor_rsrc(dx, g.dx_bytes);

  uint4 zq[D][2], yq[D][2], xq[2];
  auto load = [&](int slot, int t, int kc) {
    const int c = kc * 32 + lcol;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int m = t * kPwPix + lrow + 16 * i;
      const unsigned off = t < g.tiles && m < g.M && c < g.C ? ((unsigned)m * g.C + c) * 2u : kOutOfRange;
      zq[slot][i] = buffer_load16(zr, off);
      yq[slot][i] = buffer_load16(yr, off);
    }
  };
  auto load_x = [&](int t) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int m = t * kPwPix + lrow + 16 * i;
      xq[i] = buffer_load16(xr, t < g.tiles && m < g.M && lcol < g.cin ? ((unsigned)m * g.cin + lcol) * 2u : kOutOfRange);
    }
  };

  f32x16 acc[WGRAD ? NC : 1];
#pragma unroll
  for (int k = 0; k < (WGRAD ? NC : 1); ++k)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[k][v] = 0.f;

  // fragment addresses: rows as they lie (8 channels of a pixel), and transposed (8 pixels of a channel)
  const int r32 = lane & 31, half = lane >> 5;
  const int row_frag = r32 * kPwPitch + half * 8;
  const int s16 = lane & 15, gl = lane >> 4;
  const int tr_frag = (8 * (gl >> 1) + (s16 >> 2)) * kPwPitch + 16 * (gl & 1) + 4 * (s16 & 3);
  const int w_frag = r32 * WP + half * 8;

  int t = (int)blockIdx.x * kPwWaves + wave;
  if (WGRAD) load_x(t);
  __builtin_amdgcn_sched_barrier(0);                  // (requested in the order in which they are waited for)
#pragma unroll
  for (int k = 0; k < D; ++k) {
    load(k, t, k);
    __builtin_amdgcn_sched_barrier(0);
  }
  for (; t < g.tiles; t += stride) {
    const unsigned in0 = t * kPwPix + lrow < g.M ? ~0u : 0u, in1 = t * kPwPix + lrow + 16 < g.M ? ~0u : 0u;
    bf16x8 xf[2];
    if constexpr (WGRAD) {
#pragma unroll
      for (int i = 0; i < 2; ++i) *reinterpret_cast<uint4*>(xs + (lrow + 16 * i) * kPwPitch + lcol) = xq[i];
      load_x(t + stride);
      wave_lds_fence();
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) xf[ks] = lds_read_tr8(xs + tr_frag + ks * 16 * kPwPitch, kPwPitch);
    }
    const int m = t * kPwPix + r32;                   // lane: pixel r32, input channels 8 q + 4 half .. + 3
    unsigned dx_off[4];
    u32x2 old[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      dx_off[q] = m < g.M && q * 8 < g.cin ? ((unsigned)m * g.cin + q * 8 + 4 * half) * 2u : kOutOfRange;
      old[q] = __builtin_amdgcn_raw_buffer_load_b64(dr, (int)(g.accumulate ? dx_off[q] : kOutOfRange), 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    f32x16 dxa;
#pragma unroll
    for (int v = 0; v < 16; ++v) dxa[v] = 0.f;
#pragma unroll
    for (int kc = 0; kc < NC; ++kc) {
      constexpr int kD = D;
      const int slot = kc % kD;
      uint4 o[2];
#pragma unroll
      for (int h = 0; h < 4; ++h) {                   // two channels at a time
        const float* p = cf + kc * 32 + lcol + 2 * h;
        const float2 mu = dw_pair(p), a = dw_pair(p + CP), b = dw_pair(p + 2 * CP), fp = dw_pair(p + 3 * CP), fq = dw_pair(p + 4 * CP);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const unsigned dw = dw_word(zq[slot][i], h), yw = dw_word(yq[slot][i], h);
          const float y0 = bf_lo(yw) - mu.x, y1 = bf_hi(yw) - mu.y;
          const float d0 = dw_pass(fmaf(y0, a.x, b.x), bf_lo(dw), limit), d1 = dw_pass(fmaf(y1, a.y, b.y), bf_hi(dw), limit);
          const unsigned v = pack_bf2(bn_bwd_dy(y0, d0, a.x, fp.x, fq.x), bn_bwd_dy(y1, d1, a.y, fp.y, fq.y)) & (i ? in1 : in0);
          if (h == 0) o[i].x = v; else if (h == 1) o[i].y = v; else if (h == 2) o[i].z = v; else o[i].w = v;
        }
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) *reinterpret_cast<uint4*>(ds + (lrow + 16 * i) * kPwPitch + lcol) = o[i];
      load(slot, kc + kD < NC ? t : t + stride, (kc + kD) % NC);
      __builtin_amdgcn_sched_barrier(0);
      wave_lds_fence();
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const bf16x8 df = *reinterpret_cast<const bf16x8*>(ds + row_frag + ks * 16);
        const bf16x8 wf = *reinterpret_cast<const bf16x8*>(wt + w_frag + kc * 32 + ks * 16);
        dxa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, df, dxa, 0, 0, 0);
      }
      if constexpr (WGRAD) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
          acc[kc] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_read_tr8(ds + tr_frag + ks * 16 * kPwPitch, kPwPitch), xf[ks], acc[kc], 0, 0, 0);
      }
      wave_lds_fence();
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const u32x2 o = {pack_bf2(dxa[4 * q] + bf_lo(old[q].x), dxa[4 * q + 1] + bf_hi(old[q].x)),
                       pack_bf2(dxa[4 * q + 2] + bf_lo(old[q].y), dxa[4 * q + 3] + bf_hi(old[q].y))};
      __builtin_amdgcn_raw_buffer_store_b64(o, dr, (int)dx_off[q], 0, 0);
    }
  }

  if constexpr (WGRAD) {                              // the waves' sums, in wave order
    float* const sums = reinterpret_cast<float*>(tile_s);
    float* const out = part + (size_t)blockIdx.x * g.C * g.cin;
#pragma unroll
    for (int kc = 0; kc < NC; ++kc) {
      __syncthreads();
#pragma unroll
      for (int v = 0; v < 16; ++v) sums[wave * 1024 + (8 * (v >> 2) + 4 * half + (v & 3)) * 32 + r32] = acc[kc][v];
      __syncthreads();
      for (int i = tid; i < 1024; i += kPwThreads) {
        float s = sums[i];
#pragma unroll
        for (int k = 1; k < kPwWaves; ++k) s += sums[k * 1024 + i];
        const int c = kc * 32 + (i >> 5), ci = i & 31;
        if (c < g.C && ci < g.cin) out[c * g.cin + ci] = s;
      }
    }
  }
}

// The backward pass of a projection (dense 1 x 1 layer of at most 32 outputs that normalises the layer in front as it stages it, FOLD in
// conv_kernels.h) together with the first stage of that layer's batch norm.
//
// What bounds it: memory, as above; here the input side is the large one.  Separate passes move it five times (backward-data writes dz, the
// weight gradient reads the convolution output y in front, the batch-norm reduction reads both); here y is read and dz written once:
//   dz[m][c]  = sum_k dy[m][k] w[k][c]
//   dw[k][c]  = sum_m dy[m][k] z[m][c],   z = act(norm(y)) formed on the way to LDS
//   sums of dpre and dpre * xhat over the pixels, dpre = dz where the rectifier passes
// A workgroup has 64 channels (whole cache lines; dy, the small side, is read once for each 64) and every pblocks-th group of 128 pixels; a
// wave works alone on 32 pixels, two tiles requested ahead.  The filter stays in registers as fragments.
//
// Measured: 3.9 TB/s of what it has to move in the supernet's step at batch 64, 4.4 in MobileNetV2's at batch 128.  Against the separate passes:
// supernet step 30.9 -> 29.0 ms, search step 17.3 -> 16.7, MobileNetV2 22.5 -> 21.8 ms for four batches, 1.789 -> 1.765 at batch 33.
constexpr int kPjThreads = 256, kPjWaves = kPjThreads / 64, kPjCh = 64;
constexpr int kPjPitch = kPjCh + 8;                   // 144 bytes

// Two sums of a wave for each of 64 channels, 8 of which a lane has (from 8 (lane % 8) on): out[channel], out[64 + channel].
__device__ __forceinline__ void wave_channel_sums(float (&s1)[8], float (&s2)[8], float* out, int lane) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
#pragma unroll
    for (int off = 8; off < 64; off <<= 1) {
      s1[e] += __shfl_xor(s1[e], off, 64);
      s2[e] += __shfl_xor(s2[e], off, 64);
    }
    if (lane < 8) {
      out[lane * 8 + e] = s1[e];
      out[64 + lane * 8 + e] = s2[e];
    }
  }
}

struct PjBwdArgs {
  int M, C, K;              // pixels, channels of the input (a multiple of 8), outputs (8, 16, 24 or 32)
  int tiles, groups, pblocks;
  unsigned y_bytes, dy_bytes;
};

template <bool WGRAD>
__device__ __forceinline__ void pj_bwd_block(const Blk& blk, const bf16_t* __restrict__ dy, const bf16_t* __restrict__ y,
    const bf16_t* __restrict__ wt, bf16_t* __restrict__ dz, float* __restrict__ wpart, float* __restrict__ spart, PjBwdArgs g, NormFold f) {
  __shared__ __attribute__((aligned(16))) bf16_t tile_s[kPjWaves * kPwPix * (kPjPitch + kPwPitch)];
  static_assert(sizeof tile_s >= kPjWaves * 1024 * 4, "the waves' 32 x 32 sums fit where the tiles were");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  bf16_t* const zs = tile_s + wave * kPwPix * (kPjPitch + kPwPitch);     // dz, then z: 32 pixels x 64 channels
  bf16_t* const ds = zs + kPwPix * kPjPitch;                             // dy: 32 pixels x 32 outputs
  const int wg = xcd_contiguous(blk.x, blk.gx);
  const int c0 = (wg % g.groups) * kPjCh, pb = wg / g.groups;
  const __amdgpu_buffer_rsrc_t yr = tensor_rsrc(y, g.y_bytes), zr = tensor_rsrc(dz, g.y_bytes), dr = tensor_rsrc(dy, g.dy_bytes);
  const int r32 = lane & 31, half = lane >> 5;
  const int lrow = lane >> 3, lcol = (lane & 7) * 8;                     // a thread's rows lrow, lrow + 8, ... and its 8 channels
  const bool ch_in = c0 + lcol < g.C;
  const unsigned limit = dw_pass_limit(f.act);
  const float hi = f.act == ACT_RELU6 ? 6.f : __builtin_inff();

  bf16x8 wf[2][2];                                                       // 32 channels x 16 outputs each
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int c = c0 + i * 32 + r32, k = ks * 16 + half * 8;
      uint4 q = make_uint4(0, 0, 0, 0);
      if (c < g.C && k < g.K) q = *reinterpret_cast<const uint4*>(wt + (size_t)c * g.K + k);
      wf[i][ks] = __builtin_bit_cast(bf16x8, q);
    }
  float mu[8], a[8], b[8], s1[8], s2[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int c = ch_in ? c0 + lcol + e : 0;
    mu[e] = f.mean[c]; a[e] = f.gamma[c] * f.invstd[c]; b[e] = f.beta[c];
    s1[e] = s2[e] = 0.f;
  }
  f32x16 acc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
  const int s16 = lane & 15, gl = lane >> 4;
  const int tr_row = 8 * (gl >> 1) + (s16 >> 2), tr_col = 16 * (gl & 1) + 4 * (s16 & 3);

  uint4 yq[2][4], dq[2][2];
  auto load_dy = [&](int slot, int t) {
    const int m = t * kPwPix + r32;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int k = ks * 16 + half * 8;
      dq[slot][ks] = buffer_load16(dr, t < g.tiles && m < g.M && k < g.K ? ((unsigned)m * g.K + k) * 2u : kOutOfRange);
    }
  };
  auto y_off = [&](int t, int i) {
    const int m = t * kPwPix + lrow + 8 * i;
    return t < g.tiles && m < g.M && ch_in ? ((unsigned)m * g.C + c0 + lcol) * 2u : kOutOfRange;
  };
  auto load_y = [&](int slot, int t) {
#pragma unroll
    for (int i = 0; i < 4; ++i) yq[slot][i] = buffer_load16(yr, y_off(t, i));
  };
  const int stride = g.pblocks * kPjWaves;
  int t = pb * kPjWaves + wave;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    load_dy(k, t + k * stride);
    __builtin_amdgcn_sched_barrier(0);                // (requested in the order in which they are waited for)
    load_y(k, t + k * stride);
    __builtin_amdgcn_sched_barrier(0);
  }
  for (; t < g.tiles; t += 2 * stride) {
#pragma unroll
    for (int slot = 0; slot < 2; ++slot) {            // (past the last tile: nothing but zeros, and nothing stored)
      const int tt = t + slot * stride;
      const bf16x8 d0 = __builtin_bit_cast(bf16x8, dq[slot][0]), d1 = __builtin_bit_cast(bf16x8, dq[slot][1]);
#pragma unroll
      for (int i = 0; i < 2; ++i) {                   // lane: pixel r32, channels 32 i + 8 q + 4 half .. + 3
        f32x16 d;
#pragma unroll
        for (int v = 0; v < 16; ++v) d[v] = 0.f;
        d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[i][0], d0, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[i][1], d1, d, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<uint2*>(zs + r32 * kPjPitch + i * 32 + q * 8 + 4 * half) =
              make_uint2(pack_bf2(d[4 * q], d[4 * q + 1]), pack_bf2(d[4 * q + 2], d[4 * q + 3]));
      }
      if constexpr (WGRAD) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) *reinterpret_cast<uint4*>(ds + r32 * kPwPitch + ks * 16 + half * 8) = dq[slot][ks];
      }
      load_dy(slot, tt + 2 * stride);
      __builtin_amdgcn_sched_barrier(0);
      wave_lds_fence();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint4* const at = reinterpret_cast<uint4*>(zs + (lrow + 8 * i) * kPjPitch + lcol);
        const uint4 dv = *at;
        const unsigned off = y_off(tt, i), in = off == kOutOfRange ? 0u : ~0u;
        const u32x4 out = {dv.x, dv.y, dv.z, dv.w};
        __builtin_amdgcn_raw_buffer_store_b128(out, zr, (int)off, 0, 0);
        unsigned z[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          const unsigned dw = dw_word(dv, h), yw = dw_word(yq[slot][i], h);
          const float y0 = bf_lo(yw) - mu[2 * h], y1 = bf_hi(yw) - mu[2 * h + 1];
          const float p0 = fmaf(y0, a[2 * h], b[2 * h]), p1 = fmaf(y1, a[2 * h + 1], b[2 * h + 1]);
          const float g0 = dw_pass(p0, bf_lo(dw), limit), g1 = dw_pass(p1, bf_hi(dw), limit);
          s1[2 * h] += g0; s1[2 * h + 1] += g1;
          s2[2 * h] = fmaf(g0, y0, s2[2 * h]); s2[2 * h + 1] = fmaf(g1, y1, s2[2 * h + 1]);
          z[h] = pack_bf2(__builtin_amdgcn_fmed3f(p0, 0.f, hi), __builtin_amdgcn_fmed3f(p1, 0.f, hi)) & in;
        }
        if (WGRAD) *at = make_uint4(z[0], z[1], z[2], z[3]);
      }
      load_y(slot, tt + 2 * stride);
      __builtin_amdgcn_sched_barrier(0);
      wave_lds_fence();
      if constexpr (WGRAD) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          const bf16x8 df = lds_read_tr8(ds + (tr_row + ks * 16) * kPwPitch + tr_col, kPwPitch);
#pragma unroll
          for (int i = 0; i < 2; ++i)
            acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(df, lds_read_tr8(zs + (tr_row + ks * 16) * kPjPitch + i * 32 + tr_col, kPjPitch), acc[i], 0, 0, 0);
        }
        wave_lds_fence();
      }
    }
  }

  float* const sums = reinterpret_cast<float*>(tile_s);
  if constexpr (WGRAD) {                              // the waves' sums, in wave order
    float* const out = wpart + (size_t)pb * g.K * g.C;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      __syncthreads();
#pragma unroll
      for (int v = 0; v < 16; ++v) sums[wave * 1024 + (8 * (v >> 2) + 4 * half + (v & 3)) * 32 + r32] = acc[i][v];
      __syncthreads();
      for (int j = tid; j < 1024; j += kPjThreads) {
        float s = sums[j];
#pragma unroll
        for (int k = 1; k < kPjWaves; ++k) s += sums[k * 1024 + j];
        const int k = j >> 5, c = c0 + i * 32 + (j & 31);
        if (k < g.K && c < g.C) out[k * g.C + c] = s;
      }
    }
  }
  __syncthreads();
  wave_channel_sums(s1, s2, sums + wave * 128, lane);
  __syncthreads();
  if (tid < 128 && c0 + (tid & 63) < g.C) {
    float s = sums[tid];
#pragma unroll
    for (int k = 1; k < kPjWaves; ++k) s += sums[k * 128 + tid];
    const int c = c0 + (tid & 63);
    spart[(size_t)pb * 2 * g.C + (tid >> 6) * g.C + c] = tid < 64 ? s : s * f.invstd[c];
  }
}
template <bool WGRAD>
__global__ __launch_bounds__(kPjThreads, 2) void pj_bwd_kernel(const bf16_t* __restrict__ dy, const bf16_t* __restrict__ y,
    const bf16_t* __restrict__ wt, bf16_t* __restrict__ dz, float* __restrict__ wpart, float* __restrict__ spart, PjBwdArgs g, NormFold f) {
  pj_bwd_block<WGRAD>(one_block(), dy, y, wt, dz, wpart, spart, g, f);
}

// The forward pass of an expand layer (the same shapes as pw_bwd_kernel's): y = x w, and what its batch norm needs of it.
//
// What bounds it: memory, the writes of y.  The implicit GEMM walks through such a layer as load, one reduction step, staged store, one after the
// other, its tiles two or three a compute unit; here a workgroup keeps its 64 channels' filter in registers and walks the pixels, a wave works
// alone on 32 of them, its store (whole cache lines, through LDS rows of its own) beside the next tile's products.
// AFFINE (the teacher): the folded batch norm and the rectifier on the way out.  Else the batch norm's statistics of y as stored: a mean, a sum
// of squares about it and a count for each workgroup and channel, as bn_finalize_kernel<T, true> merges them.  A workgroup sums y - y0 and its
// square, y0 the output at its own first pixel: a pixel far from the others costs the precision of its own workgroup's share (M pixels with
// one of them as everybody's y0, on blank images, M times a rounding error of the variance).
//
// Measured against igemm_kernel (2.2 to 2.8 TB/s on these layers), same machine, alternating: supernet step 28.96 -> 28.33 ms, search step
// 16.71 -> 16.30, MobileNetV2 21.75 -> 21.35 ms for four batches, 1.762 -> 1.737 at batch 33.
constexpr int kPwfThreads = 256, kPwfWaves = kPwfThreads / 64;

struct PwFwdArgs {
  int M, K, C;              // pixels, inputs (8, 16, 24 or 32), outputs (a multiple of 8)
  int tiles, groups, pblocks;
  unsigned x_bytes, y_bytes;
};

template <bool AFFINE>
__device__ __forceinline__ void pw_fwd_block(const Blk& blk, const bf16_t* __restrict__ x, const bf16_t* __restrict__ w, bf16_t* __restrict__ y,
    const float* __restrict__ ea, const float* __restrict__ eb, int act, float* __restrict__ spart, PwFwdArgs g) {
  __shared__ __attribute__((aligned(16))) bf16_t tile_s[kPwfWaves * kPwPix * kPjPitch];
  __shared__ __attribute__((aligned(16))) float ep_s[AFFINE ? 2 * kPjCh : 4];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  bf16_t* const ys = tile_s + wave * kPwPix * kPjPitch;                  // y: 32 pixels x 64 channels
  const int wg = xcd_contiguous(blk.x, blk.gx);
  const int c0 = (wg % g.groups) * kPjCh, pb = wg / g.groups;
  const __amdgpu_buffer_rsrc_t xr = tensor_rsrc(x, g.x_bytes), yr = tensor_rsrc(y, g.y_bytes);
  const int r32 = lane & 31, half = lane >> 5;
  const int lrow = lane >> 3, lcol = (lane & 7) * 8;                     // a thread's rows lrow, lrow + 8, ... and its 8 channels
  const bool ch_in = c0 + lcol < g.C;

  bf16x8 wf[2][2];                                                       // 32 channels x 16 inputs each
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int c = c0 + i * 32 + r32, k = ks * 16 + half * 8;
      uint4 q = make_uint4(0, 0, 0, 0);
      if (c < g.C && k < g.K) q = *reinterpret_cast<const uint4*>(w + (size_t)c * g.K + k);
      wf[i][ks] = __builtin_bit_cast(bf16x8, q);
    }
  if (AFFINE) {
    if (tid < kPjCh) {
      ep_s[tid] = c0 + tid < g.C ? ea[c0 + tid] : 0.f;
      ep_s[kPjCh + tid] = c0 + tid < g.C ? eb[c0 + tid] : 0.f;
    }
    __syncthreads();
  }
  auto load = [&](uint4 (&q)[2], int m, bool in) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int k = ks * 16 + half * 8;
      q[ks] = buffer_load16(xr, in && k < g.K ? ((unsigned)m * g.K + k) * 2u : kOutOfRange);
    }
  };
  auto product = [&](const uint4 (&q)[2]) {           // lane: pixel r32, channels 32 i + 8 q + 4 half .. + 3
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      f32x16 d;
#pragma unroll
      for (int v = 0; v < 16; ++v) d[v] = 0.f;
      d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[i][0], __builtin_bit_cast(bf16x8, q[0]), d, 0, 0, 0);
      d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[i][1], __builtin_bit_cast(bf16x8, q[1]), d, 0, 0, 0);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int col = i * 32 + u * 8 + 4 * half;
        float o[4] = {d[4 * u], d[4 * u + 1], d[4 * u + 2], d[4 * u + 3]};
        if (AFFINE) {
          const float4 a = *reinterpret_cast<const float4*>(ep_s + col), b = *reinterpret_cast<const float4*>(ep_s + kPjCh + col);
          o[0] = apply_act(fmaf(o[0], a.x, b.x), act); o[1] = apply_act(fmaf(o[1], a.y, b.y), act);
          o[2] = apply_act(fmaf(o[2], a.z, b.z), act); o[3] = apply_act(fmaf(o[3], a.w, b.w), act);
        }
        *reinterpret_cast<uint2*>(ys + r32 * kPjPitch + col) = make_uint2(pack_bf2(o[0], o[1]), pack_bf2(o[2], o[3]));
      }
    }
  };

  uint4 xq[2][2];
  float y0[8], s1[8], s2[8];
  if constexpr (!AFFINE) {                            // the outputs at the workgroup's first pixel, in every row
    load(xq[0], pb * kPwfWaves * kPwPix, true);
    product(xq[0]);
    wave_lds_fence();
    IO<bf16_t>::unpack(*reinterpret_cast<const uint4*>(ys + lcol), y0);
    wave_lds_fence();
#pragma unroll
    for (int e = 0; e < 8; ++e) s1[e] = s2[e] = 0.f;
  }
  const int stride = g.pblocks * kPwfWaves;
  int t = pb * kPwfWaves + wave;
  auto load_tile = [&](uint4 (&q)[2], int tt) { load(q, tt * kPwPix + r32, tt < g.tiles && tt * kPwPix + r32 < g.M); };
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    load_tile(xq[k], t + k * stride);
    __builtin_amdgcn_sched_barrier(0);                // (requested in the order in which they are waited for)
  }
  for (; t < g.tiles; t += 2 * stride) {
#pragma unroll
    for (int slot = 0; slot < 2; ++slot) {            // (past the last tile: nothing is stored or summed)
      const int tt = t + slot * stride;
      product(xq[slot]);
      load_tile(xq[slot], tt + 2 * stride);
      __builtin_amdgcn_sched_barrier(0);
      wave_lds_fence();
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint4 v = *reinterpret_cast<const uint4*>(ys + (lrow + 8 * i) * kPjPitch + lcol);
        const int m = tt * kPwPix + lrow + 8 * i;
        const bool in = tt < g.tiles && m < g.M && ch_in;
        const u32x4 out = {v.x, v.y, v.z, v.w};
        __builtin_amdgcn_raw_buffer_store_b128(out, yr, (int)(in ? ((unsigned)m * g.C + c0 + lcol) * 2u : kOutOfRange), 0, 0);
        if constexpr (!AFFINE) {
          if (in) {
            float f[8];
            IO<bf16_t>::unpack(v, f);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              f[e] -= y0[e];
              s1[e] += f[e];
              s2[e] = fmaf(f[e], f[e], s2[e]);
            }
          }
        }
      }
      wave_lds_fence();
    }
  }
  if constexpr (!AFFINE) {
    float* const sums = reinterpret_cast<float*>(tile_s);
    __syncthreads();
    wave_channel_sums(s1, s2, sums + wave * 128, lane);
    if (tid < 8) {
#pragma unroll
      for (int e = 0; e < 8; ++e) sums[kPwfWaves * 128 + tid * 8 + e] = y0[e];
    }
    __syncthreads();
    if (tid < 64 && c0 + tid < g.C) {
      float a = sums[tid], b = sums[64 + tid];
#pragma unroll
      for (int k = 1; k < kPwfWaves; ++k) { a += sums[k * 128 + tid]; b += sums[k * 128 + 64 + tid]; }
      // the workgroup's tiles (tile t is that of workgroup t / waves mod pblocks), the last of all perhaps not full
      const int own = g.tiles / stride * kPwfWaves + min(max(g.tiles % stride - pb * kPwfWaves, 0), kPwfWaves);
      const int missing = (g.tiles - 1) / kPwfWaves % g.pblocks == pb ? g.tiles * kPwPix - g.M : 0;
      const float n = (float)(own * kPwPix - missing), shift = a / n;
      float* const out = spart + (size_t)pb * 3 * g.C + c0 + tid;
      out[0] = sums[kPwfWaves * 128 + tid] + shift;
      out[g.C] = fmaxf(b - a * shift, 0.f);
      out[2 * g.C] = n;
    }
  }
}
template <bool AFFINE>
__global__ __launch_bounds__(kPwfThreads, 3) void pw_fwd_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w, bf16_t* __restrict__ y,
    const float* __restrict__ ea, const float* __restrict__ eb, int act, float* __restrict__ spart, PwFwdArgs g) {
  pw_fwd_block<AFFINE>(one_block(), x, w, y, ea, eb, act, spart, g);
}

}  // namespace pbd
