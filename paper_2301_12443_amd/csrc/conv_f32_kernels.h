// float32 dense convolutions on the fp32 matrix cores (v_mfma_f32_32x32x2_f32: fp32 products and fp32 sums, twice the
// vector ALUs' rate), channel-last tensors.
//
// An MFMA of this shape takes ONE float per lane and operand, lanes 0..31 one reduction element of the 32 rows,
// lanes 32..63 another, and which reduction element that is does not matter as long as both operands agree.  So
// both operands go from memory straight to registers, with no LDS staging and no transposition:
//  * igemm_f32_kernel (forward, backward-data): a lane loads 16 bytes, four consecutive channels of its pixel; half 0 the first
//    four of a run of eight, half 1 the other four; four MFMAs use them up.
//  * wgrad_f32_kernel (backward-weight): a lane loads 8 bytes of one pixel, two neighbouring channels; the even
//    and the odd rows / columns of a 64 x 64 tile are separate MFMAs.
// 64 cycles per MFMA against 8 to 16 bytes per lane: what a wave loads costs the L1 path a quarter of the time
// its matrix instructions take.  What bounds the small layers this precision is used on is latency, so the
// reduction is cut over the eight waves of a workgroup, each with a batch of loads in flight while the one before
// is multiplied, and the partial tiles meet in LDS in a fixed order (bit-reproducible).
//  Against one thread per result (conv_direct_*): VGG-16 at 64 x 32 x 32, forward 2516 -> 27 us a layer (72 TFLOP/s on
// the 64-wide tiles), backward-weight 3968 -> 9.6, backward-data 97 -> 9.7; its whole step 90.8 -> 1.53 ms, the
// four-layer network at 8 x 32 x 32 1943 -> 258 us.  Each result is also closer to the exact sum (eight shorter
// chains instead of one): relative error of a 64-channel 3 x 3 layer 4.1e-7 -> 1.6e-7.
#pragma once
#include "conv_kernels.h"

namespace pbd {

constexpr int kF32Threads = 512;                  // eight waves
constexpr int kF32Pitch = 36;                     // floats per staged row of 32: 16-byte accesses of neighbouring rows spread over the banks

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 buffer_load_f4(__amdgpu_buffer_rsrc_t r, unsigned byte_off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte_off, 0, 0));
}
__device__ __forceinline__ f32x2 buffer_load_f2(__amdgpu_buffer_rsrc_t r, unsigned byte_off) {
  return __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)byte_off, 0, 0));
}
__device__ __forceinline__ float buffer_load_f1(__amdgpu_buffer_rsrc_t r, unsigned byte_off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)byte_off, 0, 0));
}

// Same view as igemm_kernel: Out[m][j] = sum_kk Agather(m, kk) * W(j, kk), rows m = pixels of an [N][HO][WO] grid,
// kk = (r*S + s)*CA + c.  MODE 0 reads the weights as they lie, [NC][R][S][CA]; MODE 1 reads the forward filter
// [CA][R][S][NC] (the 32 columns of a tile are then contiguous), so there is no transposed copy to keep.
//   A wave owns MT x NT tiles of 32 pixels x 32 channels; of the eight waves KW share a tile and cut its reduction,
// the others take the next rows.  The workgroup's tile is (8 / KW) * 32 * MT rows x 32 * NT columns.
struct F32Args {
  IgemmArgs g;
  int kw_log2;            // 1, 2, 4 or 8 waves per tile
  int accumulate;         // Out += (backward-data into a value that already has a gradient)
};

template <int MODE, int MT, int NT>
__global__ __launch_bounds__(kF32Threads) void igemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ Bw,
                                                               float* __restrict__ Out, const float* __restrict__ ep_a,
                                                               const float* __restrict__ ep_b, int act, F32Args fa) {
  // reduction runs of 8 channels per batch: two batches in registers, the next one in flight
  constexpr int UNR = MT * NT == 1 ? 4 : 2;
  const IgemmArgs& g = fa.g;
  __shared__ __attribute__((aligned(16))) float part[8][32 * kF32Pitch];
  const int tid = threadIdx.x, lane = tid & 63, row = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kw = 1 << fa.kw_log2, ks = wave & (kw - 1), mw = wave >> fa.kw_log2, rows_wg = (8 >> fa.kw_log2) * 32 * MT;
  const int tile = xcd_contiguous(blockIdx.x, g.tiles_m * g.tiles_n);
  const int m0 = tile / g.tiles_n * rows_wg, n0 = tile % g.tiles_n * 32 * NT;
  const int sh = g.stride == 2 ? 1 : 0, smask = g.stride - 1;

  int rbase[MT], rh[MT], rw[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    const int m = m0 + (mw * MT + i) * 32 + row;
    const int mm = m < g.M ? m : 0;
    const int b_ = mm % g.WO, t = mm / g.WO, a_ = t % g.HO;
    rbase[i] = (t / g.HO) * g.HA * g.WA;
    rh[i] = MODE == 0 ? a_ * g.stride - g.pad : a_ + g.pad;
    rw[i] = MODE == 0 ? b_ * g.stride - g.pad : b_ + g.pad;
    if (m >= g.M) rh[i] = -(1 << 24);             // (fails every range test)
  }
  const __amdgpu_buffer_rsrc_t ra = tensor_rsrc(A, g.a_bytes), rb = tensor_rsrc(Bw, g.b_bytes);
  const int RS = g.R * g.S;
  unsigned bbase[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int col = n0 + j * 32 + row;
    bbase[j] = col >= g.NC ? kOutOfRange : (unsigned)(MODE == 0 ? col * g.Kred + 4 * half : 4 * half * RS * g.NC + col) * 4u;
  }

  // this wave's runs of 8: [run0, run1) of Kred / 8; the tap of a run is the same for all lanes
  const int runs = g.Kred >> 3, per = (runs + kw - 1) >> fa.kw_log2;
  const int run0 = min(runs, ks * per), run1 = min(runs, run0 + per);
  int r, s, c;
  {
    const int kk = run0 * 8, rs = kk / g.CA;
    c = kk - rs * g.CA; r = rs / g.S; s = rs - r * g.S;
  }
  f32x4 av[2][UNR][MT], bv[2][UNR][NT];
  int at = run0;
  auto load = [&](auto stage) {
    constexpr int S_ = decltype(stage)::value;
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const bool live = at < run1;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        int h = MODE == 0 ? rh[i] + r : rh[i] - r, w = MODE == 0 ? rw[i] + s : rw[i] - s;
        bool ok = live;
        if (MODE == 1) { ok = ok && ((h | w) & smask) == 0; h >>= sh; w >>= sh; }
        ok = ok && (unsigned)h < (unsigned)g.HA && (unsigned)w < (unsigned)g.WA;
        const unsigned off = (unsigned)((rbase[i] + h * g.WA + w) * g.CA + c + 4 * half) * 4u;
        av[S_][u][i] = buffer_load_f4(ra, ok ? off : kOutOfRange);
      }
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        if (MODE == 0) {
          bv[S_][u][j] = buffer_load_f4(rb, live ? bbase[j] + (unsigned)at * 32u : kOutOfRange);
        } else {
          // channels c .. c + 3 (+ 4 in half 1) of the reduction: one row of the forward filter each
          const unsigned step = (unsigned)(RS * g.NC) * 4u;
          const unsigned off = live ? bbase[j] + (unsigned)((c * RS + r * g.S + s) * g.NC) * 4u : kOutOfRange;
          bv[S_][u][j].x = buffer_load_f1(rb, off);
          bv[S_][u][j].y = buffer_load_f1(rb, live ? off + step : kOutOfRange);
          bv[S_][u][j].z = buffer_load_f1(rb, live ? off + 2 * step : kOutOfRange);
          bv[S_][u][j].w = buffer_load_f1(rb, live ? off + 3 * step : kOutOfRange);
        }
      }
      ++at;
      c += 8;
      if (c >= g.CA) { c = 0; if (++s == g.S) { s = 0; ++r; } }
    }
  };
  f32x16 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  auto multiply = [&](auto stage) {
    constexpr int S_ = decltype(stage)::value;
#pragma unroll
    for (int u = 0; u < UNR; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int j = 0; j < NT; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(bv[S_][u][j][e], av[S_][u][i][e], acc[i][j], 0, 0, 0);
  };
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  const int batches = (run1 - run0 + UNR - 1) / UNR;
  if (batches > 0) load(S0{});
  for (int t = 0; t < batches; t += 2) {
    if (t + 1 < batches) load(S1{});
    __builtin_amdgcn_sched_barrier(0);            // (the loads above are in flight while the batch before is multiplied)
    multiply(S0{});
    if (t + 1 >= batches) break;
    if (t + 2 < batches) load(S0{});
    __builtin_amdgcn_sched_barrier(0);
    multiply(S1{});
  }

  // a tile at a time: the KW partial tiles side by side in LDS, added in wave order, stored as whole rows
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      if (i + j > 0) __syncthreads();
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(&part[wave][row * kF32Pitch + 8 * q + 4 * half]) =
            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
      __syncthreads();
      for (int t = tid; t < (8 >> fa.kw_log2) * 256; t += kF32Threads) {
        const int w0 = t >> 8, px = (t >> 3) & 31, ch = (t & 7) * 4;
        const int m = m0 + (w0 * MT + i) * 32 + px, col = n0 + j * 32 + ch;
        if (m >= g.M || col >= g.NC) continue;    // NC % 8 == 0: a group of four is in or out as a whole
        float o[4] = {0.f, 0.f, 0.f, 0.f};
        for (int k = 0; k < kw; ++k) {
          const float4 p = *reinterpret_cast<const float4*>(&part[(w0 << fa.kw_log2) + k][px * kF32Pitch + ch]);
          o[0] += p.x; o[1] += p.y; o[2] += p.z; o[3] += p.w;
        }
        float4* dst = reinterpret_cast<float4*>(Out + (size_t)m * g.NC + col);
        if (ep_a) {
          const float4 ea = *reinterpret_cast<const float4*>(ep_a + col), eb = *reinterpret_cast<const float4*>(ep_b + col);
          o[0] = apply_act(fmaf(o[0], ea.x, eb.x), act); o[1] = apply_act(fmaf(o[1], ea.y, eb.y), act);
          o[2] = apply_act(fmaf(o[2], ea.z, eb.z), act); o[3] = apply_act(fmaf(o[3], ea.w, eb.w), act);
        } else if (fa.accumulate) {
          const float4 p = *dst;
          o[0] += p.x; o[1] += p.y; o[2] += p.z; o[3] += p.w;
        }
        *dst = make_float4(o[0], o[1], o[2], o[3]);
      }
    }
}

// dW[k][j] = sum over pixels of dy[m][k] * xcol[m][j]: 64 x 64 tiles, the pixels of a split dealt to the eight waves
// in turns of 2 * UNR, partial tiles added in LDS in wave order; `part` gets one [K][J] matrix per split.
template <int UNR>
__global__ __launch_bounds__(kF32Threads) void wgrad_f32_kernel(const float* __restrict__ dy, const float* __restrict__ x,
                                                               float* __restrict__ part, WgradTrArgs g) {
  constexpr int PITCH = 68;
  __shared__ __attribute__((aligned(16))) float red[8][32 * PITCH];
  const int tid = threadIdx.x, lane = tid & 63, row = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tile = xcd_contiguous(blockIdx.x, g.tiles_k * g.tiles_j * g.splits);
  const int slice = tile / (g.tiles_k * g.tiles_j);
  const int k0 = ((tile / g.tiles_j) % g.tiles_k) * 64, j0 = (tile % g.tiles_j) * 64;
  const int mbeg = slice * g.pix_per_split, mend = min(g.M, mbeg + g.pix_per_split);
  const __amdgpu_buffer_rsrc_t rd = tensor_rsrc(dy, g.dy_bytes), rx = tensor_rsrc(x, g.x_bytes);

  const int kcol = k0 + 2 * row, jcol = j0 + 2 * row;             // (both even: a pair is in or out as a whole)
  const bool k_ok = kcol < g.K, j_ok = jcol < g.J;
  int br, bs, bc;
  {
    const int rs = j_ok ? jcol / g.C : 0;
    bc = j_ok ? jcol - rs * g.C : 0;
    br = rs / g.S;
    bs = rs - br * g.S;
  }
  br -= g.pad; bs -= g.pad;
  // pixel of load u: mbeg + (turn * 8 + wave) * 2 UNR + 2 u + half, advanced by 16 UNR pixels a turn without divisions
  int pm[UNR], pn[UNR], pp[UNR], pq[UNR];
#pragma unroll
  for (int u = 0; u < UNR; ++u) {
    pm[u] = mbeg + wave * 2 * UNR + 2 * u + half;
    pq[u] = pm[u] % g.Q;
    const int t = pm[u] / g.Q;
    pp[u] = t % g.P;
    pn[u] = t / g.P;
  }
  f32x2 dv[2][UNR], xv[2][UNR];
  auto load = [&](auto stage) {
    constexpr int S_ = decltype(stage)::value;
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const bool live = pm[u] < mend;
      const int h = pp[u] * g.stride + br, w = pq[u] * g.stride + bs;
      const bool ok = live && j_ok && (unsigned)h < (unsigned)g.H && (unsigned)w < (unsigned)g.W;
      dv[S_][u] = buffer_load_f2(rd, live && k_ok ? (unsigned)(pm[u] * g.K + kcol) * 4u : kOutOfRange);
      xv[S_][u] = buffer_load_f2(rx, ok ? (unsigned)(((pn[u] * g.H + h) * g.W + w) * g.C + bc) * 4u : kOutOfRange);
      pm[u] += 16 * UNR;
      int q = pq[u] + g.dq;
      const int c1 = q >= g.Q ? 1 : 0;
      pq[u] = q - (c1 ? g.Q : 0);
      int p = pp[u] + g.dp + c1;
      const int c2 = p >= g.P ? 1 : 0;
      pp[u] = p - (c2 ? g.P : 0);
      pn[u] += g.dn + c2;
    }
  };
  f32x16 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
  auto multiply = [&](auto stage) {
    constexpr int S_ = decltype(stage)::value;
#pragma unroll
    for (int u = 0; u < UNR; ++u)
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(dv[S_][u][a], xv[S_][u][b], acc[a][b], 0, 0, 0);
  };
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  const int turns = (mend - mbeg + 16 * UNR - 1) / (16 * UNR);
  load(S0{});
  for (int t = 0; t < turns; t += 2) {
    if (t + 1 < turns) load(S1{});
    __builtin_amdgcn_sched_barrier(0);
    multiply(S0{});
    if (t + 1 >= turns) break;
    if (t + 2 < turns) load(S0{});
    __builtin_amdgcn_sched_barrier(0);
    multiply(S1{});
  }
  // even channels of the 64, then the odd ones: rows k0 + 2 i + a, all 64 columns
  float* out = part + (size_t)slice * g.K * g.J;
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    if (a) __syncthreads();
#pragma unroll
    for (int v = 0; v < 16; ++v)
      *reinterpret_cast<float2*>(&red[wave][(8 * (v >> 2) + 4 * half + (v & 3)) * PITCH + 2 * row]) = make_float2(acc[a][0][v], acc[a][1][v]);
    __syncthreads();
    const int i = tid >> 4, col = (tid & 15) * 4;                 // 512 threads: 32 rows x 16 groups of four columns
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      const float4 p = *reinterpret_cast<const float4*>(&red[w][i * PITCH + col]);
      o.x += p.x; o.y += p.y; o.z += p.z; o.w += p.w;
    }
    const int k = k0 + 2 * i + a, j = j0 + col;
    if (k < g.K && j < g.J) *reinterpret_cast<float4*>(out + (size_t)k * g.J + j) = o;
  }
}

}  // namespace pbd
