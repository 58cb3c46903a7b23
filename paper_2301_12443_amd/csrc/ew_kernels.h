// Bandwidth-bound kernels of the blockwise-distillation step for gfx950:
// layout/cast, batch normalisation (statistics, apply, backward), activations,
// max-pool, residual add, candidate mix, depthwise convolution, fused MSE loss +
// gradient, fused SGD-momentum.  Tensors are channel-last (NHWC); a thread owns
// one vector of 8 consecutive channels, so a wavefront touches contiguous
// 1 KiB (bf16) or 2 KiB (fp32) runs and every access is a 16-byte transaction.
// All reductions are two-stage and ordered (no atomics), which keeps a step
// bit-reproducible and independent of the order in which blocks are trained
// (Sec. IV-B: blocks share no parameters).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "many.h"

namespace pbd {

typedef __bf16 bf16_t;
enum { ACT_NONE = 0, ACT_RELU = 1, ACT_RELU6 = 2 };

__device__ __forceinline__ float bf_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }
// round-to-nearest-even pair conversion (v_cvt_pk_bf16_f32 on gfx950)
__device__ __forceinline__ uint32_t pack_bf2(float a, float b) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  f2 v = {a, b};
  b2 r = __builtin_convertvector(v, b2);
  return __builtin_bit_cast(uint32_t, r);
}

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Raw buffer descriptor over a whole tensor: a load whose byte offset lies outside [0, bytes) returns
// zeros in hardware, which turns padding, ragged tiles and the reduction tail into plain offsets
// (no branches, no selects).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tensor_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
__device__ __forceinline__ uint4 buffer_load16(__amdgpu_buffer_rsrc_t r, unsigned byte_off) {
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte_off, 0, 0);
  return make_uint4(v.x, v.y, v.z, v.w);
}
constexpr unsigned kOutOfRange = 0x80000000u;   // byte offset beyond any tensor (they are < 2^31 elements)

template <class T> struct IO;
// ld_raw() only starts the 16- or 32-byte load, unpack() converts later: a loop that calls ld_raw() for all its rows,
// then __builtin_amdgcn_sched_barrier(0), then unpack() has every load in flight before the first wait (left to
// itself the scheduler pairs each load with its conversion and the loads go out one at a time).
template <> struct IO<float> {
  struct Raw { float4 a, b; };
  static __device__ __forceinline__ Raw ld_raw(const float* p) {
    Raw q; q.a = reinterpret_cast<const float4*>(p)[0]; q.b = reinterpret_cast<const float4*>(p)[1]; return q;
  }
  template <bool STREAM> static __device__ __forceinline__ Raw ld_raw_t(const float* p) { return ld_raw(p); }
  template <bool STREAM> static __device__ __forceinline__ void st_t(float* p, const float v[8]) { st(p, v); }
  static __device__ __forceinline__ void unpack(const Raw& q, float v[8]) {
    v[0] = q.a.x; v[1] = q.a.y; v[2] = q.a.z; v[3] = q.a.w; v[4] = q.b.x; v[5] = q.b.y; v[6] = q.b.z; v[7] = q.b.w;
  }
  static __device__ __forceinline__ void ld(const float* p, float v[8]) {
    const float4 a = reinterpret_cast<const float4*>(p)[0], b = reinterpret_cast<const float4*>(p)[1];
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
  static __device__ __forceinline__ void st(float* p, const float v[8]) {
    reinterpret_cast<float4*>(p)[0] = make_float4(v[0], v[1], v[2], v[3]);
    reinterpret_cast<float4*>(p)[1] = make_float4(v[4], v[5], v[6], v[7]);
  }
};
template <> struct IO<bf16_t> {
  typedef uint4 Raw;
  static __device__ __forceinline__ Raw ld_raw(const bf16_t* p) { return *reinterpret_cast<const uint4*>(p); }
  // STREAM: nontemporal forms for the passes over tensors far larger than the caches: a line that is read or
  // written once per pass does not push out what the convolutions running beside the pass keep in L2
  typedef unsigned int u32x4_nt __attribute__((ext_vector_type(4)));
  template <bool STREAM> static __device__ __forceinline__ Raw ld_raw_t(const bf16_t* p) {
    if (!STREAM) return ld_raw(p);
    const u32x4_nt q = __builtin_nontemporal_load(reinterpret_cast<const u32x4_nt*>(p));
    return make_uint4(q.x, q.y, q.z, q.w);
  }
  template <bool STREAM> static __device__ __forceinline__ void st_t(bf16_t* p, const float v[8]) {
    if (!STREAM) { st(p, v); return; }
    u32x4_nt q = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7])};
    __builtin_nontemporal_store(q, reinterpret_cast<u32x4_nt*>(p));
  }
  static __device__ __forceinline__ void unpack(const Raw& u, float v[8]) {
    v[0] = bf_lo(u.x); v[1] = bf_hi(u.x); v[2] = bf_lo(u.y); v[3] = bf_hi(u.y);
    v[4] = bf_lo(u.z); v[5] = bf_hi(u.z); v[6] = bf_lo(u.w); v[7] = bf_hi(u.w);
  }
  static __device__ __forceinline__ void ld(const bf16_t* p, float v[8]) {
    const uint4 u = *reinterpret_cast<const uint4*>(p);
    v[0] = bf_lo(u.x); v[1] = bf_hi(u.x); v[2] = bf_lo(u.y); v[3] = bf_hi(u.y);
    v[4] = bf_lo(u.z); v[5] = bf_hi(u.z); v[6] = bf_lo(u.w); v[7] = bf_hi(u.w);
  }
  static __device__ __forceinline__ void st(bf16_t* p, const float v[8]) {
    uint4 u;
    u.x = pack_bf2(v[0], v[1]); u.y = pack_bf2(v[2], v[3]);
    u.z = pack_bf2(v[4], v[5]); u.w = pack_bf2(v[6], v[7]);
    *reinterpret_cast<uint4*>(p) = u;
  }
};

// Gathered 8-channel loads through a buffer descriptor: issue() only starts the load (an invalid
// position becomes an out-of-range offset and reads as zeros), unpack() converts later, so that a
// whole stencil of loads is in flight before the first use.
template <class T> struct BufIO;
template <> struct BufIO<bf16_t> {
  typedef uint4 Raw;
  static __device__ __forceinline__ Raw issue(__amdgpu_buffer_rsrc_t r, unsigned elem, bool ok) {
    return buffer_load16(r, ok ? elem * 2u : kOutOfRange);
  }
  static __device__ __forceinline__ Raw pack(const float v[8]) {
    return make_uint4(pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7]));
  }
  static __device__ __forceinline__ Raw slab_read(const uint4* s, int, int r) { return s[r]; }
  static __device__ __forceinline__ void slab_write(uint4* s, int, int r, const Raw& u) { s[r] = u; }
  static __device__ __forceinline__ void unpack(const Raw& u, float v[8]) {
    v[0] = bf_lo(u.x); v[1] = bf_hi(u.x); v[2] = bf_lo(u.y); v[3] = bf_hi(u.y);
    v[4] = bf_lo(u.z); v[5] = bf_hi(u.z); v[6] = bf_lo(u.w); v[7] = bf_hi(u.w);
  }
};
template <> struct BufIO<float> {
  struct Raw { uint4 a, b; };
  static __device__ __forceinline__ Raw issue(__amdgpu_buffer_rsrc_t r, unsigned elem, bool ok) {
    Raw q;
    q.a = buffer_load16(r, ok ? elem * 4u : kOutOfRange);
    q.b = buffer_load16(r, ok ? elem * 4u + 16u : kOutOfRange);
    return q;
  }
  static __device__ __forceinline__ Raw pack(const float v[8]) {
    return Raw{make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])),
               make_uint4(__float_as_uint(v[4]), __float_as_uint(v[5]), __float_as_uint(v[6]), __float_as_uint(v[7]))};
  }
  // (two planes: neighbouring lanes' rows lie 16 bytes apart in each)
  static __device__ __forceinline__ Raw slab_read(const uint4* s, int plane, int r) { return Raw{s[r], s[plane + r]}; }
  static __device__ __forceinline__ void slab_write(uint4* s, int plane, int r, const Raw& u) { s[r] = u.a; s[plane + r] = u.b; }
  static __device__ __forceinline__ void unpack(const Raw& u, float v[8]) {
    v[0] = __uint_as_float(u.a.x); v[1] = __uint_as_float(u.a.y); v[2] = __uint_as_float(u.a.z);
    v[3] = __uint_as_float(u.a.w); v[4] = __uint_as_float(u.b.x); v[5] = __uint_as_float(u.b.y);
    v[6] = __uint_as_float(u.b.z); v[7] = __uint_as_float(u.b.w);
  }
};

// Written as selects on two values derived from `act` (a clamp bound that no value reaches unless the layer is a
// ReLU6, and "no rectifier at all"), not as a branch per case: `act` is a launch argument, the kernels call this
// per element inside their loops, and the compiler keeps a branch chain per element otherwise.  Same value as the
// case-by-case definition for every input, NaN and infinities included:
//   ReLU: v > 0 ? v : 0;  ReLU6: v > 0 ? min(v, 6) : 0;  none: v
__device__ __forceinline__ float apply_act(float v, int act) {
  const bool all = act != ACT_RELU && act != ACT_RELU6;
  const float hi = act == ACT_RELU6 ? 6.f : __builtin_nanf("");     // (v >= NaN never holds)
  const float t = v >= hi ? hi : v;
  return (all || v > 0.f) ? t : 0.f;
}
// slope of the activation at pre-activation v (1 where it passes the gradient):
//   ReLU: v > 0;  ReLU6: 0 < v < 6;  none: always
__device__ __forceinline__ bool act_pass(float v, int act) {
  const bool all = act != ACT_RELU && act != ACT_RELU6;
  const float hi = act == ACT_RELU6 ? 6.f : __builtin_nanf("");
  return all || (v > 0.f && !(v >= hi));
}
// ---------------------------------------------------------------------------
// layout / cast:  x float32 NCHW  ->  A_0  T NHWC with Cp channels (pads = 0)
// ---------------------------------------------------------------------------
template <class T>
__global__ void cast_input_kernel(const float* __restrict__ x, T* __restrict__ out, int N, int C,
                                  int HW, int Cp) {
  const long nvec = (long)N * HW * (Cp / 8);
  const int ncv = Cp / 8;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nvec; i += (long)gridDim.x * blockDim.x) {
    const int cv = (int)(i % ncv);
    const long pix = i / ncv;
    const int n = (int)(pix / HW), hw = (int)(pix % HW);
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int c = cv * 8 + k;
      v[k] = c < C ? x[((long)n * C + c) * HW + hw] : 0.f;
    }
    IO<T>::st(out + i * 8, v);
  }
}

// ---------------------------------------------------------------------------
// Space-to-depth form of a 3-channel input for a 7 x 7 stride-2 stem (pad 3):
//   x float32 NCHW  ->  x2 T [N][H/2][W/2][16],  x2[n][i][j][(dy*2 + dx)*3 + c] = x[n][c][2i + dy][2j + dx], lanes 12..15 = 0.
// With the filter repacked the same way (pack_stem_weights_kernel) the stem is a 4 x 4 stride-1 convolution
// over 16 channels with two rows / columns of padding in front:
//   out[a][b] = sum_{r,s,c} W[r][s][c] x[2a-3+r][2b-3+s][c],  row 2a-3+r = 2 (a-2+br) + dy  <=>  r = 2 br + dy - 1,
// a reduction of 4*4*16 = 256 elements (147 of them real) instead of 7*7*8 = 392 with the channels padded to 8.
// ---------------------------------------------------------------------------
template <class T>
__global__ void s2d_input_kernel(const float* __restrict__ x, T* __restrict__ out, int N, int C, int H, int W) {
  const int H2 = H / 2, W2 = W / 2;
  const long npix = (long)N * H2 * W2;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < npix; i += (long)gridDim.x * blockDim.x) {
    const int j = (int)(i % W2);
    const long t = i / W2;
    const int ii = (int)(t % H2), n = (int)(t / H2);
    float v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = 0.f;
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
      for (int c = 0; c < C; ++c) {                  // (C <= 4)
        const float2 p = *reinterpret_cast<const float2*>(x + (((long)n * C + c) * H + 2 * ii + dy) * W + 2 * j);
        v[(dy * 2 + 0) * C + c] = p.x;
        v[(dy * 2 + 1) * C + c] = p.y;
      }
    IO<T>::st(out + i * 16, v);
    IO<T>::st(out + i * 16 + 8, v + 8);
  }
}
// w [K][7][7][8] (channel lanes >= C are zero) -> w2 [K][4][4][16] as above; one thread per element of w2
template <class T>
__global__ void pack_stem_weights_kernel(const T* __restrict__ w, T* __restrict__ w2, int K, int C) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= K * 256) return;
  const int lane = i & 15, bs = (i >> 4) & 3, br = (i >> 6) & 3, k = i >> 8;
  const int q = lane / C, c = lane % C;              // q = dy*2 + dx
  const int r = 2 * br + (q >> 1) - 1, s_ = 2 * bs + (q & 1) - 1;
  T v = T(0);
  if (lane < 4 * C && r >= 0 && s_ >= 0) v = w[((k * 7 + r) * 7 + s_) * 8 + c];
  w2[i] = v;
}
// the inverse on the weight gradient: dw2 float32 [K][4][4][16] -> dw float32 [K][7][7][8] (lanes >= C zero)
__global__ void unpack_stem_grad_kernel(const float* __restrict__ dw2, float* __restrict__ dw, int K, int C) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= K * 392) return;
  const int c = i & 7, t = i >> 3, s_ = t % 7, r = (t / 7) % 7, k = t / 49;
  float v = 0.f;
  if (c < C) {
    const int br = (r + 1) >> 1, dy = (r + 1) & 1, bs = (s_ + 1) >> 1, dx = (s_ + 1) & 1;
    v = dw2[((k * 4 + br) * 4 + bs) * 16 + (dy * 2 + dx) * C + c];
  }
  dw[i] = v;
}

// ---------------------------------------------------------------------------
// inference-mode BN folded to  y = a*x + b  (teacher; Sec. II-A: the teacher is
// pretrained and only evaluated)
// ---------------------------------------------------------------------------
__global__ void bn_fold_kernel(const float* gamma, const float* beta, const float* rmean,
                               const float* rvar, float* a, float* b, int C, float eps) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= C) return;
  const float s = gamma[c] / sqrtf(rvar[c] + eps);
  a[c] = s;
  b[c] = beta[c] - rmean[c] * s;
}

// ---------------------------------------------------------------------------
// per-channel column reductions over the M = N*H*W rows of an NHWC matrix.
// Block = 256 threads = cvl channel-vector lanes x (256/cvl) row lanes; grid =
// (column slabs, row chunks).  Each block writes one ordered partial.
// ---------------------------------------------------------------------------
struct ColGrid {
  int cvl;        // channel-vector lanes per block (<= 32); 256 / cvl row lanes, the rest of the block idles
  int slabs;      // ceil(ncv / cvl)
  int chunks;     // row chunks (gridDim.y)
  long rows_per_chunk;
  bool join64 = false;   // the row lanes' sums are added in double (block_col_reduce64)
};

// in-block reduction of NV floats per thread over the row lanes.  Threads are numbered
// row_lane * cvl + cv_lane (row lanes 0 .. 256/cvl - 1 take part).  The association is fixed in both
// forms, so the result never depends on scheduling.  smem: at least 256 * NV floats.
//  * cvl a power of two: the lanes of a wave that share a channel vector are cvl apart, so a butterfly
//    (lane ^ cvl, ^ 2 cvl, ... ^ 32) adds them without leaving the registers; the four waves' sums then
//    meet in LDS and are added as (w0 + w1) + (w2 + w3).
//  * any other cvl (channel counts such as 48, 96, 144): every thread leaves its sums in LDS as
//    [row_lane][cv_lane][NV]; thread o adds column o over the row lanes in order.
template <int NV>
__device__ __forceinline__ void block_col_reduce(float (&acc)[NV], float* smem, int cvl, int cv_lane,
                                                 int row_lane, float* out /*[NV]*/, bool& owner) {
  owner = row_lane == 0;
  if ((cvl & (cvl - 1)) == 0) {
    for (int off = cvl; off < 64; off <<= 1) {
#pragma unroll
      for (int k = 0; k < NV; ++k) acc[k] += __shfl_xor(acc[k], off, 64);
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane < cvl) {
      float* mine = smem + (wave * cvl + lane) * NV;
#pragma unroll
      for (int k = 0; k < NV; ++k) mine[k] = acc[k];
    }
    __syncthreads();
    if (owner) {   // wave 0, lane == cv_lane
      const float* w0 = smem + cv_lane * NV;
      const int ws = cvl * NV;
#pragma unroll
      for (int k = 0; k < NV; ++k) out[k] = (w0[k] + w0[ws + k]) + (w0[2 * ws + k] + w0[3 * ws + k]);
    }
    __syncthreads();
    return;
  }
  const int rl = 256 / cvl, nout = cvl * NV;
  if (row_lane < rl) {
    float* mine = smem + (row_lane * cvl + cv_lane) * NV;
#pragma unroll
    for (int k = 0; k < NV; ++k) mine[k] = acc[k];
  }
  __syncthreads();
  for (int o = threadIdx.x; o < nout; o += 256) {
    float sum = smem[o];
    for (int r = 1; r < rl; ++r) sum += smem[r * nout + o];
    smem[o] = sum;       // column o of row 0 is read by this thread only
  }
  __syncthreads();
  if (owner) {
#pragma unroll
    for (int k = 0; k < NV; ++k) out[k] = smem[cv_lane * NV + k];
  }
  __syncthreads();
}

// training-mode BN + activation:  z = act((y - mean) * (gamma*invstd) + beta).
// Column-grid launch: a thread keeps its 8 channels' coefficients in registers and streams rows.
// what a value reads back as after it was stored in T
template <class T> __device__ __forceinline__ float as_stored(float v);
template <> __device__ __forceinline__ float as_stored<float>(float v) { return v; }
template <> __device__ __forceinline__ float as_stored<bf16_t>(float v) { return bf_lo(pack_bf2(v, 0.f)); }

// res (optional): a residual add fused into the pass, z = res_act(stored(act(bn(y))) + res): the same
// numbers as storing the normalised tensor and adding in a second kernel, without that tensor
template <class T, bool STREAM>
__device__ __forceinline__ void bn_apply_rows(const T* __restrict__ y, T* __restrict__ z, const float (&mu)[8], const float (&a)[8], const float (&b)[8],
                                              int cv, int ncv, long r, long r1, int rl, int act, const T* __restrict__ res, int res_act) {
  for (; r + 3 * rl < r1; r += 4 * rl) {             // four rows (with a residual: eight loads) in flight
    typename IO<T>::Raw yr[4], sr[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) yr[u] = IO<T>::template ld_raw_t<STREAM>(y + ((r + u * rl) * ncv + cv) * 8);
    if (res) {
#pragma unroll
      for (int u = 0; u < 4; ++u) sr[u] = IO<T>::template ld_raw_t<STREAM>(res + ((r + u * rl) * ncv + cv) * 8);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float v[8];
      IO<T>::unpack(yr[u], v);
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = apply_act(fmaf(v[k] - mu[k], a[k], b[k]), act);
      if (res) {
        float s[8];
        IO<T>::unpack(sr[u], s);
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = apply_act(as_stored<T>(v[k]) + s[k], res_act);
      }
      IO<T>::template st_t<STREAM>(z + ((r + u * rl) * ncv + cv) * 8, v);
    }
  }
  for (; r < r1; r += rl) {
    float v[8];
    IO<T>::ld(y + (r * ncv + cv) * 8, v);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = apply_act(fmaf(v[k] - mu[k], a[k], b[k]), act);
    if (res) {
      float s[8];
      IO<T>::ld(res + (r * ncv + cv) * 8, s);
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = apply_act(as_stored<T>(v[k]) + s[k], res_act);
    }
    IO<T>::template st_t<STREAM>(z + (r * ncv + cv) * 8, v);
  }
}
template <class T, bool STREAM>
__device__ __forceinline__ void bn_apply_block(const Blk& blk, const T* __restrict__ y, T* __restrict__ z,
                                                       const float* __restrict__ mean,
                                                       const float* __restrict__ invstd,
                                                       const float* __restrict__ gamma,
                                                       const float* __restrict__ beta, long M, int Cp,
                                                       int act, ColGrid g, const T* __restrict__ res, int res_act) {
  const int ncv = Cp / 8;
  const int cv_lane = threadIdx.x % g.cvl, row_lane = threadIdx.x / g.cvl, rl = 256 / g.cvl;
  const int cv = blk.x * g.cvl + cv_lane;
  if (cv >= ncv || row_lane >= rl) return;
  const long r0 = blk.y * g.rows_per_chunk;
  const long r1 = min(M, r0 + g.rows_per_chunk);
  float mu[8], a[8], b[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int c = cv * 8 + k;
    mu[k] = mean[c]; a[k] = gamma[c] * invstd[c]; b[k] = beta[c];
  }
  bn_apply_rows<T, STREAM>(y, z, mu, a, b, cv, ncv, r0 + row_lane, r1, rl, act, res, res_act);
}
template <class T, bool STREAM = false>
__global__ __launch_bounds__(256) void bn_apply_kernel(const T* __restrict__ y,
    T* __restrict__ z, const float* __restrict__ mean, const float* __restrict__ invstd, const float* __restrict__ gamma,
    const float* __restrict__ beta, long M, int Cp, int act, ColGrid g, const T* __restrict__ res, int res_act) {
  bn_apply_block<T, STREAM>(one_block(), y, z, mean, invstd, gamma, beta, M, Cp, act, g, res, res_act);
}

// The same for at most 16 channel-vector lanes, the row lanes' sums added in double: a chunk of few, long row lanes (bn_apply_sums_kernel) then rounds
// once, where it is stored.  2-norm of a float32 mean's distance from 64 bits, in standard deviations, 8085 rows of 48 channels: 5.5e-9; lanes added in
// float 1.5e-8, the 256 shorter chunks of the separate passes 8.4e-9 (16384 of 64: 4.4, 5.3 and 4.4e-9); a weight gradient of the batch norm, 2185 rows
// of 72, relative: 1.8, 2.6 and 2.0e-8.  No slower (VGG-16 at batch 85 861 / 855 us a step).  256 / (cvl NV) threads share a column.
template <int NV>
__device__ __forceinline__ void block_col_reduce64(float (&acc)[NV], float* smem, int cvl, int cv_lane, int row_lane, float* out /*[NV]*/, bool& owner) {
  owner = row_lane == 0;
  const int t = threadIdx.x, rl = 256 / cvl, nout = cvl * NV, shares = 256 / nout, share = t / nout;
  if (row_lane < rl) {
    float* mine = smem + (row_lane * cvl + cv_lane) * NV;
#pragma unroll
    for (int k = 0; k < NV; ++k) mine[k] = acc[k];
  }
  __syncthreads();
  double sum = 0.0;
  if (share < shares)
    for (int r = share; r < rl; r += shares) sum += (double)smem[r * nout + t % nout];
  __syncthreads();
  double* joint = reinterpret_cast<double*>(smem);
  joint[t] = sum;
  __syncthreads();
  if (t < nout)
    for (int q = 1; q < shares; ++q) sum += joint[q * nout + t];
  __syncthreads();
  if (t < nout) smem[t] = (float)sum;
  __syncthreads();
  if (owner) {
#pragma unroll
    for (int k = 0; k < NV; ++k) out[k] = smem[cv_lane * NV + k];
  }
}

// part[chunk][0][c] = sum (y - piv), part[chunk][1][c] = sum (y - piv)^2 with the pivot
// piv[c] = y[row 0][c]: shifting by a sample of the channel keeps the variance free of the
// cancellation that  E[y^2] - mean^2  suffers when |mean| >> std
template <class T, bool STREAM>
__device__ __forceinline__ void bn_stats_block(const Blk& blk, const T* __restrict__ y, float* __restrict__ part,
                                                       long M, int Cp, ColGrid g) {
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int ncv = Cp / 8;
  const int cv_lane = threadIdx.x % g.cvl, row_lane = threadIdx.x / g.cvl, rl = 256 / g.cvl;
  const int cv = blk.x * g.cvl + cv_lane;
  const long r0 = blk.y * g.rows_per_chunk;
  const long r1 = min(M, r0 + g.rows_per_chunk);
  float acc[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) acc[k] = 0.f;
  if (cv < ncv && row_lane < rl) {
    float piv[8];
    IO<T>::ld(y + (long)cv * 8, piv);
    long r = r0 + row_lane;
    for (; r + 3 * rl < r1; r += 4 * rl) {           // four rows in flight
      typename IO<T>::Raw yr[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) yr[u] = IO<T>::template ld_raw_t<STREAM>(y + ((r + u * rl) * ncv + cv) * 8);
      __builtin_amdgcn_sched_barrier(0);
      float v[4][8];
#pragma unroll
      for (int u = 0; u < 4; ++u) IO<T>::unpack(yr[u], v[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float d = v[u][k] - piv[k];
          acc[k] += d;
          acc[8 + k] = fmaf(d, d, acc[8 + k]);
        }
    }
    for (; r < r1; r += rl) {
      float v[8];
      IO<T>::ld(y + (r * ncv + cv) * 8, v);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float d = v[k] - piv[k];
        acc[k] += d;
        acc[8 + k] = fmaf(d, d, acc[8 + k]);
      }
    }
  }
  float out[16];
  bool owner;
  if (g.join64) block_col_reduce64<16>(acc, smem, g.cvl, cv_lane, row_lane, out, owner);
  else block_col_reduce<16>(acc, smem, g.cvl, cv_lane, row_lane, out, owner);
  if (owner && cv < ncv) {
    float* p = part + (long)blk.y * 2 * Cp + cv * 8;
#pragma unroll
    for (int k = 0; k < 8; ++k) { p[k] = out[k]; p[Cp + k] = out[8 + k]; }
  }
}
template <class T, bool STREAM = false>
__global__ __launch_bounds__(256) void bn_stats_kernel(const T* __restrict__ y,
    float* __restrict__ part, long M, int Cp, ColGrid g) {
  bn_stats_block<T, STREAM>(one_block(), y, part, M, Cp, g);
}

// Finalize kernels run 8 channels x 32 lanes per block (thread = lane * 8 + channel): lane l adds
// chunks l, l+32, ... in order, the 8 lanes of a channel inside one wave are added by a butterfly and
// the 4 waves in a fixed order (fixed association, independent of scheduling).  Few chunks per lane, eight of them requested at a time,
// keep the chain of dependent loads short: these kernels sit between two passes over the tensor.
// GROUPS: the chunks hold a mean, a sum of squares about it and a number of rows each (part[chunk][3][Cp]) instead of two
// sums; s1 and s2 come out as the sums of y and y^2, in double.
constexpr int kFinalizeChannels = 8;
template <bool GROUPS = false>
__device__ __forceinline__ void finalize_sums(const float* __restrict__ part, int chunks, int Cp, int c,
                                              int lane, double& s1, double& s2) {
  __shared__ double red1[4][kFinalizeChannels], red2[4][kFinalizeChannels];
  const int cl = threadIdx.x & (kFinalizeChannels - 1);
  double a = 0.0, b = 0.0;
  if (c < Cp) {
    // (a batch of loads in flight before the first addition; past the last chunk: the last one, not added)
    constexpr int U = 8, W = GROUPS ? 3 : 2;
    for (int k0 = lane; k0 < chunks; k0 += 32 * U) {
      float v[U][W];
#pragma unroll
      for (int i = 0; i < U; ++i) {
        const float* p = part + (long)min(k0 + 32 * i, chunks - 1) * W * Cp + c;
#pragma unroll
        for (int w = 0; w < W; ++w) v[i][w] = p[(long)w * Cp];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < U; ++i) {
        const bool in = k0 + 32 * i < chunks;
        if (GROUPS) {
          const double mu = (double)v[i][0], n = (double)v[i][W - 1];
          const double a1 = n * mu, b1 = (double)v[i][1] + n * mu * mu;
          a += in ? a1 : 0.0;
          b += in ? b1 : 0.0;
        } else {
          a += in ? (double)v[i][0] : 0.0;
          b += in ? (double)v[i][1] : 0.0;
        }
      }
    }
  }
#pragma unroll
  for (int off = kFinalizeChannels; off < 64; off <<= 1) {
    a += __shfl_xor(a, off, 64);
    b += __shfl_xor(b, off, 64);
  }
  if ((threadIdx.x & 63) < kFinalizeChannels) {
    red1[threadIdx.x >> 6][cl] = a;
    red2[threadIdx.x >> 6][cl] = b;
  }
  __syncthreads();
  s1 = (red1[0][cl] + red1[1][cl]) + (red1[2][cl] + red1[3][cl]);
  s2 = (red2[0][cl] + red2[1][cl]) + (red2[2][cl] + red2[3][cl]);
}

// mean, biased variance -> inv std; running statistics
//   rm <- (1-rho) rm + rho mean,  rv <- (1-rho) rv + rho var m/(m-1)
// keep (optional): [2][Cp] copies of gamma and beta as the step's normalisation uses them (the update overwrites both),
// for a normalised tensor that is not written and may be asked for later
template <class T, bool GROUPS>
__device__ __forceinline__ void bn_finalize_block(const Blk& blk, const float* __restrict__ part, const T* __restrict__ y, int chunks,
                                   int Cp, double m, float* mean, float* invstd, float* rmean,
                                   float* rvar, float eps, float rho, const float* gamma, const float* beta, float* keep) {
  const int c = blk.x * kFinalizeChannels + (threadIdx.x & (kFinalizeChannels - 1)), lane = threadIdx.x >> 3;
  double s1, s2;
  const int cl = min(c, Cp - 1);                     // (what the end needs besides the sums, requested ahead of them)
  const float pivot = y ? (float)y[cl] : 0.f, ga = gamma[cl], be = beta[cl], rm = rmean[cl], rv = rvar[cl];   // y: the row the sums were shifted by, if any
  finalize_sums<GROUPS>(part, chunks, Cp, c, lane, s1, s2);
  if (c >= Cp || lane != 0) return;
  const double shift = s1 / m;
  const double mu = (double)pivot + shift;
  double var = s2 / m - shift * shift;
  if (var < 0.0) var = 0.0;
  if (keep) { keep[c] = ga; keep[Cp + c] = be; }
  mean[c] = (float)mu;
  invstd[c] = (float)(1.0 / sqrt(var + (double)eps));
  rmean[c] = (1.f - rho) * rm + rho * (float)mu;
  rvar[c] = (1.f - rho) * rv + rho * (float)(var * m / (m - 1.0));
}
template <class T, bool GROUPS = false>
__global__ void bn_finalize_kernel(const float* __restrict__ part, const T* __restrict__ y,
    int chunks, int Cp, double m, float* mean, float* invstd, float* rmean, float* rvar, float eps, float rho, const float* gamma,
    const float* beta, float* keep) {
  bn_finalize_block<T, GROUPS>(one_block(), part, y, chunks, Cp, m, mean, invstd, rmean, rvar, eps, rho, gamma, beta, keep);
}

// out[g][i] = sum of part[k][i] over the `per` chunks of group g, in order: shortens the list of partial
// sums that a finalize kernel walks through when a convolution's row tiles delivered thousands of them
constexpr int kStatGroupsMax = 1024;   // partial sums a batch-norm finalize walks through at most
__device__ __forceinline__ void regroup_partials_block(const Blk& blk, const float* __restrict__ part, float* __restrict__ out, int chunks, int n, int per) {
  const int i = blk.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int k0 = blk.y * per, k1 = min(chunks, k0 + per);
  float s = 0.f;
  for (int k = k0; k < k1; ++k) s += part[(long)k * n + i];
  out[(long)blk.y * n + i] = s;
}
__global__ void regroup_partials_kernel(const float* __restrict__ part, float* __restrict__ out, int chunks, int n, int per) {
  regroup_partials_block(one_block(), part, out, chunks, n, per);
}

// The elementwise passes of small tensors add the partial sums themselves: no finalize launch between the reduction and them, and instead of the
// whole-column kernels where a column is long.  A workgroup has at most 64 channels (whole 128-byte lines of bf16) and adds their sums,
// kSumChunksMax partial sums at most, in double: thread = (lane, channel), lane l adds chunks l, l + lanes, ... and the lanes are added in order.
// All workgroups of a slab come to the same numbers; those of the first row chunk store them.
// What bounds them is the launch: 8 MB tensors stream in ~2 us, the sums of 64 chunks are two rounds of loads from the caches.
constexpr int kSumChunksMax = 128, kSumChannels = 64;
struct SlabSums { double part[2][256]; float co[2][kSumChannels]; };
__device__ __forceinline__ void slab_sums(SlabSums& s, const float* __restrict__ part, int chunks, int Cp, int c0, int n, double& s1, double& s2) {
  const int ch = threadIdx.x % n, lane = threadIdx.x / n, lanes = 256 / n;
  double a = 0.0, b = 0.0;
  if (c0 + ch < Cp && lane < lanes) {
    const float* p = part + c0 + ch;
    for (int k = lane; k < chunks; k += 8 * lanes) {
      float u[8], v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {                  // (past the last chunk: the last one, not added)
        const long at = (long)min(k + i * lanes, chunks - 1) * 2 * Cp;
        u[i] = p[at]; v[i] = p[at + Cp];
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const bool in = k + i * lanes < chunks;
        a += in ? (double)u[i] : 0.0;
        b += in ? (double)v[i] : 0.0;
      }
    }
  }
  s.part[0][threadIdx.x] = a;
  s.part[1][threadIdx.x] = b;
  __syncthreads();
  s1 = s2 = 0.0;
  if ((int)threadIdx.x < n)
    for (int l = 0; l < lanes; ++l) { s1 += s.part[0][l * n + threadIdx.x]; s2 += s.part[1][l * n + threadIdx.x]; }
}
// bn_finalize_kernel and bn_apply_kernel (pivot: the row that the sums were shifted by, if any)
template <class T>
__device__ __forceinline__ void bn_apply_sums_block(const Blk& blk, const T* __restrict__ y, T* __restrict__ z, const float* __restrict__ part,
    const T* __restrict__ pivot, int chunks, double m, float* mean, float* invstd, float* rmean, float* rvar, float eps, float rho,
    const float* __restrict__ gamma, const float* __restrict__ beta, long M, int Cp, int act, ColGrid g, const T* __restrict__ res, int res_act) {
  __shared__ SlabSums sh;
  const int n = g.cvl * 8, c0 = blk.x * n, t = threadIdx.x;
  double s1, s2;
  slab_sums(sh, part, chunks, Cp, c0, n, s1, s2);
  if (t < n && c0 + t < Cp) {
    const int c = c0 + t;
    const double shift = s1 / m, mu = (pivot ? (double)(float)pivot[c] : 0.0) + shift;
    double var = s2 / m - shift * shift;
    if (var < 0.0) var = 0.0;
    const float is = (float)(1.0 / sqrt(var + (double)eps));
    sh.co[0][t] = (float)mu;
    sh.co[1][t] = is;
    if (blk.y == 0) {
      mean[c] = (float)mu;
      invstd[c] = is;
      rmean[c] = (1.f - rho) * rmean[c] + rho * (float)mu;
      rvar[c] = (1.f - rho) * rvar[c] + rho * (float)(var * m / (m - 1.0));
    }
  }
  __syncthreads();
  const int ncv = Cp / 8, cv_lane = t % g.cvl, row_lane = t / g.cvl, rl = 256 / g.cvl, cv = blk.x * g.cvl + cv_lane;
  if (cv >= ncv || row_lane >= rl) return;
  const long r0 = blk.y * g.rows_per_chunk;
  float mu[8], a[8], b[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int c = cv * 8 + k;
    mu[k] = sh.co[0][cv_lane * 8 + k]; a[k] = gamma[c] * sh.co[1][cv_lane * 8 + k]; b[k] = beta[c];
  }
  bn_apply_rows<T, false>(y, z, mu, a, b, cv, ncv, r0 + row_lane, min(M, r0 + g.rows_per_chunk), rl, act, res, res_act);
}
template <class T>
__global__ __launch_bounds__(256) void bn_apply_sums_kernel(const T* __restrict__ y, T* __restrict__ z, const float* __restrict__ part,
    const T* __restrict__ pivot, int chunks, double m, float* mean, float* invstd, float* rmean, float* rvar, float eps, float rho,
    const float* __restrict__ gamma, const float* __restrict__ beta, long M, int Cp, int act, ColGrid g, const T* __restrict__ res, int res_act) {
  bn_apply_sums_block<T>(one_block(), y, z, part, pivot, chunks, m, mean, invstd, rmean, rvar, eps, rho, gamma, beta, M, Cp, act, g, res, res_act);
}

// BN backward, stage 1: with xhat = (y - mean)*invstd, pre = gamma*xhat + beta and
// dpre = [act passes at pre] * dz:  part[chunk][0][c] = sum dpre, part[chunk][1][c] = sum dpre*xhat
// RES: the layer's output went straight into a two-input add (fused into its normalisation pass on the way
// forward).  dz is then the gradient of the add's output and zres that output: the gradient passes where the
// add's activation res_act does (zres == nullptr: no activation), is stored to dstore (the gradient of both
// inputs of the add: the backward pass of the add itself, done here) and enters the sums.
// LOSS (with RES and zres): the add's output is the block's output S.  dz is then the teacher's activation A,
// the gradient of the add's output is 2 (S - A) / M rounded as it would be stored (Sec. II-A, the loss of the
// block's output), and loss_part[workgroup] = sum (S - A)^2 over the workgroup's elements (rows and threads joined in double where the grid
// says so for the column sums: bfloat16 losses of 15376 x 40, relative, 2-norm, 2.5e-8 from 64 bits, in float 4.5e-8).
template <class T, bool RES, bool LOSS, bool STREAM>
__device__ __forceinline__ void bn_bwd_reduce_block(const Blk& blk, const T* __restrict__ dz, const T* __restrict__ y, const float* __restrict__ gamma,
    const float* __restrict__ beta, const float* __restrict__ mean, const float* __restrict__ invstd,
    float* __restrict__ part, long M, int Cp, int act, ColGrid g, const T* __restrict__ zres,
    int res_act, T* __restrict__ dstore, float* __restrict__ loss_part,
    float two_over_m) {
  static_assert(RES || !LOSS, "the loss rides only where the add does");
  float lacc = 0.f;
  double lsum = 0.0;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int ncv = Cp / 8;
  const int cv_lane = threadIdx.x % g.cvl, row_lane = threadIdx.x / g.cvl, rl = 256 / g.cvl;
  const int cv = blk.x * g.cvl + cv_lane;
  const long r0 = blk.y * g.rows_per_chunk;
  const long r1 = min(M, r0 + g.rows_per_chunk);
  float acc[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) acc[k] = 0.f;
  if (cv < ncv && row_lane < rl) {
    float av[8], bv[8], mv[8], iv[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      av[k] = gamma[cv * 8 + k]; bv[k] = beta[cv * 8 + k]; mv[k] = mean[cv * 8 + k]; iv[k] = invstd[cv * 8 + k];
    }
    float sc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) sc[k] = av[k] * iv[k];
    long r = r0 + row_lane;
    for (; r + 3 * rl < r1; r += 4 * rl) {           // four rows (eight loads, twelve with an add's output) in flight
      typename IO<T>::Raw dr[4], yr[4], zr[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        dr[u] = IO<T>::template ld_raw_t<STREAM>(dz + ((r + u * rl) * ncv + cv) * 8);
        yr[u] = IO<T>::template ld_raw_t<STREAM>(y + ((r + u * rl) * ncv + cv) * 8);
      }
      if (RES && zres) {
#pragma unroll
        for (int u = 0; u < 4; ++u) zr[u] = IO<T>::template ld_raw_t<STREAM>(zres + ((r + u * rl) * ncv + cv) * 8);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        float d[8], v[8];
        IO<T>::unpack(dr[u], d);
        IO<T>::unpack(yr[u], v);
        if (RES) {
          if (zres) {
            float z[8];
            IO<T>::unpack(zr[u], z);
            if (LOSS) {
#pragma unroll
              for (int k = 0; k < 8; ++k) {
                const float e = z[k] - d[k];
                lacc = fmaf(e, e, lacc);
                d[k] = as_stored<T>(e * two_over_m);
              }
              if (g.join64) { lsum += (double)lacc; lacc = 0.f; }
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) d[k] = act_pass(z[k], res_act) ? d[k] : 0.f;
          }
          IO<T>::template st_t<STREAM>(dstore + ((r + u * rl) * ncv + cv) * 8, d);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float yc = v[k] - mv[k];
          const float dp = act_pass(fmaf(yc, sc[k], bv[k]), act) ? d[k] : 0.f;
          acc[k] += dp;
          acc[8 + k] = fmaf(dp, yc * iv[k], acc[8 + k]);
        }
      }
    }
    for (; r < r1; r += rl) {
      float d[8], v[8];
      IO<T>::ld(dz + (r * ncv + cv) * 8, d);
      IO<T>::ld(y + (r * ncv + cv) * 8, v);
      if (RES) {
        if (zres) {
          float z[8];
          IO<T>::ld(zres + (r * ncv + cv) * 8, z);
          if (LOSS) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              const float e = z[k] - d[k];
              lacc = fmaf(e, e, lacc);
              d[k] = as_stored<T>(e * two_over_m);
            }
            if (g.join64) { lsum += (double)lacc; lacc = 0.f; }
          }
#pragma unroll
          for (int k = 0; k < 8; ++k) d[k] = act_pass(z[k], res_act) ? d[k] : 0.f;
        }
        IO<T>::template st_t<STREAM>(dstore + (r * ncv + cv) * 8, d);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float yc = v[k] - mv[k];
        const float dp = act_pass(fmaf(yc, sc[k], bv[k]), act) ? d[k] : 0.f;
        acc[k] += dp;
        acc[8 + k] = fmaf(dp, yc * iv[k], acc[8 + k]);
      }
    }
  }
  float out[16];
  bool owner;
  if (g.join64) block_col_reduce64<16>(acc, smem, g.cvl, cv_lane, row_lane, out, owner);
  else block_col_reduce<16>(acc, smem, g.cvl, cv_lane, row_lane, out, owner);
  if (owner && cv < ncv) {
    float* p = part + (long)blk.y * 2 * Cp + cv * 8;
#pragma unroll
    for (int k = 0; k < 8; ++k) { p[k] = out[k]; p[Cp + k] = out[8 + k]; }
  }
  if (LOSS) {                                        // the workgroup's share of sum (S - A)^2, added in a fixed order
    __syncthreads();
    auto join = [&](auto* sums, auto mine) {
      sums[threadIdx.x] = mine;
      __syncthreads();
      for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) sums[threadIdx.x] += sums[threadIdx.x + h];
        __syncthreads();
      }
      if (threadIdx.x == 0) loss_part[blk.y * blk.gx + blk.x] = (float)sums[0];
    };
    if (g.join64) join(reinterpret_cast<double*>(smem), lsum);
    else join(smem, lacc);
  }
}
template <class T, bool RES = false, bool LOSS = false, bool STREAM = false>
__global__ __launch_bounds__(256) void bn_bwd_reduce_kernel(
    const T* __restrict__ dz, const T* __restrict__ y, const float* __restrict__ gamma, const float* __restrict__ beta,
    const float* __restrict__ mean, const float* __restrict__ invstd, float* __restrict__ part, long M, int Cp, int act, ColGrid g,
    const T* __restrict__ zres = nullptr, int res_act = 0, T* __restrict__ dstore = nullptr, float* __restrict__ loss_part = nullptr,
    float two_over_m = 0.f) {
  bn_bwd_reduce_block<T, RES, LOSS, STREAM>(one_block(), dz, y, gamma, beta, mean, invstd, part, M, Cp, act, g, zres, res_act, dstore, loss_part, two_over_m);
}

// stage 2: dbeta, dgamma (the parameter gradients) and the per-channel terms
// k2 = dbeta/m, k3 = dgamma/m of  dy = gamma*invstd*(dpre - k2 - xhat*k3)
__device__ __forceinline__ void bn_bwd_finalize_block(const Blk& blk, const float* __restrict__ part, int chunks, int Cp, double m,
                                       float* g_gamma, float* g_beta, float* k2, float* k3) {
  const int c = blk.x * kFinalizeChannels + (threadIdx.x & (kFinalizeChannels - 1)), lane = threadIdx.x >> 3;
  double sb, sg;
  finalize_sums(part, chunks, Cp, c, lane, sb, sg);
  if (c >= Cp || lane != 0) return;
  g_beta[c] = (float)sb;
  g_gamma[c] = (float)sg;
  k2[c] = (float)(sb / m);
  k3[c] = (float)(sg / m);
}
__global__ void bn_bwd_finalize_kernel(const float* __restrict__ part, int chunks, int Cp, double m, float* g_gamma, float* g_beta,
    float* k2, float* k3) {
  bn_bwd_finalize_block(one_block(), part, chunks, Cp, m, g_gamma, g_beta, k2, k3);
}

// stage 3: gradient w.r.t. the convolution output, written to dy (dy == dz: in place; column-grid launch, each
// thread reads its elements before it writes them)
struct BnBwdCoef { float mu[8], a[8], b[8], is[8], c2[8], c3[8]; };
template <class T, bool STREAM>
__device__ __forceinline__ void bn_bwd_apply_rows(const T* dz, T* dy, const T* __restrict__ y, const BnBwdCoef& f, int cv, int ncv, long r, long r1, int rl, int act) {
  const auto &mu = f.mu, &a = f.a, &b = f.b, &is = f.is, &c2 = f.c2, &c3 = f.c3;
  for (; r + 3 * rl < r1; r += 4 * rl) {             // four rows (eight loads) in flight
    typename IO<T>::Raw dr[4], yr[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      dr[u] = IO<T>::template ld_raw_t<STREAM>(dz + ((r + u * rl) * ncv + cv) * 8);
      yr[u] = IO<T>::template ld_raw_t<STREAM>(y + ((r + u * rl) * ncv + cv) * 8);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float d[8], v[8];
      IO<T>::unpack(dr[u], d);
      IO<T>::unpack(yr[u], v);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float yc = v[k] - mu[k];
        const float dp = act_pass(fmaf(yc, a[k], b[k]), act) ? d[k] : 0.f;
        d[k] = a[k] * (dp - c2[k] - yc * is[k] * c3[k]);
      }
      IO<T>::template st_t<STREAM>(dy + ((r + u * rl) * ncv + cv) * 8, d);
    }
  }
  for (; r < r1; r += rl) {
    float d[8], v[8];
    IO<T>::ld(dz + (r * ncv + cv) * 8, d);
    IO<T>::ld(y + (r * ncv + cv) * 8, v);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float yc = v[k] - mu[k];
      const float dp = act_pass(fmaf(yc, a[k], b[k]), act) ? d[k] : 0.f;
      d[k] = a[k] * (dp - c2[k] - yc * is[k] * c3[k]);
    }
    IO<T>::template st_t<STREAM>(dy + (r * ncv + cv) * 8, d);
  }
}
template <class T, bool STREAM>
__device__ __forceinline__ void bn_bwd_apply_block(const Blk& blk, const T* dz, T* dy, const T* __restrict__ y, const float* __restrict__ gamma,
    const float* __restrict__ beta, const float* __restrict__ mean, const float* __restrict__ invstd,
    const float* __restrict__ k2, const float* __restrict__ k3, long M, int Cp, int act, ColGrid g) {
  const int ncv = Cp / 8;
  const int cv_lane = threadIdx.x % g.cvl, row_lane = threadIdx.x / g.cvl, rl = 256 / g.cvl;
  const int cv = blk.x * g.cvl + cv_lane;
  if (cv >= ncv || row_lane >= rl) return;
  const long r0 = blk.y * g.rows_per_chunk;
  const long r1 = min(M, r0 + g.rows_per_chunk);
  BnBwdCoef f;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int c = cv * 8 + k;
    f.mu[k] = mean[c]; f.is[k] = invstd[c]; f.a[k] = gamma[c] * f.is[k]; f.b[k] = beta[c];
    f.c2[k] = k2[c]; f.c3[k] = k3[c];
  }
  bn_bwd_apply_rows<T, STREAM>(dz, dy, y, f, cv, ncv, r0 + row_lane, r1, rl, act);
}
// bn_bwd_finalize_kernel and bn_bwd_apply_kernel
template <class T>
__device__ __forceinline__ void bn_bwd_apply_sums_block(const Blk& blk, const T* dz, T* dy, const T* __restrict__ y, const float* __restrict__ part, int chunks,
    double m, float* g_gamma, float* g_beta, const float* __restrict__ gamma, const float* __restrict__ beta, const float* __restrict__ mean,
    const float* __restrict__ invstd, float* k2, float* k3, long M, int Cp, int act, ColGrid g) {
  __shared__ SlabSums sh;
  const int n = g.cvl * 8, c0 = blk.x * n, t = threadIdx.x;
  double sb, sg;
  slab_sums(sh, part, chunks, Cp, c0, n, sb, sg);
  if (t < n && c0 + t < Cp) {
    const int c = c0 + t;
    const float v2 = (float)(sb / m), v3 = (float)(sg / m);
    sh.co[0][t] = v2;
    sh.co[1][t] = v3;
    if (blk.y == 0) {
      g_beta[c] = (float)sb;
      g_gamma[c] = (float)sg;
      k2[c] = v2;
      k3[c] = v3;
    }
  }
  __syncthreads();
  const int ncv = Cp / 8, cv_lane = t % g.cvl, row_lane = t / g.cvl, rl = 256 / g.cvl, cv = blk.x * g.cvl + cv_lane;
  if (cv >= ncv || row_lane >= rl) return;
  const long r0 = blk.y * g.rows_per_chunk;
  BnBwdCoef f;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int c = cv * 8 + k;
    f.mu[k] = mean[c]; f.is[k] = invstd[c]; f.a[k] = gamma[c] * f.is[k]; f.b[k] = beta[c];
    f.c2[k] = sh.co[0][cv_lane * 8 + k]; f.c3[k] = sh.co[1][cv_lane * 8 + k];
  }
  bn_bwd_apply_rows<T, false>(dz, dy, y, f, cv, ncv, r0 + row_lane, min(M, r0 + g.rows_per_chunk), rl, act);
}
template <class T>
__global__ __launch_bounds__(256) void bn_bwd_apply_sums_kernel(const T* dz, T* dy, const T* __restrict__ y, const float* __restrict__ part, int chunks,
    double m, float* g_gamma, float* g_beta, const float* __restrict__ gamma, const float* __restrict__ beta, const float* __restrict__ mean,
    const float* __restrict__ invstd, float* k2, float* k3, long M, int Cp, int act, ColGrid g) {
  bn_bwd_apply_sums_block<T>(one_block(), dz, dy, y, part, chunks, m, g_gamma, g_beta, gamma, beta, mean, invstd, k2, k3, M, Cp, act, g);
}
template <class T, bool STREAM = false>
__global__ __launch_bounds__(256) void bn_bwd_apply_kernel(const T* dz, T* dy,
    const T* __restrict__ y, const float* __restrict__ gamma, const float* __restrict__ beta, const float* __restrict__ mean,
    const float* __restrict__ invstd, const float* __restrict__ k2, const float* __restrict__ k3, long M, int Cp, int act, ColGrid g) {
  bn_bwd_apply_block<T, STREAM>(one_block(), dz, dy, y, gamma, beta, mean, invstd, k2, k3, M, Cp, act, g);
}

// ---------------------------------------------------------------------------
// Whole-column kernels for short matrices (M <= 4096 rows).  One block of 512 threads owns an
// 8-channel slab over ALL rows and keeps its (at most 8) rows per thread in registers, so
// statistics, their finalisation and the elementwise pass are one launch and one read instead of
// three launches and two reads: at these sizes the launches, not the bytes, are the cost.
// ---------------------------------------------------------------------------
constexpr int kSmallThreads = 512;                   // 8 waves: up to 256 registers per thread
constexpr int kSmallRows = 8;                        // rows per thread

// consecutive slabs go to the same XCD (blocks are dealt round-robin over 8 XCDs), so each cache
// line of a row is pulled into one L2 only
__device__ __forceinline__ int xcd_slab(int b, int nslab) {
  return (nslab & 7) == 0 ? (b & 7) * (nslab >> 3) + (b >> 3) : b;
}

// Sum of 16 per-thread values over the block, result in every thread.  In the wave: a
// reduce-scatter butterfly (exchange half of the values with lane^32, a quarter with lane^16, ...:
// 17 cross-lane moves instead of 96), float.  Across the waves: added in order, in double (BN
// backward subtracts these means from the gradient and what is left feeds weight gradients whose
// own sum cancels, so the totals want more than float).  A fixed association throughout.
__device__ __forceinline__ void block_sum16(const float (&v)[16], double (&out)[16], float (*red)[16], double* tot) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float w8[8], w4[4], w2[2], w1;
  const bool h32 = lane & 32, h16 = lane & 16, h8 = lane & 8, h4 = lane & 4;
#pragma unroll
  for (int i = 0; i < 8; ++i) w8[i] = (h32 ? v[8 + i] : v[i]) + __shfl_xor(h32 ? v[i] : v[8 + i], 32, 64);
#pragma unroll
  for (int i = 0; i < 4; ++i) w4[i] = (h16 ? w8[4 + i] : w8[i]) + __shfl_xor(h16 ? w8[i] : w8[4 + i], 16, 64);
#pragma unroll
  for (int i = 0; i < 2; ++i) w2[i] = (h8 ? w4[2 + i] : w4[i]) + __shfl_xor(h8 ? w4[i] : w4[2 + i], 8, 64);
  w1 = (h4 ? w2[1] : w2[0]) + __shfl_xor(h4 ? w2[0] : w2[1], 4, 64);
  w1 += __shfl_xor(w1, 2, 64);
  w1 += __shfl_xor(w1, 1, 64);
  if ((lane & 3) == 0) red[wave][(h32 ? 8 : 0) + (h16 ? 4 : 0) + (h8 ? 2 : 0) + (h4 ? 1 : 0)] = w1;
  __syncthreads();
  if (threadIdx.x < 16) {
    double t = (double)red[0][threadIdx.x];
#pragma unroll 1
    for (int w = 1; w < kSmallThreads / 64; ++w) t += (double)red[w][threadIdx.x];
    tot[threadIdx.x] = t;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) out[k] = tot[k];
}

struct SmallLds {
  float red[kSmallThreads / 64][16];
  double tot[16];
  float coef[3][8];
};
struct ColFwd { const float *gamma, *beta; float *mean, *invstd, *rmean, *rvar; int act; };
struct ColBwd { const float *gamma, *beta, *mean, *invstd; float *g_gamma, *g_beta; int act; };
struct SmallTerms { float mu[8], a[8], b[8]; };

// Batch statistics of a thread's rows (pivot-shifted sums as in bn_stats_kernel), running statistics, and the terms of
// z = act((y - mean) * (gamma*invstd) + beta)
template <class T, int N>
__device__ __forceinline__ void small_stats(const typename BufIO<T>::Raw (&raw)[N], const float (&piv)[8], const ColFwd& bn, SmallTerms& t,
                                            SmallLds& lds, int cv, int M, float eps, float rho) {
  const int tid = threadIdx.x;
  float acc[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) acc[k] = 0.f;
#pragma unroll
  for (int u = 0; u < N; ++u) {
    if (u * kSmallThreads + (tid & ~63) >= M) continue;     // no lane of this wave owns the row
    const bool ok = u * kSmallThreads + tid < M;
    float v[8];
    BufIO<T>::unpack(raw[u], v);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float d = ok ? v[k] - piv[k] : 0.f;
      acc[k] += d;
      acc[8 + k] = fmaf(d, d, acc[8 + k]);
    }
  }
  double sum[16];
  block_sum16(acc, sum, lds.red, lds.tot);
  // thread k < 8 finalises channel k in double (once, not in every thread) and hands the float
  // coefficients to the block through LDS
  if (tid < 8) {
    const int c = cv * 8 + tid;
    const double m = (double)M;
    double s1 = 0.0, s2 = 0.0;
    float pv = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (k == tid) { s1 = sum[k]; s2 = sum[8 + k]; pv = piv[k]; }
    const double shift = s1 / m;
    const double mean_d = (double)pv + shift;
    double var = s2 / m - shift * shift;
    if (var < 0.0) var = 0.0;
    const float is = (float)(1.0 / sqrt(var + (double)eps));
    const float muf = (float)mean_d;
    bn.mean[c] = muf;
    bn.invstd[c] = is;
    bn.rmean[c] = (1.f - rho) * bn.rmean[c] + rho * muf;
    bn.rvar[c] = (1.f - rho) * bn.rvar[c] + rho * (float)(var * m / (m - 1.0));
    lds.coef[0][tid] = muf; lds.coef[1][tid] = bn.gamma[c] * is; lds.coef[2][tid] = bn.beta[c];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 8; ++k) { t.mu[k] = lds.coef[0][k]; t.a[k] = lds.coef[1][k]; t.b[k] = lds.coef[2][k]; }
}

template <class T>
__device__ __forceinline__ void bn_small_fwd_block(const Blk& blk, const T* __restrict__ y, T* __restrict__ z, const float* __restrict__ gamma, const float* __restrict__ beta,
    float* __restrict__ mean, float* __restrict__ invstd, float* __restrict__ rmean, float* __restrict__ rvar,
    int M, int Cp, float eps, float rho, int act, unsigned bytes) {
  __shared__ SmallLds lds;
  const int ncv = Cp / 8, cv = xcd_slab(blk.x, ncv), tid = threadIdx.x;
  const __amdgpu_buffer_rsrc_t ry = tensor_rsrc(y, bytes);
  typename BufIO<T>::Raw raw[kSmallRows];
#pragma unroll
  for (int u = 0; u < kSmallRows; ++u) {
    const int r = u * kSmallThreads + tid;
    raw[u] = BufIO<T>::issue(ry, (unsigned)(r * ncv + cv) * 8u, r < M);
  }
  float piv[8];
  IO<T>::ld(y + (long)cv * 8, piv);
  SmallTerms t;
  small_stats<T>(raw, piv, ColFwd{gamma, beta, mean, invstd, rmean, rvar, act}, t, lds, cv, M, eps, rho);
#pragma unroll
  for (int u = 0; u < kSmallRows; ++u) {
    const int r = u * kSmallThreads + tid;
    if (r >= M) continue;
    float v[8];
    BufIO<T>::unpack(raw[u], v);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = apply_act(fmaf(v[k] - t.mu[k], t.a[k], t.b[k]), act);
    IO<T>::st(z + ((long)r * ncv + cv) * 8, v);
  }
}
template <class T>
__global__ __launch_bounds__(kSmallThreads) void bn_small_fwd_kernel(const T* __restrict__ y, T* __restrict__ z,
    const float* __restrict__ gamma, const float* __restrict__ beta, float* __restrict__ mean, float* __restrict__ invstd,
    float* __restrict__ rmean, float* __restrict__ rvar, int M, int Cp, float eps, float rho, int act, unsigned bytes) {
  bn_small_fwd_block<T>(one_block(), y, z, gamma, beta, mean, invstd, rmean, rvar, M, Cp, eps, rho, act, bytes);
}

// BN backward of a thread's rows: sums of dpre and dpre*xhat, the parameter gradients, then
// dy = gamma*invstd*(dpre - dbeta/m - xhat*dgamma/m), handed out row by row (rows past M: dz = 0, they add nothing)
template <class T, int N, class F>
__device__ __forceinline__ void small_bwd(const typename BufIO<T>::Raw (&rawd)[N], const typename BufIO<T>::Raw (&rawy)[N], const ColBwd& bn,
                                          SmallLds& lds, int cv, int M, F&& out) {
  const int tid = threadIdx.x;
  float mu[8], a[8], b[8], is[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int c = cv * 8 + k;
    mu[k] = bn.mean[c]; is[k] = bn.invstd[c]; a[k] = bn.gamma[c] * is[k]; b[k] = bn.beta[c];
  }
  float acc[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) acc[k] = 0.f;
#pragma unroll
  for (int u = 0; u < N; ++u) {
    if (u * kSmallThreads + (tid & ~63) >= M) continue;     // no lane of this wave owns the row
    float d[8], v[8];
    BufIO<T>::unpack(rawd[u], d);
    BufIO<T>::unpack(rawy[u], v);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float yc = v[k] - mu[k];
      const float dp = act_pass(fmaf(yc, a[k], b[k]), bn.act) ? d[k] : 0.f;
      acc[k] += dp;
      acc[8 + k] = fmaf(dp, yc * is[k], acc[8 + k]);
    }
  }
  double sum[16];
  block_sum16(acc, sum, lds.red, lds.tot);
  if (tid < 8) {
    double sb = 0.0, sg = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (k == tid) { sb = sum[k]; sg = sum[8 + k]; }
    const double m = (double)M;
    bn.g_beta[cv * 8 + tid] = (float)sb;
    bn.g_gamma[cv * 8 + tid] = (float)sg;
    lds.coef[0][tid] = (float)(sb / m);
    lds.coef[1][tid] = (float)(sg / m);
  }
  __syncthreads();
  float c2[8], c3[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) { c2[k] = lds.coef[0][k]; c3[k] = lds.coef[1][k]; }
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int r = u * kSmallThreads + tid;
    if (r >= M) continue;
    float d[8], v[8];
    BufIO<T>::unpack(rawd[u], d);
    BufIO<T>::unpack(rawy[u], v);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float yc = v[k] - mu[k];
      const float dp = act_pass(fmaf(yc, a[k], b[k]), bn.act) ? d[k] : 0.f;
      d[k] = a[k] * (dp - c2[k] - yc * is[k] * c3[k]);
    }
    out(u, r, d);
  }
}

template <class T>
__device__ __forceinline__ void bn_small_bwd_block(const Blk& blk, T* dz, const T* __restrict__ y, const float* __restrict__ gamma, const float* __restrict__ beta,
    const float* __restrict__ mean, const float* __restrict__ invstd, float* __restrict__ g_gamma,
    float* __restrict__ g_beta, int M, int Cp, int act, unsigned bytes) {
  __shared__ SmallLds lds;
  const int ncv = Cp / 8, cv = xcd_slab(blk.x, ncv), tid = threadIdx.x;
  const __amdgpu_buffer_rsrc_t ry = tensor_rsrc(y, bytes), rd = tensor_rsrc(dz, bytes);
  typename BufIO<T>::Raw rawd[kSmallRows], rawy[kSmallRows];
#pragma unroll
  for (int u = 0; u < kSmallRows; ++u) {
    const int r = u * kSmallThreads + tid;
    rawd[u] = BufIO<T>::issue(rd, (unsigned)(r * ncv + cv) * 8u, r < M);
    rawy[u] = BufIO<T>::issue(ry, (unsigned)(r * ncv + cv) * 8u, r < M);
  }
  small_bwd<T>(rawd, rawy, ColBwd{gamma, beta, mean, invstd, g_gamma, g_beta, act}, lds, cv, M,
               [&](int, int r, const float (&d)[8]) { IO<T>::st(dz + ((long)r * ncv + cv) * 8, d); });
}
template <class T>
__global__ __launch_bounds__(kSmallThreads) void bn_small_bwd_kernel(T* dz, const T* __restrict__ y,
    const float* __restrict__ gamma, const float* __restrict__ beta, const float* __restrict__ mean, const float* __restrict__ invstd,
    float* __restrict__ g_gamma, float* __restrict__ g_beta, int M, int Cp, int act, unsigned bytes) {
  bn_small_bwd_block<T>(one_block(), dz, y, gamma, beta, mean, invstd, g_gamma, g_beta, M, Cp, act, bytes);
}

// A 3 x 3 depthwise layer of a short column with the batch norms around it.  A workgroup of the whole-column kernels owns 8 channels of every
// image, which is all that a depthwise layer needs of its input: so the normalisation in front (PRE), the convolution and the normalisation
// behind it are one launch, with the column between them in LDS.
//   forward:  y1 -> z1 (stored) -> y2 (stored) -> z2;   backward:  dz2, y2 -> dy2 (in place) -> dz1, y1 -> dy1
// Bound by the launches, which follow one another in a block's chain: 4 to 6 us each, three of them here, of which the arithmetic is one or two.
// Every value that went through memory is rounded as it was there, and the taps are added in dw_slide_kernel's order, zeros outside
// the image included, so the bits are those of the separate launches.
// Up to 2048 rows.  A step of VGG-16 at 32 x 32, whose last block has six of these layers at 4 x 4 and 2 x 2, separate / fused: batch 85 (1360
// rows) 824 / 784 us, float32 at batch 64 (1024) 1277 / 1204.  Eight rows a thread, up to 4096 rows: batch 16 (256) 621 / 575, 85 825 / 804, 128 (2048) 938
// / 935, four batches of 256 (4096) in a pipeline 4829 / 4850: there the rows of one workgroup take longer than the launches that they save.
constexpr int kDwSmallRows = 4;                          // rows per thread
template <class T> struct DwSmall {
  static constexpr int ROWS = kDwSmallRows * kSmallThreads;
  static constexpr int PLANE = ROWS + 1;                            // the last one is zeros: what lies outside the image
  uint4 slab[PLANE * (int)sizeof(T) / 2];
  uint4 first[2];
  SmallLds lds;
};

// this thread's rows of a stride-1 3 x 3 convolution of the slab, rounded as a store rounds them (rows past M: zeros)
template <class T, bool FLIP>
__device__ __forceinline__ void dw_small_conv(typename BufIO<T>::Raw (&raw)[kDwSmallRows], const uint4* slab, const T* __restrict__ w, int cv, int ncv, int M, int H, int W) {
  constexpr int ROWS = DwSmall<T>::ROWS, PLANE = DwSmall<T>::PLANE;
  float f[9][8];
#pragma unroll
  for (int t = 0; t < 9; ++t) IO<T>::ld(w + ((long)(FLIP ? 8 - t : t) * ncv + cv) * 8, f[t]);
  const int lane_row = threadIdx.x;
#pragma unroll
  for (int u = 0; u < kDwSmallRows; ++u) {
    const int m = u * kSmallThreads + lane_row;
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    if (m < M) {
      const int q = m % W, h = (m / W) % H;
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          const bool in = (unsigned)(h + r - 1) < (unsigned)H && (unsigned)(q + t - 1) < (unsigned)W;
          float v[8];
          BufIO<T>::unpack(BufIO<T>::slab_read(slab, PLANE, in ? m + (r - 1) * W + t - 1 : ROWS), v);
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] = fmaf(v[e], f[r * 3 + t][e], acc[e]);
        }
    }
    raw[u] = BufIO<T>::pack(acc);
  }
}

template <class T, bool PRE>
__global__ __launch_bounds__(kSmallThreads) void dw_small_fwd_kernel(const T* __restrict__ x, T* __restrict__ z1, ColFwd pre, const T* __restrict__ w,
    T* __restrict__ y2, T* __restrict__ z2, ColFwd bn, int M, int H, int W, int Cp, float eps, float rho, unsigned bytes) {
  typedef BufIO<T> B;
  typedef typename B::Raw Raw;
  constexpr int ROWS = DwSmall<T>::ROWS, PLANE = DwSmall<T>::PLANE;
  __shared__ DwSmall<T> sm;
  const int ncv = Cp / 8, cv = xcd_slab(blockIdx.x, ncv), tid = threadIdx.x;
  const __amdgpu_buffer_rsrc_t rx = tensor_rsrc(x, bytes);
  Raw raw[kDwSmallRows];
#pragma unroll
  for (int u = 0; u < kDwSmallRows; ++u) {
    const int r = u * kSmallThreads + tid;
    raw[u] = B::issue(rx, (unsigned)(r * ncv + cv) * 8u, r < M);
  }
  auto at = [&](T* p, int r) { return reinterpret_cast<Raw*>(p + ((long)r * ncv + cv) * 8); };
  float piv[8];
  SmallTerms t;
  if constexpr (PRE) {
    IO<T>::ld(x + (long)cv * 8, piv);
    small_stats<T>(raw, piv, pre, t, sm.lds, cv, M, eps, rho);
  }
#pragma unroll
  for (int u = 0; u < kDwSmallRows; ++u) {
    const int r = u * kSmallThreads + tid;
    if (r >= M) continue;
    if constexpr (PRE) {
      float v[8];
      B::unpack(raw[u], v);
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = apply_act(fmaf(v[k] - t.mu[k], t.a[k], t.b[k]), pre.act);
      raw[u] = B::pack(v);
      *at(z1, r) = raw[u];
    }
    B::slab_write(sm.slab, PLANE, r, raw[u]);
  }
  const float zero[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (tid == 0) B::slab_write(sm.slab, PLANE, ROWS, B::pack(zero));
  __syncthreads();
  dw_small_conv<T, false>(raw, sm.slab, w, cv, ncv, M, H, W);
  if (tid == 0) B::slab_write(sm.first, 1, 0, raw[0]);
#pragma unroll
  for (int u = 0; u < kDwSmallRows; ++u) {
    const int r = u * kSmallThreads + tid;
    if (r < M) *at(y2, r) = raw[u];
  }
  __syncthreads();
  B::unpack(B::slab_read(sm.first, 1, 0), piv);
  small_stats<T>(raw, piv, bn, t, sm.lds, cv, M, eps, rho);
#pragma unroll
  for (int u = 0; u < kDwSmallRows; ++u) {
    const int r = u * kSmallThreads + tid;
    if (r >= M) continue;
    float v[8];
    B::unpack(raw[u], v);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = apply_act(fmaf(v[k] - t.mu[k], t.a[k], t.b[k]), bn.act);
    IO<T>::st(z2 + ((long)r * ncv + cv) * 8, v);
  }
}

template <class T, bool PRE>
__global__ __launch_bounds__(kSmallThreads) void dw_small_bwd_kernel(T* __restrict__ dz2, const T* __restrict__ y2, ColBwd bn, const T* __restrict__ w, T* __restrict__ dx,
    const T* __restrict__ y1, ColBwd pre, int M, int H, int W, int Cp, unsigned bytes) {
  typedef BufIO<T> B;
  typedef typename B::Raw Raw;
  constexpr int ROWS = DwSmall<T>::ROWS, PLANE = DwSmall<T>::PLANE;
  __shared__ DwSmall<T> sm;
  const int ncv = Cp / 8, cv = xcd_slab(blockIdx.x, ncv), tid = threadIdx.x;
  const __amdgpu_buffer_rsrc_t rd = tensor_rsrc(dz2, bytes), ry = tensor_rsrc(y2, bytes);
  Raw rawd[kDwSmallRows], rawy[kDwSmallRows];
#pragma unroll
  for (int u = 0; u < kDwSmallRows; ++u) {
    const int r = u * kSmallThreads + tid;
    rawd[u] = B::issue(rd, (unsigned)(r * ncv + cv) * 8u, r < M);
    rawy[u] = B::issue(ry, (unsigned)(r * ncv + cv) * 8u, r < M);
  }
  auto at = [&](T* p, int r) { return reinterpret_cast<Raw*>(p + ((long)r * ncv + cv) * 8); };
  small_bwd<T>(rawd, rawy, bn, sm.lds, cv, M, [&](int, int r, const float (&d)[8]) {
    const Raw q = B::pack(d);
    *at(dz2, r) = q;
    B::slab_write(sm.slab, PLANE, r, q);
  });
  if constexpr (PRE) {                                   // in flight behind the convolution
    const __amdgpu_buffer_rsrc_t rp = tensor_rsrc(y1, bytes);
#pragma unroll
    for (int u = 0; u < kDwSmallRows; ++u) {
      const int r = u * kSmallThreads + tid;
      rawy[u] = B::issue(rp, (unsigned)(r * ncv + cv) * 8u, r < M);
    }
  }
  const float zero[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (tid == 0) B::slab_write(sm.slab, PLANE, ROWS, B::pack(zero));
  __syncthreads();
  dw_small_conv<T, true>(rawd, sm.slab, w, cv, ncv, M, H, W);
  if constexpr (PRE) {
    small_bwd<T>(rawd, rawy, pre, sm.lds, cv, M, [&](int, int r, const float (&d)[8]) { *at(dx, r) = B::pack(d); });
  } else {
#pragma unroll
    for (int u = 0; u < kDwSmallRows; ++u) {
      const int r = u * kSmallThreads + tid;
      if (r < M) *at(dx, r) = rawd[u];
    }
  }
}

// ---------------------------------------------------------------------------
// max-pool; idx keeps the window position r*k+t of the first maximum
// ---------------------------------------------------------------------------
// The producing layer's normalisation and activation applied to every element a pool reads (mean == nullptr: x is
// read as it is): x is then that layer's convolution output, each element becomes what bn_apply_kernel would have
// stored (same arithmetic, same rounding), and the normalised tensor, which only the pool reads, is never written.
struct NormFold { const float* mean; const float* invstd; const float* gamma; const float* beta; int act; };

template <class T>
__global__ void maxpool_fwd_kernel(const T* __restrict__ x, T* __restrict__ z, uint8_t* __restrict__ idx,
                                   int N, int H, int W, int P, int Q, int ncv, int k, int stride, int pad,
                                   NormFold fold) {
  const long nvec = (long)N * P * Q * ncv;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nvec; i += (long)gridDim.x * blockDim.x) {
    const int cv = (int)(i % ncv);
    long pix = i / ncv;
    const int q = (int)(pix % Q); pix /= Q;
    const int p = (int)(pix % P);
    const int n = (int)(pix / P);
    float best[8];
    int bi[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { best[e] = 0.f; bi[e] = -1; }
    float mu[8], fa[8], fb[8];
    if (fold.mean) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int ch = cv * 8 + e;
        mu[e] = fold.mean[ch]; fa[e] = fold.gamma[ch] * fold.invstd[ch]; fb[e] = fold.beta[ch];
      }
    }
    for (int r = 0; r < k; ++r) {
      const int h = p * stride + r - pad;
      if (h < 0 || h >= H) continue;
      for (int t = 0; t < k; ++t) {
        const int w = q * stride + t - pad;
        if (w < 0 || w >= W) continue;
        float v[8];
        IO<T>::ld(x + ((((long)n * H + h) * W + w) * ncv + cv) * 8, v);
        if (fold.mean) {
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = as_stored<T>(apply_act(fmaf(v[e] - mu[e], fa[e], fb[e]), fold.act));
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (bi[e] < 0 || v[e] > best[e]) { best[e] = v[e]; bi[e] = r * k + t; }
      }
    }
    IO<T>::st(z + i * 8, best);
    if (idx) {
      uint2 pk;
      pk.x = (uint32_t)bi[0] | ((uint32_t)bi[1] << 8) | ((uint32_t)bi[2] << 16) | ((uint32_t)bi[3] << 24);
      pk.y = (uint32_t)bi[4] | ((uint32_t)bi[5] << 8) | ((uint32_t)bi[6] << 16) | ((uint32_t)bi[7] << 24);
      *reinterpret_cast<uint2*>(idx + i * 8) = pk;
    }
  }
}

// The 3 x 3, stride-2, pad-1 pool (the ResNet stem's) with all nine taps of a window loaded before the first is looked at
// (out-of-range taps read a clamped position and are skipped): one memory latency per window instead of one per
// tap.  Same values and window positions as maxpool_fwd_kernel.
template <class T>
__global__ void maxpool_fwd_k3s2_kernel(const T* __restrict__ x, T* __restrict__ z, uint8_t* __restrict__ idx,
                                        int N, int H, int W, int P, int Q, int ncv, NormFold fold) {
  const long nvec = (long)N * P * Q * ncv;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nvec; i += (long)gridDim.x * blockDim.x) {
    const int cv = (int)(i % ncv);
    long pix = i / ncv;
    const int q = (int)(pix % Q); pix /= Q;
    const int p = (int)(pix % P);
    const int n = (int)(pix / P);
    float mu[8], fa[8], fb[8];
    if (fold.mean) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int ch = cv * 8 + e;
        mu[e] = fold.mean[ch]; fa[e] = fold.gamma[ch] * fold.invstd[ch]; fb[e] = fold.beta[ch];
      }
    }
    typename IO<T>::Raw raw[9];
    unsigned ok = 0;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int h = 2 * p - 1 + tap / 3, w = 2 * q - 1 + tap % 3;
      if (h >= 0 && h < H && w >= 0 && w < W) ok |= 1u << tap;
      const int hc = min(max(h, 0), H - 1), wc = min(max(w, 0), W - 1);
      raw[tap] = IO<T>::ld_raw(x + ((((long)n * H + hc) * W + wc) * ncv + cv) * 8);
    }
    __builtin_amdgcn_sched_barrier(0);
    float best[8];
    int bi[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { best[e] = 0.f; bi[e] = -1; }
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      if (!(ok >> tap & 1)) continue;
      float v[8];
      IO<T>::unpack(raw[tap], v);
      if (fold.mean) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = as_stored<T>(apply_act(fmaf(v[e] - mu[e], fa[e], fb[e]), fold.act));
      }
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (bi[e] < 0 || v[e] > best[e]) { best[e] = v[e]; bi[e] = tap; }
    }
    IO<T>::st(z + i * 8, best);
    if (idx) {
      uint2 pk;
      pk.x = (uint32_t)bi[0] | ((uint32_t)bi[1] << 8) | ((uint32_t)bi[2] << 16) | ((uint32_t)bi[3] << 24);
      pk.y = (uint32_t)bi[4] | ((uint32_t)bi[5] << 8) | ((uint32_t)bi[6] << 16) | ((uint32_t)bi[7] << 24);
      *reinterpret_cast<uint2*>(idx + i * 8) = pk;
    }
  }
}

// Its backward pass: an input pixel lies in one window per direction when its coordinate is even (tap 1) and in two when
// it is odd (taps 0 and 2), so at most four windows, whose positions and gradients are all loaded before the first
// comparison; contributions are added in the tap order of maxpool_bwd_kernel.
template <class T>
__global__ void maxpool_bwd_k3s2_kernel(const T* __restrict__ dz, const uint8_t* __restrict__ idx,
                                        T* __restrict__ dx, int N, int H, int W, int P, int Q, int ncv, int accumulate) {
  const long nvec = (long)N * H * W * ncv;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nvec; i += (long)gridDim.x * blockDim.x) {
    const int cv = (int)(i % ncv);
    long pix = i / ncv;
    const int w = (int)(pix % W); pix /= W;
    const int h = (int)(pix % H);
    const int n = (int)(pix / H);
    // candidate windows per direction, in tap order: odd coordinate: tap 0 of window (c + 1) / 2, tap 2 of (c - 1) / 2;
    // even: tap 1 of window c / 2
    int pr[2], rr[2], qc[2], tc[2];
    bool pv[2], qv[2];
    if (h & 1) { rr[0] = 0; pr[0] = (h + 1) >> 1; pv[0] = pr[0] < P; rr[1] = 2; pr[1] = (h - 1) >> 1; pv[1] = pr[1] < P; }
    else { rr[0] = 1; pr[0] = h >> 1; pv[0] = pr[0] < P; rr[1] = 0; pr[1] = 0; pv[1] = false; }
    if (w & 1) { tc[0] = 0; qc[0] = (w + 1) >> 1; qv[0] = qc[0] < Q; tc[1] = 2; qc[1] = (w - 1) >> 1; qv[1] = qc[1] < Q; }
    else { tc[0] = 1; qc[0] = w >> 1; qv[0] = qc[0] < Q; tc[1] = 0; qc[1] = 0; qv[1] = false; }
    uint2 pk[4];
    typename IO<T>::Raw raw[4];
    bool valid[4];
    uint32_t me[4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int k = a * 2 + b;
        valid[k] = pv[a] && qv[b];
        const int pp = min(pr[a], P - 1), qq = min(qc[b], Q - 1);
        const long o = ((((long)n * P + pp) * Q + qq) * ncv + cv) * 8;
        pk[k] = *reinterpret_cast<const uint2*>(idx + o);
        raw[k] = IO<T>::ld_raw(dz + o);
        me[k] = (uint32_t)(rr[a] * 3 + tc[b]);
      }
    float acc[8];
    if (accumulate) IO<T>::ld(dx + i * 8, acc);
    else {
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float d[8];
      IO<T>::unpack(raw[k], d);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t word = e < 4 ? pk[k].x : pk[k].y;
        if (valid[k] && ((word >> (8 * (e & 3))) & 0xffu) == me[k]) acc[e] += d[e];
      }
    }
    IO<T>::st(dx + i * 8, acc);
  }
}

// gather form: every input pixel collects from the windows that chose it
template <class T>
__global__ void maxpool_bwd_kernel(const T* __restrict__ dz, const uint8_t* __restrict__ idx,
                                   T* __restrict__ dx, int N, int H, int W, int P, int Q, int ncv,
                                   int k, int stride, int pad, int accumulate) {
  const long nvec = (long)N * H * W * ncv;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nvec; i += (long)gridDim.x * blockDim.x) {
    const int cv = (int)(i % ncv);
    long pix = i / ncv;
    const int w = (int)(pix % W); pix /= W;
    const int h = (int)(pix % H);
    const int n = (int)(pix / H);
    float acc[8];
    if (accumulate) IO<T>::ld(dx + i * 8, acc);
    else {
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    }
    for (int r = 0; r < k; ++r) {
      const int ph = h + pad - r;
      if (ph < 0 || ph % stride) continue;
      const int p = ph / stride;
      if (p >= P) continue;
      for (int t = 0; t < k; ++t) {
        const int qw = w + pad - t;
        if (qw < 0 || qw % stride) continue;
        const int q = qw / stride;
        if (q >= Q) continue;
        const long o = ((((long)n * P + p) * Q + q) * ncv + cv) * 8;
        const uint2 pk = *reinterpret_cast<const uint2*>(idx + o);
        float d[8];
        IO<T>::ld(dz + o, d);
        const uint32_t me = (uint32_t)(r * k + t);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint32_t word = e < 4 ? pk.x : pk.y;
          if (((word >> (8 * (e & 3))) & 0xffu) == me) acc[e] += d[e];
        }
      }
    }
    IO<T>::st(dx + i * 8, acc);
  }
}

// ---------------------------------------------------------------------------
// joins: z = act(sum_k p_k v_k) forward; backward fans  s_k*[act passes at z]*dz
// out to up to 8 destinations, each either written or accumulated
// ---------------------------------------------------------------------------
struct Join {
  const void* src[8];
  void* dst[8];
  float p[8];
  const float* pdev;     // when set, the weights are read from device memory instead (trainable mix)
  int accumulate[8];
  int n;
};

__device__ __forceinline__ void join_weights(const Join& j, float (&p)[8]) {
#pragma unroll
  for (int k = 0; k < 8; ++k) p[k] = k < j.n ? (j.pdev ? j.pdev[k] : j.p[k]) : 0.f;
}

template <class T>
__global__ void join_fwd_kernel(Join j, T* __restrict__ z, long nvec, int act) {
  float p[8];
  join_weights(j, p);
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nvec; i += (long)gridDim.x * blockDim.x) {
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (k >= j.n) break;
      float v[8];
      IO<T>::ld(static_cast<const T*>(j.src[k]) + i * 8, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = fmaf(p[k], v[e], acc[e]);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = apply_act(acc[e], act);
    IO<T>::st(z + i * 8, acc);
  }
}

// z is the post-activation output: for ReLU the gradient passes where z > 0
template <class T>
__global__ void join_bwd_kernel(Join j, const T* __restrict__ dz, const T* __restrict__ z, long nvec, int act) {
  float p[8];
  join_weights(j, p);
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nvec; i += (long)gridDim.x * blockDim.x) {
    float d[8];
    IO<T>::ld(dz + i * 8, d);
    if (act != ACT_NONE) {
      float v[8];
      IO<T>::ld(z + i * 8, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) d[e] = act_pass(v[e], act) ? d[e] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (k >= j.n) break;
      T* dst = static_cast<T*>(j.dst[k]);
      if (!dst) continue;
      float o[8];
      if (j.accumulate[k]) {
        IO<T>::ld(dst + i * 8, o);
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = fmaf(p[k], d[e], o[e]);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = p[k] * d[e];
      }
      IO<T>::st(dst + i * 8, o);
    }
  }
}

// ---------------------------------------------------------------------------
// architecture round of a supernet (Sec. VI-A, neural architecture search): a mix op computes
// z = act(sum_k p_k y_k) with p = softmax(alpha).  With d = dL/dz masked by the activation,
//   g_k = <d, y_k>,   dL/dalpha_j = p_j (g_j - sum_k p_k g_k).
// mix_dot_kernel leaves one partial g per workgroup; mix_alpha_update_kernel sums them in a fixed
// order, forms the gradient, applies  v <- mu v + g ; alpha <- alpha - lr v  and writes the new p.
// One mix op owns 32 floats of state: alpha[8], momentum[8], gradient[8], p[8].
// ---------------------------------------------------------------------------
constexpr int kMixState = 32, kMixAlpha = 0, kMixMom = 8, kMixGrad = 16, kMixP = 24;
constexpr int kMixDotBlocks = 512;

template <class T>
__global__ __launch_bounds__(256) void mix_dot_kernel(Join j, const T* __restrict__ dz, const T* __restrict__ z,
                                                      float* __restrict__ part, long nvec, int act) {
  __shared__ float red[4][8];
  float acc[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) acc[k] = 0.f;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nvec; i += (long)gridDim.x * blockDim.x) {
    float d[8];
    IO<T>::ld(dz + i * 8, d);
    if (act != ACT_NONE) {
      float v[8];
      IO<T>::ld(z + i * 8, v);
#pragma unroll
      for (int e = 0; e < 8; ++e) d[e] = act_pass(v[e], act) ? d[e] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (k >= j.n) break;
      float v[8];
      IO<T>::ld(static_cast<const T*>(j.src[k]) + i * 8, v);
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) s = fmaf(d[e], v[e], s);
      acc[k] += s;
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    float v = acc[k];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if (lane == 0) red[wave][k] = v;
  }
  __syncthreads();
  if (threadIdx.x < 8) part[blockIdx.x * 8 + threadIdx.x] = (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
}

// one workgroup of 256 threads; state = the mix op's 32 floats; update == 0 leaves alpha, momentum and p
__global__ __launch_bounds__(256) void mix_alpha_update_kernel(const float* __restrict__ part, int nblocks,
                                                               float* __restrict__ state, int n,
                                                               const float* __restrict__ lr_ptr, float mu, int update) {
  __shared__ double red[32][8];
  __shared__ double g[8];
  __shared__ float alpha[8];
  const int k = threadIdx.x & 7, row = threadIdx.x >> 3;
  double s = 0.0;
  for (int b = row; b < nblocks; b += 32) s += (double)part[b * 8 + k];
  red[row][k] = s;
  __syncthreads();
  for (int h = 16; h > 0; h >>= 1) {
    if (row < h) red[row][k] += red[row + h][k];
    __syncthreads();
  }
  if (threadIdx.x < 8) g[threadIdx.x] = red[0][threadIdx.x];
  __syncthreads();
  if ((int)threadIdx.x < n) {
    // the g_q nearly agree, and the stored p sum to one only to float32 rounding: without the division their
    // common part would stay in the difference (times that rounding, 1e-4 of the gradient where they agree to 1e-3)
    double mean = 0.0, sum_p = 0.0;
    for (int q = 0; q < n; ++q) { mean += (double)state[kMixP + q] * g[q]; sum_p += (double)state[kMixP + q]; }
    const float grad = (float)((double)state[kMixP + threadIdx.x] * (g[threadIdx.x] - mean / sum_p));
    state[kMixGrad + threadIdx.x] = grad;
    float a = state[kMixAlpha + threadIdx.x];
    if (update) {
      const float v = fmaf(mu, state[kMixMom + threadIdx.x], grad);
      a -= *lr_ptr * v;
      state[kMixMom + threadIdx.x] = v;
      state[kMixAlpha + threadIdx.x] = a;
    }
    alpha[threadIdx.x] = a;
  }
  __syncthreads();   // every read of the old p is done; alpha[] is complete
  if (update && (int)threadIdx.x < n) {
    float top = alpha[0];
    for (int q = 1; q < n; ++q) top = fmaxf(top, alpha[q]);
    float sum = 0.f;
    for (int q = 0; q < n; ++q) sum += expf(alpha[q] - top);
    state[kMixP + threadIdx.x] = expf(alpha[threadIdx.x] - top) / sum;
  }
}

// ---------------------------------------------------------------------------
// fused MSE loss + gradient (Sec. II-A, L(delta output)):
//   part[block] = sum (s-t)^2 ;  ds = 2 (s-t) / M ;  loss = sum(part) / M
// ---------------------------------------------------------------------------
template <class T>
__global__ __launch_bounds__(256) void mse_kernel(const T* __restrict__ s, const T* __restrict__ t,
                                                  T* __restrict__ ds, float* __restrict__ part,
                                                  long nvec, float two_over_m) {
  __shared__ float red[256];
  float acc = 0.f;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nvec; i += (long)gridDim.x * blockDim.x) {
    float a[8], b[8];
    IO<T>::ld(s + i * 8, a);
    IO<T>::ld(t + i * 8, b);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float d = a[e] - b[e];
      acc = fmaf(d, d, acc);
      a[e] = d * two_over_m;
    }
    IO<T>::st(ds + i * 8, a);
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s2 = 128; s2 > 0; s2 >>= 1) {
    if ((int)threadIdx.x < s2) red[threadIdx.x] += red[threadIdx.x + s2];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(256) void mse_final_kernel(const float* __restrict__ part, int n, double inv_m,
                                                        float* loss) {
  __shared__ double red[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) s += (double)part[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = (float)(red[0] * inv_m);
}

// ---------------------------------------------------------------------------
// fused SGD-momentum over one block's flat parameter arena (Algorithm 1,
// update_weight; Sec. IV-B):  v <- mu v + g ; w <- w - lr v ; compute copy <- rne(w)
// ---------------------------------------------------------------------------
template <class T>
__global__ void sgd_momentum_kernel(float* __restrict__ w, float* __restrict__ v,
                                    const float* __restrict__ g, T* __restrict__ wc, long n4,
                                    const float* __restrict__ lr_ptr, float mu) {
  const float lr = *lr_ptr;  // device scalar: a captured graph stays valid when the rate changes
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n4; i += (long)gridDim.x * blockDim.x) {
    float4 wv = reinterpret_cast<float4*>(w)[i], vv = reinterpret_cast<float4*>(v)[i];
    const float4 gv = reinterpret_cast<const float4*>(g)[i];
    vv.x = fmaf(mu, vv.x, gv.x); vv.y = fmaf(mu, vv.y, gv.y);
    vv.z = fmaf(mu, vv.z, gv.z); vv.w = fmaf(mu, vv.w, gv.w);
    wv.x -= lr * vv.x; wv.y -= lr * vv.y; wv.z -= lr * vv.z; wv.w -= lr * vv.w;
    reinterpret_cast<float4*>(v)[i] = vv;
    reinterpret_cast<float4*>(w)[i] = wv;
    if (wc) {
      uint2 pk;
      pk.x = pack_bf2(wv.x, wv.y);
      pk.y = pack_bf2(wv.z, wv.w);
      reinterpret_cast<uint2*>(wc)[i] = pk;
    }
  }
}

__global__ void set_scalar_kernel(float* p, float v) { *p = v; }

// compute copy <- rne(master) without an update (after parameters were loaded)
__global__ void cast_params_kernel(const float* __restrict__ w, bf16_t* __restrict__ wc, long n4) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n4; i += (long)gridDim.x * blockDim.x) {
    const float4 wv = reinterpret_cast<const float4*>(w)[i];
    uint2 pk;
    pk.x = pack_bf2(wv.x, wv.y);
    pk.y = pack_bf2(wv.z, wv.w);
    reinterpret_cast<uint2*>(wc)[i] = pk;
  }
}

// Transposed weight copies for backward-data: src [K][RS][C] -> dst [C][RS][K].
struct TransposeEntry { long src, dst; int K, RS, C; };
template <class T>
__global__ __launch_bounds__(256) void transpose_weights_kernel(const T* __restrict__ wc, T* __restrict__ wt,
                                                                const TransposeEntry* __restrict__ table) {
  // 64 x 64 tiles of one filter tap through LDS: rows of 64 consecutive c are read, rows of 64 consecutive k
  // written, both whole cache lines per wave
  __shared__ T tile[64][65];
  const TransposeEntry e = table[blockIdx.y];
  const int tk = (e.K + 63) / 64, tc = (e.C + 63) / 64;
  const long ntiles = (long)tk * tc * e.RS;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (long t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const int k0 = (int)(t % tk) * 64;
    const long r = t / tk;
    const int c0 = (int)(r % tc) * 64, rs = (int)(r / tc);
    T v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {                  // all sixteen loads in flight
      const int k = k0 + ty + 4 * j, c = c0 + tx;
      v[j] = (k < e.K && c < e.C) ? wc[e.src + ((long)k * e.RS + rs) * e.C + c] : T(0);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) tile[ty + 4 * j][tx] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int c = c0 + ty + 4 * j, k = k0 + tx;
      if (k < e.K && c < e.C) wt[e.dst + ((long)c * e.RS + rs) * e.K + k] = tile[tx][ty + 4 * j];
    }
    __syncthreads();
  }
}

// out[j] = sum_s part[s*n + j]   (ordered second stage of split reductions); n % 4 == 0.
// Block = (256/SL) float4 outputs x SL split lanes: lane l adds splits l, l+SL, ... in order (four
// loads in flight), then the SL lane sums are added in order, so the result does not depend on
// scheduling.  SL = 8 for a few partials of a large tensor, 32 for many partials of a small one.
template <int SL>
__device__ __forceinline__ void sum_partials_body(const Blk& blk, const float* __restrict__ part, float* __restrict__ out, long n, int splits,
                                                  float4* red /*[256]*/) {
  constexpr int NO = 256 / SL;
  const int o = threadIdx.x % NO, l = threadIdx.x / NO;
  const long n4 = n / 4;
  for (long base = (long)blk.x * NO; base < n4; base += (long)blk.gx * NO) {
    const long i = base + o;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < n4) {
      int k = l;
      for (; k + 3 * SL < splits; k += 4 * SL) {
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const float4*>(part + (long)(k + u * SL) * n + i * 4);
#pragma unroll
        for (int u = 0; u < 4; ++u) { s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w; }
      }
      for (; k < splits; k += SL) {
        const float4 v = *reinterpret_cast<const float4*>(part + (long)k * n + i * 4);
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
      }
    }
    red[l * NO + o] = s;
    __syncthreads();
    if (l == 0 && i < n4) {
      float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int k = 0; k < SL; ++k) {
        const float4 v = red[k * NO + o];
        t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
      }
      *reinterpret_cast<float4*>(out + i * 4) = t;
    }
    __syncthreads();
  }
}
constexpr int kManySplits = 64;       // from here on SL = 32
template <int SL>
__device__ __forceinline__ void sum_partials_block(const Blk& blk, const float* __restrict__ part, float* __restrict__ out, long n, int splits) {
  __shared__ float4 red[256];
  sum_partials_body<SL>(blk, part, out, n, splits, red);
}
template <int SL>
__global__ __launch_bounds__(256) void sum_partials_kernel(const float* __restrict__ part, float* __restrict__ out,
    long n, int splits) {
  sum_partials_block<SL>(one_block(), part, out, n, splits);
}
// The same for many layers in one launch, blockIdx.y = layer: the weight gradients of a student block, whose partial
// sums wait side by side until the update reads them.  A launch of its own per layer is 4 us for a few microseconds' worth of
// memory traffic or less: 52 of 435 launches of a MobileNetV2 step, 224 of 3670 us of kernel time at batch 33.
struct SumEntry { long part, out, n; int splits, pad; };   // float32 element offsets
__global__ __launch_bounds__(256) void sum_partials_batch_kernel(const float* __restrict__ parts, float* __restrict__ outs,
                                                                 const SumEntry* __restrict__ table) {
  __shared__ float4 red[256];
  const SumEntry e = table[blockIdx.y];
  if (e.splits >= kManySplits) sum_partials_body<32>(one_block(), parts + e.part, outs + e.out, e.n, e.splits, red);
  else sum_partials_body<8>(one_block(), parts + e.part, outs + e.out, e.n, e.splits, red);
}

// ---------------------------------------------------------------------------
// depthwise convolution, weights [k*k][Cp] (channel-last)
// ---------------------------------------------------------------------------
// Forward: one thread = 8 channels of one output pixel; all k*k taps are requested before the
// first multiply.  KK = k*k.
template <class T, int KK>
__global__ __launch_bounds__(256) void dw_fwd_kernel(const T* __restrict__ x, const T* __restrict__ w,
                                                     T* __restrict__ y, const float* __restrict__ a,
                                                     const float* __restrict__ b, int act, int N, int H, int W,
                                                     int P, int Q, int ncv, int k, int stride, int pad,
                                                     unsigned x_elems) {
  const long nvec = (long)N * P * Q * ncv;
  const __amdgpu_buffer_rsrc_t xr = tensor_rsrc(x, x_elems * (unsigned)sizeof(T));
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nvec; i += (long)gridDim.x * blockDim.x) {
    const int cv = (int)(i % ncv);
    long pix = i / ncv;
    const int q = (int)(pix % Q); pix /= Q;
    const int p = (int)(pix % P);
    const int n = (int)(pix / P);
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    constexpr int G = KK < 25 ? KK : 25;     // taps in flight at once (bounds the register footprint)
#pragma unroll
    for (int t0 = 0; t0 < KK; t0 += G) {
      typename BufIO<T>::Raw raw[G];
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const int t = t0 + u;
        const int r = t / k, s = t - r * k;    // k is uniform: scalar arithmetic after unrolling
        const int h = p * stride + r - pad, ww = q * stride + s - pad;
        const bool ok = t < KK && (unsigned)h < (unsigned)H && (unsigned)ww < (unsigned)W;
        raw[u] = BufIO<T>::issue(xr, (unsigned)(((n * H + h) * W + ww) * ncv + cv) * 8u, ok);
      }
#pragma unroll
      for (int u = 0; u < G; ++u) {
        if (t0 + u >= KK) continue;
        float v[8], f[8];
        BufIO<T>::unpack(raw[u], v);
        IO<T>::ld(w + ((long)(t0 + u) * ncv + cv) * 8, f);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = fmaf(v[e], f[e], acc[e]);
      }
    }
    if (a) {  // folded inference-mode BN + activation (teacher)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = apply_act(fmaf(acc[e], a[cv * 8 + e], b[cv * 8 + e]), act);
    }
    IO<T>::st(y + i * 8, acc);
  }
}

// Sliding-window forward / stride-1 backward-data: one thread = 8 channels of WS consecutive output
// pixels of one row.  Per filter row it loads the (WS-1)*STRIDE + K input pixels once and uses each
// for up to K outputs, so the loads per output drop from K*K to K*((WS-1)*STRIDE+K)/WS: the vector
// memory pipeline, not HBM, is what a one-pixel-per-thread depthwise kernel saturates.
// FLIP: read the filter mirrored (backward-data of a stride-1 convolution is the same sliding
// sum with taps (K-1-r, K-1-s)); `accumulate` then adds to what dst holds.
template <class T, int K, int STRIDE, int WS, bool FLIP>
__device__ __forceinline__ void dw_slide_block(const Blk& blk, const T* __restrict__ x, const T* __restrict__ w,
                                                       T* dst, const float* __restrict__ a,
                                                       const float* __restrict__ b, int act, int accumulate,
                                                       int N, int H, int W, int P, int Q, int ncv, int pad,
                                                       unsigned x_elems) {
  constexpr int NIN = (WS - 1) * STRIDE + K;
  const int QS = (Q + WS - 1) / WS;
  const long nitem = (long)N * P * QS * ncv;
  const __amdgpu_buffer_rsrc_t xr = tensor_rsrc(x, x_elems * (unsigned)sizeof(T));
  for (long i = blk.x * (long)blockDim.x + threadIdx.x; i < nitem; i += (long)blk.gx * blockDim.x) {
    const int cv = (int)(i % ncv);
    long seg = i / ncv;
    const int qs = (int)(seg % QS); seg /= QS;
    const int p = (int)(seg % P);
    const int n = (int)(seg / P);
    const int q0 = qs * WS, w0 = q0 * STRIDE - pad;
    float ea[8], eb[8];                // folded BN terms, fetched ahead of the taps they follow
    if (a) {
#pragma unroll
      for (int e = 0; e < 8; ++e) { ea[e] = a[cv * 8 + e]; eb[e] = b[cv * 8 + e]; }
    }
    float acc[WS][8];
#pragma unroll
    for (int o = 0; o < WS; ++o)
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[o][e] = 0.f;
#pragma unroll(K == 3 ? 3 : 1)
    for (int r = 0; r < K; ++r) {      // 5x5 and 7x7: one filter row at a time bounds the registers
      const int h = p * STRIDE + r - pad;
      const bool row_ok = (unsigned)h < (unsigned)H;
      const unsigned rowoff = (unsigned)((n * H + h) * W + w0) * (unsigned)ncv + (unsigned)cv;
      typename BufIO<T>::Raw raw[NIN];
#pragma unroll
      for (int j = 0; j < NIN; ++j)
        raw[j] = BufIO<T>::issue(xr, (rowoff + (unsigned)(j * ncv)) * 8u, row_ok && (unsigned)(w0 + j) < (unsigned)W);
      float f[K][8];
#pragma unroll
      for (int t = 0; t < K; ++t) {
        const int tap = FLIP ? (K - 1 - r) * K + (K - 1 - t) : r * K + t;
        IO<T>::ld(w + ((long)tap * ncv + cv) * 8, f[t]);
      }
#pragma unroll
      for (int j = 0; j < NIN; ++j) {
        float v[8];
        BufIO<T>::unpack(raw[j], v);
#pragma unroll
        for (int o = 0; o < WS; ++o) {
          const int t = j - o * STRIDE;       // compile-time after unrolling
          if (t < 0 || t >= K) continue;
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[o][e] = fmaf(v[e], f[t][e], acc[o][e]);
        }
      }
    }
#pragma unroll
    for (int o = 0; o < WS; ++o) {
      if (q0 + o >= Q) continue;
      T* out = dst + ((((long)n * P + p) * Q + q0 + o) * ncv + cv) * 8;
      if (a) {  // folded inference-mode BN + activation (teacher)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[o][e] = apply_act(fmaf(acc[o][e], ea[e], eb[e]), act);
      }
      if (accumulate) {
        float old[8];
        IO<T>::ld(out, old);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[o][e] += old[e];
      }
      IO<T>::st(out, acc[o]);
    }
  }
}
template <class T, int K, int STRIDE, int WS, bool FLIP>
__global__ __launch_bounds__(256) void dw_slide_kernel(const T* __restrict__ x,
    const T* __restrict__ w, T* dst, const float* __restrict__ a, const float* __restrict__ b, int act, int accumulate, int N, int H,
    int W, int P, int Q, int ncv, int pad, unsigned x_elems) {
  dw_slide_block<T, K, STRIDE, WS, FLIP>(one_block(), x, w, dst, a, b, act, accumulate, N, H, W, P, Q, ncv, pad, x_elems);
}

// LDS-tiled stride-1 3 x 3 depthwise convolution on the vector ALUs (bf16): a block stages the (8+K-1) x (16+K-1) input
// pixels x 64 channels behind an 8 x 16 output tile in LDS with ONE round of global loads (all in
// flight together), then every thread slides over 4 outputs reading LDS.  Each input element is
// fetched once per tile instead of ~K*K/2 times, which takes the kernel off the vector-memory
// pipeline and onto HBM.  LDS pixel pitch 160 B: the two 4-pixel segments of a 16-lane group land
// 128 B apart modulo the 256 B bank span.  FLIP / accumulate as in dw_slide_kernel.
//  Whole 128-byte lines of whole 64-channel groups, read and written (nontemporally: the tensors are far larger than the
// caches) by one workgroup: bound by memory on tensors the caches do not hold, where dw_mfma_kernel's workgroups of 32 channels share
// each line with a neighbour and lose to it.  Backward-data in us against dw_mfma_kernel: 128 x 56 x 56 x 192 64 and 77,
// 64 x 56 x 56 x 192 35 and 40, 128 x 40 x 40 x 384 68 and 83, 128 x 28 x 28 x 384 37 and 40, 128 x 24 x 24 x 960 65 and 72,
// 64 x 112 x 112 x 64 40 and 48; on smaller tensors or channel counts that leave a group part empty it is the other way round (64 x 28
// x 28 x 192 13 and 10, 128 x 14 x 14 x 960 24 and 20, 128 x 56 x 56 x 144 76 and 60).
constexpr int kDwTileH = 8, kDwTileW = 16, kDwTileCv = 8, kDwTilePitch = kDwTileCv * 16 + 32;

template <bool FLIP>
__global__ __launch_bounds__(256) void dw_tile_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w,
                                                      bf16_t* dst, const float* __restrict__ a,
                                                      const float* __restrict__ b, int act, int accumulate,
                                                      int N, int H, int W, int ncv, int tiles_h, int tiles_w,
                                                      unsigned x_bytes) {
  constexpr int K = 3, TH = kDwTileH, TW = kDwTileW, WS = 4, CVB = kDwTileCv, PIXB = kDwTilePitch;
  constexpr int IH = TH + K - 1, IW = TW + K - 1, NIN = WS + K - 1, pad = K / 2;
  constexpr int TOTAL = IH * IW * CVB, NLOAD = (TOTAL + 255) / 256;
  __shared__ __attribute__((aligned(16))) unsigned char tile[IH * IW * PIXB];
  __shared__ __attribute__((aligned(16))) float wl[K * K * CVB * 8];   // the block's filters, unpacked once
  const int tid = threadIdx.x;
  int t = blockIdx.x;
  const int tw = t % tiles_w; t /= tiles_w;
  const int th_ = t % tiles_h;
  const int n = t / tiles_h;
  const int h0 = th_ * TH, w0 = tw * TW, cv0 = blockIdx.y * CVB;
  const __amdgpu_buffer_rsrc_t xr = tensor_rsrc(x, x_bytes);

  uint4 raw[NLOAD];
#pragma unroll
  for (int i = 0; i < NLOAD; ++i) {
    const int c = tid + i * 256;
    const int pix = c / CVB, cvl = c % CVB;
    const int ih = pix / IW, iw = pix % IW;
    const int h = h0 - pad + ih, ww = w0 - pad + iw;
    const bool ok = c < TOTAL && (unsigned)h < (unsigned)H && (unsigned)ww < (unsigned)W && cv0 + cvl < ncv;
    raw[i] = buffer_load16(xr, ok ? (unsigned)(((n * H + h) * W + ww) * ncv + cv0 + cvl) * 16u : kOutOfRange);
  }
  constexpr int NW = (K * K * CVB + 255) / 256;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int c = tid + i * 256;
    if (c < K * K * CVB) {
      const int tap = c / CVB, wcv = cv0 + c % CVB;
      float f[8];
      if (wcv < ncv) IO<bf16_t>::ld(w + ((long)tap * ncv + wcv) * 8, f);
      else {
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = 0.f;
      }
      float* dstw = &wl[((FLIP ? K * K - 1 - tap : tap) * CVB + c % CVB) * 8];
      *reinterpret_cast<float4*>(dstw) = make_float4(f[0], f[1], f[2], f[3]);
      *reinterpret_cast<float4*>(dstw + 4) = make_float4(f[4], f[5], f[6], f[7]);
    }
  }
#pragma unroll
  for (int i = 0; i < NLOAD; ++i) {
    const int c = tid + i * 256;
    if (c < TOTAL) *reinterpret_cast<uint4*>(&tile[(c / CVB) * PIXB + (c % CVB) * 16]) = raw[i];
  }
  __syncthreads();

  const int cvl = tid % CVB, seg = (tid / CVB) % (TW / WS), th = tid / (CVB * (TW / WS));
  const int cv = cv0 + cvl;
  if (cv >= ncv) return;
  float ea[8], eb[8];                  // folded BN terms, fetched ahead of the taps they follow
  if (a) {
#pragma unroll
    for (int e = 0; e < 8; ++e) { ea[e] = a[cv * 8 + e]; eb[e] = b[cv * 8 + e]; }
  }
  float acc[WS][8];
#pragma unroll
  for (int o = 0; o < WS; ++o)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[o][e] = 0.f;
#pragma unroll 1
  for (int r = 0; r < K; ++r) {
    const unsigned char* rowp = &tile[((th + r) * IW + seg * WS) * PIXB + cvl * 16];
    uint4 in[NIN];
#pragma unroll
    for (int j = 0; j < NIN; ++j) in[j] = *reinterpret_cast<const uint4*>(rowp + j * PIXB);
    float f[K][8];
#pragma unroll
    for (int tt = 0; tt < K; ++tt) {
      const float* wr = &wl[((r * K + tt) * CVB + cvl) * 8];
      const float4 lo = *reinterpret_cast<const float4*>(wr), hi = *reinterpret_cast<const float4*>(wr + 4);
      f[tt][0] = lo.x; f[tt][1] = lo.y; f[tt][2] = lo.z; f[tt][3] = lo.w;
      f[tt][4] = hi.x; f[tt][5] = hi.y; f[tt][6] = hi.z; f[tt][7] = hi.w;
    }
#pragma unroll
    for (int j = 0; j < NIN; ++j) {
      float v[8];
      BufIO<bf16_t>::unpack(in[j], v);
#pragma unroll
      for (int o = 0; o < WS; ++o) {
        const int tt = j - o;
        if (tt < 0 || tt >= K) continue;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[o][e] = fmaf(v[e], f[tt][e], acc[o][e]);
      }
    }
  }
  const int h = h0 + th;
  if (h >= H) return;
#pragma unroll
  for (int o = 0; o < WS; ++o) {
    const int ww = w0 + seg * WS + o;
    if (ww >= W) continue;
    bf16_t* out = dst + ((((long)n * H + h) * W + ww) * ncv + cv) * 8;
    if (a) {
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[o][e] = apply_act(fmaf(acc[o][e], ea[e], eb[e]), act);
    }
    if (accumulate) {
      float old[8];
      IO<bf16_t>::ld(out, old);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[o][e] += old[e];
    }
    IO<bf16_t>::st_t<true>(out, acc[o]);
  }
}

// Backward-data in gather form: dx[h,w] (+)= sum_taps dy[(h+pad-r)/st, (w+pad-s)/st] * w[r][s]
template <class T, int KK>
__global__ __launch_bounds__(256) void dw_dgrad_kernel(const T* __restrict__ dy, const T* __restrict__ w,
                                                       T* __restrict__ dx, int N, int H, int W, int P, int Q,
                                                       int ncv, int k, int stride, int pad, int accumulate,
                                                       unsigned dy_elems) {
  const long nvec = (long)N * H * W * ncv;
  const __amdgpu_buffer_rsrc_t dr = tensor_rsrc(dy, dy_elems * (unsigned)sizeof(T));
  const int sh = stride == 2 ? 1 : 0, smask = stride - 1;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nvec; i += (long)gridDim.x * blockDim.x) {
    const int cv = (int)(i % ncv);
    long pix = i / ncv;
    const int ww = (int)(pix % W); pix /= W;
    const int h = (int)(pix % H);
    const int n = (int)(pix / H);
    float acc[8];
    if (accumulate) IO<T>::ld(dx + i * 8, acc);
    else {
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    }
    constexpr int G = KK < 25 ? KK : 25;
#pragma unroll
    for (int t0 = 0; t0 < KK; t0 += G) {
      typename BufIO<T>::Raw raw[G];
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const int t = t0 + u;
        const int r = t / k, s = t - r * k;
        const int ph = h + pad - r, qw = ww + pad - s;
        const int p = ph >> sh, q = qw >> sh;
        const bool ok = t < KK && ((ph | qw) & smask) == 0 && (unsigned)p < (unsigned)P && (unsigned)q < (unsigned)Q;
        raw[u] = BufIO<T>::issue(dr, (unsigned)(((n * P + p) * Q + q) * ncv + cv) * 8u, ok);
      }
#pragma unroll
      for (int u = 0; u < G; ++u) {
        if (t0 + u >= KK) continue;
        float d[8], f[8];
        BufIO<T>::unpack(raw[u], d);
        IO<T>::ld(w + ((long)(t0 + u) * ncv + cv) * 8, f);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = fmaf(d[e], f[e], acc[e]);
      }
    }
    IO<T>::st(dx + i * 8, acc);
  }
}

// Backward-data of a stride-2 depthwise convolution: an input pixel only meets the taps whose
// parity matches its own, (K+1)/2 per dimension, so only those are visited (K*K/4 instead of K*K
// masked loads).
template <class T, int K>
__device__ __forceinline__ void dw_dgrad_s2_block(const Blk& blk, const T* __restrict__ dy, const T* __restrict__ w,
                                                          T* __restrict__ dx, int N, int H, int W, int P, int Q,
                                                          int ncv, int pad, int accumulate, unsigned dy_elems) {
  constexpr int HK = (K + 1) / 2;
  const long nvec = (long)N * H * W * ncv;
  const __amdgpu_buffer_rsrc_t dr = tensor_rsrc(dy, dy_elems * (unsigned)sizeof(T));
  for (long i = blk.x * (long)blockDim.x + threadIdx.x; i < nvec; i += (long)blk.gx * blockDim.x) {
    const int cv = (int)(i % ncv);
    long pix = i / ncv;
    const int ww = (int)(pix % W); pix /= W;
    const int h = (int)(pix % H);
    const int n = (int)(pix / H);
    const int ph = h + pad, qw = ww + pad, r0 = ph & 1, s0 = qw & 1;
    float acc[8];
    if (accumulate) IO<T>::ld(dx + i * 8, acc);
    else {
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    }
    typename BufIO<T>::Raw raw[HK * HK];
#pragma unroll
    for (int a = 0; a < HK; ++a)
#pragma unroll
      for (int b = 0; b < HK; ++b) {
        const int r = r0 + 2 * a, s = s0 + 2 * b;
        const int p = (ph - r) >> 1, q = (qw - s) >> 1;
        const bool ok = r < K && s < K && (unsigned)p < (unsigned)P && (unsigned)q < (unsigned)Q;
        raw[a * HK + b] = BufIO<T>::issue(dr, (unsigned)(((n * P + p) * Q + q) * ncv + cv) * 8u, ok);
      }
#pragma unroll
    for (int a = 0; a < HK; ++a)
#pragma unroll
      for (int b = 0; b < HK; ++b) {
        const int r = min(r0 + 2 * a, K - 1), s = min(s0 + 2 * b, K - 1);   // clamped taps carry zeros
        float d[8], f[8];
        BufIO<T>::unpack(raw[a * HK + b], d);
        IO<T>::ld(w + ((long)(r * K + s) * ncv + cv) * 8, f);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = fmaf(d[e], f[e], acc[e]);
      }
    IO<T>::st(dx + i * 8, acc);
  }
}
template <class T, int K>
__global__ __launch_bounds__(256) void dw_dgrad_s2_kernel(const T* __restrict__ dy, const T* __restrict__ w,
    T* __restrict__ dx, int N, int H, int W, int P, int Q, int ncv, int pad, int accumulate, unsigned dy_elems) {
  dw_dgrad_s2_block<T, K>(one_block(), dy, w, dx, N, H, W, P, Q, ncv, pad, accumulate, dy_elems);
}

// dW[r][t][c] = sum over output pixels dY * X(shifted).  ROWS tap rows per block: 3x3 filters keep all
// 9 x 8 accumulators in registers and read dY / X once; larger filters take one tap row per
// blockIdx.z (grid = (slabs, chunks, k / ROWS)).  All taps of a pixel are requested before use.
template <class T, int KMAX, int ROWS>
__device__ __forceinline__ void dw_wgrad_block(const Blk& blk, const T* __restrict__ dy, const T* __restrict__ x,
                                                       float* __restrict__ part, int N, int H, int W,
                                                       int P, int Q, int Cp, int k, int stride, int pad,
                                                       ColGrid g, unsigned x_elems) {
  extern __shared__ float smem[];
  const int ncv = Cp / 8;
  const int cv_lane = threadIdx.x % g.cvl, row_lane = threadIdx.x / g.cvl, rl = 256 / g.cvl;
  const int cv = blk.x * g.cvl + cv_lane;
  const int rbase = blk.z * ROWS;
  const long M = (long)N * P * Q;
  const long r0 = blk.y * g.rows_per_chunk;
  const long r1 = min(M, r0 + g.rows_per_chunk);
  const __amdgpu_buffer_rsrc_t xr = tensor_rsrc(x, x_elems * (unsigned)sizeof(T));
  float acc[ROWS][KMAX * 8];
#pragma unroll
  for (int a = 0; a < ROWS; ++a)
#pragma unroll
    for (int t = 0; t < KMAX * 8; ++t) acc[a][t] = 0.f;
  if (cv < ncv && row_lane < rl && r0 + row_lane < r1) {
    // (n, p, q) of this thread's first row, then advanced by rl rows per step without divisions
    long pix = r0 + row_lane;
    int q = (int)(pix % Q); pix /= Q;
    int p = (int)(pix % P);
    int n = (int)(pix / P);
    const int dq = rl % Q, dp = (rl / Q) % P, dn = rl / (Q * P);
    for (long m = r0 + row_lane; m < r1; m += rl) {
      typename BufIO<T>::Raw raw[ROWS][KMAX];
#pragma unroll
      for (int a = 0; a < ROWS; ++a)
#pragma unroll
        for (int t = 0; t < KMAX; ++t) {
          const int h = p * stride + rbase + a - pad, ww = q * stride + t - pad;
          const bool ok = rbase + a < k && t < k && (unsigned)h < (unsigned)H && (unsigned)ww < (unsigned)W;
          raw[a][t] = BufIO<T>::issue(xr, (unsigned)(((n * H + h) * W + ww) * ncv + cv) * 8u, ok);
        }
      float d[8];
      IO<T>::ld(dy + (m * ncv + cv) * 8, d);
#pragma unroll
      for (int a = 0; a < ROWS; ++a)
#pragma unroll
        for (int t = 0; t < KMAX; ++t) {
          float v[8];
          BufIO<T>::unpack(raw[a][t], v);
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[a][t * 8 + e] = fmaf(d[e], v[e], acc[a][t * 8 + e]);
        }
      q += dq;
      if (q >= Q) { q -= Q; ++p; }
      p += dp;
      if (p >= P) { p -= P; ++n; }
      n += dn;
    }
  }
  // tree reduction over the row lanes, one tap row (KMAX x 8 values) at a time
#pragma unroll
  for (int a = 0; a < ROWS; ++a) {
    if (rbase + a >= k) continue;   // uniform over the block
    float out[KMAX * 8];
    bool owner;
    block_col_reduce<KMAX * 8>(acc[a], smem, g.cvl, cv_lane, row_lane, out, owner);
    if (owner && cv < ncv) {
#pragma unroll
      for (int t = 0; t < KMAX; ++t) {
        if (t >= k) continue;
        float* pp = part + ((long)blk.y * k * k + (rbase + a) * k + t) * Cp + cv * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) pp[e] = out[t * 8 + e];
      }
    }
  }
}
template <class T, int KMAX, int ROWS>
__global__ __launch_bounds__(256) void dw_wgrad_kernel(const T* __restrict__ dy,
    const T* __restrict__ x, float* __restrict__ part, int N, int H, int W, int P, int Q, int Cp, int k, int stride, int pad, ColGrid g,
    unsigned x_elems) {
  dw_wgrad_block<T, KMAX, ROWS>(one_block(), dy, x, part, N, H, W, P, Q, Cp, k, stride, pad, g, x_elems);
}

}  // namespace pbd
