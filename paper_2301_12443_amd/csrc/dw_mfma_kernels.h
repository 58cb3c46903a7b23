// Depthwise convolutions (bf16, stride 1, 3 x 3 / 5 x 5 / 7 x 7) on the matrix cores.
//
// v_mfma_f32_4x4x4_16b_bf16 multiplies sixteen independent 4 x 4 matrices in 8 cycles: one per channel.  A row of a
// depthwise filter applied to a run of pixels is a product with a banded (Toeplitz) matrix,
//   out[n] = sum_k T[n][k] x[k],  T[n][k] = w[k - n],   n = 0..3 output columns,  k = 0..3 of a quad of input columns,
// so four output columns meet K + 3 input columns in NT = ceil((K + 3) / 4) products per filter row: 28 of 48
// multiply-adds are real at K = 7, 20 of 32 at K = 5, 12 of 32 at K = 3, at 128 multiply-adds a cycle and SIMD against
// 16 of the vector ALUs.  Products of bf16 numbers are exact in float32 and sums are kept there, as in the kernels on the
// vector ALUs.
//  A tap outside the filter is a product with zero, which an infinity or NaN among the inputs turns into NaN, up to three columns
// further than the filter reaches.  The forward pass of a layer whose normalisation is folded in (the frozen teacher's, with
// running statistics) therefore forms every result that came out as NaN once more from the filter's own taps.  In a student's
// layer the value goes into the batch statistics, and the whole channel is NaN either way; so is, in its backward pass, the
// gradient of the whole channel.
//
// Layout.  An operand lane holds four consecutive pixels of ONE channel, so tiles lie in LDS channel by channel,
// [channel][row][column]; the 4 pixels x 8 channels that a thread loads (four 16-byte chunks) are transposed in
// registers on their way there (16 byte permutes per 32 elements).  Pitches (bytes): CHP = 8 odd, ROWP so that
// the 16 lanes of an LDS cycle (4 channels x 4 row strips) hit 16 different 8-byte banks.
// A workgroup of four waves owns 16 x 16 outputs x 32 channels: wave = (16 channels) x (8 of 16 columns).  Lane
// 4 c + j of the data operand is channel c and row strip j (output rows 4 j .. 4 j + 3), so one 8-byte LDS read of input row
// 4 j + y serves every (output row, filter row) pair with the sum y: 40 reads for 168 products at K = 7.
#pragma once
#include "conv_kernels.h"

namespace pbd {

constexpr int kDwTile = 16;           // output rows and columns of a tile
constexpr int kDwCh = 32;             // channels of a workgroup

typedef short dw_s16x4 __attribute__((ext_vector_type(4)));
typedef float dw_f32x4 __attribute__((ext_vector_type(4)));

template <int K> struct DwGeom {
  static constexpr int IN = kDwTile + K - 1;            // input rows and columns behind a tile
  static constexpr int NQ = (IN + 3) / 4;               // quads of input columns
  static constexpr int NT = (K + 6) / 4;                // quads that four output columns meet
  static constexpr int ROWP = K == 7 ? 56 : 40;         // bytes per row of a channel: 4 ROWP = 32 odd (mod 128)
  static constexpr int CHP = (IN * ROWP + 31) / 32 * 32 + 8;   // bytes per channel: 8 (mod 32)
  static constexpr int ITEMS = IN * NQ * (kDwCh / 8);   // 4 pixels x 8 channels each
  static constexpr int NLOAD = (ITEMS + 255) / 256;
  static constexpr int WROW = K == 3 ? 8 : 16;          // bytes of a filter row in LDS
};
constexpr int kDwOutP = kDwCh * 2 + 16;                 // staged output: bytes per pixel ...
constexpr int kDwOutRow = kDwTile * kDwOutP + 16;       // ... and per row of 16

__device__ __forceinline__ unsigned dw_lo2(unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }  // low halves
__device__ __forceinline__ unsigned dw_hi2(unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }  // high halves
// A lane's shift by n = 0..3 elements over a run of element pairs: whole pairs by a bit-wise select on all-ones or
// all-zeros (n >= 2), the odd element by a byte permute with the lane's own selector.  (Written as conditional expressions
// on the run's elements the compiler keeps the run in scratch memory and indexes it.)
__device__ __forceinline__ unsigned dw_sel(unsigned mask, unsigned set, unsigned clear) { return (set & mask) | (clear & ~mask); }
constexpr unsigned kDwSelLow = 0x03020100u, kDwSelMid = 0x05040302u, kDwSelHigh = 0x07060504u;   // lo | lo.hi, hi.lo | hi

// the four 16-byte chunks (8 channels) of four neighbouring pixels -> eight channels of four pixels, CH_PITCH bytes apart
template <int CH_PITCH>
__device__ __forceinline__ void dw_store_transposed(unsigned char* dst, const uint4 (&p)[4]) {
  const unsigned a[4][4] = {{p[0].x, p[0].y, p[0].z, p[0].w}, {p[1].x, p[1].y, p[1].z, p[1].w},
                            {p[2].x, p[2].y, p[2].z, p[2].w}, {p[3].x, p[3].y, p[3].z, p[3].w}};
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    *reinterpret_cast<uint2*>(dst + (2 * m) * CH_PITCH) = make_uint2(dw_lo2(a[0][m], a[1][m]), dw_lo2(a[2][m], a[3][m]));
    *reinterpret_cast<uint2*>(dst + (2 * m + 1) * CH_PITCH) = make_uint2(dw_hi2(a[0][m], a[1][m]), dw_hi2(a[2][m], a[3][m]));
  }
}

// The producer's batch norm and rectifier, applied to what a kernel stages (FOLD): the input is then the producing layer's
// convolution output y, and the normalised tensor z = act((y - mean) * (gamma * invstd) + beta) is neither written nor read.  The
// arithmetic and the rounding are bn_apply_kernel's, so every value is what it would have stored; pixels outside the image
// stay zero.  ~45 vector operations per 8 channels and pixel (halo included) beside matrix instructions that leave the vector
// ALUs idle.
struct DwFold { float mu[kDwCh], a[kDwCh], b[kDwCh]; };
__device__ __forceinline__ void dw_fold_load(DwFold& f, const NormFold& fold, int c0, int C, int tid) {
  if (tid < kDwCh) {
    const int c = c0 + tid;
    const bool in = c < C;
    f.mu[tid] = in ? fold.mean[c] : 0.f;
    f.a[tid] = in ? fold.gamma[c] * fold.invstd[c] : 0.f;
    f.b[tid] = in ? fold.beta[c] : 0.f;
  }
}
// p: four pixels x 8 channels as loaded; bit i of ok: pixel i lies in the image.  ReLU or ReLU6 (hi = infinity or 6)
__device__ __forceinline__ void dw_fold_apply(uint4 (&p)[4], const DwFold& f, int c8, unsigned ok, float hi) {
  float mu[8], a[8], b[8];
#pragma unroll
  for (int e = 0; e < 8; e += 4) {
    const float4 m4 = *reinterpret_cast<const float4*>(f.mu + c8 + e), a4 = *reinterpret_cast<const float4*>(f.a + c8 + e),
                 b4 = *reinterpret_cast<const float4*>(f.b + c8 + e);
    mu[e] = m4.x; mu[e + 1] = m4.y; mu[e + 2] = m4.z; mu[e + 3] = m4.w;
    a[e] = a4.x; a[e + 1] = a4.y; a[e + 2] = a4.z; a[e + 3] = a4.w;
    b[e] = b4.x; b[e + 1] = b4.y; b[e + 2] = b4.z; b[e + 3] = b4.w;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float v[8];
    IO<bf16_t>::unpack(p[i], v);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = fminf(fmaxf(fmaf(v[e] - mu[e], a[e], b[e]), 0.f), hi);
    const bool in = (ok >> i) & 1u;
    p[i] = in ? make_uint4(pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7])) : make_uint4(0u, 0u, 0u, 0u);
  }
}

// Work items: (tile, channel group), group fastest (neighbouring groups share the 128-byte lines of a pixel), a
// workgroup takes `per_block` tiles of one group one after the other (its filters stay in registers).
struct DwArgs {
  int N, H, W, ncv;             // images, height, width, 8-channel vectors
  int tiles_h, tiles_w, tiles;  // tiles = N * tiles_h * tiles_w
  int groups, per_block;        // channel groups, tiles per workgroup
  unsigned bytes;               // of the input tensor (and of the output: the shapes agree at stride 1)
  float* stats;                 // forward, STATS: [2 x chunks][3][8 ncv] mean, sum of squares about it, pixels
  int P, Q;                     // stride 2: height, width and bytes of dy (tiles are counted over it)
  unsigned dy_bytes;
};

// y = x * w (FLIP: mirrored filter, the backward-data pass of the same layer), optionally a folded batch norm and
// activation behind it.
// Bound by the latency of load - stage - multiply - stage - store at three to four workgroups per compute unit (no unit is
// busy all the time).  Launch averages over the supernet step (batch 64) against a tile kernel on the vector ALUs: backward-data
// 7 x 7 72 -> 34 us, 5 x 5 41 -> 24, 3 x 3 26 -> 20; forward with FOLD and STATS, two passes over the tensor less beside it,
// 73 -> 44, 41 -> 34, 25 -> 31 (MobileNetV2's teacher at batch 33, plain 3 x 3 forward: 11.1 -> 8.5).
// Stores go through the caches whatever the tensor's size: a workgroup writes 64 of the 128 bytes of a line, its neighbour the
// others, and past the caches the halves reach memory one by one (128 x 56 x 56 x 144, 3 x 3: backward-data 97 us nontemporal, 60
// through the caches; 128 x 40 x 40 x 384, 7 x 7 120 and 111; the supernet step 41.21 and 41.03 ms).
// Slower: the next tile's loads in flight behind the products (K = 7 40 us, K = 5 31: the registers cost a workgroup per
// compute unit); 64 channels a workgroup (K = 5 31 us, batch 33 12.6 against 11.4).
// ACC (backward-data into a value that already has a gradient): the result is added to what dst holds, in float32, and rounded
// once.  What dst holds is loaded ahead of the products and passes through LDS the way the result does.
template <int K, bool FLIP, bool FOLD, bool STATS, bool ACC>
__device__ __forceinline__ void dw_mfma_block(const Blk& blk, const bf16_t* __restrict__ x, const bf16_t* __restrict__ w,
                                                         bf16_t* __restrict__ dst, const float* __restrict__ a,
                                                         const float* __restrict__ b, int act, DwArgs g, NormFold fold) {
  typedef DwGeom<K> G;
  constexpr int NT = G::NT, pad = K / 2;
  constexpr int LDS = G::CHP * kDwCh > kDwOutRow * kDwTile ? G::CHP * kDwCh : kDwOutRow * kDwTile;
  static_assert(kDwCh * K * G::WROW <= LDS, "the filters fit where the tile goes");
  __shared__ __attribute__((aligned(16))) unsigned char smem[LDS];
  __shared__ __attribute__((aligned(16))) DwFold folded;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slice = wave & 1, half = wave >> 1;
  const int wg = xcd_contiguous(blk.x, blk.gx);
  const int cv0 = (wg % g.groups) * (kDwCh / 8);
  const int tile_begin = (wg / g.groups) * g.per_block, tile_end = min(g.tiles, tile_begin + g.per_block);
  const __amdgpu_buffer_rsrc_t xr = tensor_rsrc(x, g.bytes);
  const int ch = slice * 16 + (lane >> 2), strip = lane & 3;         // (strip: also this lane's output column of the filter operand)

  if (FOLD) dw_fold_load(folded, fold, cv0 * 8, g.ncv * 8, tid);
  const float hi = fold.act == ACT_RELU6 ? 6.f : __builtin_inff();
  // ---- filters: [channel][filter row][tap] in LDS, then each lane's Toeplitz rows into registers ----
  for (int i = tid; i < K * K * (kDwCh / 2); i += 256) {
    const int tap = i / (kDwCh / 2), c2 = i % (kDwCh / 2);
    const int t = FLIP ? K * K - 1 - tap : tap;
    unsigned v = 0;
    if (cv0 * 8 + 2 * c2 < g.ncv * 8) v = *reinterpret_cast<const unsigned*>(w + (size_t)tap * g.ncv * 8 + cv0 * 8 + 2 * c2);
    unsigned short* p = reinterpret_cast<unsigned short*>(smem + (2 * c2 * K + t / K) * G::WROW) + t % K;
    p[0] = (unsigned short)v;
    p[K * G::WROW / 2] = (unsigned short)(v >> 16);
  }
  __syncthreads();
  const unsigned far = strip >= 2 ? ~0u : 0u, odd = strip & 1 ? kDwSelMid : kDwSelHigh;
  dw_s16x4 wt[K][NT];
#pragma unroll
  for (int r = 0; r < K; ++r) {
    // element pairs P[-2 .. 2 NT - 1] of the filter row with zeros around it
    unsigned P[2 * NT + 2];
#pragma unroll
    for (int i = 0; i < 2 * NT + 2; ++i) P[i] = 0u;
    const unsigned char* row = smem + (ch * K + r) * G::WROW;
    const uint2 q0 = *reinterpret_cast<const uint2*>(row);
    P[2] = q0.x; P[3] = K == 3 ? q0.y & 0xffffu : q0.y;              // (the last tap's partner was never written)
    if (K > 3) {
      const uint2 q1 = *reinterpret_cast<const uint2*>(row + 8);
      P[4] = K == 5 ? q1.x & 0xffffu : q1.x;
      if (K > 5) P[5] = q1.y & 0xffffu;
    }
    // T[n][k] of quad t = tap 4 t + k - n, n = this lane's column: two pairs further back for n >= 2, half a pair for odd n
    unsigned E[2 * NT + 1];
#pragma unroll
    for (int i = 0; i < 2 * NT + 1; ++i) E[i] = dw_sel(far, P[i], P[i + 1]);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const unsigned d0 = __builtin_amdgcn_perm(E[2 * t + 1], E[2 * t], odd);
      const unsigned d1 = __builtin_amdgcn_perm(E[2 * t + 2], E[2 * t + 1], odd);
      wt[r][t] = __builtin_bit_cast(dw_s16x4, make_uint2(d0, d1));
    }
  }
  float ea = 1.f, eb = 0.f;
  if (a && cv0 * 8 + ch < g.ncv * 8) { ea = a[cv0 * 8 + ch]; eb = b[cv0 * 8 + ch]; }
  // STATS: this lane's sums of (y - pivot) and (y - pivot)^2 over the stored outputs of its channel, the pivot being the wave's first
  // output of the channel that lies in the image (no cancellation when |mean| is far above the deviation)
  float pivot = 0.f, s1 = 0.f, s2 = 0.f, cnt = 0.f;
  bool pivoted = false;                                  // (the same for the whole wave)

  for (int tile = tile_begin; tile < tile_end; ++tile) {
    int t_ = tile;
    const int tw = t_ % g.tiles_w; t_ /= g.tiles_w;
    const int th = t_ % g.tiles_h, n = t_ / g.tiles_h;
    const int h0 = th * kDwTile, w0 = tw * kDwTile;
    // ---- the tile's input, all loads in flight together ----
    uint4 raw[G::NLOAD][4];
    unsigned ok = 0;                                     // bit 4 i + p: pixel p of item i lies in the image
#pragma unroll
    for (int i = 0; i < G::NLOAD; ++i) {
      const int c = tid + i * 256;
      const int cvl = c % (kDwCh / 8), quad = (c / (kDwCh / 8)) % G::NQ, row = c / (kDwCh / 8) / G::NQ;
      const int h = h0 - pad + row, w_ = w0 - pad + 4 * quad;
      const bool rok = c < G::ITEMS && (unsigned)h < (unsigned)g.H && cv0 + cvl < g.ncv;
      const unsigned off = (unsigned)(((n * g.H + h) * g.W + w_) * g.ncv + cv0 + cvl) * 16u;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const bool in = rok && 4 * quad + p < G::IN && (unsigned)(w_ + p) < (unsigned)g.W;
        raw[i][p] = buffer_load16(xr, in ? off + (unsigned)(p * g.ncv) * 16u : kOutOfRange);
        if (FOLD) ok |= (in ? 1u : 0u) << (4 * i + p);
      }
    }
    __syncthreads();                                     // the previous tile (or the filters) has been read
#pragma unroll
    for (int i = 0; i < G::NLOAD; ++i) {
      const int c = tid + i * 256;
      const int cvl = c % (kDwCh / 8), quad = (c / (kDwCh / 8)) % G::NQ, row = c / (kDwCh / 8) / G::NQ;
      if (FOLD) dw_fold_apply(raw[i], folded, cvl * 8, ok >> (4 * i), hi);
      if (c < G::ITEMS) dw_store_transposed<G::CHP>(smem + cvl * 8 * G::CHP + row * G::ROWP + quad * 8, raw[i]);
    }
    __syncthreads();

    // this thread's chunks of the output: 8 channels of a pixel each
    constexpr int NOUT = kDwTile * kDwTile * (kDwCh / 8) / 256;
    auto chunk = [&](int i, int& at, size_t& out) {      // its place in LDS and in dst; whether it lies in the image
      const int c = tid + i * 256;
      const int cvl = c % (kDwCh / 8), col = (c / (kDwCh / 8)) % kDwTile, row = c / (kDwCh / 8) / kDwTile;
      const int h = h0 + row, w_ = w0 + col;
      at = row * kDwOutRow + col * kDwOutP + cvl * 16;
      out = ((((size_t)n * g.H + h) * g.W + w_) * g.ncv + cv0 + cvl) * 8;
      return h < g.H && w_ < g.W && cv0 + cvl < g.ncv;
    };
    uint4 old[ACC ? NOUT : 1];
    if constexpr (ACC) {
#pragma unroll
      for (int i = 0; i < NOUT; ++i) {
        int at; size_t out;
        old[i] = chunk(i, at, out) ? *reinterpret_cast<const uint4*>(dst + out) : make_uint4(0u, 0u, 0u, 0u);
      }
    }

    // ---- products: acc[rho][q] = output rows 4 strip + rho, output columns 8 half + 4 q + 0..3 ----
    dw_f32x4 acc[4][2];
#pragma unroll
    for (int o = 0; o < 4; ++o)
#pragma unroll
      for (int q = 0; q < 2; ++q) acc[o][q] = dw_f32x4{0.f, 0.f, 0.f, 0.f};
    const unsigned char* in = smem + ch * G::CHP + 4 * strip * G::ROWP + half * 16;
#pragma unroll
    for (int c = 0; c < NT + 1; ++c)
#pragma unroll
      for (int y = 0; y < K + 3; ++y) {
        const dw_s16x4 d = *reinterpret_cast<const dw_s16x4*>(in + y * G::ROWP + c * 8);
#pragma unroll
        for (int o = 0; o < 4; ++o) {
          const int r = y - o;
          if (r < 0 || r >= K) continue;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int t = c - q;
            if (t < 0 || t >= NT) continue;
            acc[o][q] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(wt[r][t], d, acc[o][q], 0, 0, 0);
          }
        }
      }

    if constexpr (!FLIP && !FOLD && !STATS) {
      float s = 0.f;                                     // NaN if any of them is (or infinities cancel)
#pragma unroll
      for (int o = 0; o < 4; ++o)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int m = 0; m < 4; ++m) s += acc[o][q][m];
      if (s != s && cv0 * 8 + ch < g.ncv * 8) {
#pragma unroll
        for (int o = 0; o < 4; ++o)
#pragma unroll
          for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
              if (acc[o][q][m] == acc[o][q][m]) continue;
              float v = 0.f;
#pragma unroll 1
              for (int i = 0; i < K * K; ++i) {
                const int r = i / K, t = i % K;
                v = fmaf((float)*reinterpret_cast<const bf16_t*>(in + (o + r) * G::ROWP + (4 * q + m + t) * 2),
                         (float)w[(size_t)i * g.ncv * 8 + cv0 * 8 + ch], v);
              }
              acc[o][q][m] = v;
            }
      }
    }

    // ---- output through LDS: pixel-major, then 16-byte stores ----
    if (a) {                                             // folded inference-mode BN + activation (teacher)
#pragma unroll
      for (int o = 0; o < 4; ++o)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int m = 0; m < 4; ++m) acc[o][q][m] = apply_act(fmaf(acc[o][q][m], ea, eb), act);
    }
    if (STATS) {
      const int rows = min(4, g.H - h0 - 4 * strip);     // of this lane's outputs (none or negative: below the image)
      const int cols = min(8, g.W - w0 - half * 8);      // (the same for the whole wave; none where a row's last tile ends in the left half)
      if (!pivoted && cols > 0) {
        pivot = as_stored<bf16_t>(__shfl(acc[0][0][0], lane & ~3, 64));
        pivoted = true;
      }
#pragma unroll
      for (int o = 0; o < 4; ++o) {
        const bool row_in = o < rows;
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            const float v = as_stored<bf16_t>(acc[o][q][m]) - pivot;
            const float d = row_in && q * 4 + m < cols ? v : 0.f;
            s1 += d;
            s2 = fmaf(d, d, s2);
          }
        __builtin_amdgcn_sched_barrier(0);               // (one row's temporaries at a time)
      }
      cnt += (float)(max(rows, 0) * max(cols, 0));
    }
    __syncthreads();                                     // every wave has read the input tile
    if constexpr (ACC) {
#pragma unroll
      for (int i = 0; i < NOUT; ++i) {
        int at; size_t out;
        chunk(i, at, out);
        *reinterpret_cast<uint4*>(smem + at) = old[i];
      }
      __syncthreads();
    }
    // lanes 4 apart hold neighbouring channels: the even channel packs columns 0 and 1 of both, the odd one columns 2 and 3
    unsigned char* so = smem + (ch >> 1) * 4 + ((ch & 1) * 2 + half * 8) * kDwOutP;
#pragma unroll
    for (int o = 0; o < 4; ++o)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const int v0 = __float_as_int(acc[o][q][m]), v2 = __float_as_int(acc[o][q][m + 2]);
          const int lo = __builtin_amdgcn_update_dpp(v0, v2, 0x114, 0xf, 0xa, false);   // row_shr:4 into the odd channels
          const int hi = __builtin_amdgcn_update_dpp(v2, v0, 0x104, 0xf, 0x5, false);   // row_shl:4 into the even channels
          unsigned* slot = reinterpret_cast<unsigned*>(so + (4 * strip + o) * kDwOutRow + (q * 4 + m) * kDwOutP);
          if constexpr (ACC) *slot = pack_bf2(__int_as_float(lo) + bf_lo(*slot), __int_as_float(hi) + bf_hi(*slot));
          else *slot = pack_bf2(__int_as_float(lo), __int_as_float(hi));
        }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NOUT; ++i) {
      int at; size_t out;
      if (!chunk(i, at, out)) continue;
      *reinterpret_cast<uint4*>(dst + out) = *reinterpret_cast<const uint4*>(smem + at);
    }
  }
  if (STATS) {
#pragma unroll
    for (int off = 1; off < 4; off <<= 1) {              // the four row strips of a channel
      s1 += __shfl_xor(s1, off, 64);
      s2 += __shfl_xor(s2, off, 64);
      cnt += __shfl_xor(cnt, off, 64);
    }
    if (strip == 0 && cv0 * 8 + ch < g.ncv * 8) {
      const float shift = cnt > 0.f ? s1 / cnt : 0.f;
      float* p = g.stats + (size_t)((wg / g.groups) * 2 + half) * 3 * (g.ncv * 8) + cv0 * 8 + ch;
      p[0] = pivot + shift;
      p[g.ncv * 8] = fmaxf(s2 - s1 * shift, 0.f);
      p[2 * g.ncv * 8] = cnt;
    }
  }
}
template <int K, bool FLIP, bool FOLD = false, bool STATS = false, bool ACC = false>
__global__ __launch_bounds__(256, K == 7 || ACC ? 3 : 4) void dw_mfma_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ w, bf16_t* __restrict__ dst, const float* __restrict__ a,
    const float* __restrict__ b, int act, DwArgs g, NormFold fold) {
  dw_mfma_block<K, FLIP, FOLD, STATS, ACC>(one_block(), x, w, dst, a, b, act, g, fold);
}

// Backward-weight of the same layers: dW[r][s] = sum over pixels of x[p + r][q + s] dy[p][q], per channel.
// A product takes four neighbouring columns of one input row: A[i][k] = x[y][4 c + i + k] (s = i + 4 it: the four lanes of a
// channel read the same quads and shift them by their own i), B[k][j] = dy[y - j - 4 jt][4 c + k] (r = j + 4 jt), so
// D[i][j] accumulates filter tap (r, s): 49 of 64 multiply-adds are real at K = 7, 25 of 64 at K = 5, 9 of 16 at K = 3, and
// x and dy are read once for all taps.  A shifted quad of x meets dy's quads c (it = 0) and c - 1 (it = 1).  Rows of dy
// outside the tile are a row of zeros.  A workgroup walks per_block tiles with its accumulators in registers; the two
// column halves meet in LDS at the end; one partial result per workgroup as in the other kernels.  Bound by the shifts and
// LDS reads.  Launch averages over the supernet step, with FOLD, against a tile kernel on the vector ALUs that read the
// normalised tensor: 7 x 7 91 -> 47 us, 5 x 5 72 -> 41, 3 x 3 37 -> 32.
template <int K, bool FOLD>
__device__ __forceinline__ void dw_wgrad_mfma_block(const Blk& blk, const bf16_t* __restrict__ dy, const bf16_t* __restrict__ x,
                                                               float* __restrict__ part, DwArgs g, NormFold fold) {
  typedef DwGeom<K> G;
  constexpr int pad = K / 2, NIT = K == 3 ? 1 : 2, QS = K == 7 ? 1 : 2;    // (QS: accumulators per tap block, one per quad column where registers allow)
  constexpr int ROWX = G::NQ * 8, CHX = (G::IN * ROWX + 31) / 32 * 32 + 8;          // x: rows of whole quads
  constexpr int ROWD = kDwTile * 2, CHD = kDwTile * ROWD + 8;                        // dy: 16 x 16 pixels a channel
  constexpr int ZERO = CHX * kDwCh + CHD * kDwCh;                                    // a row of zeros
  __shared__ __attribute__((aligned(16))) unsigned char smem[ZERO + ROWD];
  __shared__ __attribute__((aligned(16))) DwFold folded;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slice = wave & 1, half = wave >> 1;
  const int wg = xcd_contiguous(blk.x, blk.gx);
  const int cv0 = (wg % g.groups) * (kDwCh / 8), chunk = wg / g.groups;
  const int tile_begin = chunk * g.per_block, tile_end = min(g.tiles, tile_begin + g.per_block);
  const __amdgpu_buffer_rsrc_t xr = tensor_rsrc(x, g.bytes), dr = tensor_rsrc(dy, g.bytes);
  const int ch = slice * 16 + (lane >> 2), n4 = lane & 3;             // n4: s offset of the x operand, r offset of the dy operand
  const unsigned far = n4 >= 2 ? ~0u : 0u, odd = n4 & 1 ? kDwSelMid : kDwSelLow;
  if (tid < ROWD / 8) *reinterpret_cast<uint2*>(smem + ZERO + tid * 8) = make_uint2(0u, 0u);

  dw_f32x4 sum[NIT][NIT];                                // over the tiles, each summed on its own first (shorter chains of additions)
#pragma unroll
  for (int i = 0; i < NIT; ++i)
#pragma unroll
    for (int j = 0; j < NIT; ++j) sum[i][j] = dw_f32x4{0.f, 0.f, 0.f, 0.f};

  if (FOLD) dw_fold_load(folded, fold, cv0 * 8, g.ncv * 8, tid);     // (visible behind the first tile's barrier)
  const float hi = fold.act == ACT_RELU6 ? 6.f : __builtin_inff();
  uint4 rx[G::NLOAD][4], rd[4];
  unsigned ok = 0;                                       // bit 4 i + p: pixel p of item i of rx lies in the image
  auto load_tile = [&](int tile) {
    ok = 0;
    int t_ = tile;
    const int tw = t_ % g.tiles_w; t_ /= g.tiles_w;
    const int th = t_ % g.tiles_h, n = t_ / g.tiles_h;
    const int h0 = th * kDwTile, w0 = tw * kDwTile;
#pragma unroll
    for (int i = 0; i < G::NLOAD; ++i) {
      const int c = tid + i * 256;
      const int cvl = c % (kDwCh / 8), quad = (c / (kDwCh / 8)) % G::NQ, row = c / (kDwCh / 8) / G::NQ;
      const int h = h0 - pad + row, w_ = w0 - pad + 4 * quad;
      const bool rok = c < G::ITEMS && (unsigned)h < (unsigned)g.H && cv0 + cvl < g.ncv;
      const unsigned off = (unsigned)(((n * g.H + h) * g.W + w_) * g.ncv + cv0 + cvl) * 16u;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const bool in = rok && 4 * quad + p < G::IN && (unsigned)(w_ + p) < (unsigned)g.W;
        rx[i][p] = buffer_load16(xr, in ? off + (unsigned)(p * g.ncv) * 16u : kOutOfRange);
        if (FOLD) ok |= (in ? 1u : 0u) << (4 * i + p);
      }
    }
    const int cvl = tid % (kDwCh / 8), quad = (tid / (kDwCh / 8)) % 4, drow = tid / (kDwCh / 8) / 4;
    const int h = h0 + drow, w_ = w0 + 4 * quad;
    const unsigned off = (unsigned)(((n * g.H + h) * g.W + w_) * g.ncv + cv0 + cvl) * 16u;
#pragma unroll
    for (int p = 0; p < 4; ++p)
      rd[p] = buffer_load16(dr, h < g.H && w_ + p < g.W && cv0 + cvl < g.ncv ? off + (unsigned)(p * g.ncv) * 16u : kOutOfRange);
  };

  if (tile_begin < tile_end) load_tile(tile_begin);
  for (int tile = tile_begin; tile < tile_end; ++tile) {
    __syncthreads();                                     // the previous tile has been read
#pragma unroll
    for (int i = 0; i < G::NLOAD; ++i) {
      const int c = tid + i * 256;
      const int cvl = c % (kDwCh / 8), quad = (c / (kDwCh / 8)) % G::NQ, row = c / (kDwCh / 8) / G::NQ;
      if (FOLD) dw_fold_apply(rx[i], folded, cvl * 8, ok >> (4 * i), hi);
      if (c < G::ITEMS) dw_store_transposed<CHX>(smem + cvl * 8 * CHX + row * ROWX + quad * 8, rx[i]);
    }
    dw_store_transposed<CHD>(smem + CHX * kDwCh + (tid % (kDwCh / 8)) * 8 * CHD + (tid / (kDwCh / 8) / 4) * ROWD + ((tid / (kDwCh / 8)) % 4) * 8, rd);
    __syncthreads();
    if (tile + 1 < tile_end) load_tile(tile + 1);        // in flight behind this tile's products

    const unsigned char* xp = smem + ch * CHX + half * 16;
    const unsigned char* dp = smem + CHX * kDwCh + ch * CHD + half * 16;
    const unsigned char* zp = smem + ZERO + half * 16;
    dw_f32x4 acc[NIT][NIT][QS];
#pragma unroll
    for (int i = 0; i < NIT; ++i)
#pragma unroll
      for (int j = 0; j < NIT; ++j)
#pragma unroll
        for (int q = 0; q < QS; ++q) acc[i][j][q] = dw_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
    for (int y = 0; y < G::IN; ++y) {
      const unsigned char* db[NIT];
#pragma unroll
      for (int jt = 0; jt < NIT; ++jt) {
        const int row = y - n4 - 4 * jt;
        db[jt] = (unsigned)row < (unsigned)kDwTile ? dp + row * ROWD : zp;
      }
      dw_s16x4 d[NIT][2];
#pragma unroll
      for (int jt = 0; jt < NIT; ++jt)
#pragma unroll
        for (int q = 0; q < 2; ++q) d[jt][q] = *reinterpret_cast<const dw_s16x4*>(db[jt] + q * 8);
      // the shifted quads of the input row: c = 0 .. NIT of this half (two quads of dy each)
      uint2 xq[NIT + 2];
#pragma unroll
      for (int c = 0; c < NIT + 2; ++c) xq[c] = *reinterpret_cast<const uint2*>(xp + y * ROWX + c * 8);
      unsigned D[2 * (NIT + 2)];
#pragma unroll
      for (int c = 0; c < NIT + 2; ++c) { D[2 * c] = xq[c].x; D[2 * c + 1] = xq[c].y; }
      unsigned E[2 * (NIT + 1) + 1];
#pragma unroll
      for (int i = 0; i < 2 * (NIT + 1) + 1; ++i) E[i] = dw_sel(far, D[i + 1], D[i]);
#pragma unroll
      for (int c = 0; c < NIT + 1; ++c) {
        const unsigned s0 = __builtin_amdgcn_perm(E[2 * c + 1], E[2 * c], odd);
        const unsigned s1 = __builtin_amdgcn_perm(E[2 * c + 2], E[2 * c + 1], odd);
        const dw_s16x4 xs = __builtin_bit_cast(dw_s16x4, make_uint2(s0, s1));
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
          const int q = c - it;
          if (q < 0 || q > 1) continue;
#pragma unroll
          for (int jt = 0; jt < NIT; ++jt)
            acc[it][jt][q % QS] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(xs, d[jt][q], acc[it][jt][q % QS], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < NIT; ++i)
#pragma unroll
      for (int j = 0; j < NIT; ++j) sum[i][j] += QS == 2 ? acc[i][j][0] + acc[i][j][QS - 1] : acc[i][j][0];
  }
  // ---- the two column halves of a slice meet in LDS; lane 4 c + j holds taps (r = 4 jt + j, s = 4 it + v) of channel c ----
  __syncthreads();
  float* red = reinterpret_cast<float*>(smem);
  if (half) {
#pragma unroll
    for (int it = 0; it < NIT; ++it)
#pragma unroll
      for (int jt = 0; jt < NIT; ++jt)
        *reinterpret_cast<dw_f32x4*>(red + ((slice * NIT * NIT + it * NIT + jt) * 64 + lane) * 4) = sum[it][jt];
  }
  __syncthreads();
  if (half || cv0 * 8 + ch >= g.ncv * 8) return;
#pragma unroll
  for (int it = 0; it < NIT; ++it)
#pragma unroll
    for (int jt = 0; jt < NIT; ++jt) {
      const dw_f32x4 o = *reinterpret_cast<const dw_f32x4*>(red + ((slice * NIT * NIT + it * NIT + jt) * 64 + lane) * 4);
      const int r = 4 * jt + n4;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int s = 4 * it + v;
        if (r < K && s < K) part[((size_t)chunk * K * K + r * K + s) * (g.ncv * 8) + cv0 * 8 + ch] = sum[it][jt][v] + o[v];
      }
    }
}
template <int K, bool FOLD = false>
__global__ __launch_bounds__(256, 3) void dw_wgrad_mfma_kernel(const bf16_t* __restrict__ dy,
    const bf16_t* __restrict__ x, float* __restrict__ part, DwArgs g, NormFold fold) {
  dw_wgrad_mfma_block<K, FOLD>(one_block(), dy, x, part, g, fold);
}

// The whole backward pass of a stride-1 layer between two batch norms, y1 -> z1 = act(bn(y1)) -> y2 = z1 * w -> z2 = act(bn(y2)), in one
// pass over the tensors: reads dz2, y2 (with the filter's halo) and y1, forms dy2 from dz2 and y2 as it stages them (bn_bwd_dy), and from
// that one tile the gradient of z1 (stored), the filter's (one partial result per workgroup) and the two
// sums of y1's batch-norm backward pass (bn_bwd_reduce_kernel's; one pair per workgroup and channel).  As passes of their own these read and
// write the layer's tensor ten times (apply 3, backward-data 2, backward-weight 2, reduce 2, and dy2's halo), here it is four.
// The weight gradient is taken over the pixels p of x = z1 so that x needs no halo and dy2's tile serves both products:
// dW[r][s] = sum over p of x[p] dy2[p + pad - (r, s)], i.e. dw_wgrad_mfma_kernel with the operands' roles changed and the taps mirrored.
// Bound by the vector ALUs (73 % of their cycles at 3 x 3 and 5 x 5, 60 % at 7 x 7, whose tile leaves room for two workgroups a
// compute unit): a third of the instructions form dy2, halo included (1.3, 1.6 and 1.9 elements for one).  Against the passes it replaces,
// 64 x 56 x 56 x 144: 3 x 3 115 -> 76 us, 5 x 5 134 -> 91, 7 x 7 158 -> 134; 64 x 14 x 14 x 384: 33 -> 20, 35 -> 24, 40 -> 31; 128 x 6 x 6 x 960,
// 5 x 5, 77 -> 69; all such layers of a supernet step at batch 64 11.6 -> 7.9 ms.  Tried: the filters' Toeplitz rows held in registers
// (20 of them at 5 x 5, spilled), x shifted by selects instead of by its LDS address (13 instructions a row more).
struct BnBwd { const float* mean; const float* invstd; const float* gamma; const float* beta; const float* k2; const float* k3; int act; };
struct DwBnBwd { float mu[kDwCh], a[kDwCh], b[kDwCh], p[kDwCh], q[kDwCh]; };   // (BnBwdTerms of the channels)
// The last stage of a batch norm's backward pass as every kernel has it that forms dy as it stages it, and bn_bwd_form_kernel, which forms the
// tensor for those who ask for it: dy = a dpre + (p (y - mu) + q), dpre = dz where the activation passes, two roundings an element
// (bn_bwd_apply_kernel: a (dpre - k2 - (y - mu) invstd k3), the same to within their last bits).
struct BnBwdTerms { float mu, a, b, p, q; };
__device__ __forceinline__ BnBwdTerms bn_bwd_terms(const BnBwd& f, int c) {
  const float is = f.invstd[c], a = f.gamma[c] * is;
  return {f.mean[c], a, f.beta[c], -a * (is * f.k3[c]), -a * f.k2[c]};
}
__device__ __forceinline__ float bn_bwd_dy(float yc, float dpre, float a, float p, float q) { return fmaf(a, dpre, fmaf(p, yc, q)); }
__device__ __forceinline__ unsigned dw_word(const uint4& v, int m) { return m == 0 ? v.x : m == 1 ? v.y : m == 2 ? v.z : v.w; }
// all ones where bit i is set (a conditional expression on it becomes a branch around the arithmetic)
__device__ __forceinline__ unsigned dw_bit(unsigned v, int i) { return (unsigned)((int)(v << (31 - i)) >> 31); }
// act_pass as one integer comparison (0 < v, 0 < v < 6, always: positive floats order like their bits, NaN lies above infinity);
// the two float comparisons meet in scalar registers, which a chain of them waits for
__device__ __forceinline__ unsigned dw_pass_limit(int act) {
  return act == ACT_RELU6 ? 0x40bfffffu - 1u : act == ACT_RELU ? 0x7f800000u - 1u : ~0u;
}
__device__ __forceinline__ float dw_pass(float v, float d, unsigned limit) { return __float_as_uint(v) - 1u <= limit ? d : 0.f; }
__device__ __forceinline__ float2 dw_pair(const float* p) { return *reinterpret_cast<const float2*>(p); }
// Four pixels x 8 channels of dz2 and y2 -> dy2, transposed into the tile; bit i of ok: pixel i lies in the image (elsewhere dy2 is
// zero).  Two channels at a time: their coefficients are few enough to leave three workgroups a compute unit.
template <int CH_PITCH>
__device__ __forceinline__ void dw_bn_bwd_store(unsigned char* dst, const uint4 (&d)[4], const uint4 (&y)[4], const DwBnBwd& f, int c8, unsigned ok, unsigned limit,
                                                bool store) {
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const float2 mu = dw_pair(f.mu + c8 + 2 * m), a = dw_pair(f.a + c8 + 2 * m), b = dw_pair(f.b + c8 + 2 * m),
                 fp = dw_pair(f.p + c8 + 2 * m), fq = dw_pair(f.q + c8 + 2 * m);
    unsigned o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned dw = dw_word(d[i], m), yw = dw_word(y[i], m);
      const float y0 = bf_lo(yw) - mu.x, y1 = bf_hi(yw) - mu.y;
      const float d0 = dw_pass(fmaf(y0, a.x, b.x), bf_lo(dw), limit), d1 = dw_pass(fmaf(y1, a.y, b.y), bf_hi(dw), limit);
      const float t0 = bn_bwd_dy(y0, d0, a.x, fp.x, fq.x), t1 = bn_bwd_dy(y1, d1, a.y, fp.y, fq.y);
      o[i] = pack_bf2(t0, t1) & dw_bit(ok, i);
    }
    if (store) {
      *reinterpret_cast<uint2*>(dst + (2 * m) * CH_PITCH) = make_uint2(dw_lo2(o[0], o[1]), dw_lo2(o[2], o[3]));
      *reinterpret_cast<uint2*>(dst + (2 * m + 1) * CH_PITCH) = make_uint2(dw_hi2(o[0], o[1]), dw_hi2(o[2], o[3]));
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}
// dy as a tensor, bit for bit what the kernels form (pbd_read_grad_value)
__global__ __launch_bounds__(256) void bn_bwd_form_kernel(const bf16_t* __restrict__ dz, const bf16_t* __restrict__ y, bf16_t* __restrict__ dy, long nvec,
                                                          int ncv, BnBwd f) {
  const unsigned limit = dw_pass_limit(f.act);
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nvec; i += (long)gridDim.x * blockDim.x) {
    const uint4 d = *reinterpret_cast<const uint4*>(dz + i * 8), v = *reinterpret_cast<const uint4*>(y + i * 8);
    unsigned o[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int c = (int)(i % ncv) * 8 + 2 * m;
      const BnBwdTerms t0 = bn_bwd_terms(f, c), t1 = bn_bwd_terms(f, c + 1);
      const unsigned dw = dw_word(d, m), yw = dw_word(v, m);
      const float y0 = bf_lo(yw) - t0.mu, y1 = bf_hi(yw) - t1.mu;
      const float d0 = dw_pass(fmaf(y0, t0.a, t0.b), bf_lo(dw), limit), d1 = dw_pass(fmaf(y1, t1.a, t1.b), bf_hi(dw), limit);
      o[m] = pack_bf2(bn_bwd_dy(y0, d0, t0.a, t0.p, t0.q), bn_bwd_dy(y1, d1, t1.a, t1.p, t1.q));
    }
    *reinterpret_cast<uint4*>(dy + i * 8) = make_uint4(o[0], o[1], o[2], o[3]);
  }
}
// the same for x = z1 from y1 (dw_fold_apply's arithmetic)
template <int CH_PITCH>
__device__ __forceinline__ void dw_fold_store(unsigned char* dst, const uint4 (&y)[4], const DwFold& f, int c8, unsigned ok, float hi) {
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const float2 mu = dw_pair(f.mu + c8 + 2 * m), a = dw_pair(f.a + c8 + 2 * m), b = dw_pair(f.b + c8 + 2 * m);
    unsigned o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned yw = dw_word(y[i], m);
      const float z0 = fminf(fmaxf(fmaf(bf_lo(yw) - mu.x, a.x, b.x), 0.f), hi), z1 = fminf(fmaxf(fmaf(bf_hi(yw) - mu.y, a.y, b.y), 0.f), hi);
      o[i] = pack_bf2(z0, z1) & dw_bit(ok, i);
    }
    *reinterpret_cast<uint2*>(dst + (2 * m) * CH_PITCH) = make_uint2(dw_lo2(o[0], o[1]), dw_lo2(o[2], o[3]));
    *reinterpret_cast<uint2*>(dst + (2 * m + 1) * CH_PITCH) = make_uint2(dw_hi2(o[0], o[1]), dw_hi2(o[2], o[3]));
    __builtin_amdgcn_sched_barrier(0);
  }
}

// WGRAD false: the architecture round, which leaves the filters alone.
template <int K, bool WGRAD>
__device__ __forceinline__ void dw_bwd_mfma_block(const Blk& blk, const bf16_t* __restrict__ dz, const bf16_t* __restrict__ y2, const bf16_t* __restrict__ y1, const bf16_t* __restrict__ w,
    bf16_t* __restrict__ dx, float* __restrict__ wpart, float* __restrict__ spart, DwArgs g, BnBwd f2, NormFold f1) {
  typedef DwGeom<K> G;
  constexpr int NT = G::NT, pad = K / 2, NIT = K == 3 ? 1 : 2, QS = K == 3 ? 2 : 1;
  constexpr int DY = G::CHP * kDwCh > kDwOutRow * kDwTile ? G::CHP * kDwCh : kDwOutRow * kDwTile;   // dy2's tile, then dz1's
  constexpr int ROWD = kDwTile * 2, CHD = kDwTile * ROWD + 8;                        // x: 16 x 16 pixels a channel
  constexpr int ZERO = DY + (WGRAD ? CHD * kDwCh : 0);                               // a row of zeros
  __shared__ __attribute__((aligned(16))) unsigned char smem[ZERO + ROWD];
  __shared__ __attribute__((aligned(16))) unsigned char filt[kDwCh * K * G::WROW];
  __shared__ __attribute__((aligned(16))) DwBnBwd c2;
  __shared__ __attribute__((aligned(16))) DwFold c1;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slice = wave & 1, half = wave >> 1;
  const int wg = xcd_contiguous(blk.x, blk.gx);
  const int cv0 = (wg % g.groups) * (kDwCh / 8), chunk = wg / g.groups, C = g.ncv * 8;
  const int tile_begin = chunk * g.per_block, tile_end = min(g.tiles, tile_begin + g.per_block);
  const __amdgpu_buffer_rsrc_t zr = tensor_rsrc(dz, g.bytes), y2r = tensor_rsrc(y2, g.bytes), y1r = tensor_rsrc(y1, g.bytes);
  int ch = slice * 16 + (lane >> 2), n4 = lane & 3;          // n4: output row strip, column of the filter operand, tap offset
  const float hi1 = f1.act == ACT_RELU6 ? 6.f : __builtin_inff();
  const unsigned limit1 = dw_pass_limit(f1.act), limit2 = dw_pass_limit(f2.act);

  if (tid < kDwCh) {
    const int c = cv0 * 8 + tid;
    const BnBwdTerms t = c < C ? bn_bwd_terms(f2, c) : BnBwdTerms{};
    c2.mu[tid] = t.mu; c2.a[tid] = t.a; c2.b[tid] = t.b; c2.p[tid] = t.p; c2.q[tid] = t.q;
  }
  dw_fold_load(c1, f1, cv0 * 8, C, tid);
  if (tid < ROWD / 8) *reinterpret_cast<uint2*>(smem + ZERO + tid * 8) = make_uint2(0u, 0u);

  // ---- mirrored filters: [channel][filter row][tap] in LDS, from where every tile forms its Toeplitz rows anew ----
  for (int i = tid; i < K * K * (kDwCh / 2); i += 256) {
    const int tap = i / (kDwCh / 2), cc = i % (kDwCh / 2), t = K * K - 1 - tap;
    unsigned v = 0;
    if (cv0 * 8 + 2 * cc < C) v = *reinterpret_cast<const unsigned*>(w + (size_t)tap * C + cv0 * 8 + 2 * cc);
    unsigned short* p = reinterpret_cast<unsigned short*>(filt + (2 * cc * K + t / K) * G::WROW) + t % K;
    p[0] = (unsigned short)v;
    p[K * G::WROW / 2] = (unsigned short)(v >> 16);
  }
  dw_f32x4 wsum[NIT][NIT];                               // over the tiles, each summed on its own first
#pragma unroll
  for (int i = 0; i < NIT; ++i)
#pragma unroll
    for (int j = 0; j < NIT; ++j) wsum[i][j] = dw_f32x4{0.f, 0.f, 0.f, 0.f};
  float sb[8], sg[8];                                    // this thread's channels: sum dpre1, sum dpre1 (y1 - mean1)
#pragma unroll
  for (int e = 0; e < 8; ++e) sb[e] = sg[e] = 0.f;
  // this thread's four pixels of the tile (of x, and of the stored gradient): columns 4 xq .. 4 xq + 3 of row xrow
  const int cvl = tid % (kDwCh / 8), xq = (tid / (kDwCh / 8)) % 4, xrow = tid / (kDwCh / 8) / 4;

  for (int tile = tile_begin; tile < tile_end; ++tile) {
    int t_ = tile;
    const int tw = t_ % g.tiles_w; t_ /= g.tiles_w;
    const int th = t_ % g.tiles_h, n = t_ / g.tiles_h;
    const int h0 = th * kDwTile, w0 = tw * kDwTile;
    // ---- all loads of the tile in flight together ----
    uint4 rz[G::NLOAD][4], ry[G::NLOAD][4], rx[4];
    unsigned ok = 0;                                     // bit 4 i + p: pixel p of item i lies in the image
    // (places formed anew in every phase: kept over the tile they cost the registers that the loads in flight need)
    int at0 = tid;
    asm volatile("" : "+v"(at0));
#pragma unroll
    for (int i = 0; i < G::NLOAD; ++i) {
      const int c = at0 + i * 256, quad = (c / (kDwCh / 8)) % G::NQ, row = c / (kDwCh / 8) / G::NQ;
      const int h = h0 - pad + row, w_ = w0 - pad + 4 * quad;
      const bool rok = c < G::ITEMS && (unsigned)h < (unsigned)g.H && cv0 + cvl < g.ncv;
      const unsigned off = (unsigned)(((n * g.H + h) * g.W + w_) * g.ncv + cv0 + cvl) * 16u;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const bool in = rok && 4 * quad + p < G::IN && (unsigned)(w_ + p) < (unsigned)g.W;
        const unsigned at = in ? off + (unsigned)(p * g.ncv) * 16u : kOutOfRange;
        rz[i][p] = buffer_load16(zr, at);
        ry[i][p] = buffer_load16(y2r, at);
        ok |= (in ? 1u : 0u) << (4 * i + p);
      }
    }
    unsigned xok = 0;                                    // bit p: pixel p of x lies in the image
    const unsigned xoff = (unsigned)(((n * g.H + h0 + xrow) * g.W + w0 + 4 * xq) * g.ncv + cv0 + cvl) * 16u;
    asm volatile("" : "+v"(at0), "+v"(n4), "+v"(ch));
    __syncthreads();                                     // the previous tile's result (or the filters) has been read
#pragma unroll
    for (int i = 0; i < G::NLOAD; ++i) {
      const int c = at0 + i * 256, quad = (c / (kDwCh / 8)) % G::NQ, row = c / (kDwCh / 8) / G::NQ;
      unsigned char* dst = smem + cvl * 8 * G::CHP + row * G::ROWP + quad * 8;
      if (__builtin_amdgcn_ballot_w64((ok >> (4 * i) & 15u) != 0u))
        dw_bn_bwd_store<G::CHP>(dst, rz[i], ry[i], c2, cvl * 8, ok >> (4 * i), limit2, c < G::ITEMS);
      else if (c < G::ITEMS) {                           // rows outside the image: a third of the tile on a 14 x 14 image
#pragma unroll
        for (int e = 0; e < 8; ++e) *reinterpret_cast<uint2*>(dst + e * G::CHP) = make_uint2(0u, 0u);
      }
      if (i == 0) {                                      // (in flight behind the other items, in the first one's registers)
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const bool in = h0 + xrow < g.H && w0 + 4 * xq + p < g.W && cv0 + cvl < g.ncv;
          rx[p] = buffer_load16(y1r, in ? xoff + (unsigned)(p * g.ncv) * 16u : kOutOfRange);
          xok |= (in ? 1u : 0u) << p;
        }
      }
    }
    if constexpr (WGRAD) dw_fold_store<CHD>(smem + DY + cvl * 8 * CHD + xrow * ROWD + xq * 8, rx, c1, cvl * 8, xok, hi1);
    __syncthreads();

    // ---- weight gradient (dw_wgrad_mfma_kernel, dy2 in the role of x): D[r'][s'] = sum x[p] dy2tile[p + (r', s')] ----
    if constexpr (WGRAD) {
      const unsigned odd = n4 & 1 ? kDwSelMid : kDwSelLow;
      // (a lane's whole pairs of shift are in the address: LDS reads of two words)
      const unsigned char* xp = smem + ch * G::CHP + half * 16 + (n4 >> 1) * 4;
      const unsigned char* dp = smem + DY + ch * CHD + half * 16 - n4 * ROWD;
      const unsigned char* zp = smem + ZERO + half * 16;
      dw_f32x4 acc[NIT][NIT][QS];
#pragma unroll
      for (int i = 0; i < NIT; ++i)
#pragma unroll
        for (int j = 0; j < NIT; ++j)
#pragma unroll
          for (int q = 0; q < QS; ++q) acc[i][j][q] = dw_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int y = 0; y < G::IN; ++y) {
        // row y - n4 - 4 jt of x, n4 = 0..3: none, some or all of the four lie in the tile
        dw_s16x4 d[NIT][2];
#pragma unroll
        for (int jt = 0; jt < NIT; ++jt) {
          const int top = y - 4 * jt;
          const unsigned char* db = dp + top * ROWD;
          if (top < 3) db = n4 <= top ? db : zp;
          if (top > kDwTile - 1) db = n4 > top - kDwTile ? db : zp;
          if (top < 0 || top > kDwTile + 2) continue;
#pragma unroll
          for (int q = 0; q < 2; ++q) d[jt][q] = *reinterpret_cast<const dw_s16x4*>(db + q * 8);
        }
        unsigned E[2 * (NIT + 1) + 1];
#pragma unroll
        for (int i = 0; i < 2 * (NIT + 1) + 1; ++i) E[i] = *reinterpret_cast<const unsigned*>(xp + y * G::ROWP + i * 4);
#pragma unroll
        for (int c = 0; c < NIT + 1; ++c) {
          const dw_s16x4 xs = __builtin_bit_cast(dw_s16x4, make_uint2(__builtin_amdgcn_perm(E[2 * c + 1], E[2 * c], odd),
                                                                      __builtin_amdgcn_perm(E[2 * c + 2], E[2 * c + 1], odd)));
#pragma unroll
          for (int it = 0; it < NIT; ++it) {
            const int q = c - it;
            if (q < 0 || q > 1) continue;
#pragma unroll
            for (int jt = 0; jt < NIT; ++jt)
              if (y - 4 * jt >= 0 && y - 4 * jt <= kDwTile + 2)
                acc[it][jt][q % QS] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(xs, d[jt][q], acc[it][jt][q % QS], 0, 0, 0);
          }
        }
        if (y % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < NIT; ++i)
#pragma unroll
        for (int j = 0; j < NIT; ++j) wsum[i][j] += QS == 2 ? acc[i][j][0] + acc[i][j][QS - 1] : acc[i][j][0];
      __builtin_amdgcn_sched_barrier(0);
    }

    // ---- backward-data (dw_mfma_kernel, FLIP): acc[o][q] = rows 4 n4 + o, columns 8 half + 4 q + 0..3 ----
    dw_s16x4 wt[K][NT];                                  // (not held over the tile: 20 registers at 5 x 5)
    {
      const unsigned far = n4 >= 2 ? ~0u : 0u, odd = n4 & 1 ? kDwSelMid : kDwSelHigh;
#pragma unroll
      for (int r = 0; r < K; ++r) {
        unsigned P[2 * NT + 2];
#pragma unroll
        for (int i = 0; i < 2 * NT + 2; ++i) P[i] = 0u;
        const unsigned char* row = filt + (ch * K + r) * G::WROW;
        const uint2 q0 = *reinterpret_cast<const uint2*>(row);
        P[2] = q0.x; P[3] = K == 3 ? q0.y & 0xffffu : q0.y;
        if (K > 3) {
          const uint2 q1 = *reinterpret_cast<const uint2*>(row + 8);
          P[4] = K == 5 ? q1.x & 0xffffu : q1.x;
          if (K > 5) P[5] = q1.y & 0xffffu;
        }
        unsigned E[2 * NT + 1];
#pragma unroll
        for (int i = 0; i < 2 * NT + 1; ++i) E[i] = dw_sel(far, P[i], P[i + 1]);
#pragma unroll
        for (int t = 0; t < NT; ++t)
          wt[r][t] = __builtin_bit_cast(dw_s16x4, make_uint2(__builtin_amdgcn_perm(E[2 * t + 1], E[2 * t], odd),
                                                             __builtin_amdgcn_perm(E[2 * t + 2], E[2 * t + 1], odd)));
      }
    }
    dw_f32x4 acc[4][2];
#pragma unroll
    for (int o = 0; o < 4; ++o)
#pragma unroll
      for (int q = 0; q < 2; ++q) acc[o][q] = dw_f32x4{0.f, 0.f, 0.f, 0.f};
    const unsigned char* in = smem + ch * G::CHP + 4 * n4 * G::ROWP + half * 16;
#pragma unroll
    for (int c = 0; c < NT + 1; ++c)
#pragma unroll
      for (int y = 0; y < K + 3; ++y) {
        const dw_s16x4 d = *reinterpret_cast<const dw_s16x4*>(in + y * G::ROWP + c * 8);
#pragma unroll
        for (int o = 0; o < 4; ++o) {
          const int r = y - o;
          if (r < 0 || r >= K) continue;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int t = c - q;
            if (t < 0 || t >= NT) continue;
            acc[o][q] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(wt[r][t], d, acc[o][q], 0, 0, 0);
          }
        }
        if (K > 3 && y % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // (not every read of the tile in registers at once)
      }
    __syncthreads();                                     // every wave has read dy2's tile
    unsigned char* so = smem + (ch >> 1) * 4 + ((ch & 1) * 2 + half * 8) * kDwOutP;
#pragma unroll
    for (int o = 0; o < 4; ++o)
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const int v0 = __float_as_int(acc[o][q][m]), v2 = __float_as_int(acc[o][q][m + 2]);
          const int lo = __builtin_amdgcn_update_dpp(v0, v2, 0x114, 0xf, 0xa, false);   // row_shr:4 into the odd channels
          const int hi = __builtin_amdgcn_update_dpp(v2, v0, 0x104, 0xf, 0x5, false);   // row_shl:4 into the even channels
          *reinterpret_cast<unsigned*>(so + (4 * n4 + o) * kDwOutRow + (q * 4 + m) * kDwOutP) = pack_bf2(__int_as_float(lo), __int_as_float(hi));
        }
    __syncthreads();
    // ---- store, and the sums of y1's batch-norm backward pass over what was stored ----
    uint4 out[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      out[p] = *reinterpret_cast<const uint4*>(smem + xrow * kDwOutRow + (4 * xq + p) * kDwOutP + cvl * 16);
      if ((xok >> p) & 1u) *reinterpret_cast<uint4*>(reinterpret_cast<unsigned char*>(dx) + xoff + (unsigned)(p * g.ncv) * 16u) = out[p];
      else out[p] = make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const float2 mu = dw_pair(c1.mu + cvl * 8 + 2 * m), a = dw_pair(c1.a + cvl * 8 + 2 * m), b = dw_pair(c1.b + cvl * 8 + 2 * m);
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const unsigned dw = dw_word(out[p], m), yw = dw_word(rx[p], m);
        const float y0 = bf_lo(yw) - mu.x, y1_ = bf_hi(yw) - mu.y;
        const float d0 = dw_pass(fmaf(y0, a.x, b.x), bf_lo(dw), limit1), d1 = dw_pass(fmaf(y1_, a.y, b.y), bf_hi(dw), limit1);
        sb[2 * m] += d0;
        sb[2 * m + 1] += d1;
        sg[2 * m] = fmaf(d0, y0, sg[2 * m]);
        sg[2 * m + 1] = fmaf(d1, y1_, sg[2 * m + 1]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // ---- sums: lanes 4 apart hold the same channels; then the four waves ----
  __syncthreads();
  float* red = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int off = 4; off < 64; off <<= 1) {
      sb[e] += __shfl_xor(sb[e], off, 64);
      sg[e] += __shfl_xor(sg[e], off, 64);
    }
  if (lane < kDwCh / 8) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      red[(wave * 2) * kDwCh + lane * 8 + e] = sb[e];
      red[(wave * 2 + 1) * kDwCh + lane * 8 + e] = sg[e];
    }
  }
  __syncthreads();
  if (tid < 2 * kDwCh && cv0 * 8 + tid % kDwCh < C) {
    const int c = cv0 * 8 + tid % kDwCh;
    const float v = (red[tid] + red[2 * kDwCh + tid]) + (red[4 * kDwCh + tid] + red[6 * kDwCh + tid]);
    spart[((size_t)chunk * 2 + tid / kDwCh) * C + c] = tid < kDwCh ? v : v * f1.invstd[c];
  }
  if constexpr (!WGRAD) return;
  // ---- the two column halves of a slice meet; lane 4 c + j holds taps (r' = 4 jt + j, s' = 4 it + v) of channel c, mirrored ----
  __syncthreads();
  if (half) {
#pragma unroll
    for (int it = 0; it < NIT; ++it)
#pragma unroll
      for (int jt = 0; jt < NIT; ++jt)
        *reinterpret_cast<dw_f32x4*>(red + ((slice * NIT * NIT + it * NIT + jt) * 64 + lane) * 4) = wsum[it][jt];
  }
  __syncthreads();
  if (half || cv0 * 8 + ch >= C) return;
#pragma unroll
  for (int it = 0; it < NIT; ++it)
#pragma unroll
    for (int jt = 0; jt < NIT; ++jt) {
      const dw_f32x4 o = *reinterpret_cast<const dw_f32x4*>(red + ((slice * NIT * NIT + it * NIT + jt) * 64 + lane) * 4);
      const int r = K - 1 - (4 * jt + n4);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int s = K - 1 - (4 * it + v);
        if (r >= 0 && s >= 0) wpart[((size_t)chunk * K * K + r * K + s) * C + cv0 * 8 + ch] = wsum[it][jt][v] + o[v];
      }
    }
}
template <int K, bool WGRAD>
__global__ __launch_bounds__(256, WGRAD ? (K == 7 ? 2 : 3) : (K == 7 ? 3 : 4)) void dw_bwd_mfma_kernel(
    const bf16_t* __restrict__ dz, const bf16_t* __restrict__ y2, const bf16_t* __restrict__ y1, const bf16_t* __restrict__ w,
    bf16_t* __restrict__ dx, float* __restrict__ wpart, float* __restrict__ spart, DwArgs g, BnBwd f2, NormFold f1) {
  dw_bwd_mfma_block<K, WGRAD>(one_block(), dz, y2, y1, w, dx, wpart, spart, g, f2, f1);
}

// Backward-weight of a stride-2 layer, dW[r][s] = sum x[2 p + r - pad][2 q + s - pad] dy[p][q].  Columns (and rows) of x of one
// parity are a stride-1 problem with at most (K + 1) / 2 <= 4 taps, so one product covers all taps of a parity pair: the four
// pixels a thread loads lie two columns apart, LDS holds [channel][row][column parity][column], and with y the row of
// x in the tile, A[i][k] = x[y][parity][4 c + i + k] (s = 2 i + parity), B[k][j] = dy[(y >> 1) - j][4 c + k] (r = 2 j + (y & 1)).
// Tile: 8 x 16 pixels of dy, 32 channels; wave = (16 channels) x (column parity), so no two waves share a tap.
// Bound by the shifts (vector ALUs) and LDS reads at 8 waves per compute unit; against one thread per 8 channels and filter
// row (dw_wgrad_kernel): 5 x 5, MobileNetV2 batch 128 69 -> 41 us a launch, batch 33 28 -> 13; 7 x 7, supernet 52 -> 30.  3 x 3 only
// wins on few tiles (a third of the products are real there, and the shifts cost the same).
constexpr int kDwS2TileH = 8;
template <int K>
__device__ __forceinline__ void dw_wgrad_s2_mfma_block(const Blk& blk, const bf16_t* __restrict__ dy, const bf16_t* __restrict__ x,
                                                                  float* __restrict__ part, DwArgs g) {
  constexpr int pad = K / 2, IH = 2 * kDwS2TileH - 2 + K, NQ = 5, CVB = kDwCh / 8;
  constexpr int ROWX = 2 * NQ * 8, CHX = (IH * ROWX + 31) / 32 * 32 + 8;
  constexpr int ROWD = kDwTile * 2, CHD = kDwS2TileH * ROWD + 8;
  constexpr int ITEMS = IH * 2 * NQ * CVB, NLOAD = (ITEMS + 255) / 256;
  constexpr int DITEMS = kDwS2TileH * 4 * CVB;                        // (128: half of the threads)
  constexpr int ZERO = CHX * kDwCh + CHD * kDwCh;                     // a row of zeros
  __shared__ __attribute__((aligned(16))) unsigned char smem[ZERO + ROWD];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slice = wave & 1, par = wave >> 1;
  const int wg = xcd_contiguous(blk.x, blk.gx);
  const int cv0 = (wg % g.groups) * CVB, chunk = wg / g.groups;
  const int tile_begin = chunk * g.per_block, tile_end = min(g.tiles, tile_begin + g.per_block);
  const __amdgpu_buffer_rsrc_t xr = tensor_rsrc(x, g.bytes), dr = tensor_rsrc(dy, g.dy_bytes);
  const int ch = slice * 16 + (lane >> 2), n4 = lane & 3;
  const unsigned far = n4 >= 2 ? ~0u : 0u, odd = n4 & 1 ? kDwSelMid : kDwSelLow;
  if (tid < ROWD / 8) *reinterpret_cast<uint2*>(smem + ZERO + tid * 8) = make_uint2(0u, 0u);

  dw_f32x4 sum[2];                                       // by row parity; over the tiles, each summed on its own first
  sum[0] = sum[1] = dw_f32x4{0.f, 0.f, 0.f, 0.f};
  uint4 rx[NLOAD][4], rd[4];
  auto load_tile = [&](int tile) {
    int t_ = tile;
    const int tw = t_ % g.tiles_w; t_ /= g.tiles_w;
    const int th = t_ % g.tiles_h, n = t_ / g.tiles_h;
    const int p0 = th * kDwS2TileH, q0 = tw * kDwTile;
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      const int c = tid + i * 256;
      const int cvl = c % CVB, quad = (c / CVB) % NQ, rp = c / CVB / NQ;   // rp = row * 2 + column parity
      const int h = 2 * p0 - pad + (rp >> 1), w_ = 2 * q0 - pad + 8 * quad + (rp & 1);
      const bool rok = c < ITEMS && (unsigned)h < (unsigned)g.H && cv0 + cvl < g.ncv;
      const unsigned off = (unsigned)(((n * g.H + h) * g.W + w_) * g.ncv + cv0 + cvl) * 16u;
#pragma unroll
      for (int p = 0; p < 4; ++p)
        rx[i][p] = buffer_load16(xr, rok && (unsigned)(w_ + 2 * p) < (unsigned)g.W ? off + (unsigned)(2 * p * g.ncv) * 16u : kOutOfRange);
    }
    const int cvl = tid % CVB, quad = (tid / CVB) % 4, drow = tid / CVB / 4;
    const int h = p0 + drow, w_ = q0 + 4 * quad;
    const unsigned off = (unsigned)(((n * g.P + h) * g.Q + w_) * g.ncv + cv0 + cvl) * 16u;
#pragma unroll
    for (int p = 0; p < 4; ++p)
      rd[p] = buffer_load16(dr, tid < DITEMS && h < g.P && w_ + p < g.Q && cv0 + cvl < g.ncv ? off + (unsigned)(p * g.ncv) * 16u : kOutOfRange);
  };

  if (tile_begin < tile_end) load_tile(tile_begin);
  for (int tile = tile_begin; tile < tile_end; ++tile) {
    __syncthreads();                                     // the previous tile has been read
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      const int c = tid + i * 256;
      const int cvl = c % CVB, quad = (c / CVB) % NQ, rp = c / CVB / NQ;
      if (c < ITEMS) dw_store_transposed<CHX>(smem + cvl * 8 * CHX + rp * (NQ * 8) + quad * 8, rx[i]);
    }
    if (tid < DITEMS)
      dw_store_transposed<CHD>(smem + CHX * kDwCh + (tid % CVB) * 8 * CHD + (tid / CVB / 4) * ROWD + ((tid / CVB) % 4) * 8, rd);
    __syncthreads();
    if (tile + 1 < tile_end) load_tile(tile + 1);        // in flight behind this tile's products

    const unsigned char* xp = smem + ch * CHX + par * (NQ * 8);
    const unsigned char* dp = smem + CHX * kDwCh + ch * CHD;
    const unsigned char* zp = smem + ZERO;
    dw_f32x4 acc[2];
    acc[0] = acc[1] = dw_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int y2 = 0; y2 < (IH + 1) / 2; ++y2) {
      const int row = y2 - n4;
      const unsigned char* db = (unsigned)row < (unsigned)kDwS2TileH ? dp + row * ROWD : zp;
      dw_s16x4 d[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) d[q] = *reinterpret_cast<const dw_s16x4*>(db + q * 8);
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int y = min(2 * y2 + e, IH - 1);           // (IH is odd: the last odd row is the last row once more, into taps r >= K)
        unsigned D[2 * NQ];
#pragma unroll
        for (int c = 0; c < NQ; ++c) {
          const uint2 v = *reinterpret_cast<const uint2*>(xp + y * ROWX + c * 8);
          D[2 * c] = v.x; D[2 * c + 1] = v.y;
        }
        unsigned E[2 * NQ - 1];
#pragma unroll
        for (int i = 0; i < 2 * NQ - 1; ++i) E[i] = dw_sel(far, D[i + 1], D[i]);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const unsigned s0 = __builtin_amdgcn_perm(E[2 * c + 1], E[2 * c], odd);
          const unsigned s1 = __builtin_amdgcn_perm(E[2 * c + 2], E[2 * c + 1], odd);
          acc[e] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(dw_s16x4, make_uint2(s0, s1)), d[c], acc[e], 0, 0, 0);
        }
      }
    }
    sum[0] += acc[0];
    sum[1] += acc[1];
  }
  if (cv0 * 8 + ch >= g.ncv * 8) return;
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 2 * n4 + e, s = 2 * v + par;
      if (r < K && s < K) part[((size_t)chunk * K * K + r * K + s) * (g.ncv * 8) + cv0 * 8 + ch] = sum[e][v];
    }
}
template <int K>
__global__ __launch_bounds__(256, 2) void dw_wgrad_s2_mfma_kernel(const bf16_t* __restrict__ dy,
    const bf16_t* __restrict__ x, float* __restrict__ part, DwArgs g) {
  dw_wgrad_s2_mfma_block<K>(one_block(), dy, x, part, g);
}

}  // namespace pbd
