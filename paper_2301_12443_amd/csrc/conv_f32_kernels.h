// float32 dense convolutions on the fp32 matrix cores, channel-last tensors, bit for bit the results of the direct kernels
// (conv_direct_* in conv_kernels.h).
//
// v_mfma_f32_32x32x2_f32 and v_mfma_f32_16x16x4_f32 add their two / four products to the accumulator one after the other, in
// the order of the lanes that hold them, as fused multiply-adds that round each time, subnormals included (checked against
// fmaf over chains of up to 4096).  One result's chain therefore stays ONE chain in the order of the direct kernels: no cut of
// the reduction over waves or workgroups, and the lanes 0..31 / 32..63 (or the four groups of sixteen) of an operand hold
// CONSECUTIVE reduction elements.  A tap outside the image, which the direct kernels leave out, is a product with zero and
// changes no chain of finite numbers; a result that comes out as NaN is formed once more the direct way, so an infinity or NaN in a
// weight that the image's edge never meets stays there.
//   Why the order matters: a rectifier's mask, and everything behind it, hangs on the last bit of some pre-activations, so another
// order of summation, closer to the exact sum or not, moves single gradients by percents and a few steps' results with them.
//
// An MFMA takes one float per lane and operand: 64 cycles for 32 x 32 results and two reduction elements, 32 cycles for 16 x 16 and
// four.  Both run at the same rate, but a chain of n elements takes 32 n cycles on the one and 8 n on the other, and the
// small layers this precision is used on are bound by the length of the chain.  So the 16-wide tiles are taken wherever the
// 32-wide ones would not give every compute unit a workgroup.
//
// Measured, VGG-16 at 64 x 32 x 32: against one thread per result the whole step takes 1.77 ms instead of 91.1, the four-layer
// network's at 8 x 32 x 32 0.24 instead of 1.94 ms.  Forward 64 -> 64, 3 x 3, 65536 pixels 57 us (84 TFLOP/s), 512 -> 512 at 1024
// pixels 81 us (60), the weight gradient of a 1 x 1 layer over 65536 pixels 440 us.  Cutting a reduction over eight waves and
// adding the parts (other bits) took 1.50 ms a step.
#pragma once
#include "conv_kernels.h"

namespace pbd {

typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 buffer_load_f4(__amdgpu_buffer_rsrc_t r, unsigned byte_off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte_off, 0, 0));
}

// exchange of lane rows of two registers: odd rows of 16 of `a` with even rows of `b`; lanes 32..63 of `a` with 0..31 of `b`
__device__ __forceinline__ void swap_rows16(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap_rows32(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
}

template <int TILE> struct F32Tile;
template <> struct F32Tile<32> {
  typedef f32x16 Acc;
  static constexpr int GROUPS = 2, VALUES = 16;       // reduction elements per MFMA, results per lane
  static constexpr int COLP = 64;                     // floats per reduction element staged [element][channel]
  // tile row of a lane's four results 4 q .. 4 q + 3
  static __device__ __forceinline__ int row(int q, int group) { return 8 * q + 4 * group; }
  static __device__ __forceinline__ Acc mfma(float a, float b, Acc c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
  // v[e] of lane group g = element 4 g + e of a run of eight -> element 2 e + g
  static __device__ __forceinline__ void in_order(float (&v)[4]) {
    swap_rows32(v[0], v[1]);                          // 0 1 | 4 5
    swap_rows32(v[2], v[3]);                          // 2 3 | 6 7
    const float t = v[1]; v[1] = v[2]; v[2] = t;
  }
};
template <> struct F32Tile<16> {
  typedef f32x4 Acc;
  static constexpr int GROUPS = 4, VALUES = 4;
  static constexpr int COLP = 48;                     // (two elements that a half wave reads lie on different banks)
  static __device__ __forceinline__ int row(int, int group) { return 4 * group; }
  static __device__ __forceinline__ Acc mfma(float a, float b, Acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  // element 4 g + e of a run of sixteen -> element 4 e + g: a 4 x 4 transposition
  static __device__ __forceinline__ void in_order(float (&v)[4]) {
    swap_rows16(v[0], v[1]); swap_rows16(v[2], v[3]);
    swap_rows32(v[0], v[2]); swap_rows32(v[1], v[3]);
  }
};

// The product both kernels share.  A workgroup of four waves owns EDGE x EDGE = 2 x 2 tiles of Out[p][q] = sum_e P[p][e] Q[q][e] and
// their whole reduction, in stages of BK elements (sixteen MFMAs).  Two passes of all threads load a stage of an operand, four
// floats each, into registers and from there into LDS:
//  * ROWS: the operand's memory is contiguous along the reduction; staged [p][element], ROWP = BK + 4 floats a row, a lane
//    reads four elements of its row at once and neighbouring lane groups exchange them;
//  * else contiguous along p (or q): staged [element][p], a lane reads one element at a time.
// While stage t is multiplied from registers, stage t + 1 goes from LDS to the other register set, stage t + 2 from
// registers to LDS, and t + 3 to t + 6 are on their way from memory.  Sixteen dependent 16-wide products take 512 cycles, a stage of
// the 65536-pixel weight gradient about 1030: the barrier, the LDS reads behind it and the products' own latency are what is left
// (1570 before the staging was dealt out between the products and the waits counted loads exactly).
template <int TILE> struct F32Gemm {
  typedef F32Tile<TILE> F;
  static constexpr int EDGE = 2 * TILE, BK = 16 * F::GROUPS, ROWP = BK + 4, COLP = F::COLP;    // 32 and 64, 64 and 32
  template <bool ROWS> static constexpr int floats = ROWS ? EDGE * ROWP : BK * COLP;             // per stage in LDS
  // what thread tid stages in pass i: row / element, and the first of its four elements / rows
  static constexpr int PER = 256 / (BK / 4), PER_COL = 256 / (EDGE / 4);
  template <bool ROWS> static __device__ __forceinline__ int major(int tid, int i) { return ROWS ? tid / (BK / 4) + i * PER : tid / (EDGE / 4) + i * PER_COL; }
  template <bool ROWS> static __device__ __forceinline__ int minor(int tid) { return (ROWS ? tid % (BK / 4) : tid % (EDGE / 4)) * 4; }
  static_assert(2 * PER == EDGE && 2 * PER_COL == BK, "two passes stage a stage");

  template <bool ROWS> static __device__ __forceinline__ void put(float* buf, f32x4 v, int i, int tid) {
    *reinterpret_cast<f32x4*>(buf + major<ROWS>(tid, i) * (ROWS ? ROWP : COLP) + minor<ROWS>(tid)) = v;
  }
  // operands 4 v .. 4 v + 3 of the lane whose tile row is `at`
  template <bool ROWS> static __device__ __forceinline__ void get(const float* buf, float (&f)[4], int v, int at, int group) {
    if constexpr (ROWS) {
      const f32x4 q = *reinterpret_cast<const f32x4*>(buf + at * ROWP + v * 4 * F::GROUPS + 4 * group);
#pragma unroll
      for (int e = 0; e < 4; ++e) f[e] = q[e];
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) f[e] = buf[((4 * v + e) * F::GROUPS + group) * COLP + at];
    }
  }
  // load_p(i), load_q(i): pass i = 0, 1 of the next stage of an operand
  template <bool P_ROWS, bool Q_ROWS, class LP, class LQ>
  static __device__ __forceinline__ void run(LP&& load_p, LQ&& load_q, typename F::Acc& acc, int stages, int tid) {
    __shared__ __attribute__((aligned(16))) float sp[2][floats<P_ROWS>], sq[2][floats<Q_ROWS>];
    const int lane = tid & 63, group = lane / TILE, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int at_p = (wave >> 1) * TILE + lane % TILE, at_q = (wave & 1) * TILE + lane % TILE;
    f32x4 gp[4][2], gq[4][2];                          // stage n waits in set n % 4 and goes through LDS buffer n % 2
    float fp[2][4][4], fq[2][4][4];
    // quarter v of a stage's staging: one pass of one operand.  (No branch around a load, and the order pinned: the compiler
    // then knows how many loads are younger than the one it waits for.)
    auto load = [&](auto set, int v) {
      constexpr int S_ = decltype(set)::value;
      if (v < 2) gp[S_][v] = load_p(v); else gq[S_][v - 2] = load_q(v - 2);
    };
    auto store = [&](auto set, int v) {
      constexpr int S_ = decltype(set)::value;
      if (v < 2) put<P_ROWS>(sp[S_ & 1], gp[S_][v], v, tid); else put<Q_ROWS>(sq[S_ & 1], gq[S_][v - 2], v - 2, tid);
    };
    auto order = [&](int set, int v) {
      if (P_ROWS) F::in_order(fp[set][v]);
      if (Q_ROWS) F::in_order(fq[set][v]);
    };
    auto turn = [&](auto set) {
      constexpr int S_ = decltype(set)::value, CUR = S_ & 1, NXT = CUR ^ 1;
      const std::integral_constant<int, (S_ + 2) & 3> ahead{};
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        get<P_ROWS>(sp[NXT], fp[NXT][v], v, at_p, group);
        get<Q_ROWS>(sq[NXT], fq[NXT][v], v, at_q, group);
        order(v < 3 ? CUR : NXT, (v + 1) & 3);         // (what the next four products read)
        store(ahead, v);
        load(ahead, v);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = F::mfma(fp[CUR][v][e], fq[CUR][v][e], acc);
        // addresses and LDS traffic of the coming stages issue between the products, which wait for each other
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                              // an MFMA
          __builtin_amdgcn_sched_group_barrier(0x100, P_ROWS || Q_ROWS ? 2 : 1, 0);       // LDS reads
          __builtin_amdgcn_sched_group_barrier(0x006, 12, 0);                             // vector and scalar ALU
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      __syncthreads();
    };
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;
    using S2 = std::integral_constant<int, 2>;
    using S3 = std::integral_constant<int, 3>;
    auto load_all = [&](auto set) {
#pragma unroll
      for (int v = 0; v < 4; ++v) load(set, v);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto store_all = [&](auto set) {
#pragma unroll
      for (int v = 0; v < 4; ++v) store(set, v);
      __builtin_amdgcn_sched_barrier(0);
    };
    load_all(S0{}); load_all(S1{}); load_all(S2{}); load_all(S3{});
    store_all(S0{});
    load_all(S0{});
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) { get<P_ROWS>(sp[0], fp[0][v], v, at_p, group); get<Q_ROWS>(sq[0], fq[0][v], v, at_q, group); }
    order(0, 0);
    store_all(S1{});
    load_all(S1{});
    __syncthreads();
    // (whole rounds of the four sets in a loop without exits; what is staged behind the last stage, zeros, is not multiplied)
    for (int t = 0; t < stages >> 2; ++t) { turn(S0{}); turn(S1{}); turn(S2{}); turn(S3{}); }
    if (stages & 3) {
      turn(S0{});
      if ((stages & 3) > 1) turn(S1{});
      if ((stages & 3) > 2) turn(S2{});
    }
  }
};

// Same view as igemm_kernel: Out[m][j] = sum_kk Agather(m, kk) * W(j, kk), rows m = pixels of an [N][HO][WO] grid,
// kk = (r*S + s)*CA + c.  MODE 0 reads the weights as they lie, [NC][R][S][CA]; MODE 1 reads the forward filter
// [CA][R][S][NC], so there is no transposed copy to keep.
template <int MODE, int TILE>
__global__ __launch_bounds__(256) void igemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ Bw,
                                                       float* Out, const float* __restrict__ ep_a,
                                                       const float* __restrict__ ep_b, int act, int accumulate, IgemmArgs g) {
  typedef F32Tile<TILE> F;
  typedef F32Gemm<TILE> G;
  constexpr bool W_ROWS = MODE == 0;
  const int tid = threadIdx.x, lane = tid & 63, group = lane / TILE, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tile = xcd_contiguous(blockIdx.x, g.tiles_m * g.tiles_n);
  const int m0 = tile / g.tiles_n * G::EDGE, n0 = tile % g.tiles_n * G::EDGE;
  const int sh = g.stride == 2 ? 1 : 0, smask = g.stride - 1;
  const __amdgpu_buffer_rsrc_t ra = tensor_rsrc(A, g.a_bytes), rb = tensor_rsrc(Bw, g.b_bytes);
  const int RS = g.R * g.S;

  // a thread's reduction element kk = tap * CA + c, moved on by a stage at a time (CA % 8 == 0: its four elements share a tap)
  // off: what the tap and channel add to an element's offset, advanced by additions like the rest
  struct Tap { int kk, c, r, s, off; };
  auto tap_of = [&](int kk) {
    const int rs = kk / g.CA, r = rs / g.S, q = rs % g.S, c = kk - rs * g.CA;
    return Tap{kk, c, r, q, MODE == 0 ? (r * g.WA + q) * g.CA + c : c - ((r * g.WA + q) * g.CA >> sh)};
  };
  const int dtap = G::BK / g.CA, dc = G::BK % g.CA, dr = dtap / g.S, ds = dtap % g.S;   // BK in the mixed radix of (r, s, c)
  // (a channel count run out is the next tap of the row: the same offset at MODE 0.  MODE 1 forms it anew: with stride 2 the taps of a row are
  // half a pixel apart)
  const int d_off = (dr * g.WA + ds) * g.CA + dc, row_off = (g.WA - g.S) * g.CA;
  auto next_stage = [&](Tap& t) {
    t.kk += G::BK;
    const int c = t.c + dc, c1 = c >= g.CA ? 1 : 0, s = t.s + ds + c1, c2 = s >= g.S ? 1 : 0;
    t.c = c - (c1 ? g.CA : 0);
    t.s = s - (c2 ? g.S : 0);
    t.r += dr + c2;
    if (MODE == 0) t.off += d_off + (c2 ? row_off : 0);
    else t.off = t.c - ((t.r * g.WA + t.s) * g.CA >> sh);
  };
  // pixels: two rows of four elements a stage
  Tap ta = tap_of(G::template minor<true>(tid));
  int at[2], rh[2], rw[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = m0 + G::template major<true>(tid, i), mm = m < g.M ? m : 0;
    const int b_ = mm % g.WO, t = mm / g.WO, a_ = t % g.HO;
    rh[i] = MODE == 0 ? a_ * g.stride - g.pad : a_ + g.pad;
    rw[i] = MODE == 0 ? b_ * g.stride - g.pad : b_ + g.pad;
    at[i] = (t / g.HO) * g.HA * g.WA * g.CA + ((rh[i] * g.WA + rw[i]) * g.CA >> (MODE == 1 ? sh : 0));
    if (m >= g.M) rh[i] = -(1 << 24);                  // (fails every range test)
  }
  auto load_pixels = [&](int i) {
    int h = MODE == 0 ? rh[i] + ta.r : rh[i] - ta.r, w = MODE == 0 ? rw[i] + ta.s : rw[i] - ta.s;
    bool ok = ta.kk < g.Kred;
    if (MODE == 1) { ok &= ((h | w) & smask) == 0; h >>= sh; w >>= sh; }
    ok &= ((unsigned)h < (unsigned)g.HA) & ((unsigned)w < (unsigned)g.WA);
    const unsigned off = (unsigned)(at[i] + ta.off) * 4u;
    if (i == 1) next_stage(ta);
    return buffer_load_f4(ra, ok ? off : kOutOfRange);
  };
  // weights: MODE 0 two channels' four elements, MODE 1 two elements' four channels (NC % 8 == 0: in or out as a whole).  Offsets of the elements
  // kk and, MODE 1, channel and tap of each, advanced by additions; an element past the last is out of range there or not asked for.
  int wk[2], wc[2], woff[2];
  bool w_in[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    wk[i] = MODE == 0 ? G::template minor<true>(tid) : G::template major<false>(tid, i);
    const int bat = n0 + (MODE == 0 ? G::template major<true>(tid, i) : G::template minor<false>(tid));
    w_in[i] = bat < g.NC;
    wc[i] = wk[i] % g.CA;
    woff[i] = MODE == 0 ? bat * g.Kred + wk[i] : (wc[i] * RS + wk[i] / g.CA) * g.NC + bat;
  }
  const int w_step = (dc * RS + dtap) * g.NC, w_wrap = (1 - g.CA * RS) * g.NC;
  auto load_weights = [&](int i) {
    const unsigned off = w_in[i] & (wk[i] < g.Kred) ? (unsigned)woff[i] * 4u : kOutOfRange;
    wk[i] += G::BK;
    if (MODE == 0) {
      woff[i] += G::BK;
    } else {
      const int c = wc[i] + dc;
      const bool wrap = c >= g.CA;
      wc[i] = c - (wrap ? g.CA : 0);
      woff[i] += w_step + (wrap ? w_wrap : 0);
    }
    return buffer_load_f4(rb, off);
  };

  // a lane holds runs of four consecutive channels of one pixel (NC % 8 == 0: in or out as a whole)
  const int m = m0 + (wave & 1) * TILE + lane % TILE, col0 = n0 + (wave >> 1) * TILE;
  typename F::Acc acc;
#pragma unroll
  for (int q = 0; q < F::VALUES / 4; ++q) {
    // the direct kernel's chain starts from the value that is added to
    const int col = col0 + F::row(q, group);
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
    if (accumulate && m < g.M && col < g.NC) o = *reinterpret_cast<const float4*>(Out + (size_t)m * g.NC + col);
    acc[4 * q] = o.x; acc[4 * q + 1] = o.y; acc[4 * q + 2] = o.z; acc[4 * q + 3] = o.w;
  }
  G::template run<W_ROWS, true>(load_weights, load_pixels, acc, (g.Kred + G::BK - 1) / G::BK, tid);

#pragma unroll
  for (int q = 0; q < F::VALUES / 4; ++q) {
    const int col = col0 + F::row(q, group);
    if (m >= g.M || col >= g.NC) continue;
    float4* dst = reinterpret_cast<float4*>(Out + (size_t)m * g.NC + col);
    float o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = acc[4 * q + e];
    if (o[0] != o[0] || o[1] != o[1] || o[2] != o[2] || o[3] != o[3]) {
      const int b_ = m % g.WO, t = m / g.WO, a_ = t % g.HO, n = t / g.HO;
      const ConvGeom d = MODE == 0 ? ConvGeom{g.N, g.HA, g.WA, g.CA, g.HO, g.WO, g.NC, g.R, g.S, g.stride, g.pad}
                                   : ConvGeom{g.N, g.HO, g.WO, g.NC, g.HA, g.WA, g.CA, g.R, g.S, g.stride, g.pad};
      const float4 old = accumulate ? *dst : make_float4(0.f, 0.f, 0.f, 0.f);
      const float init[4] = {old.x, old.y, old.z, old.w};
#pragma unroll
      for (int e = 0; e < 4; ++e)
        o[e] = MODE == 0 ? conv_direct_fwd_at(A, Bw, d, n, a_, b_, col + e) : conv_direct_dgrad_at(A, Bw, d, n, a_, b_, col + e, init[e]);
    }
    if (MODE == 0) {
      if (ep_a) {
        const float4 ea = *reinterpret_cast<const float4*>(ep_a + col), eb = *reinterpret_cast<const float4*>(ep_b + col);
        o[0] = fmaf(o[0], ea.x, eb.x); o[1] = fmaf(o[1], ea.y, eb.y); o[2] = fmaf(o[2], ea.z, eb.z); o[3] = fmaf(o[3], ea.w, eb.w);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = apply_act(o[e], act);
    }
    *dst = make_float4(o[0], o[1], o[2], o[3]);
  }
}

// dW[k][j] = sum over pixels of dy[m][k] * xcol[m][j], in pixel order (so bound by the chain on layers of many pixels and few
// weights: 16 cycles a pixel, 8 of them the products').  Both operands are contiguous along their channels; a gathered pixel is addressed once per
// four channels of a tap.
template <int TILE>
__device__ __forceinline__ void wgrad_f32_block(const Blk& blk, const float* __restrict__ dy, const float* __restrict__ x,
                                                float* __restrict__ dw, WgradTrArgs g) {
  typedef F32Tile<TILE> F;
  typedef F32Gemm<TILE> G;
  const int tid = threadIdx.x, lane = tid & 63, group = lane / TILE, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tile = xcd_contiguous(blk.x, g.tiles_k * g.tiles_j);
  const int k0 = (tile / g.tiles_j) * G::EDGE, j0 = (tile % g.tiles_j) * G::EDGE;
  const __amdgpu_buffer_rsrc_t rd = tensor_rsrc(dy, g.dy_bytes), rx = tensor_rsrc(x, g.x_bytes);

  const int kcol = k0 + G::template minor<false>(tid), jcol = j0 + G::template minor<false>(tid);   // (K, J, C are multiples of 8: four are in or out)
  const bool k_ok = kcol < g.K;
  // the two pixels of the next stage: of dy, of x, both advanced by additions (pixels past the end lie past both tensors: zeros)
  const WgradSteps steps = wgrad_steps<4>(g);
  WgradPixel px[2];
  unsigned dm[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = G::template major<false>(tid, i);
    px[i].template init<4>(g, jcol, m);
    dm[i] = (unsigned)(m * g.K + kcol) * 4u;
  }
  const unsigned d_step = (unsigned)(G::BK * g.K) * 4u;
  auto load_dy = [&](int i) {
    const unsigned off = dm[i];
    dm[i] += d_step;
    return buffer_load_f4(rd, k_ok ? off : kOutOfRange);
  };
  auto load_x = [&](int i) {
    const unsigned off = px[i].in_image(steps) ? px[i].off : kOutOfRange;
    px[i].advance(steps);
    return buffer_load_f4(rx, off);
  };
  typename F::Acc acc;
#pragma unroll
  for (int v = 0; v < F::VALUES; ++v) acc[v] = 0.f;
  G::template run<false, false>(load_x, load_dy, acc, (g.M + G::BK - 1) / G::BK, tid);

  // lane: row k of dW, runs of four columns
  const int k = k0 + (wave & 1) * TILE + lane % TILE;
#pragma unroll
  for (int q = 0; q < F::VALUES / 4; ++q) {
    const int j = j0 + (wave >> 1) * TILE + F::row(q, group);
    if (k >= g.K || j >= g.J) continue;
    float o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = acc[4 * q + e];
    if (o[0] != o[0] || o[1] != o[1] || o[2] != o[2] || o[3] != o[3]) {
      const ConvGeom d{g.N, g.H, g.W, g.C, g.P, g.Q, g.K, g.R, g.S, g.stride, g.pad};
      const int rs = j / g.C;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = conv_direct_wgrad_at(dy, x, d, k, rs / g.S, rs % g.S, j - rs * g.C + e);
    }
    *reinterpret_cast<float4*>(dw + (size_t)k * g.J + j) = make_float4(o[0], o[1], o[2], o[3]);
  }
}
template <int TILE>
__global__ __launch_bounds__(256) void wgrad_f32_kernel(const float* __restrict__ dy, const float* __restrict__ x,
                                                       float* __restrict__ dw, WgradTrArgs g) {
  wgrad_f32_block<TILE>(one_block(), dy, x, dw, g);
}

}  // namespace pbd
