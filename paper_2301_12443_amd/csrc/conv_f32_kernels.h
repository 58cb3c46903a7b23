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
// Measured, us, with the addresses and lane exchanges in the multiplying waves / with loaders: forward 64 -> 64, 3 x 3, 65536 pixels 57 / 51 (95
// TFLOP/s), 256 -> 256, 4096 60 / 48, 512 -> 512, 1024 79 / 52 (93), 256 pixels 46 / 25; weight gradient of 64 -> 64, 1 x 1 over 65536 pixels 420 /
// 284 (10.4 cycles a pixel), of 8 -> 16, 3 x 3 over 8192 55 / 38; VGG-16 at 64 x 32 x 32 1655 / 1295 a step with six stages throughout (91 ms with one thread per result).
// Cutting a reduction over eight waves and adding the parts (other bits) is faster still where the chain is long.
#pragma once
#include "conv_kernels.h"

namespace pbd {

typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 buffer_load_f4(__amdgpu_buffer_rsrc_t r, unsigned byte_off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte_off, 0, 0));
}

template <int TILE> struct F32Tile;
template <> struct F32Tile<32> {
  typedef f32x16 Acc;
  static constexpr int GROUPS = 2, VALUES = 16;       // reduction elements per MFMA, results per lane
  // tile row of a lane's four results 4 q .. 4 q + 3
  static __device__ __forceinline__ int row(int q, int group) { return 8 * q + 4 * group; }
  static __device__ __forceinline__ Acc mfma(float a, float b, Acc c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
};
template <> struct F32Tile<16> {
  typedef f32x4 Acc;
  static constexpr int GROUPS = 4, VALUES = 4;
  static __device__ __forceinline__ int row(int, int group) { return 4 * group; }
  static __device__ __forceinline__ Acc mfma(float a, float b, Acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};

__device__ __forceinline__ void pin(float& v) { asm volatile("" : "+v"(v)); }
// the result arrives later: only use it behind wait_lgkmcnt + pin()
template <int OFF> __device__ __forceinline__ float lds_read4_async(unsigned addr) {
  static_assert(OFF >= 0 && OFF < 65536, "a 16-bit offset");
  float v;
  asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
// f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>)
template <class F, int... I> __device__ __forceinline__ void unrolled(F&& f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F> __device__ __forceinline__ void unrolled(F&& f) { unrolled(f, std::make_integer_sequence<int, N>{}); }

// The product both kernels share.  A workgroup owns EDGE x EDGE = 2 x 2 tiles of Out[p][q] = sum_e P[p][e] Q[q][e] and their whole
// reduction, in stages of BK elements (sixteen MFMAs).  Four waves multiply, one tile each; four others, one on each SIMD beside them, bring
// the operands from memory straight into a ring of NS stages in LDS.
//   Why waves of their own: an MFMA that needs the one before follows it after 32 (64) cycles, and LDS reads, scalar operations and
// waits between the two are free, but one vector operation costs 14 cycles and every further one 4 (measured on chains of 1024).  With the
// addresses and the exchange of lanes in the same waves a product took 64 cycles; here the chain has nothing between its
// products but two LDS reads, all of whose addresses are a register and a constant.
//  * ROWS: the operand's memory is contiguous along the reduction, [p][element] in LDS; else along p, [element][p].  A load brings a block of
//    1 KiB: rows (elements) of 4 TILE .. bytes, their 16-byte chunks permuted.  ROWS: chunk c of row r in slot c ^ (r % 4 or r / 2 % 4), blocks 64
//    bytes apart; else chunk c of element e in slot c ^ half a row where element bit 1 (TILE 32: bit 0) is set.  The lanes of a read, one float
//    each, go 32 at a time to 32 banks; they lie on 16 of them (TILE 32, ROWS: on 8), so a read takes 4 (8) LDS cycles instead of 2 (counted:
//    SQ_LDS_IDX_ACTIVE, 50 and 75 % of it conflicts).  Beside the 32 (64) of a product on each of four SIMDs that just fits.
// A stage's barrier: the loaders have seen its loads land, the multiplying waves have read the stage before.  They read stage t while
// they multiply stage t - 1.
constexpr int kF32Threads = 512;
constexpr int f32_stage(int tile) { return tile == 32 ? 32 : 64; }      // elements of the reduction a stage
template <int TILE, int NS> struct F32Gemm {
  typedef F32Tile<TILE> F;
  static constexpr int EDGE = 2 * TILE, BK = f32_stage(TILE);                                    // 32 and 64, 64 and 32
  static_assert(BK == 16 * F::GROUPS, "sixteen products a stage");
  template <bool ROWS> static constexpr int block_bytes() { return ROWS ? 1024 + 64 : 1024; }
  template <bool P_ROWS, bool Q_ROWS> static constexpr int stage_bytes() { return 8 * (block_bytes<P_ROWS>() + block_bytes<Q_ROWS>()); }
  // what lane `lane` of loader w brings in pass i = 0, 1 (block w + 4 i): row / element, and the first of its four elements / rows
  template <bool ROWS> static __device__ __forceinline__ int major(int lane, int w, int i) {
    return (ROWS ? TILE == 16 : TILE == 32) ? 4 * (w + 4 * i) + lane / 16 : 8 * (w + 4 * i) + lane / 8;
  }
  template <bool ROWS> static __device__ __forceinline__ int minor(int lane) {
    if (ROWS) return 4 * (TILE == 16 ? (lane % 16) ^ (lane / 16) : (lane % 8) ^ (lane / 16));
    return 4 * (TILE == 16 ? (lane % 8) ^ (4 * (lane / 16 % 2)) : (lane % 16) ^ (8 * (lane / 16 % 2)));
  }
  // A multiplying lane's LDS address of reduction element (s, group) of its row `at` of the EDGE: address register s % 4 (ROWS) or 0 ...
  template <bool ROWS> static __device__ __forceinline__ unsigned base(int at, int group, int r) {
    if (!ROWS) return TILE == 16 ? (unsigned)(group * 128 + ((at ^ (group / 2 * 16)) * 4)) : (unsigned)(group * 256 + ((at ^ (group * 32)) * 4));
    if (TILE == 16) return (unsigned)(at / 4 * block_bytes<true>() + at % 4 * 256 + (r ^ (at % 4)) * 16 + group * 4);
    return (unsigned)(at / 8 * block_bytes<true>() + at % 8 * 128 + (r ^ (at / 2 % 4)) * 16 + group * 4);
  }
  // ... and constant.  (TILE 32, ROWS: two products share a chunk)
  template <bool ROWS> static constexpr int reg(int s) { return !ROWS ? 0 : TILE == 16 ? s % 4 : s / 2 % 4; }
  template <bool ROWS> static constexpr int offset(int s) { return !ROWS ? s * 512 : TILE == 16 ? s / 4 * 64 : s / 8 * 64 + s % 2 * 8; }

  // The loaders' part.  load_p(i, at), load_q(i, at): bring pass i = 0, 1 of the next stage of an operand to the 1 KiB from `at` on
  template <bool P_ROWS, bool Q_ROWS, class LP, class LQ>
  static __device__ __forceinline__ void bring(unsigned char* ring, LP&& load_p, LQ&& load_q, int stages, int w) {
    constexpr int STAGE = stage_bytes<P_ROWS, Q_ROWS>(), BP = block_bytes<P_ROWS>(), BQ = block_bytes<Q_ROWS>();
    int slot = 0;
    auto load = [&] {
      unsigned char* at = ring + slot * STAGE;
#pragma unroll
      for (int i = 0; i < 2; ++i) load_p(i, at + (w + 4 * i) * BP);
#pragma unroll
      for (int i = 0; i < 2; ++i) load_q(i, at + 8 * BP + (w + 4 * i) * BQ);
      slot = slot + 1 == NS ? 0 : slot + 1;
    };
    for (int t = 0; t < min(NS - 1, stages); ++t) load();
    for (int t = 0; t < stages; ++t) {
      if (t + NS - 2 < stages) wait_vmcnt<4 * (NS - 2)>(); else wait_vmcnt<0>();
      block_barrier();                                 // stage t is in LDS, stage t - 1 has been read
      if (t + NS - 1 < stages) load();
    }
  }
  // The multiplying waves' part: wave 0 .. 3
  template <bool P_ROWS, bool Q_ROWS>
  static __device__ __forceinline__ void multiply(const unsigned char* ring, typename F::Acc& acc, int stages, int lane, int wave) {
    constexpr int STAGE = stage_bytes<P_ROWS, Q_ROWS>(), HALF = 3;      // (slots within reach of a constant)
    static_assert(NS % HALF == 0 && HALF * STAGE <= 65536, "every slot is a register and a constant");
    static_assert(6 % NS == 0, "a round of six turns leaves the slots where they were");
    const int group = lane / TILE, at_p = (wave >> 1) * TILE + lane % TILE, at_q = (wave & 1) * TILE + lane % TILE;
    unsigned ap[NS / HALF][4], aq[NS / HALF][4];
    const unsigned ring_at = (unsigned)(size_t)(lds_void_ptr)ring;
#pragma unroll
    for (int h = 0; h < NS / HALF; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        ap[h][r] = ring_at + h * HALF * STAGE + base<P_ROWS>(at_p, group, r);
        aq[h][r] = ring_at + h * HALF * STAGE + 8 * block_bytes<P_ROWS>() + base<Q_ROWS>(at_q, group, r);
      }
    float fp[2][16], fq[2][16];
    // one stage: set t % 2 is read from its slot while the other set, the stage before, is multiplied
    auto turn = [&](auto number, auto multiplies) {
      constexpr int T = decltype(number)::value, SET = T % 2, SLOT = T % NS, H = SLOT / HALF, AT = SLOT % HALF * STAGE;
      constexpr bool MUL = decltype(multiplies)::value;
      block_barrier();
      unrolled<16>([&](auto m) {
        constexpr int M = decltype(m)::value;
        if constexpr (MUL) acc = F::mfma(fp[SET ^ 1][M], fq[SET ^ 1][M], acc);
        __builtin_amdgcn_sched_barrier(0);
        unrolled<3>([&](auto u) {                      // (all of them requested by the eleventh product: the others cover the last's way)
          constexpr int R = 3 * M + decltype(u)::value, S = R / 2;
          if constexpr (R < 32) {
            if constexpr (R % 2 == 0) fp[SET][S] = lds_read4_async<AT + offset<P_ROWS>(S)>(ap[H][reg<P_ROWS>(S)]);
            else fq[SET][S] = lds_read4_async<AT + offset<Q_ROWS>(S)>(aq[H][reg<Q_ROWS>(S)]);
          }
        });
        __builtin_amdgcn_sched_barrier(0);
      });
      // (what was multiplied lives to here, so that no read lands in a register that a product on its way still takes)
      if constexpr (MUL) {
#pragma unroll
        for (int m = 0; m < 16; ++m) asm volatile("" ::"v"(fp[SET ^ 1][m]), "v"(fq[SET ^ 1][m]));
      }
      wait_lgkmcnt<0>();
#pragma unroll
      for (int m = 0; m < 16; ++m) { pin(fp[SET][m]); pin(fq[SET][m]); }
    };
    auto last = [&](auto number) {                     // the products of stage `number`
      constexpr int SET = decltype(number)::value % 2;
#pragma unroll
      for (int m = 0; m < 16; ++m) acc = F::mfma(fp[SET][m], fq[SET][m], acc);
    };
    using Yes = std::true_type;
    turn(std::integral_constant<int, 0>{}, std::false_type{});
    int t = 1;
    for (; t + 6 <= stages; t += 6) unrolled<6>([&](auto u) { turn(std::integral_constant<int, (1 + decltype(u)::value) % 6>{}, Yes{}); });
    // 0 .. 5 stages are left, numbered 1 .. 5 (mod 6); then the products of the last
    const int left = stages - t;
    unrolled<5>([&](auto u) { if (left > decltype(u)::value) turn(std::integral_constant<int, 1 + decltype(u)::value>{}, Yes{}); });
    if (left % 2 == 0) last(std::integral_constant<int, 0>{}); else last(std::integral_constant<int, 1>{});
  }
};

// Same view as igemm_kernel: Out[m][j] = sum_kk Agather(m, kk) * W(j, kk), rows m = pixels of an [N][HO][WO] grid,
// kk = (r*S + s)*CA + c.  MODE 0 reads the weights as they lie, [NC][R][S][CA]; MODE 1 reads the forward filter
// [CA][R][S][NC], so there is no transposed copy to keep.
template <int MODE, int TILE, int NS>
__global__ __launch_bounds__(512) void igemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ Bw,
                                                       float* Out, const float* __restrict__ ep_a,
                                                       const float* __restrict__ ep_b, int act, int accumulate, IgemmArgs g) {
  typedef F32Tile<TILE> F;
  typedef F32Gemm<TILE, NS> G;
  constexpr bool W_ROWS = MODE == 0;
  __shared__ __attribute__((aligned(16))) unsigned char ring[NS * G::template stage_bytes<W_ROWS, true>()];
  const int tid = threadIdx.x, lane = tid & 63, group = lane / TILE, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tile = xcd_contiguous(blockIdx.x, g.tiles_m * g.tiles_n);
  const int m0 = tile / g.tiles_n * G::EDGE, n0 = tile % g.tiles_n * G::EDGE;
  const int sh = g.stride == 2 ? 1 : 0, smask = g.stride - 1;
  const __amdgpu_buffer_rsrc_t ra = tensor_rsrc(A, g.a_bytes), rb = tensor_rsrc(Bw, g.b_bytes);
  const int stages = (g.Kred + G::BK - 1) / G::BK, RS = g.R * g.S;
  if (wave >= 4) {                                     // a loader
    const int w = wave - 4, c4 = G::template minor<true>(lane);
    // pixels: two rows of four elements a stage
    int at[2], rh[2], rw[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int m = m0 + G::template major<true>(lane, w, i), mm = m < g.M ? m : 0;
      const int b_ = mm % g.WO, t = mm / g.WO, a_ = t % g.HO;
      rh[i] = MODE == 0 ? a_ * g.stride - g.pad : a_ + g.pad;
      rw[i] = MODE == 0 ? b_ * g.stride - g.pad : b_ + g.pad;
      at[i] = (t / g.HO) * g.HA * g.WA * g.CA + ((rh[i] * g.WA + rw[i]) * g.CA >> (MODE == 1 ? sh : 0));
      if (m >= g.M) rh[i] = -(1 << 24);                // (fails every range test)
    }
    const unsigned hlim = MODE == 0 ? (unsigned)g.HA : (unsigned)g.HA << sh, wlim = MODE == 0 ? (unsigned)g.WA : (unsigned)g.WA << sh;
    if (g.CA % G::BK == 0) {
      // A stage lies inside one tap: its position is scalar, and whether the tap lies in the image is two bits of a mask that is set up
      // once, its row's and its column's.  The few vector operations matter: beside a chain of products on the same SIMD one takes ~13 cycles.
      unsigned skip[2], aoff[2];
      unsigned woff[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        unsigned in = 0;
        for (int q = 0; q < g.S; ++q) {
          const int x = MODE == 0 ? rw[i] + q : rw[i] - q;
          in |= ((unsigned)x < wlim && (MODE == 0 || (x & smask) == 0) ? 1u : 0u) << q;
        }
        for (int q = 0; q < g.R; ++q) {
          const int y = MODE == 0 ? rh[i] + q : rh[i] - q;
          in |= ((unsigned)y < hlim && (MODE == 0 || (y & smask) == 0) ? 1u : 0u) << (g.S + q);
        }
        skip[i] = ~in;
        aoff[i] = (unsigned)(at[i] + c4) * 4u;
        const int k = MODE == 0 ? c4 : G::template major<false>(lane, w, i);
        const int bat = n0 + (MODE == 0 ? G::template major<true>(lane, w, i) : G::template minor<false>(lane));
        woff[i] = bat < g.NC ? (unsigned)(MODE == 0 ? bat * g.Kred + k : k * RS * g.NC + bat) * 4u : kOutOfRange;
      }
      int r = 0, q = 0, c = 0;
      auto load_weights = [&](int i, unsigned char* dst) {
        const int tap = r * g.S + q;
        dma_load16(rb, dst, woff[i], (unsigned)(MODE == 0 ? tap * g.CA + c : (c * RS + tap) * g.NC) * 4u);
      };
      auto load_pixels = [&](int i, unsigned char* dst) {
        const unsigned here = 1u << q | 1u << (g.S + r);
        const int add = MODE == 0 ? (r * g.WA + q) * g.CA + c : c - ((r * g.WA + q) * g.CA >> sh);
        dma_load16(ra, dst, skip[i] & here ? kOutOfRange : aoff[i] + (unsigned)(add * 4));
        if (i == 0) return;
        c += G::BK;                                    // (the pixels come last)
        if (c == g.CA) { c = 0; if (++q == g.S) { q = 0; ++r; } }
      };
      G::template bring<W_ROWS, true>(ring, load_weights, load_pixels, stages, w);
      return;
    }
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
    Tap ta = tap_of(c4);
    auto load_pixels = [&](int i, unsigned char* dst) {
      int h = MODE == 0 ? rh[i] + ta.r : rh[i] - ta.r, w = MODE == 0 ? rw[i] + ta.s : rw[i] - ta.s;
      bool ok = ta.kk < g.Kred;
      if (MODE == 1) { ok &= ((h | w) & smask) == 0; h >>= sh; w >>= sh; }
      ok &= ((unsigned)h < (unsigned)g.HA) & ((unsigned)w < (unsigned)g.WA);
      const unsigned off = (unsigned)(at[i] + ta.off) * 4u;
      if (i == 1) next_stage(ta);
      dma_load16(ra, dst, ok ? off : kOutOfRange);
    };
    // weights: MODE 0 two channels' four elements, MODE 1 two elements' four channels (NC % 8 == 0: in or out as a whole).  Offsets of the elements
    // kk and, MODE 1, channel and tap of each, advanced by additions; an element past the last is out of range there or not asked for.
    int wk[2], wc[2], woff[2];
    bool w_in[2];
  #pragma unroll
    for (int i = 0; i < 2; ++i) {
      wk[i] = MODE == 0 ? G::template minor<true>(lane) : G::template major<false>(lane, w, i);
      const int bat = n0 + (MODE == 0 ? G::template major<true>(lane, w, i) : G::template minor<false>(lane));
      w_in[i] = bat < g.NC;
      wc[i] = wk[i] % g.CA;
      woff[i] = MODE == 0 ? bat * g.Kred + wk[i] : (wc[i] * RS + wk[i] / g.CA) * g.NC + bat;
    }
    const int w_step = (dc * RS + dtap) * g.NC, w_wrap = (1 - g.CA * RS) * g.NC;
    auto load_weights = [&](int i, unsigned char* dst) {
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
      dma_load16(rb, dst, off);
    };
    G::template bring<W_ROWS, true>(ring, load_weights, load_pixels, stages, w);
    return;
  }

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
  G::template multiply<W_ROWS, true>(ring, acc, stages, lane, wave);

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
// weights: 10 cycles a pixel, 8 of them the products').  Both operands are contiguous along their channels; a gathered pixel is addressed once per
// four channels of a tap.
template <int TILE, int NS>
__device__ __forceinline__ void wgrad_f32_block(const Blk& blk, const float* __restrict__ dy, const float* __restrict__ x,
                                                float* __restrict__ dw, WgradTrArgs g) {
  typedef F32Tile<TILE> F;
  typedef F32Gemm<TILE, NS> G;
  __shared__ __attribute__((aligned(16))) unsigned char ring[NS * G::template stage_bytes<false, false>()];
  const int tid = threadIdx.x, lane = tid & 63, group = lane / TILE, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tile = xcd_contiguous(blk.x, g.tiles_k * g.tiles_j);
  const int k0 = (tile / g.tiles_j) * G::EDGE, j0 = (tile % g.tiles_j) * G::EDGE;
  const __amdgpu_buffer_rsrc_t rd = tensor_rsrc(dy, g.dy_bytes), rx = tensor_rsrc(x, g.x_bytes);

  const int stages = (g.M + G::BK - 1) / G::BK;
  if (wave >= 4) {                                     // a loader
    const int w = wave - 4, c4 = G::template minor<false>(lane);
    const int kcol = k0 + c4, jcol = j0 + c4;          // (K, J, C are multiples of 8: four are in or out)
    // the two pixels of the next stage: of dy, and of x where one pixel of x meets one of dy, a scalar moves on (pixels past the end lie past
    // both tensors: zeros); else those of x are advanced by additions
    unsigned dm[2], xm[2], d_at = 0, x_at = 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int m = G::template major<false>(lane, w, i);
      dm[i] = kcol < g.K ? (unsigned)(m * g.K + kcol) * 4u : kOutOfRange;
      xm[i] = jcol < g.J ? (unsigned)(m * g.C + jcol) * 4u : kOutOfRange;
    }
    auto load_dy = [&](int i, unsigned char* dst) {
      dma_load16(rd, dst, dm[i], d_at);
      if (i == 1) d_at += (unsigned)(G::BK * g.K) * 4u;
    };
    if (g.R * g.S == 1 && g.stride == 1 && g.pad == 0) {
      auto load_x = [&](int i, unsigned char* dst) {
        dma_load16(rx, dst, xm[i], x_at);
        if (i == 1) x_at += (unsigned)(G::BK * g.C) * 4u;
      };
      G::template bring<false, false>(ring, load_x, load_dy, stages, w);
      return;
    }
    // Whole rows of the image a stage, and whole stages an image (or whole images a stage), as in images of 2^n pixels: a lane's column stays, its row moves
    // on by a scalar, and four vector operations are left of eighteen (chain of 8192 pixels, 3 x 3, 32 x 32 images: 51 -> 38 us)
    const int rows = G::BK / g.Q;
    if (G::BK % g.Q == 0 && (g.P % rows == 0 || rows % g.P == 0)) {
      int h[2], off[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int m = G::template major<false>(lane, w, i), rs = jcol / g.C, c = jcol - rs * g.C;
        const int wx = m % g.Q * g.stride + rs % g.S - g.pad, p = m / g.Q % g.P, n = m / (g.P * g.Q);
        h[i] = p * g.stride + rs / g.S - g.pad;
        off[i] = (((n * g.H + h[i]) * g.W + wx) * g.C + c) * 4;
        if (jcol >= g.J || (unsigned)wx >= (unsigned)g.W) h[i] = 1 << 30;        // (fails every range test)
      }
      int row = 0, image = 0;                          // of dy, of the stage's first pixel
      auto load_x = [&](int i, unsigned char* dst) {
        const int ahead = ((image * g.H + row * g.stride) * g.W * g.C) * 4;
        dma_load16(rx, dst, (unsigned)(h[i] + row * g.stride) < (unsigned)g.H ? (unsigned)(off[i] + ahead) : kOutOfRange);
        if (i == 0) return;
        if (rows > g.P) image += rows / g.P;
        else if ((row += rows) == g.P) { row = 0; ++image; }
      };
      G::template bring<false, false>(ring, load_x, load_dy, stages, w);
      return;
    }
    const WgradSteps steps = wgrad_steps<4>(g);
    WgradPixel px[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) px[i].template init<4>(g, jcol, G::template major<false>(lane, w, i));
    auto load_x = [&](int i, unsigned char* dst) {
      dma_load16(rx, dst, px[i].in_image(steps) ? px[i].off : kOutOfRange);
      px[i].advance(steps);
    };
    G::template bring<false, false>(ring, load_x, load_dy, stages, w);
    return;
  }
  typename F::Acc acc;
#pragma unroll
  for (int v = 0; v < F::VALUES; ++v) acc[v] = 0.f;
  G::template multiply<false, false>(ring, acc, stages, lane, wave);

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
template <int TILE, int NS>
__global__ __launch_bounds__(512) void wgrad_f32_kernel(const float* __restrict__ dy, const float* __restrict__ x,
                                                       float* __restrict__ dw, WgradTrArgs g) {
  wgrad_f32_block<TILE, NS>(one_block(), dy, x, dw, g);
}

}  // namespace pbd
