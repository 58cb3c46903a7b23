// One launch for several independent problems of the same kernel: the candidates of a mixed layer, whose chains of small kernels
// (48 to 300 workgroups of a few microseconds each) would otherwise follow one another.  Six candidates a layer, search step of the
// MobileNetV2 supernet at batch 16: 4204 profiled launches and 37.7 ms of kernel time -> 1491 and 24.6 (an empty launch behind another costs
// 2.4 us, and a grid of one candidate leaves most of the chip idle), 23.5 -> 18.6 ms; the weight step at batch 64 35.6 -> 34.0 ms.
//
// A kernel that takes part is written as a __device__ function K_block(blk, arguments ...) that reads its place in the grid from `blk`;
// its __global__ form is K_kernel.  many_kernel<K_block, ...> runs the workgroups of up to kManyMax problems one after the other in
// one grid: workgroup w belongs to the last problem p with start[p] <= w and is workgroup w - start[p] of that problem's own grid.
// Every start is a multiple of 8, so a workgroup meets the same XCD as in a launch of its own (xcd_contiguous).
#pragma once
#include <hip/hip_runtime.h>

namespace pbd {

struct Blk { int x, y, z, gx, gy; };       // place in the grid, and the grid's width and height
__device__ __forceinline__ Blk one_block() { return Blk{(int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z, (int)gridDim.x, (int)gridDim.y}; }

// a kernel's arguments as one plain value
template <class... A> struct Pack {};
template <class H, class... T> struct Pack<H, T...> { H head; Pack<T...> tail; };
inline void pack_up(Pack<>&) {}
template <class H, class... T> inline void pack_up(Pack<H, T...>& p, const H& h, const T&... t) { p.head = h; pack_up(p.tail, t...); }
// f(values before ..., the pack's values ...)
template <class F, class... D> __host__ __device__ __forceinline__ void unpack_to(F&& f, const Pack<>&, const D&... d) { f(d...); }
template <class F, class H, class... T, class... D>
__host__ __device__ __forceinline__ void unpack_to(F&& f, const Pack<H, T...>& p, const D&... d) { unpack_to(f, p.tail, d..., p.head); }

constexpr int kManyMax = 8;
template <class P> struct Many {
  int n, start[kManyMax + 1], size[kManyMax];     // problems; first workgroup (a multiple of 8) and workgroups of each
  int gx[kManyMax], gy[kManyMax];
  P args[kManyMax];
};
// (the arguments stay in the kernel-argument segment: a problem's are read through scalar loads at its index)
template <auto Block, int THREADS, int WAVES, class P>
__global__ __launch_bounds__(THREADS, WAVES) void many_kernel(Many<P> m) {
  int p = 0;
  while (p + 1 < m.n && (int)blockIdx.x >= m.start[p + 1]) ++p;
  const int w = (int)blockIdx.x - m.start[p];
  if (w >= m.size[p]) return;
  const int gx = m.gx[p], gy = m.gy[p], yz = w / gx;
  const Blk blk{w - yz * gx, yz % gy, yz / gy, gx, gy};
  unpack_to([&](auto&... a) { Block(blk, a...); }, m.args[p]);
}

}  // namespace pbd
