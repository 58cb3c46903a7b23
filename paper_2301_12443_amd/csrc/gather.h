// Offsets of what the direct-to-LDS convolution kernel gathers, plain C++: the kernel, the launch rule and the CPU tests use the same functions.
#pragma once

namespace pbd {

// The byte range of the gathered tensor's descriptor, and the offset of a lane that is to get zeros.  The hardware passes a load whose
// vector offset is below the range less its scalar offset (never wrapped: both end at the range).
constexpr unsigned kGatherRange = 0xC0000000u;

// The descriptor begins `before` elements ahead of the tensor, so that a tap's offset, the scalar one, is never negative; the row's is
// fixed.  A load's byte is row + tap - 2 before.
struct Gather {
  bool forward;          // else backward-data: the taps go backwards from the row's pixel
  int R, S, pad;
  int width;             // pixels of a row of the tensor
  int column;            // elements from one column to the next: a pixel; backward-data of stride 2, which counts dx's, half a pixel of dy
  constexpr unsigned elems(int row, int col) const { return ((unsigned)row * (unsigned)width + (unsigned)col) * (unsigned)column; }
  constexpr unsigned before() const { return forward ? elems(pad, pad) : elems(R - 1, S - 1); }
  // the window's corner (backward-data: dx's pixel and the padding) in the image that begins at element `image`, channel c
  constexpr unsigned row(unsigned image, int h, int w, int c) const { return (image + elems(h, w) + (unsigned)c + (forward ? before() : 0u)) * 2u; }
  constexpr unsigned tap(int r, int s, int c) const { return ((forward ? elems(r, s) : before() - elems(r, s)) + (unsigned)c) * 2u; }
  // Does every load of a tensor of this many bytes, whose taps are `run` elements long, keep to the range?  What lies ahead of the tensor
  // counts too, and so does the last tap: a few image rows, which is nothing unless the whole batch has no more (batch x height 1: 3 x 3 up to
  // 1.5 GiB forward and 1 GiB backward, 5 x 5 0.75 and 0.6 GiB).
  constexpr bool in_range(long bytes, int run) const {
    const long ahead = forward ? ((long)pad * width + pad) * column : ((long)(R - 1) * width + S - 1) * column;
    const long tap = (forward ? ((long)(R - 1) * width + S - 1) * column : ahead) + run;
    return bytes + 2 * ahead <= (long)kGatherRange && 2 * tap <= (long)kGatherRange;
  }
};

}  // namespace pbd
