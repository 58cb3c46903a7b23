"""The direct-to-LDS convolution kernel's offsets (csrc/gather.h, compiled here for the host) against the range of its descriptor: a load reaches its
byte if its row's offset is below the range less its tap's, and a lane outside the image gets zeros if the range itself is not.  Where in_range
says so every load must keep to that, on tensors of up to the library's 2 GiB with few rows in the whole batch above all; where it does not, one
does not keep to it."""
import ctypes as C
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2301_12443_amd", "csrc")
RANGE = 0xC0000000
GIB = 1 << 30
LIMIT = 2 * GIB - 4096                # tensors end below this

SOURCE = """
#include "gather.h"
#define G pbd::Gather{f != 0, R, S, pad, w, c}
extern "C" {
unsigned range() { return pbd::kGatherRange; }
unsigned before(int f, int R, int S, int pad, int w, int c) { return G.before(); }
unsigned row(int f, int R, int S, int pad, int w, int c, unsigned image, int h, int x, int ch) { return G.row(image, h, x, ch); }
unsigned tap(int f, int R, int S, int pad, int w, int c, int r, int s, int ch) { return G.tap(r, s, ch); }
int in_range(int f, int R, int S, int pad, int w, int c, long bytes, int run) { return G.in_range(bytes, run); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("gather")
    (tmp / "gather.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-shared", "-fPIC", "-I" + CSRC, str(tmp / "gather.cpp"), "-o", str(tmp / "gather.so")], check=True)
    L = C.CDLL(str(tmp / "gather.so"))
    for f in (L.range, L.before, L.row, L.tap):
        f.restype = C.c_uint
    L.in_range.argtypes = [C.c_int] * 6 + [C.c_long, C.c_int]
    assert L.range() == RANGE
    return L


def _ends(n, k):
    return sorted(i for i in {*range(k + 1), n // 2, n // 2 + 1, *range(n - k - 1, n)} if 0 <= i < n)


def _keeps(lib, forward, n, rows, width, ch, k, stride, run=1):
    """Whether every load keeps to the range.  The gathered tensor is n x rows x width pixels of ch channels (forward: x; else dy, and the
    windows are dx's pixels); run: neighbouring pixels a tap reads as one (forward)."""
    pad, S = k // 2, 1 if run > 1 else k
    g = (int(forward), k, S, pad, width, ch if forward else ch // stride)
    before = lib.before(*g)
    grid_h = (rows + 2 * pad - k) // stride + 1 if forward else rows * stride
    grid_w = (width + 2 * pad - (run if run > 1 else k)) // stride + 1 if forward else width * stride
    for image in sorted({0, n // 2, n - 1}):
        for a in _ends(grid_h, k):
            for b in _ends(grid_w, k):
                h0, w0 = (a * stride - pad, b * stride - pad) if forward else (a + pad, b + pad)
                at = {c: lib.row(*g, image * rows * width * ch, h0, w0, c) for c in (0, ch - 8)}
                for r in range(k):
                    for s in range(S):
                        uni = lib.tap(*g, r, s, 0)
                        if uni > RANGE:                  # (the difference is negative: everything passes)
                            return False
                        for x in range(run):
                            p, q = (h0 + r, w0 + s + x) if forward else (h0 - r, w0 - s)
                            inside = forward or (p % stride == 0 and q % stride == 0)
                            p, q = (p, q) if forward else (p // stride, q // stride)
                            if not inside or not (0 <= p < rows and 0 <= q < width):
                                continue                 # the range itself: never below what is left of it
                            for c, off in at.items():
                                byte = ((image * rows + p) * width + q) * ch * 2 + c * 2
                                u = uni + x * ch * 2
                                if u > RANGE or not off < RANGE - u or off + u - 2 * before != byte:
                                    return False
    return True


def _in_range(lib, forward, n, rows, width, ch, k, stride, run=1):
    S = 1 if run > 1 else k
    return bool(lib.in_range(int(forward), k, S, k // 2, width, ch if forward else ch // stride, n * rows * width * ch * 2, ch * run))


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7])
@pytest.mark.parametrize("forward,stride", [(True, 1), (True, 2), (False, 1), (False, 2)])
@pytest.mark.parametrize("n,rows", [(1, 1), (1, 2), (2, 1), (1, 3), (4, 1), (1, 7), (3, 5), (1, 64)])
def test_every_load_in_range_or_the_layer_refused(lib, n, rows, forward, stride, k):
    last = True
    for size in (0.05, 0.3, 0.45, 0.55, 0.63, 0.72, 0.8, 0.95, 1.05, 1.25, 1.4, 1.6, 1.8, 2.0):
        ch = 64
        width = int(min(size * GIB, LIMIT)) // (n * rows * ch * 2)
        if not forward and stride == 2:
            width -= width % 2
        shape = (forward, n, rows, width, ch, k, stride)
        ok = _in_range(lib, *shape)
        assert last or not ok                            # the larger, the sooner
        last = ok
        assert ok == _keeps(lib, *shape), (size, ok)


def test_space_to_depth_stems(lib):
    for n, rows, size in ((1, 1, 0.5), (1, 1, 0.95), (2, 1, 0.95), (16, 112, 0.95), (1, 1, 0.03)):
        width = int(size * GIB) // (n * rows * 16 * 2)
        shape = (True, n, rows, width, 16, 4, 1, 4)
        ok = _in_range(lib, *shape)
        assert ok or n * rows < 3
        if ok:
            assert _keeps(lib, *shape)


@pytest.mark.parametrize("n,rows,width,ch,k,stride", [(256, 56, 56, 64, 3, 1), (256, 28, 28, 384, 3, 2), (256, 14, 14, 2048, 1, 1), (1, 224, 224, 64, 7, 1),
                                                      (1, 1, 8200, 64, 3, 1), (660, 56, 56, 512, 1, 1), (1490, 28, 28, 768, 3, 1)])
def test_ordinary_layers_are_in_range(lib, n, rows, width, ch, k, stride):
    for forward in (True, False):
        assert _in_range(lib, forward, n, rows, width, ch, k, stride) and _keeps(lib, forward, n, rows, width, ch, k, stride)
