"""The library's host-side choices by size (csrc/acc_plan.h), compiled with the host compiler: which kernel a call takes."""
import collections
import ctypes
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_SOURCE = r'''
#include "paper_2605_01255_amd/csrc/acc_plan.h"
using namespace acc;
extern "C" {
int gemm_tile(int64_t M, int64_t N, int64_t K, int persist_ok) { return (int)pick_gemm_tile(M, N, K, persist_ok != 0).tile; }
int gemm_one_round(int64_t M, int64_t N, int64_t K, int persist_ok) { return pick_gemm_tile(M, N, K, persist_ok != 0).one_round; }
int f32_tile(int64_t M, int64_t N, int64_t splits, int all_tiles) { return (int)pick_f32_tile(M, N, 0, splits, all_tiles != 0).tile; }
int f32_four_stages(int64_t M, int64_t N, int64_t k, int splits) { return pick_f32_tile(M, N, k, splits, true).deep; }
int factor_tile(int64_t M, int64_t N, int64_t K, int form) { return (int)pick_factor_tile(M, N, K, (form & 1) != 0, (form & 2) != 0); }
void sketch(int64_t n, int64_t channels, int64_t r, int64_t ld, int bf16_factor, int* out) {
  const SketchPlan p = plan_sketch(n, channels, r, ld, true, bf16_factor != 0, false);
  const int v[] = {p.fast, p.ch, p.rc, p.n_cslab * p.n_js, p.G, p.tokens_per_split, p.two_sums, p.room};
  for (int i = 0; i < 8; ++i) out[i] = v[i];
}
int raised_capacity() { return RaisedLimits::kKernels; }
int raised_lost(int kernels, int devices) {  // entries the table has forgotten after all were added
  static RaisedLimits table;
  int lost = 0;
  for (int d = 0; d < devices; ++d)
    for (int k = 1; k <= kernels; ++k) {
      if (table.has((const void*)(intptr_t)k, d)) ++lost;   // not added yet
      table.add((const void*)(intptr_t)k, d);
    }
  for (int d = 0; d < devices; ++d)
    for (int k = 1; k <= kernels; ++k) lost += table.has((const void*)(intptr_t)k, d) ? 0 : 1;
  return lost;
}
int f32_sketch_splits(int64_t n, int64_t channels, int64_t r, int f32_factor) {  // 0: the generic form
  const F32SketchPlan p = plan_f32_sketch(n, channels, r, f32_factor != 0);
  return p.stored ? (int)p.splits : 0;
}
int f32_shared_launch(int64_t M, int64_t N, int64_t n, int64_t out_n, int splits) { return f32_pair(M, N, splits, n, out_n); }
int f32_sketch_fits(int64_t n, int64_t channels, int64_t r, int f32_factor) {
  const F32SketchPlan p = plan_f32_sketch(n, channels, r, f32_factor != 0);
  const int64_t partials = p.splits == 1 && f32_factor ? 0 : p.splits * channels * r;
  return !p.stored || n * r + partials <= generic_sketch_splits(n, channels, r) * channels * r;
}
}
'''


@functools.lru_cache(maxsize=None)
def lib():
    with tempfile.TemporaryDirectory() as tmp:
        src, out = os.path.join(tmp, "plan.cpp"), os.path.join(tmp, "plan.so")
        with open(src, "w") as f:
            f.write(_SOURCE)
        subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-shared", "-fPIC", "-I" + ROOT, src, "-o", out], check=True)
        so = ctypes.CDLL(out)
    for name in ("gemm_tile", "gemm_one_round", "f32_tile", "f32_sketch_splits", "f32_sketch_fits", "factor_tile", "f32_four_stages"):
        getattr(so, name).argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int]
    so.sketch.argtypes = [ctypes.c_int64] * 4 + [ctypes.c_int, ctypes.c_void_p]
    so.f32_shared_launch.argtypes = [ctypes.c_int64] * 4 + [ctypes.c_int]
    return so


def gemm_tile(m, n, k, float_or_sum=False):
    """(tile of the bfloat16 product, whether it is one round): as fast_gemm chooses on the ring and persistent kernels."""
    persist = not float_or_sum and k > 128
    names = ("256x256", "256x192", "192x128", "128x128", "128x64", "64x64")
    return names[lib().gemm_tile(m, n, k, persist)], bool(lib().gemm_one_round(m, n, k, persist))


def f32_tile(m, n, splits=1, both_f32=True):
    return ("64x64", "32x32", "128x64", "64x32")[lib().f32_tile(m, n, splits, both_f32)]


def f32_four_stages(m, n, k, splits=1):
    """Whether a float32 product on 32 x 32 or 64 x 32 tiles has four stages, two otherwise."""
    return bool(lib().f32_four_stages(m, n, k, splits))


def f32_sketch_splits(n, channels, r, f32_factor=True):
    """Token splits of a float32 layer's sketch with a stored S; 0 when the generic form runs."""
    return lib().f32_sketch_splits(n, channels, r, f32_factor)


def f32_sketch_fits(n, channels, r, f32_factor=True):
    """Whether S and the partial products fit the workspace of the generic form."""
    return bool(lib().f32_sketch_fits(n, channels, r, f32_factor))


def f32_pair(n, channels, other, r, f32_factor=True):
    """Token splits of a float32 layer's sketch (of `channels` columns) that shares a launch with the product of n tokens by
    `other` columns; 0: they do not share one."""
    splits = f32_sketch_splits(n, channels, r, f32_factor)
    return splits if splits and lib().f32_shared_launch(channels, r, n, other, splits) else 0


def factor_tile(m, n, k, bf16_c=True, added=False):
    """Kernel of a product of two gradient factors."""
    names = ("64x64", "128x64", "128x128", "192x128", "three-stage", "persistent", "")
    return names[lib().factor_tile(m, n, k, int(bf16_c) + 2 * int(added))] or gemm_tile(m, n, k, added or not bf16_c)[0]


Sketch = collections.namedtuple("Sketch", "tuned slab columns tiles splits tokens two_sums room")


def sketch(n, channels, r, bf16_factor=True, ld=0):
    """Plan of the bfloat16 sketch: channels of a slab and sketch columns of a tile, tiles, token splits, tokens of a split, whether it
    has two running sums, partial tiles that the workspace holds."""
    out = (ctypes.c_int * 8)()
    lib().sketch(n, channels, r, ld or channels, int(bf16_factor), out)
    return Sketch(bool(out[0]), *out[1:6], bool(out[6]), out[7])
