"""Tile choice and tile heights of the expert products, from the rule itself
(tiles.hpp compiled for the host), and the heights a call really used, from the
schedule it left at the start of its workspace."""
import ctypes
import os
import subprocess
import tempfile

import numpy as np

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2205_01848_amd", "csrc")
SRC = '''#include "tiles.hpp"
using namespace moe;
extern "C" int pays(int E, int64_t R, int64_t most, int N, int K, int gated, int act, int km, int64_t pa, int64_t pb, int cus) {
  return mid_pays({E, R, most, N, K, gated != 0, act != 0, km != 0, pa, pb}, cus);
}
// the schedule's choice: least time, the larger height on a tie
extern "C" int height(int E, const int* rows, int N, int K, int gated, int km, int64_t pa, int64_t pb, int f32, int cus) {
  int64_t best = 0;
  int pick = 0;
  for (int h = 1; h <= kMidMaxH; ++h) {
    int64_t n = 0;
    int hm = 0;
    for (int e = 0; e < E; ++e) {
      const int units = (rows[e] + kMidUnit - 1) / kMidUnit, t = (units + h - 1) / h;
      n += t;
      if (t && (units + t - 1) / t > hm) hm = (units + t - 1) / t;
    }
    const int tn = gated ? kMidN / 2 : kMidN, ks = f32 ? 32 : 64;
    const int64_t v = mid_time(n * ((N + tn - 1) / tn), hm, 2 * cus, (K + ks - 1) / ks,
                               f32 ? kStepF32 : step16(pa, pb, km != 0));
    if (h == 1 || v <= best) best = v, pick = h;
  }
  return pick;
}
'''
_lib = None


def lib():
    global _lib
    if _lib is None:
        tmp = tempfile.mkdtemp()
        src, so = os.path.join(tmp, "t.cpp"), os.path.join(tmp, "t.so")
        with open(src, "w") as f:
            f.write(SRC)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, src, "-o", so],
                       check=True)
        _lib = ctypes.CDLL(so)
        i, l = ctypes.c_int, ctypes.c_int64
        _lib.pays.argtypes = [i, l, l, i, i, i, i, i, l, l, i]
        _lib.height.argtypes = [i, ctypes.c_void_p, i, i, i, i, l, l, i, i]
    return _lib


def products(d, f, swiglu, es=2, wcopy=False):
    """(N, K, gated, act, K-major, A pitch, B pitch) of H, Y, dA and dX."""
    F = 2 * f if swiglu else f
    return [(f, d, int(swiglu), 1, 0, es * d, es * d), (d, f, 0, 0, 0, es * f, es * f),
            (f, d, 0, 1, 1, es * d, es * f), (d, F, 0, 0, int(not wcopy), es * F, es * (F if wcopy else d))]


def pays(E, R, product, cus=256, most=None):
    N, K, gated, act, km, pa, pb = product
    return bool(lib().pays(E, R, R if most is None else most, N, K, gated, act, km, pa, pb, cus))


def heights(rows, d, f, swiglu, f32, wcopy=False, cus=256):
    """The largest tile heights (units of 32 rows) of H, Y, dA and dX by the rule."""
    r = np.ascontiguousarray(rows, dtype=np.int32)
    out = []
    for N, K, gated, _, km, pa, pb in products(d, f, swiglu, 4 if f32 else 2, wcopy):
        h = lib().height(len(r), r.ctypes.data, N, K, gated, km, pa, pb, int(f32), cus)
        units = -(-r.astype(np.int64) // 32)
        n = -(-units // h)
        out.append(int((-(-units[n > 0] // n[n > 0])).max()) if (n > 0).any() else 0)
    return out


def used_heights(ws, E, R):
    """The largest heights of the two tile lists (N = f, N = d) in a workspace."""
    w = ws.detach().cpu().numpy().view(np.int32)
    up = lambda b: -(-b // 256) * 256
    n = w[1:3]
    mid = up(up(4 * (5 + 3 * 64)) + 8 * (-(-R // 256) + E)) // 4
    max_mid = -(-R // 32) + E
    return [int((w[mid + 2 * l * max_mid:][:2 * n[l]:2] >> 8).max()) if n[l] else 0 for l in range(2)]
