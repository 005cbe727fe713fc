"""The library's choice of tiles (csrc/gemm_choice.h, host code) for tests: compiled on its own, no GPU needed."""
import ctypes
import functools
import os
import subprocess
import tempfile
from collections import namedtuple

from paper_2409_12210_amd import build as B

SRC = """
#include <algorithm>
#include <cstring>
#include "gemm_choice.h"
extern "C" void choice(int d, int N, const int* f, int k, int T, int dtype, int epilogue, int* out) {
  LayerDims L;
  std::memset(&L, 0, sizeof L);
  L.d = d; L.N = N; L.k = k; L.T = T;
  for (int e = 0; e < N; ++e) { L.f[e] = f[e]; L.foff[e + 1] = L.foff[e] + f[e]; L.order[e] = e; }
  std::stable_sort(L.order, L.order + N, [&](int a, int b) { return L.f[a] > L.f[b]; });
  const auto c = modse_gemm::gemm_choice(L, (modse_dtype)dtype, epilogue);
  out[0] = c.tile.bm; out[1] = c.tile.bn; out[2] = c.kchunk;
}
extern "C" int by_hist(int d, int N, int k, int T, int elem_size, int with_rows) {
  LayerDims L;
  std::memset(&L, 0, sizeof L);
  L.d = d; L.N = N; L.k = k; L.T = T;
  return permute_by_hist(L, elem_size, with_rows != 0);
}
"""
GEMMS = {"up": 2, "down": 0, "dh": 3, "dx": 4, "wgrad": 1}  # the GemmEpilogue that names each of the five products
Choice = namedtuple("Choice", "bm bn kchunk")               # kchunk: 0 = K not split


@functools.lru_cache(None)
def _lib():
    out = tempfile.mkdtemp()
    src, so = os.path.join(out, "probe.hip"), os.path.join(out, "probe.so")
    with open(src, "w") as f:
        f.write(SRC)
    subprocess.run([B._hipcc(), "-x", "hip", "--offload-host-only", "-std=c++17", "-shared", "-fPIC",
                    "-I" + os.path.join(B.ROOT, "include"), "-I" + B.CSRC, src, "-o", so], check=True)
    return ctypes.CDLL(so)


def choice(gemm, d, d_ff, k, T, dtype):
    out = (ctypes.c_int * 3)()
    _lib().choice(d, len(d_ff), (ctypes.c_int * len(d_ff))(*d_ff), k, T, 0 if dtype == "f32" else 1, GEMMS[gemm], out)
    return Choice(*out)


def permute_by_hist(d, n_experts, k, T, dtype, with_rows):
    return bool(_lib().by_hist(d, n_experts, k, T, 4 if dtype == "f32" else 2, int(with_rows)))
