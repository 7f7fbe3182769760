"""The tile choice of the bf16 products (csrc/gemm_plan.h) compiled for the host."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TILES = ["32x32", "32x64", "64x64", "64x128", "128x128", "pair", "persistent"]
RING_STAGES = {"32x32": 16, "32x64": 6, "64x64": 4, "64x128": 6, "128x128": 4}
SRC = """
#include "gemm_plan.h"
extern "C" int plan_tile(int M, int N, int K, long long ld, int n_cu) {
  return tx::pick_tile(M, N, K, tx::persistent_shape(M, N, K, ld), n_cu);
}
extern "C" int plan_rows(int M, int N, int K, int n_cu) { return tx::persistent_rows(M, N, K, n_cu); }
"""


class Plan:
    def __init__(self, folder):
        src, out = os.path.join(str(folder), "plan.cpp"), os.path.join(str(folder), "plan.so")
        with open(src, "w") as f:
            f.write(SRC)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-Wno-unused-variable", "-shared", "-fPIC",
                        "-I" + os.path.join(ROOT, "paper_2607_28940_amd", "csrc"), src, "-o", out], check=True)
        self.lib = ctypes.CDLL(out)
        self.lib.plan_tile.argtypes = [ctypes.c_int] * 3 + [ctypes.c_longlong, ctypes.c_int]
        self.lib.plan_rows.argtypes = [ctypes.c_int] * 4

    def tile(self, M, N, K):
        return TILES[self.lib.plan_tile(M, N, K, max(N, K), 256)]

    def rows(self, M, N, K):
        """Rows the persistent kernel takes of a product of M."""
        return self.lib.plan_rows(M, N, K, 256)

    def launches(self, M, N, K):
        """(tile, rows) of each launch of a product."""
        out = []
        while M > 0:
            t = self.tile(M, N, K)
            m = self.rows(M, N, K) if t == "persistent" else M
            out.append((t, m))
            M -= m
        return out
