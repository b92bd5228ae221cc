"""The launch rules of ``csrc/launch_rules.h`` for tests: host code without a GPU, compiled on its own with g++."""
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_20438_amd", "csrc")
SHIM = """#include "launch_rules.h"
extern "C" int splits(int dtype, int R, int Hk, int hd, int kv_max) {
  return ham::attn_decode_splits(dtype, R, Hk, hd, kv_max);
}
extern "C" int prompt_keys(int R, int s0, int T, int H, int Hk) { return ham::prompt_attn_grid(R, s0, T, H, Hk).keys; }
extern "C" int prompt_blocks(int R, int s0, int T, int H, int Hk) { return ham::prompt_attn_grid(R, s0, T, H, Hk).blocks; }
extern "C" int rows_takes(int M, int N) { return ham::gemm_rows_takes(M, N); }
"""


@functools.lru_cache(None)
def rules():
    """Library with ``splits(dtype, rows, n_kv_heads, head_dim, kv_max)``, ``rows_takes(M, N)`` and ``prompt_keys`` /
    ``prompt_blocks(rows, first input, inputs of a sequence, n_heads, n_kv_heads)``."""
    with tempfile.TemporaryDirectory() as d:
        src, out = os.path.join(d, "rules.cpp"), os.path.join(d, "rules.so")
        with open(src, "w") as f:
            f.write(SHIM)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, src, "-o", out], check=True)
        return ctypes.CDLL(out)
