"""The launch plans (host headers of the library without HIP) compiled with g++ for tests that run
without a GPU.  Test infrastructure only."""
from __future__ import annotations

import ctypes
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include "ahead_plan.h"
#include "attention_plan.h"
extern "C" {
size_t t_least(int B, int N_pad, int Hq, int Hkv, int Dh, int L) { return talon::attention_least_workspace(B, N_pad, Hq, Hkv, Dh, L); }
double t_us(int waves, long long wgs, int run, int splits, int Dh, size_t bytes) { return talon::plan_us(waves, wgs, run, splits, Dh, bytes); }
void t_ahead(int B, int N, int blocks, int k, int K_init, int init_layers, int max_depth, int resident, int* out) {
  const talon::AheadPlan p = talon::ahead_plan(B, N, blocks, k, K_init, init_layers, max_depth, resident);
  const int v[] = {p.layered, p.rows, p.head, p.chunks_head, p.chunks, p.scanners};
  for (int i = 0; i < 6; ++i) out[i] = v[i];
}
int t_literal_layered(int N, int K_init, int init_layers, int least, long long blocks, int resident, int capped, int cap_tried) {
  return talon::literal_layered(N, K_init, init_layers, least, blocks, resident, capped != 0, cap_tried);
}
void t_plan(int B, int N_pad, int Hq, int Hkv, int Dh, int L, size_t bytes, long long* out) {
  const talon::AttnPlan p = talon::attention_plan(B, N_pad, Hq, Hkv, Dh, L, bytes);
  const long long v[] = {p.waves, p.row_tiles, p.run_bound, p.split_max, p.split_likely, p.capacity_per_head, p.balance, p.run_single,
                         static_cast<long long>(p.partial), static_cast<long long>(p.bytes)};
  for (int i = 0; i < 10; ++i) out[i] = v[i];
}
}
"""
FIELDS = ("waves", "row_tiles", "run_bound", "split_max", "split_likely", "capacity_per_head", "balance", "run_single", "partial", "bytes")


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "plans.cpp"), os.path.join(d, "plans.so")
        with open(src, "w") as f:
            f.write(SHIM)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2601_07353_amd", "csrc"), src, "-o", so], check=True)
        lib = ctypes.CDLL(so)      # (the mapping outlives the file)
    lib.t_least.restype = ctypes.c_size_t
    lib.t_us.restype = ctypes.c_double
    lib.t_us.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_size_t]
    lib.t_literal_layered.argtypes = [ctypes.c_int] * 4 + [ctypes.c_longlong] + [ctypes.c_int] * 3
    lib.t_plan.argtypes = [ctypes.c_int] * 6 + [ctypes.c_size_t, ctypes.c_void_p]
    return lib


def least_workspace(B, N_pad, Hq, Hkv, Dh, L):
    return _lib().t_least(B, N_pad, Hq, Hkv, Dh, L)


def attention_plan(B, N_pad, Hq, Hkv, Dh, L, nbytes=None):
    """The plan of a call; by default with the workspace that the library's query asks for."""
    if nbytes is None:
        nbytes = 2 ** 64 - 1
    out = (ctypes.c_longlong * 10)()
    _lib().t_plan(B, N_pad, Hq, Hkv, Dh, L, nbytes, out)
    return dict(zip(FIELDS, out))


def plan_us(B, N_pad, Hq, Hkv, Dh, L, waves, splits):
    """The estimate for a number of splits."""
    row_tiles = -(-N_pad * (Hq // Hkv) // (32 * waves))
    wgs = B * Hkv * row_tiles * splits
    return _lib().t_us(waves, wgs, -(-((L + 63) // 64 + N_pad // 64) // splits), splits, Dh,
                       wgs * 32 * waves * (2 * Dh + 8) if splits > 1 else 256)


def ahead_plan(B, N, vocab, dtype, k, max_depth, K_init=None, init_layers=1, resident=1024):
    """The plan of talon_build_tree_ahead (resident: four workgroups on each of 256 compute units)."""
    out = (ctypes.c_int * 6)()
    per_block = 4096 if dtype == "f32" else 8192
    _lib().t_ahead(B, N, -(-vocab // per_block), k, K_init or k, init_layers, max_depth, resident, out)
    p = dict(zip(("layered", "rows", "head", "chunks_head", "chunks", "scanners"), out))
    return dict(p, blocks=-(-vocab // per_block))


def literal_layered(B, N, vocab, dtype, layers, K_init=8, init_layers=1, resident=1024):
    """Does the uncapped call with all rows in place go layer by layer?"""
    p = ahead_plan(B, N, vocab, dtype, 16, N, K_init, init_layers, resident)
    return bool(_lib().t_literal_layered(N, K_init, init_layers, layers, B * p["rows"] * p["blocks"], resident, N <= 64, 32))
