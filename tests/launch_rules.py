"""The library's own launch rules (csrc/launch_rules.h, csrc/tw_plan.h: host code without HIP), compiled with
the host compiler, so that a test can state which kernel its sizes run (not collected by pytest)."""
import ctypes
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2408_16978_amd", "csrc")
SHIM = """
#include "launch_rules.h"
#include "tw_plan.h"
extern "C" int key_groups(int64_t n_q, int64_t n_k, int Hq, int causal) { return fpdt::sweep_key_groups(n_q, n_k, Hq, causal); }
extern "C" int f32_one_launch(int64_t S, int Hq, int Hkv) { return fpdt::f32_one_launch(S, Hq, Hkv); }
extern "C" int dkdv_splits(int64_t n_q, int64_t n_k, int Hq, int Hkv, int D, int causal) { return fpdt::bwd_dkdv_splits(n_q, n_k, Hq, Hkv, D, causal); }
extern "C" void product(int64_t M, int64_t N, int64_t K, int* out)
{
    const fpdt_tw::Plan p = fpdt_tw::plan_product(M, N, (int)((K < fpdt_tw::SK ? fpdt_tw::SK : K) / fpdt_tw::SK));
    const int v[] = {p.wmt, p.wnt, p.u.tiles, p.u.whole, p.u.splits, p.u.split_stages};
    for (int i = 0; i < 6; ++i) out[i] = v[i];
}
"""


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "rules.cpp"), os.path.join(d, "rules.so")
        with open(src, "w") as f:
            f.write(SHIM)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, src, "-o", so], check=True)
        L = ctypes.CDLL(so)
    i64, ci = ctypes.c_int64, ctypes.c_int
    L.key_groups.argtypes = [i64, i64, ci, ci]
    L.dkdv_splits.argtypes = [i64, i64, ci, ci, ci, ci]
    L.f32_one_launch.argtypes = [i64, ci, ci]
    L.product.argtypes = [i64, i64, i64, ctypes.POINTER(ci)]
    L.product.restype = None
    return L


def forward_key_groups(S, Hq):
    return _lib().key_groups(S, S, Hq, 1)


def dq_key_groups(rows, Hq, diagonal):
    return _lib().key_groups(rows, rows, Hq, int(diagonal))


def f32_one_launch(S, Hq, Hkv):
    return bool(_lib().f32_one_launch(S, Hq, Hkv))


def dkdv_splits(rows, Hq, Hkv, D, one_launch):
    return _lib().dkdv_splits(rows, rows, Hq, Hkv, D, int(one_launch))


def product(M, N, K):
    """(64-row units of a tile, 64-column units, "whole" / "divided" / "mixed")"""
    v = (ctypes.c_int * 6)()
    _lib().product(M, N, K, v)
    wmt, wnt, tiles, whole, splits, _ = v
    return wmt, wnt, "whole" if splits == 1 else "divided" if whole == 0 else "mixed"
