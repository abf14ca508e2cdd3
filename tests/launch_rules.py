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
extern "C" int key_groups(int64_t S, int Hq) { return fpdt::sweep_key_groups(S, Hq); }
extern "C" int dq_key_groups(int64_t rows, int Hq, int D, int diagonal) { return fpdt::dq_key_groups(rows, rows, Hq, D, diagonal); }
extern "C" int64_t prepare_blocks(int64_t S, int Hq, int Hkv) { return fpdt::bwd_prepare_blocks(S, Hq, Hkv); }
extern "C" int64_t prepare_next(int64_t first, int64_t blocks) { return fpdt::bwd_prepare_next(first, blocks); }
extern "C" int f32_one_launch(int64_t S, int Hq, int Hkv) { return fpdt::f32_one_launch(S, Hq, Hkv); }
extern "C" int dkdv_splits(int64_t n_q, int64_t n_k, int Hq, int Hkv, int D, int causal) { return fpdt::bwd_dkdv_splits(n_q, n_k, Hq, Hkv, D, causal); }
static void put(const fpdt_tw::Plan& p, int* out)
{
    const int v[] = {p.wmt, p.wnt, p.u.tiles, p.u.tiles_n, p.u.whole, p.u.splits, p.u.split_stages};
    for (int i = 0; i < 7; ++i) out[i] = v[i];
}
static int steps(int64_t K) { return (int)((K < fpdt_tw::SK ? fpdt_tw::SK : K) / fpdt_tw::SK); }
extern "C" void launched(int64_t M, int64_t N, int64_t K, int* out) { put(fpdt_tw::plan_launch(M, N, steps(K)), out); }
extern "C" void first_answer(int64_t M, int64_t N, int64_t K, int* out) { put(fpdt_tw::plan_product(M, N, steps(K)), out); }
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
    L.key_groups.argtypes = [i64, ci]
    L.dq_key_groups.argtypes = [i64, ci, ci, ci]
    L.dkdv_splits.argtypes = [i64, i64, ci, ci, ci, ci]
    L.f32_one_launch.argtypes = [i64, ci, ci]
    L.prepare_blocks.argtypes, L.prepare_blocks.restype = [i64, ci, ci], i64
    L.prepare_next.argtypes, L.prepare_next.restype = [i64, i64], i64
    for f in (L.launched, L.first_answer):
        f.argtypes, f.restype = [i64, i64, i64, ctypes.POINTER(ci)], None
    return L


def forward_key_groups(S, Hq):
    return _lib().key_groups(S, Hq)


def dq_key_groups(rows, Hq, diagonal, D=128):
    return _lib().dq_key_groups(rows, Hq, D, int(diagonal))


def prepare_launches(S, Hq, Hkv):
    """(first block, workgroups) of each launch that prepares a backward over the whole sequence"""
    blocks, first, out = _lib().prepare_blocks(S, Hq, Hkv), 0, []
    while first < blocks:
        out.append((first, _lib().prepare_next(first, blocks)))
        first += out[-1][1]
    return out


def f32_one_launch(S, Hq, Hkv):
    return bool(_lib().f32_one_launch(S, Hq, Hkv))


def dkdv_splits(rows, Hq, Hkv, D, one_launch):
    return _lib().dkdv_splits(rows, rows, Hq, Hkv, D, int(one_launch))


def _plan(f, M, N, K):
    v = (ctypes.c_int * 7)()
    f(M, N, K, v)
    return dict(zip(("wmt", "wnt", "tiles", "tiles_n", "whole", "splits", "split_stages"), v))


def launched(M, N, K):
    """The layout that a product runs (plan_launch)"""
    return _plan(_lib().launched, M, N, K)


def first_answer(M, N, K):
    """plan_product's answer, which plan_launch starts from"""
    return _plan(_lib().first_answer, M, N, K)


def kind(p):
    """(64-row units of a tile, 64-column units, "whole" / "divided" / "mixed")"""
    return p["wmt"], p["wnt"], "whole" if p["splits"] == 1 else "divided" if p["whole"] == 0 else "mixed"


def product(M, N, K):
    return kind(launched(M, N, K))
