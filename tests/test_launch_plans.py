"""Which kernel a call takes: the package's planning code (host C++ without HIP) compiled
with g++ and asked directly."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_04945_amd", "csrc")
SHIM = r"""
#include "gemm_plan.hpp"
extern "C" void gemm(int M, int N, int K, int bits, int frag, int* o) {
    const sq::Plan p = sq::gemm_plan(M, N, K, bits, frag != 0);
    const int v[9] = {p.cfg, p.bm, p.bn, p.splits, p.waves, p.kw, p.alds, p.u, p.d};
    for (int i = 0; i < 9; ++i) o[i] = v[i];
}
extern "C" size_t gemm_workspace(int M, int N, int K, int bits) { return sq::plan_workspace_bytes(M, N, K, bits); }
"""
STREAM = (3, 5, 6)                       # weights streamed into registers
K_GROUPS = (9, 10, 11, 12, 13, 14)       # tiles in k groups


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    d = tmp_path_factory.mktemp("plans")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o", so],
                   check=True)
    lib = ctypes.CDLL(so)
    lib.gemm_workspace.restype = ctypes.c_size_t
    return lib


def gemm(lib, M, N, K, bits, frag):
    o = (ctypes.c_int * 9)()
    lib.gemm(M, N, K, bits, int(frag), o)
    return dict(zip(("cfg", "bm", "bn", "splits", "waves", "kw", "alds", "u", "d"), o))


def log_uniform(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def shapes(n, seed):
    rng = random.Random(seed)
    for _ in range(n):
        bits = rng.choice((4, 8))
        yield (log_uniform(rng, 1, 4096), 8 * log_uniform(rng, 1, 8192),
               64 * log_uniform(rng, 1, 1024 if bits == 8 else 2048), bits)


def test_gemm_scratch_fits_the_workspace(plans):
    """Partial sums of a K split across workgroups fit what the interface asks for."""
    for M, N, K, bits in shapes(100000, 1):
        ws = plans.gemm_workspace(M, N, K, bits)
        assert M > 48 or ws == 0
        for frag in (False, True):
            p = gemm(plans, M, N, K, bits, frag)
            if p["splits"] > 1:
                assert p["splits"] * M * N * 4 <= ws, (M, N, K, bits, frag)
