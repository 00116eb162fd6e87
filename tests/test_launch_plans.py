"""Which kernel a call takes: the package's planning code (host C++ without HIP) compiled
with g++ and asked directly."""
import ctypes
import os
import random
import subprocess

import pytest

from gemm_kernels import KERNELS, SPLIT_K, kernel_of
from test_gpu_transform_split import SHAPES as SPLIT_TRANSFORM

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_04945_amd", "csrc")
SHIM = r"""
#include "gemm_plan.hpp"
#include "tac_plan.hpp"
#include "transform_plan.hpp"
extern "C" void gemm(int M, int N, int K, int bits, int frag, int* o) {
    const sq::Plan p = sq::gemm_plan(M, N, K, bits, frag != 0);
    const int v[9] = {p.cfg, p.bm, p.bn, p.splits, p.waves, p.kw, p.alds, p.u, p.d};
    for (int i = 0; i < 9; ++i) o[i] = v[i];
}
extern "C" int fast_tile(int M, int K) { return (int)sq::fast_tile(M, K); }
extern "C" int tac_quant_rows(int M, int K, int g) { return sq::tac_quant_rows(M, K, g); }
extern "C" int split(int M, int K, int dm, int du, int gated, int* o) {
    const sq::SplitShape s = sq::split_shape(M, K);
    o[0] = s.rb; o[1] = s.cb; o[2] = s.waves;
    return sq::split_faster(M, K, dm, du, gated != 0);
}
extern "C" size_t gemm_workspace(int M, int N, int K, int bits) { return sq::plan_workspace_bytes(M, N, K, bits); }
"""
STREAM = (3, 5, 6)                       # weights streamed into registers
K_GROUPS = (9, 10, 11, 12, 13, 14)       # tiles in k groups
FAST_TILES = ("32x32", "32x64", "64x64", "64x64 four per CU", "64x64 three per CU", "128x64", "128x128",
              "128x128 two per CU", "256x128", "256x192")


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


def test_every_gemm_kernel_is_reached(plans):
    for name, (M, N, K) in KERNELS.items():
        bits, frag = int(name[0]), "fragments" in name
        assert kernel_of(gemm(plans, M, N, K, bits, frag), M, bits, frag) == name


def test_split_shapes_split(plans):
    """What the scratch tests call does use the scratch, the first call the most of it."""
    scratch = []
    for M, N, K in SPLIT_K:
        for frag in (False, True):
            p = gemm(plans, M, N, K, 4, frag)
            assert p["splits"] > 1
            scratch.append(p["splits"] * M * N * 4)
    assert scratch == sorted(scratch, reverse=True) and scratch[0] > scratch[-1] and scratch[0] <= 16 << 20


def test_no_plan_asks_for_another_gemm_kernel(plans):
    few = [(M, 16 * g - 8, 64 * k, bits) for M in (1, 16, 17, 32, 33, 36, 40, 48)
           for g in (1, 128, 256, 257, 384, 512, 513, 768, 1023, 1024, 1025, 2400)
           for k in (*range(1, 50), *range(60, 130, 3), 160, 300, 1024) for bits in (4, 8)]
    for M, N, K, bits in (*few, *shapes(50000, 2)):
        for frag in (False, True):
            assert kernel_of(gemm(plans, M, N, K, bits, frag), M, bits, frag) in KERNELS, (M, N, K)


def test_gemm_scratch_fits_the_workspace(plans):
    """Partial sums of a K split across workgroups fit what the interface asks for."""
    for M, N, K, bits in shapes(100000, 1):
        ws = plans.gemm_workspace(M, N, K, bits)
        assert M > 48 or ws == 0
        for frag in (False, True):
            p = gemm(plans, M, N, K, bits, frag)
            if p["splits"] > 1:
                assert p["splits"] * M * N * 4 <= ws, (M, N, K, bits, frag)


# Measured on weights that come from memory, us streamed and in k groups; the call takes
# the faster one
@pytest.mark.parametrize("M,N,K,bits,frag,streamed,tiled", [
    (16, 6144, 4096, 4, True, 5.5, 6.0), (12, 4104, 4096, 8, True, 6.6, 7.7), (16, 9216, 4096, 8, True, 9.7, 11.2),
    (24, 3584, 6144, 4, True, 5.9, 7.2), (24, 3072, 4096, 8, True, 6.6, 8.5), (28, 2048, 6144, 8, False, 11.2, 12.6),
    (32, 12288, 5120, 4, True, 10.1, 10.4), (22, 10240, 3584, 8, True, 10.2, 10.6), (36, 24576, 2560, 8, True, 14.6, 16.4),
    (8, 12288, 64, 8, True, 2.6, 4.1), (32, 512, 16384, 4, True, 11.3, 13.5),
    (18, 7168, 3584, 4, True, 7.4, 6.0), (30, 7168, 9216, 8, True, 31.7, 19.3), (20, 8192, 4096, 4, False, 8.0, 6.8),
    (16, 6144, 4096, 4, False, 6.5, 6.1), (40, 4608, 9216, 4, True, 16.9, 10.9), (48, 5120, 12288, 8, True, 39.2, 23.2),
    (44, 37888, 12288, 4, True, 146.0, 55.0), (40, 20480, 3072, 8, False, 31.6, 23.3)])
def test_few_rows_take_the_faster_kernel(plans, M, N, K, bits, frag, streamed, tiled):
    assert (gemm(plans, M, N, K, bits, frag)["cfg"] in STREAM) == (streamed < tiled)


# The same for the tiles in k groups and the plans without them
@pytest.mark.parametrize("M,N,K,bits,frag,without,groups", [
    (128, 128, 64, 4, True, 3.0, 3.8), (200, 8192, 512, 4, False, 5.1, 6.1), (250, 8192, 512, 8, False, 5.7, 6.4),
    (57, 14336, 256, 4, True, 4.0, 4.8), (600, 3072, 2048, 4, True, 9.3, 9.8), (64, 2048, 9216, 8, False, 13.1, 16.6),
    (64, 64, 65536, 4, True, 17.4, 28.7), (64, 8, 65536, 8, True, 16.7, 44.1), (250, 64, 65536, 8, False, 19.3, 60.6),
    (128, 4096, 4096, 4, True, 12.5, 7.1), (50, 3584, 18944, 4, True, 17.7, 15.2), (100, 1024, 9216, 8, True, 15.2, 11.0),
    (160, 1872, 576, 8, True, 4.61, 5.12), (354, 2048, 512, 8, False, 4.56, 4.85),
    (128, 512, 512, 4, True, 3.86, 3.85), (512, 3584, 18944, 8, True, 96.4, 71.1), (300, 10240, 3072, 8, True, 23.8, 20.1)])
def test_small_grids_take_the_faster_tiles(plans, M, N, K, bits, frag, without, groups):
    assert (gemm(plans, M, N, K, bits, frag)["cfg"] in K_GROUPS) == (groups < without)


# Matrix-core transform: the faster of two tiles, us on it and on the other
@pytest.mark.parametrize("M,K,tile,us,other", [
    (16, 64, "64x64 four per CU", 3.4, 4.4), (543, 1024, "64x64", 10.8, 12.1),
    (1119, 640, "64x64 four per CU", 7.7, 9.2), (1665, 640, "64x64 four per CU", 9.7, 11.2),
    (3213, 512, "64x64 three per CU", 9.7, 11.1), (4113, 512, "64x64 three per CU", 12.0, 17.2),
    (1585, 1280, "64x64 three per CU", 20.4, 27.0), (9344, 896, "128x128 two per CU", 38.7, 47.9),
    (250, 4096, "64x64", 25.4, 29.9), (512, 4096, "128x64", 37.9, 40.9), (1024, 4096, "128x128", 64.0, 78.0),
    (4096, 4096, "256x128", 209.0, 254.0), (16384, 3584, "256x192", 667.0, 684.0), (64, 4096, "32x32", 15.0, 19.0),
    (128, 4096, "32x64", 19.6, 23.5), (3404, 3584, "128x128", 166.6, 180.0)])
def test_fast_transform_takes_the_faster_tile(plans, M, K, tile, us, other):
    assert us < other and FAST_TILES[plans.fast_tile(M, K)] == tile


# Fixed-order transform: us on the tiled kernel and on the split one with 4 x 4, 2 x 4,
# 1 x 4, 1 x 2 and 1 x 1 blocks of outputs per workgroup
SPLIT_BLOCKS = ((4, 4), (2, 4), (1, 4), (1, 2), (1, 1))


@pytest.mark.parametrize("M,K,tiled,split", [
    (2705, 1344, 95.3, (146.0, 133.6, 113.2, 120.5, 153.9)), (4029, 1280, 139.5, (183.6, 188.2, 154.4, 158.3, 223.4)),
    (2655, 2624, 358.1, (391.2, 403.9, 400.6, 436.0, 598.8)), (3612, 512, 27.7, (39.7, 23.2, 22.7, 28.0, 30.3)),
    (191, 4096, 165.5, (73.7, 74.9, 62.2, 83.7, 102.9)),
    (95, 4096, 165.9, (72.8, 40.6, 42.6, 45.2, 55.5)), (41, 4096, 165.4, (72.0, 39.2, 24.0, 30.3, 30.1)),
    (641, 4096, 268.4, (217.2, 221.0, 216.1, 284.4, 376.5)),
    # with the quantiser behind it
    (6877, 256, 26.3, (34.2, 31.2, 23.6, 24.0, 25.1)), (4946, 320, 28.0, (36.1, 31.4, 24.1, 25.8, 27.4)),
    (94, 11648, 461.1, (424.7, 328.9, 315.8, 398.7, 572.6))])
def test_fixed_order_transform_takes_the_faster_kernel(plans, M, K, tiled, split):
    o = (ctypes.c_int * 3)()
    us = split[SPLIT_BLOCKS.index((o[0], o[1]))] if plans.split(M, K, 0, 0, 0, o) else tiled
    assert us <= 1.05 * min(tiled, *split)


def test_split_transform_shapes_take_their_blocks(plans):
    o = (ctypes.c_int * 3)()
    for M, K, tile in SPLIT_TRANSFORM:
        for dm, du, gated in [(0, 0, 0), (K // 32, K // 32, 1), (0, 13, 1), (K // 2, 17, 1)]:
            assert plans.split(M, K, dm, du, gated, o) and f"{o[0]}x{o[1]}" == tile


def test_fixed_order_transform_blocks_fit(plans):
    """The blocks divide the columns, no row block is padding only, and the waves fit a workgroup."""
    o = (ctypes.c_int * 3)()
    for M in (1, 8, 9, 16, 17, 32, 33, 100, 1000, 5000):
        for K in range(64, 19009, 64):
            plans.split(M, K, 0, 0, 0, o)
            rb, cb, waves = o
            assert (rb, cb) in SPLIT_BLOCKS and K % (16 * cb) == 0 and (rb == 1 or M > 8 * rb)
            assert 1 <= waves <= min(16 if rb * cb <= 4 else 8, -(-K // 256))


# us on the tiled and on the split kernel, half of the rows in either state
@pytest.mark.parametrize("M,K,dm,du,tiled,split", [
    (384, 12288, 6016, 6016, 785, 979), (901, 6784, 3328, 3328, 448, 783), (1703, 4032, 0, 3870, 203, 509),
    (384, 12288, 384, 384, 1242, 978), (384, 12288, 0, 0, 1242, 978), (70, 4544, 760, 760, 184, 50)])
def test_fixed_order_transform_counts_the_bands(plans, M, K, dm, du, tiled, split):
    o = (ctypes.c_int * 3)()
    assert plans.split(M, K, dm, du, 1, o) == (split < tiled)
    assert plans.split(M, K, dm, du, 0, o) == plans.split(M, K, 0, 0, 1, o) == plans.split(M, K, 0, 0, 0, o)


# Fused calibration + quantisation at g = 16: us with 256 and with 512 workgroups
@pytest.mark.parametrize("M,K,us256,us512", [
    (513, 3584, 9.21, 8.67), (514, 3584, 9.16, 9.98), (700, 3584, 9.39, 10.58), (768, 3584, 9.41, 10.61),
    (800, 3584, 10.93, 10.71), (1000, 3328, 11.10, 10.93), (513, 4096, 9.47, 11.58), (1024, 4096, 11.0, 14.1),
    (2000, 4096, 17.3, 20.6), (2000, 3584, 16.4, 15.4)])
def test_tac_quantiser_takes_the_faster_grid(plans, M, K, us256, us512):
    assert plans.tac_quant_rows(M, K, 16) == -(-M // (256 if us256 < us512 else 512))


def test_tac_quantiser_rows_in_range(plans):
    for M in (0, 1, 2, 255, 256, 257, 512, 4095, 16384, 16385, 32768, 32769, 1 << 24):
        for K in (16, 512, 3520, 3584, 3648, 4096):
            for g in (1, 8, 16):
                assert 1 <= plans.tac_quant_rows(M, K, g) <= 64
