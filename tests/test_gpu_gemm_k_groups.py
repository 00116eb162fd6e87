"""GEMM on small grids, where a workgroup splits k over its waves: every tile of the
plan at ragged edges, k tails and uneven k groups, both weight orders and code
widths, and the split across workgroups that a deep K of many small tiles keeps."""
import numpy as np
import pytest

import paper_2606_04945_amd as sq
from gpu_util import assert_bits, assert_y, dev, host, say
from oracle import oracle as O

pytestmark = pytest.mark.gpu


# 4-bit tiles: 32 x 32 (one k step for twelve groups, fragments only; 31 steps), 32 x 64,
# 64 x 64 without k groups (K too shallow for them), 64 x 128 in three k groups; then few
# rows: streamed but for 64 x 64 tiles at (33, 8200, 1088) and, row-major, 32 x 64 at
# (20, 8200, 4160); 64 x 64 at 50 rows and a split across workgroups
@pytest.mark.parametrize("M,N,K", [(49, 8, 64), (50, 136, 3968), (130, 2056, 4160), (77, 4104, 192), (250, 4104, 1088),
                                   (190, 8192, 1024), (400, 3592, 8256), (1000, 2048, 16448),
                                   (9, 4616, 1088), (17, 4104, 192), (24, 136, 3968), (33, 8200, 1088), (41, 16392, 192),
                                   (20, 8200, 4160), (50, 8200, 4160), (50, 1032, 16320)])
def test_w4a4_k_groups(M, N, K):
    say(f"gemm k groups M={M} N={N} K={K}")
    rng = np.random.default_rng(M + N + K)
    Aq = rng.integers(0, 256, (M, K // 2), dtype=np.uint8)
    Wq = rng.integers(0, 256, (N, K // 2), dtype=np.uint8)
    check(Aq, Wq, K, O.gemm, 4)


# 8-bit: the same tiles, 128 x 128 in two k groups (49 steps), and (64, 4096, 10304):
# 256 tiles of 32 x 32 and 161 k steps, split across workgroups; few rows, streamed but
# for 64 x 64 and 64 x 128 tiles of row-major weights
@pytest.mark.parametrize("M,N,K", [(49, 8, 64), (50, 136, 1984), (130, 2056, 2112), (250, 4104, 576), (190, 8192, 576),
                                   (400, 3592, 4160), (600, 4104, 3136), (64, 4096, 10304), (3, 4616, 576),
                                   (17, 136, 1984), (48, 8200, 576), (33, 16392, 2112)])
def test_w8a8_k_groups(M, N, K):
    say(f"gemm k groups 8-bit M={M} N={N} K={K}")
    rng = np.random.default_rng(M + N + K)
    Aq = rng.integers(-128, 128, (M, K), dtype=np.int8)
    Wq = rng.integers(-128, 128, (N, K), dtype=np.int8)
    check(Aq, Wq, K, O.gemm_q8, 8)


def check(Aq, Wq, K, oracle, bits):
    rng = np.random.default_rng(1)
    M, N = len(Aq), len(Wq)
    s_a = rng.uniform(0.1, 2, M).astype(np.float32)
    s_w = rng.uniform(1e-3, 2e-3, N).astype(np.float32)
    ref_Y, ref_acc = oracle(Aq, s_a, Wq, s_w, threads=16)
    dA, dW, dsa, dsw = dev(Aq), dev(Wq), dev(s_a), dev(s_w)
    for name, f, W in (("rows", sq.w4a4_gemm, dW), ("fragments", sq.w4a4_gemm_frag, sq.weights_to_frag(dW))):
        Y, acc = f(dA, dsa, W, dsw, want_acc=True, bits=bits)
        assert_bits(host(acc), ref_acc, f"acc, weights in {name}")
        assert_y(host(Y), ref_Y, f"Y, weights in {name}")
