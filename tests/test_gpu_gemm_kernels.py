"""Every GEMM kernel the plans can choose, one call each, bit for bit against the oracle."""
import numpy as np
import pytest

import paper_2606_04945_amd as sq
from gemm_kernels import KERNELS
from gpu_util import assert_bits, assert_y, dev, host, say
from oracle import oracle as O

pytestmark = pytest.mark.gpu
THREADS = 16


@pytest.mark.parametrize("name", KERNELS)
def test_gemm_kernel_bit_exact(name):
    M, N, K = KERNELS[name]
    bits, frag = int(name[0]), "fragments" in name
    say(f"{name} M={M} N={N} K={K}")
    rng = np.random.default_rng(M + N + K)
    if bits == 8:
        Aq = rng.integers(-128, 128, (M, K), dtype=np.int8)
        Wq = rng.integers(-128, 128, (N, K), dtype=np.int8)
    else:
        Aq = rng.integers(0, 256, (M, K // 2), dtype=np.uint8)
        Wq = rng.integers(0, 256, (N, K // 2), dtype=np.uint8)
    s_a = rng.uniform(0.05, 2, M).astype(np.float32)
    s_w = rng.uniform(1e-4, 2e-3, N).astype(np.float32)
    dW = dev(Wq)
    gemm, W = (sq.w4a4_gemm_frag, sq.weights_to_frag(dW)) if frag else (sq.w4a4_gemm, dW)
    Y, acc = gemm(dev(Aq), dev(s_a), W, dev(s_w), want_acc=True, bits=bits)
    rows = np.arange(M) if M <= 4200 else np.unique(np.r_[0, M - 1, rng.choice(M, 500)])
    rY, racc = (O.gemm_q8 if bits == 8 else O.gemm)(Aq[rows], s_a[rows], Wq, s_w, threads=THREADS)
    assert_bits(host(acc)[rows], racc, "acc")
    assert_y(host(Y)[rows], rY)
