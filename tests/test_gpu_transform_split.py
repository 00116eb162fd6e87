"""Transform with k split over a workgroup's waves (few rows), bit for bit against
the oracle: every tile shape, one to several rounds of chunks, a last chunk of
one to three quarters, padded row blocks, and the band edges of the gate."""
import numpy as np
import pytest

import paper_2606_04945_amd as sq
from gpu_util import assert_bits, dev, host, say
from oracle import oracle as O

pytestmark = pytest.mark.gpu


# (M, K, blocks of 16 x 16 per tile as rows x columns): one wave (K = 64) up to 16
# chunks on 16 waves (4096), 17 on 16 (4160: a second round of one partial chunk)
# and 5, 9 or 16 on 8
SHAPES = [(1, 64, "1x1"), (17, 64, "1x1"), (33, 320, "1x1"), (31, 2240, "1x2"),
          (16, 4160, "1x1"), (64, 2112, "1x4"), (50, 4160, "2x4"), (128, 4096, "2x4"),
          (250, 4096, "4x4"), (1000, 512, "1x4"), (2000, 896, "1x4"), (866, 1152, "4x4")]


@pytest.mark.parametrize("M,K,tile", SHAPES)
def test_transform_split_bit_exact(M, K, tile):
    say(f"transform split M={M} K={K} tile {tile}")
    rng = np.random.default_rng(M * K)
    X = rng.standard_normal((M, K)).astype(np.float16)
    X[M // 2, ::7] *= 16
    st = (rng.random(M) < 0.5).astype(np.uint8)
    P = (rng.standard_normal((K, K)) / np.sqrt(K)).astype(np.float32)
    P[::5, 1] = -0.0
    P[:, 2] *= np.float32(1e-38)                      # subnormal products and sums
    dX, dP = dev(X), dev(P)
    plain = O.transform(X, None, P, 0, 0, threads=16)
    assert_bits(host(sq.sgat_transform(dX, None, dP)), plain, "x' ungated")
    for dm, du in [(K // 32, K // 32), (0, 13), (K // 2, 17)]:
        ref = plain.copy()
        ref[st == 0, K - dm - du:K - du] = 0.0
        ref[st != 0, K - du:] = 0.0
        assert_bits(host(sq.sgat_transform(dX, dev(st), dP, dm, du)), ref, f"x' bands {dm},{du}")
