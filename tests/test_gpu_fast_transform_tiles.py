"""Matrix-core transform: every tile of its launch rule at ragged rows and columns and
at k steps that its k groups do not divide, within the rigorous bound of the exact
product (which holds for any order of the sums), gated columns +0."""
import numpy as np
import pytest

import paper_2606_04945_amd as sq
from oracle import fast_transform as F
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


# 32 x 32 (8 and 66 k steps for eight groups), 32 x 64, 64 x 64, 128 x 64, 128 x 128
# in one round, 256 x 128, 256 x 192, 128 x 128 in three rounds, and 64 x 64 at up to 64
# rows; the tiles of a shallow K: 64 x 64 four per CU (2, 18 and 34 steps), three per CU (22)
# and 128 x 128 two per CU
@pytest.mark.parametrize("M,K", [(3, 64), (49, 2112), (200, 2112), (321, 1600), (500, 2112), (900, 3136), (1100, 3136),
                                 (2300, 3136), (1025, 9600), (1100, 10048), (41, 9600), (1001, 576), (701, 1088),
                                 (2050, 704), (9301, 896), (3, 256)])
def test_tiles_within_bound(M, K):
    say(f"transform_fast tiles M={M} K={K}")
    rng = np.random.default_rng(M * K)
    X = rng.standard_normal((M, K)).astype(np.float16)
    X[:, ::97] *= 16
    st = (rng.random(M) < 0.5).astype(np.uint8)
    P = (rng.standard_normal((K, K)) / np.sqrt(K)).astype(np.float32)
    dm, du = K // 32, 7
    Ps = sq.sgat_split_basis(dev(P))
    xp = host(sq.sgat_transform_fast(dev(X), dev(st), Ps, dm, du))
    rows = np.unique(np.concatenate([np.arange(min(M, 40)), np.arange(max(0, M - 40), M), rng.integers(0, M, 40)]))
    exact = F.exact_transform(X[rows], st[rows], P, dm, du)
    bound = F.fast_bound(X[rows], host(Ps).view(np.uint16), P)
    assert (np.abs(xp[rows] - exact) <= bound).all()
    keep = F.gate_mask(st, K, dm, du)
    assert (xp[~keep] == 0).all() and not np.signbit(xp[~keep]).any()
    assert np.isfinite(xp).all()
