"""TAC calibration where the decompositions have null spaces (constant and repeated
channels, fewer tokens than channels) or repeated eigenvalues, at every block size the
solver treats differently and token counts around its tiles of 32 and 64."""
import numpy as np
import pytest

import paper_2606_04945_amd as sq
import synth
from oracle import tac_calib as T
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


# A null eigenvalue (about 1e-16) is raised to 1e-12 on both sides, so the smallest
# singular value of M is about 1e-6 and its vectors carry M's rounding over it:
# 1e-16 / 1e-6, times the smoothing's weight.  1e-9 leaves an order and a half.
@pytest.mark.parametrize("N,C,g", [(3, 64, 2), (63, 64, 4), (64, 64, 8), (65, 128, 16), (5, 64, 16), (129, 128, 32),
                                   (97, 192, 64), (2049, 256, 128), (40, 128, 128)])
def test_null_spaces(N, C, g):
    say(f"tac_calibrate null spaces N={N} C={C} g={g}")
    zf, zq = synth.tac_calib_pair(N, C, g, synth.rng_for(980, synth.T_CALIB, N, C, g))
    zf[:, 1], zq[:, 1] = 0.25, 0.25                   # a constant channel
    if g > 2:
        zf[:, 3], zq[:, 3] = zf[:, 2], zq[:, 2]       # a repeated one
    _, _, M64, d64 = sq.tac_calibrate(dev(zf), dev(zq), g, want_fp64=True)
    rM, rd = T.calibrate(zf, zq, g)
    np.testing.assert_allclose(host(M64), rM, rtol=0, atol=1e-9 * max(1.0, np.abs(rM).max()))
    np.testing.assert_allclose(host(d64), rd, rtol=0, atol=1e-9 * max(1.0, np.abs(rd).max()))


def _hadamard(n):
    h = np.ones((1, 1))
    while len(h) < n:
        h = np.block([[h, h], [h, -h]])
    return h


def _clustered(C, g, rng):
    """[2 g][C] fp16 whose block covariances are exactly Q diag(1 or 4) Q^T: Hadamard rows and
    their negatives, scaled by 1 or 2 and turned by two reflections of dyadic entries."""
    out = np.empty((2 * g, C))
    for b in range(0, C, g):
        u, w = rng.choice([-1.0, 1.0], g), np.zeros(g)
        w[rng.choice(g, 4, replace=False)] = rng.choice([-1.0, 1.0], 4)
        q = (np.eye(g) - 2 / g * np.outer(u, u)) @ (np.eye(g) - 0.5 * np.outer(w, w))
        z = _hadamard(g) @ (rng.permutation(np.resize([1.0, 2.0], g))[:, None] * q)
        out[:g, b:b + g], out[g:, b:b + g] = z, -z
    assert (out.astype(np.float16) == out).all()
    return out.astype(np.float16)


# Two eigenvalues, each g / 2 times, in both inputs: columns of equal norm, which turn by
# any angle on rounding noise.  A decomposition taken to working precision is 1e-13 from
# LAPACK at g = 128 and 5e-15 at 16; one stopped where pairs are 1e-9 from orthogonal is
# 2e-12 to 4e-11 off.
@pytest.mark.parametrize("g", [8, 16, 32, 64, 128])
def test_repeated_eigenvalues(g):
    rng = np.random.default_rng(0)
    zf, zq = _clustered(256, g, rng), _clustered(256, g, rng)
    _, _, M64, d64 = sq.tac_calibrate(dev(zf), dev(zq), g, want_fp64=True)
    rM, rd = T.calibrate(zf, zq, g)
    say(f"tac_calibrate repeated eigenvalues g={g}: {np.abs(host(M64) - rM).max():.1e} from LAPACK")
    np.testing.assert_allclose(host(M64), rM, rtol=0, atol=1e-12)
    np.testing.assert_allclose(host(d64), rd, rtol=0, atol=1e-12)


# The same input twice and hardly any damping: M is the identity but for 1e-8, all its
# singular values alike and its columns nearly orthogonal from the start.
@pytest.mark.parametrize("g", [4, 8, 16, 32, 64, 128])
def test_equal_inputs(g):
    zf, _ = synth.tac_calib_pair(600, 256, g, synth.rng_for(981, synth.T_CALIB, g))
    _, _, M64, d64 = sq.tac_calibrate(dev(zf), dev(zf), g, rho=1e-8, want_fp64=True)
    rM, rd = T.calibrate(zf, zf, g, rho=1e-8)
    say(f"tac_calibrate equal inputs g={g}: {np.abs(host(M64) - rM).max():.1e} from LAPACK")
    np.testing.assert_allclose(host(M64), rM, rtol=0, atol=1e-12)
    np.testing.assert_allclose(host(d64), rd, rtol=0, atol=1e-12)
