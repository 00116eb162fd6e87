"""TAC calibration where the decompositions have null spaces: constant and repeated
channels and fewer tokens than channels, at every block size the solver treats
differently and token counts around its tiles of 32 and 64."""
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
