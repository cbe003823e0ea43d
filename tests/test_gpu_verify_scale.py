"""Positions and noise scale in any unit: with both multiplied by a power of two every
step of the verifier is, too, so models, scores, weights and counts are the same but for
that factor, bit for bit -- down to units where squares of single-precision residuals
leave the normal range.  The noise puts many residuals beside the limit.  Needs an MI355X."""
import numpy as np
import pytest

from paper_2605_17869_amd import synth
from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("iters", [0, 5])
@pytest.mark.parametrize("n", [90, 3000])
def test_power_of_two_units(n, iters):
    torch = require_gpu()
    from paper_2605_17869_amd import verify_batch
    a, b, _, _ = synth.homography_pairs(450 + n, n, 0.1, 4.0)
    a32, b32 = a.astype(np.float32), b.astype(np.float32)
    u = torch.from_numpy(synth.sample_numbers(451, 600)).cuda()
    rec = np.zeros((n, 4), np.int32)
    rec[:, 0] = rec[:, 1] = np.arange(n)
    rec = torch.from_numpy(rec).cuda()
    ref = None
    for k in (0, 30, -20, -40, -60, -70, -72, -73, -74, -75, -76, -78, -82, -90):
        s = 2.0 ** k
        kp = np.zeros((2, n, 12), np.float32)
        kp[0, :, :2], kp[1, :, :2] = a32 * np.float32(s), b32 * np.float32(s)
        kp = torch.from_numpy(kp.view(np.int32)).cuda()
        (r,) = verify_batch([(kp[0], kp[1], rec, None)], u, sigma_max=2.0 * s, refine_iters=iters)
        torch.cuda.synchronize()
        H, score, inliers, best, w = r.host()
        unit = np.array([[1, 1, 1 / s], [1, 1, 1 / s], [s, s, 1]])   # back to pixels
        got = (H * unit, score * s, inliers, best, w.astype(np.float64) * s)
        if ref is None:
            ref = got
            say(f"{n} correspondences: score {score}, {inliers} inliers, hypothesis {best}")
            assert inliers > n // 4
        assert got[1:4] == ref[1:4], (k, got[1:4], ref[1:4])
        assert np.array_equal(got[0], ref[0]) and np.array_equal(got[4], ref[4]), k
