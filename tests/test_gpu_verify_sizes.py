"""Verification at the sizes where its kernels change what they do, against the
FP64 reference verifier: rows of 64 and chunks of 1024 correspondences in the
scoring kernel, partial sums of 256 and the 4096 correspondences that stay in
LDS in the other two, positions far from the origin (where the single-precision
test has to let more through), and more pairs than one launch's table entries."""
import numpy as np
import pytest

from paper_2605_17869_amd import synth
from test_gpu_verify import check, gpu_verify

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4, 5, 63, 64, 65, 255, 257, 1023, 1024, 1025, 4095, 4096, 4097, 5003])
def test_sizes(n):
    a, b, _, _ = synth.homography_pairs(400 + n, n, 0.4 if n > 8 else 0.0, 0.6)
    u = synth.sample_numbers(500 + n, 203)
    got, = gpu_verify([(a, b, np.random.default_rng(n).permutation(n))], u)
    check(a, b, u, got)


@pytest.mark.parametrize("iters", [0, 1, 5])
def test_far_from_the_origin(iters):
    a, b, _, _ = synth.homography_pairs(410, 700, 0.5, 0.6)
    shift = np.array([4096.0, -4096.0])
    u = synth.sample_numbers(411, 400)
    got, = gpu_verify([(a + shift, b - shift, None)], u, refine_iters=iters)
    check(a + shift, b - shift, u, got, iters)


def test_more_pairs_than_one_launch_takes():
    cases = []
    for k in range(49):
        a, b, _, _ = synth.homography_pairs(420 + k, 20 + 7 * k, 0.3, 0.5)
        cases.append((a, b, None))
    u = synth.sample_numbers(421, 150)
    for (a, b, _), got in zip(cases, gpu_verify(cases, u)):
        check(a, b, u, got)
