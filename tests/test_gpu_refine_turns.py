"""Candidates dealt to refinement waves in the numbers that a large batch gives: 8, 18
and 64 a wave, and more of them than one turn of the waves takes.  Every image's features
as by itself.  Needs an MI355X."""
import numpy as np
import pytest

from paper_2605_17869_amd import synth
from gpu_util import digest, extract, extract_batch, require_gpu, say

pytestmark = pytest.mark.gpu


def egg_carton(h, w, k):
    """An extremum every seven pixels, amplitudes and phases varied so that none are equal."""
    y, x = np.mgrid[0:h, 0:w].astype(np.float64)
    img = np.sin(2 * np.pi * y / (14.0 + 0.3 * k)) * np.sin(2 * np.pi * x / (13.6 + 0.2 * k))
    slow = 1.0 + 0.3 * np.sin(y / 61 + k) * np.cos(x / 83 - k)
    return (0.5 + 0.2 * img * slow).astype(np.float32)


@pytest.mark.parametrize("n,slots,low,high", [
    (3, 16384, 8 * 1024, 64 * 1024),      # 9 to 64 a wave
    (12, 16384, 64 * 1024, 1 << 30),      # 64
    (20, 96, 20 * 96 - 1, 1 << 30)])      # 8 a wave, 32 waves: eight turns
def test_every_deal(n, slots, low, high):
    require_gpu()
    from paper_2605_17869_amd import Extractor
    ex = Extractor(dict(synth.BASE_SETTINGS, n_octaves=1, n_streams=1, contrast_threshold=0.002,
                        edge_ratio=40.0, max_candidates=slots, max_keypoints=2048))
    imgs = [egg_carton(480 + 8 * k, 640 - 8 * k, k) for k in range(3)]
    alone = []
    for img in imgs:
        kp, desc, nf, nc = extract(ex, img)
        alone.append(digest(kp, desc) + str((nf, nc)))
    got = extract_batch(ex, [imgs[k % 3] for k in range(n)])
    total = sum(min(int(r[3]), slots) for r in got)
    each = min(max(-(-total // 1024), 8), 64)
    turn = 4 * min(1024, -(-n * slots // 256)) * each
    say(f"{n} images: {total} candidates, {each} a wave, {turn} in a turn, {int(got[0][2])} features")
    assert low < total <= high and (slots > 96 or total > turn)
    assert min(int(r[2]) for r in got) > 20
    assert [digest(r[0], r[1]) + str((r[2], r[3])) for r in got] == [alone[k % 3] for k in range(n)]
