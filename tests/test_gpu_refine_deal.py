"""Candidates dealt to refinement waves by their number in the batch: features of an
image are bit-identical alone (8 candidates a wave) and in batches of 8 to 64 a wave
and of more than one turn.  Needs an MI355X."""
import numpy as np
import pytest

from paper_2605_17869_amd import synth
from gpu_util import digest, extract, extract_batch, require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp16", [0, 1])
@pytest.mark.parametrize("n", [1, 3, 6, 40])
def test_dealing_does_not_change_results(n, fp16):
    require_gpu()
    from paper_2605_17869_amd import Extractor
    st = dict(synth.BASE_SETTINGS, n_octaves=3, upsample=1, pyramid_fp16=fp16, n_streams=1,
              contrast_threshold=0.002, max_candidates=16384, max_keypoints=8192)
    rng = np.random.default_rng(830)
    imgs = [rng.random((232 + 8 * k, 301 - 4 * k)).astype(np.float32) for k in range(3)]
    ex = Extractor(st)
    alone = []
    for img in imgs:
        kp, desc, nf, nc = extract(ex, img)
        alone.append(digest(kp, desc) + str((nf, nc)))
    got = extract_batch(ex, [imgs[k % 3] for k in range(n)])
    say(f"n {n} fp16 {fp16}: {sum(int(r[3]) for r in got)} candidates")
    assert [digest(r[0], r[1]) + str((r[2], r[3])) for r in got] == [alone[k % 3] for k in range(n)]
