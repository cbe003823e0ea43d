"""The descriptor kernel takes a keypoint's tile streams with one wave (many
keypoints in a launch) or with the waves of a work-group (few): the same bits.
Window sizes cover one, two and four streams; odd image sizes, keypoints at the
border.  Needs an MI355X."""
import numpy as np
import pytest

from paper_2605_17869_amd import synth
from gpu_util import require_gpu, say

pytestmark = pytest.mark.gpu

POOLED = (0.5, 2.0 ** -0.5, 1.0, 2.0 ** 0.5, 2.0)


@pytest.mark.parametrize("scales,rootsift,fp16,size", [
    ((1.0,), 0, 0, (203, 331)), (POOLED, 1, 1, (240, 320)), (synth.dsp_linspace(), 1, 0, (203, 331)),
    ((0.25,), 0, 0, (150, 167)), ((6.0, 1.0), 0, 0, (203, 331))])
def test_many_and_few_keypoints_same_bits(scales, rootsift, fp16, size):
    torch = require_gpu()
    from paper_2605_17869_amd import Extractor
    settings = dict(synth.BASE_SETTINGS, n_octaves=3, dsp_scales=scales, rootsift=rootsift,
                    pyramid_fp16=fp16, max_keypoints=2048, max_candidates=2048)
    imgs = [torch.from_numpy(synth.blob_image(9100 + k, *size, 260)).cuda() for k in range(2)]
    ex = Extractor(settings, n_streams=1)   # one launch sequence for the whole batch
    alone = []
    for im in imgs:
        alone.append(ex.extract(im).host())
    per = sum(len(a[0]) for a in alone) / 2
    n = 2 * int(np.ceil(4096 / 2 / per) + 1)   # more keypoints than 4 per work-group
    out = ex.extract_batch([imgs[k % 2] for k in range(n)])
    torch.cuda.synchronize()
    say(f"{n} images, {per} keypoints each")
    assert per > 30 and n * per > 4096
    for k, f in enumerate(out):
        kp, desc, nf, nc = f.host()
        ref = alone[k % 2]
        assert (nf, nc) == ref[2:]
        assert kp.tobytes() == ref[0].tobytes()
        assert desc.tobytes() == ref[1].tobytes()
        assert np.all(np.isfinite(desc))
