"""Octaves of few pixels taken whole in one launch against one launch per level:
levels and features bit-identical in every tile size, at tile edges, for images
smaller than the halo, fp16 storage and batches up to the launch's image limit.
Needs an MI355X."""
import pytest

from paper_2605_17869_amd import synth
from gpu_util import digest, extract_batch, require_gpu, say
from test_gpu_chain import launch_labels, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size,up,fp16,octaves,wide_first", [
    ((97, 131), 0, 0, 4, False), ((104, 97), 1, 1, 4, False),   # last octave 13 pixels: halo far beyond it
    ((480, 640), 0, 0, 4, True),                                # 300 narrow tiles, 210 wide
    ((225, 481), 1, 1, 3, False), ((64, 1600), 0, 1, 3, False), ((513, 511), 0, 0, 3, True)])
def test_whole_octaves_equal_levels(size, up, fp16, octaves, wide_first):
    require_gpu()
    img = synth.blob_image(760 + size[0], *size, max(20, size[0] * size[1] // 800))
    base = dict(synth.BASE_SETTINGS, n_octaves=octaves, upsample=up, pyramid_fp16=fp16)
    labels = launch_labels(base, img)
    say(f"{size} up={up} fp16={fp16}: {labels}")
    assert sum("whole" in lab for lab in labels) >= octaves + up - 1
    narrow = -(-size[0] * (1 + up) // 32) * -(-size[1] * (1 + up) // 32)
    assert wide_first == (narrow > 256 and "whole" in labels[0])
    assert run(base, [img]) == run(dict(base, blur_chain=1), [img])


@pytest.mark.parametrize("n", [64, 65])
def test_whole_octaves_in_batches(n):
    require_gpu()
    from paper_2605_17869_amd import Extractor
    imgs = [synth.blob_image(790 + k, 60 + 7 * (k % 9), 133 - 8 * (k % 7), 40) for k in range(16)]
    imgs = [imgs[k % 16] for k in range(n)]
    base = dict(synth.BASE_SETTINGS, n_octaves=3, n_streams=1, max_candidates=4096, max_keypoints=4096)
    outs = [[digest(r[0], r[1]) + str(r[2:]) for r in extract_batch(Extractor(dict(base, blur_chain=c)), imgs)]
            for c in (0, 1)]
    assert outs[0] == outs[1] and outs[0][0] == outs[0][16]
