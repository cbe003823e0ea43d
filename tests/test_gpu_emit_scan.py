"""Emission with the band scan as a launch of its own and with the counts summed by
the emission itself, around the numbers of bands and of images where the one gives way
to the other: every image as by itself.  Needs an MI355X."""
import pytest

from paper_2605_17869_amd import synth
from gpu_util import digest, extract, extract_batch, require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 4, 5, 26, 30])
def test_images_around_the_limit(n):
    """Images of 19 and 20 bands: 4 and 5 images, 503 and 580 bands."""
    require_gpu()
    from paper_2605_17869_amd import Extractor
    sizes = [(97, 131), (97, 97), (100, 140)]
    imgs = [synth.blob_image(720 + k, *sizes[k % 3], 20 + 6 * k) for k in range(6)]
    ex = Extractor(dict(synth.BASE_SETTINGS, n_octaves=4, n_streams=1, max_candidates=12, max_keypoints=40))
    alone = []
    for im in imgs:
        kp, desc, nf, nc = extract(ex, im)
        alone.append(digest(kp, desc) + str((nf, nc)))
    got = extract_batch(ex, [imgs[k % 6] for k in range(n)])
    say(f"{n} images: {[int(r[3]) for r in got[:6]]} candidates")
    assert max(int(r[3]) for r in got) > 12   # one beyond its candidate slots
    assert [digest(r[0], r[1]) + str((r[2], r[3])) for r in got] == [alone[k % 6] for k in range(n)]


@pytest.mark.parametrize("rows", [4098, 4106, 4107])
def test_bands_around_the_limit(rows):
    """One octave of 511, 512 (the limit) and 513 bands: the same rows, counted by both
    forms, as part of one octave's candidates in order."""
    require_gpu()
    import numpy as np
    from paper_2605_17869_amd import Extractor
    img = synth.blob_image(731, 4107, 64, 700)[:rows]
    ex = Extractor(dict(synth.BASE_SETTINGS, n_octaves=1, n_streams=1))
    kp, desc, nf, nc = extract(ex, img)
    five = extract_batch(ex, [img] * 5)   # always with a scan of its own
    say(f"{rows} rows: {nc} candidates")
    assert nc > 100
    for r in five:
        assert digest(r[0], r[1]) + str((r[2], r[3])) == digest(kp, desc) + str((nf, nc))
    order = np.stack([kp["octave"], kp["src_layer"], kp["src_iy"], kp["src_ix"]])
    assert [tuple(c) for c in order.T] == sorted(tuple(c) for c in order.T)
