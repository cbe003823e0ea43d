"""Extremum detection against the definition evaluated on the kernels' own levels
in float32 (so counts are exact): bands of 1 to 8 rows, rows that end at and around
a 62-column segment, one to six layers, both storage modes and both group sizes.
Needs an MI355X."""
import numpy as np
import pytest

from oracle import sift_oracle as so
from paper_2605_17869_amd import synth
from gpu_util import extract, require_gpu, say

pytestmark = pytest.mark.gpu


def expected(ex, ws, shape, st):
    p = ex.params
    thr = np.float32(p.prefilter_ratio) * np.float32(p.contrast_threshold)
    total, b = 0, p.border
    for o in range(st["n_octaves"] + st["upsample"]):
        lv = [(ex.level(ws, *shape, o - st["upsample"], l) - 0.5).astype(np.float32)
              for l in range(p.n_scales + 3)]
        D = np.stack([y - x for x, y in zip(lv, lv[1:])])
        _, h, w = D.shape
        for i in range(1, p.n_scales + 1):
            ctr = D[i, b:h - b, b:w - b]
            near = np.stack([D[i + di, b + dr:h - b + dr, b + dc:w - b + dc]
                             for di, dr, dc in so.NEIGHBOURS])
            total += int(np.sum((np.abs(ctr) > thr) & ((ctr > near.max(0)) | (ctr < near.min(0)))))
    return total


@pytest.mark.parametrize("scales,up,fp16", [(3, 0, 0), (3, 1, 1), (1, 0, 0), (2, 1, 0), (4, 0, 1),
                                            (5, 0, 0), (6, 0, 1)])
def test_counts_equal_the_definition(scales, up, fp16):
    require_gpu()
    from paper_2605_17869_amd import Extractor
    st = dict(synth.BASE_SETTINGS, n_octaves=2, n_scales=scales, upsample=up, pyramid_fp16=fp16,
              max_candidates=65536, sigma0=0.8 if scales == 1 else 1.6)
    found = 0
    rng = np.random.default_rng(800 + scales)
    # 10 columns and rows of frame; 62 and 8 of them to a segment and a band
    for k, (h, w) in enumerate([(26, 71), (27, 72), (51, 73), (52, 133), (53, 134), (62, 135),
                                (95, 197), (33, 321)]):
        img = rng.random((h, w)).astype(np.float32)
        img[h // 2:, : w // 3] = 0.25   # equal neighbours are no extremum
        counts = []
        for waves in (4, 8):
            ex = Extractor(dict(st, detect_waves=waves))
            _, _, _, n_cand, ws = extract(ex, img, keep_ws=True)
            counts.append(int(n_cand))
        want = expected(ex, ws, img.shape, st)
        say(f"scales {scales} up {up} fp16 {fp16} {h}x{w}: {counts}, by definition {want}")
        assert counts == [want, want]
        found += want
    assert found > 0
