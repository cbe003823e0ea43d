"""Orientations beside pixels that are not a number.  A keypoint whose orientation
window reaches such samples keeps the peaks of the bins they do not enter: a sample
with one NaN gradient component goes to the diagonal of the other's sign (45, 135 or 315
degrees), with two to 0.  Against that rule in float64 on the kernels' own levels.
Needs an MI355X."""
import numpy as np
import pytest

from paper_2605_17869_amd import synth
from gpu_util import extract, require_gpu, say

pytestmark = pytest.mark.gpu


def angles_of(L, r, c, sigma, p):
    """(angles, smallest relative distance of a bin from the peak threshold)"""
    sw = p.ori_sigma_factor * sigma
    R = int(np.floor(p.ori_radius_factor * sw + 0.5))
    h, w = L.shape
    rr, cc = np.mgrid[max(r - R, 1):min(r + R, h - 2) + 1, max(c - R, 1):min(c + R, w - 2) + 1]
    gx, gy = L[rr, cc + 1] - L[rr, cc - 1], L[rr + 1, cc] - L[rr - 1, cc]
    ax, ay = np.abs(gx), np.abs(gy)
    big, small = np.fmax(ax, ay), np.fmin(ax, ay)   # of a NaN and a number the number
    a = np.where(big > 0, small / np.where(big > 0, big, 1.0), 0.0)
    th = np.arctan(a)
    th = np.where(ay > ax, np.pi / 2 - th, th)
    th = np.where(gx < 0, np.pi - th, th)
    th = np.where(gy < 0, -th, th)
    pos = np.where(th < 0, th + 2 * np.pi, th) * 36 / (2 * np.pi)
    wgt = np.exp(-((rr - r) ** 2 + (cc - c) ** 2) / (2 * sw * sw)) * np.sqrt(gx * gx + gy * gy)
    b0, f = np.floor(pos).astype(int) % 36, pos - np.floor(pos)
    hist = np.zeros(36)
    np.add.at(hist, b0, wgt * (1 - f))
    np.add.at(hist, (b0 + 1) % 36, wgt * f)
    hs = 0.25 * np.roll(hist, 1) + 0.5 * hist + 0.25 * np.roll(hist, -1)
    if np.all(np.isnan(hs)):
        return [], 1.0, np.isnan(hist).sum()
    lo, hi, top = np.roll(hs, 1), np.roll(hs, -1), np.nanmax(hs)
    out = []
    for b in np.flatnonzero((hs > lo) & (hs > hi) & (hs >= p.ori_peak_ratio * top)):
        out.append(float((b + 0.5 * (lo[b] - hi[b]) / (lo[b] - 2 * hs[b] + hi[b])) * 10 % 360))
    peaks = (hs > lo) & (hs > hi)
    margin = np.min(np.abs(hs[peaks] / top - p.ori_peak_ratio), initial=1.0)
    return out, margin, int(np.isnan(hist).sum())


@pytest.mark.parametrize("factor,fp16", [(12.0, 0), (20.0, 1)])
def test_keypoints_beside_nan(factor, fp16):
    require_gpu()
    from paper_2605_17869_amd import Extractor
    img = synth.blob_image(640, 300, 420, 260)
    for y, x in [(90, 110), (210, 300), (150, 205), (40, 330)]:
        img[y, x] = np.nan
    st = dict(synth.BASE_SETTINGS, n_octaves=2, ori_radius_factor=factor, pyramid_fp16=fp16,
              ori_peak_ratio=0.3)
    ex = Extractor(st)
    kp, desc, _, _, ws = extract(ex, img, keep_ws=True)
    all_kp = extract(Extractor(dict(st, upright=1)), img)[0]   # every accepted candidate once
    levels = {}
    checked = touched = 0
    key = lambda k: (int(k["octave"]), int(k["src_layer"]), int(k["src_iy"]), int(k["src_ix"]))
    got = {}
    for k in kp:
        got.setdefault(key(k), []).append(float(k["angle"]))
    for k in all_kp:
        o, l = int(k["octave"]), int(k["layer"])
        if (o, l) not in levels:
            levels[o, l] = ex.level(ws, *img.shape, o, l)
        want, margin, poisoned = angles_of(levels[o, l], int(k["iy"]), int(k["ix"]),
                                           float(k["sigma"]) / 2.0 ** o, ex.params)
        if margin < 1e-3:
            continue
        have = sorted(got.get(key(k), []))
        assert len(have) == len(want), (key(k), have, want)
        np.testing.assert_allclose(have, sorted(want), atol=0.05)
        checked += 1
        touched += poisoned > 0 and len(want) > 0
    say(f"factor {factor} fp16 {fp16}: {checked} of {len(all_kp)} candidates checked, {touched} keep "
        "peaks beside bins that are not a number")
    assert checked > 20 and touched > 2
