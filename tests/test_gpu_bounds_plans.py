"""The bounds-checked library on what small calls do not reach: matching by fp16 copies,
parts merged before the emission, pair tables, one set much longer than the other;
verification of a second chunk of correspondences, of more than stay in LDS, of
at most one a lane and of more pairs than one launch's arguments hold; images whose band
counts the emission sums itself or not.  No access out of range, the same bits.  Needs an
MI355X."""
import numpy as np
import pytest

from paper_2605_17869_amd import synth
from gpu_util import digest, extract_batch, require_gpu, say

pytestmark = pytest.mark.gpu


def both(run, what):
    """run(bounds) on both libraries: equal, and nothing out of range."""
    from paper_2605_17869_amd import bounds_violations
    say(f"bounds-checked: {what}")
    bounds_violations(reset=True)
    assert run(True) == run(False)
    n = bounds_violations(reset=True)
    say(f"{what}: {n} out-of-range accesses")
    assert n == 0


@pytest.mark.parametrize("sizes,counts", [
    ([(4200, 4301)], [(4199, 4298)]),                 # copies, parts
    ([(1100, 1203)], None),                           # parts merged before the emission
    ([(6000, 70)], None), ([(70, 6000)], [(1, 5999)]),
    ([(40 + 31 * k, 900 - 17 * k) for k in range(35)], None)], ids=lambda v: str(v)[:24])
def test_matching(sizes, counts):
    torch = require_gpu()
    from paper_2605_17869_amd import match_batch
    pairs = []
    for k, (na, nb) in enumerate(sizes):
        a, b = synth.descriptor_sets(970 + k, na, nb, min(na, nb) // 2, 0.1)[:2]
        cts = [None, None] if counts is None else [
            torch.tensor([c], dtype=torch.int32, device="cuda") for c in counts[k]]
        pairs.append((torch.from_numpy(a).cuda(), cts[0], torch.from_numpy(b).cuda(), cts[1]))

    def run(bounds):
        out = match_batch(pairs, bounds_checked=bounds)
        torch.cuda.synchronize()
        return [(m.host()[0].tobytes(), m.host()[1]) for m in out]
    both(run, f"matching {sizes[:3]}")


@pytest.mark.parametrize("sizes", [[64], [65, 1], [1025, 1024], [4097], [5003, 4096], [30 + k for k in range(27)]],
                         ids=lambda v: str(v)[:16])
def test_verification(sizes):
    torch = require_gpu()
    from paper_2605_17869_amd import verify_batch
    pairs = []
    for k, n in enumerate(sizes):
        a, b, _, _ = synth.homography_pairs(980 + k, n, 0.3 if n > 8 else 0.0, 0.5)
        kp = np.zeros((2, n, 12), np.float32)
        kp[0, :, :2], kp[1, :, :2] = a, b
        rec = np.zeros((n, 4), np.int32)
        rec[:, 0] = rec[:, 1] = np.arange(n)
        kp = torch.from_numpy(kp.view(np.int32)).cuda()
        pairs.append((kp[0], kp[1], torch.from_numpy(rec).cuda(), None))
    u = torch.from_numpy(synth.sample_numbers(990, 133)).cuda()

    def run(bounds):
        out = verify_batch(pairs, u, bounds_checked=bounds)
        torch.cuda.synchronize()
        return [[np.asarray(v).tobytes() for v in r.host()] for r in out]
    both(run, f"verification {sizes[:3]}")


@pytest.mark.parametrize("n", [1, 4, 5, 30])
def test_emission(n):
    require_gpu()
    from paper_2605_17869_amd import Extractor
    imgs = [synth.blob_image(992 + k % 5, 97 + 3 * (k % 5), 131 - 4 * (k % 5), 40) for k in range(n)]
    st = dict(synth.BASE_SETTINGS, n_octaves=3, n_streams=1, max_candidates=16)

    def run(bounds):
        return [digest(r[0], r[1]) + str(r[2:])
                for r in extract_batch(Extractor(st, bounds_checked=bounds), imgs)]
    both(run, f"{n} images")
