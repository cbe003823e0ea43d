"""Calls whose pairs the kernels carry in their arguments (up to 32) and calls that
read them from a table: ragged and empty sets, every pair bit-identical to a call of
its own, in plans with and without a merge of parts.  Needs an MI355X."""
import pytest

from paper_2605_17869_amd import synth
from gpu_util import require_gpu, say
from test_gpu_match import gpu_match

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 70])
@pytest.mark.parametrize("equal", [True, False])
def test_pairs_equal_single_calls(n, equal):
    require_gpu()
    sizes = [(300, 263)] * n if equal else [(1 + (37 * k) % 701, 1 + (91 * k) % 533) for k in range(n)]
    sets = []
    for k, (na, nb) in enumerate(sizes):
        sets.append(synth.descriptor_sets(600 + k % 8, na, nb, min(na, nb) // 2, 0.1)[:2])
    counts = [(na, nb * (k % 5) // 4) if k % 5 < 4 else None for k, (na, nb) in enumerate(sizes)]
    together = gpu_match(sets, counts=counts)
    for k in range(n):
        (rec, nf), = gpu_match([sets[k]], counts=[counts[k]])
        assert together[k][1] == nf and together[k][0].tobytes() == rec.tobytes(), (k, sizes[k])
    say(f"{n} pairs, {sum(r[1] for r in together)} matches")
