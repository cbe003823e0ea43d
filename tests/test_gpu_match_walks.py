"""Walks of unequal lengths (one set much longer than the other, in either order, one
row, empty sets, counts below capacity) in every plan that workspaces between the least
and the asked-for size select: against the FP64 reference matcher, and the same bits.
Needs an MI355X."""
import ctypes

import numpy as np
import pytest

from paper_2605_17869_amd import synth
from gpu_util import require_gpu, say
from test_gpu_match import check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,counts", [
    ([(3000, 40)], None), ([(40, 3000)], None), ([(1, 1500)], None), ([(1500, 1)], None),
    ([(2500, 129), (130, 1999), (0, 300), (300, 0), (128, 128)], None),
    ([(4224, 300)], [(4100, 257)]), ([(300, 4224)], [(1, 129)]), ([(4224, 300)], [(0, 300)]),
    ([(9000, 2200)], None),                                  # copied to fp16, walks of 18 and 71 tiles
    ([(1200 - 31 * k, 20 + 9 * k) for k in range(34)], None)])   # pairs in a table
def test_every_plan(sizes, counts):
    torch = require_gpu()
    from paper_2605_17869_amd import sift as sm
    lib = sm.load_library()
    sets = [synth.descriptor_sets(5100 + k, max(na, 1), max(nb, 1), min(na, nb) // 2, 0.1)[:2]
            for k, (na, nb) in enumerate(sizes)]
    dev = [tuple(torch.from_numpy(x).cuda() for x in s) for s in sets]
    cts = counts and [torch.tensor(c, dtype=torch.int32, device="cuda") for c in counts]
    n = len(sizes)
    up = lambda v: (v + 255) // 256 * 256
    need = ctypes.c_size_t()

    def call(frac):
        arr, keep = (sm.SiftMatchPair * n)(), []
        for k, (na, nb) in enumerate(sizes):
            cap = max(min(na, nb), 1)
            rec = torch.zeros((cap, 4), dtype=torch.int32, device="cuda")
            cnt = torch.zeros(2, dtype=torch.int32, device="cuda")
            keep.append((rec, cnt))
            pa, pb = (cts[k].data_ptr(), cts[k].data_ptr() + 4) if cts else (None, None)
            arr[k] = sm.SiftMatchPair(dev[k][0].data_ptr(), pa, na, dev[k][1].data_ptr(), pb, nb,
                                      rec.data_ptr(), cnt.data_ptr(), cnt.data_ptr() + 4, cap)
        assert lib.sift_match_workspace_size(n, arr, ctypes.byref(need)) == 0
        least = up(96 * n) + 2 * up(4 * n + 4) + sum(up(16 * (na + nb)) for na, nb in sizes)
        assert least <= need.value
        size = int(need.value - frac * (need.value - least)) // 256 * 256
        ws = torch.empty(size + 256, dtype=torch.uint8, device="cuda").fill_(0xff)   # NaN, -1
        st = lib.sift_match_batch(n, arr, ctypes.c_float(0.8), ctypes.c_void_p(ws.data_ptr()), size,
                                  ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == 0, sm.STATUS_NAMES[st]
        torch.cuda.synchronize()
        assert bool((ws[size:] == 0xff).all())
        return size, [(r.cpu().numpy(), c.cpu().numpy()) for r, c in keep]

    size, ref = call(0.0)
    for k, (na, nb) in enumerate(sizes):
        ca, cb = counts[k] if counts else (na, nb)
        rec, (written, found) = ref[k]
        assert written == found
        if ca and cb:
            check_against_oracle(sets[k][0][:ca], sets[k][1][:cb],
                                 rec[:written].view(sm.MATCH_DTYPE).reshape(-1), found)
        else:
            assert found == 0
    sizes_run = [size]
    for frac in (0.1, 0.4, 0.7, 0.9, 1.0):
        size, got = call(frac)
        sizes_run.append(size)
        for (r, c), (r0, c0) in zip(got, ref):
            assert r.tobytes() == r0.tobytes() and c.tobytes() == c0.tobytes(), size
    say(f"{n} pairs {sizes[0]}: workspaces {sizes_run}, {[int(c[0]) for _, c in ref[:5]]} matches")
