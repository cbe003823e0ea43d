"""The matcher's plans: sets converted tile by tile or copied to fp16 first,
walks cut into parts or not, parts merged at the emission or before it, and the
plan of a small workspace.  Every one against the FP64 reference matcher at the
edges of tiles and parts, and against each other bit for bit.  Needs an MI355X."""
import ctypes

import numpy as np
import pytest

from paper_2605_17869_amd import synth
from gpu_util import require_gpu, say
from test_gpu_match import check_against_oracle, gpu_match

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("na,nb,counts", [
    (128, 1, None), (1, 129, None), (257, 1025, None),     # one tile; a row past a tile; parts of one tile
    (1100, 1200, None),                                    # parts merged before the emission
    (4200, 4300, None), (4097, 4225, (4096, 4096)),        # copied to fp16, 256 own rows a group
    (4300, 4200, (130, 4099)), (4300, 4200, (4100, 1)),    # most parts empty
])
def test_plans_equal_oracle(na, nb, counts):
    a, b, _ = synth.descriptor_sets(4000 + na, na, nb, (2 * min(na, nb)) // 3, 0.1)
    (rec, nf), = gpu_match([(a, b)], counts=[counts])
    ca, cb = counts or (na, nb)
    n_ref, marginal = check_against_oracle(a[:ca], b[:cb], rec, nf)
    say(f"{na}x{nb} {counts}: gpu {len(rec)} oracle {n_ref} marginal rows {marginal}")


@pytest.mark.parametrize("sizes", [[(300, 263)], [(4200, 4300), (77, 900)], [(0, 50), (1500, 1700)]])
def test_small_workspace_same_bits(sizes):
    torch = require_gpu()
    from paper_2605_17869_amd import sift as sm
    lib = sm.load_library()
    sets = [synth.descriptor_sets(77 + k, max(na, 1), nb, min(na, nb) // 2, 0.1)[:2]
            for k, (na, nb) in enumerate(sizes)]
    dev = [tuple(torch.from_numpy(x).cuda() for x in s) for s in sets]
    out = []
    for least in (False, True):
        arr = (sm.SiftMatchPair * len(sizes))()
        keep = []
        for k, (na, nb) in enumerate(sizes):
            cap = max(min(na, nb), 1)
            rec = torch.zeros((cap, 4), dtype=torch.int32, device="cuda")
            cnt = torch.zeros(2, dtype=torch.int32, device="cuda")
            keep.append((rec, cnt))
            arr[k] = sm.SiftMatchPair(dev[k][0].data_ptr(), None, na, dev[k][1].data_ptr(), None, nb,
                                      rec.data_ptr(), cnt.data_ptr(), cnt.data_ptr() + 4, cap)
        need = ctypes.c_size_t()
        assert lib.sift_match_workspace_size(len(sizes), arr, ctypes.byref(need)) == 0
        # what a call needed before it could be cut into parts: tables, the
        # nearest of every row and one summary per b row and 128 a rows
        up = lambda v: (v + 255) // 256 * 256
        was = up(96 * len(sizes)) + 2 * up(4 * len(sizes) + 4) + sum(
            up(16 * na) + up(16 * nb) + up(16 * nb * ((na + 127) // 128)) for na, nb in sizes)
        size = min(was, need.value) if least else max(was, need.value)
        ws = torch.empty(size + 256, dtype=torch.uint8, device="cuda")
        ws[size:] = 0x5a
        st = lib.sift_match_batch(len(sizes), arr, ctypes.c_float(0.8), ctypes.c_void_p(ws.data_ptr()),
                                  size, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == 0, sm.STATUS_NAMES[st]
        torch.cuda.synchronize()
        assert bool((ws[size:] == 0x5a).all())
        out.append([(r.cpu().numpy().tobytes(), c.cpu().numpy().tobytes()) for r, c in keep])
    assert out[0] == out[1]
    assert any(np.frombuffer(c, np.int32)[0] > 0 for _, c in out[0])
