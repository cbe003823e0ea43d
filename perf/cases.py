"""The workloads this library is timed on: extraction (single images, batches,
graph replay, served requests), descriptor matching and geometric
verification, each through its public Python entry point.

A case is a dict of plain values.  ``kind`` is "extract", "match" or "verify".

Extraction cases: ``entry`` (extract, noalloc, batch, graph or server), ``n``
images with sides drawn from [h0, h1] x [w0, w1] (equal ends: fixed sizes; the
draw depends on the case alone, pixel values on the seed), ``blobs`` per
million pixels, ``pad`` unused columns per input row (an image that is a view
of a wider buffer), ``cap`` output rows per image, and the settings that users
change: octaves, upsampled octave, fp16 pyramid storage, pooled domain sizes
(1: none; 5: half-octave steps; 10: the linearly spaced set), RootSIFT, upright.
"""
import math

import numpy as np
import torch

from paper_2605_17869_amd import sift as sm

N_HYP = 1500        # homography hypotheses per pair
SIGMA_MAX = 2.0     # largest noise scale of verification, pixels
RATIO = 0.8


def _extract(name, entry, n, h, w, **kw):
    case = dict(name=name, kind="extract", entry=entry, n=n, h0=h[0], h1=h[1], w0=w[0], w1=w[1],
                blobs=1272, pad=0, cap=4096, octaves=4, upsample=0, fp16=0, dsp=1, rootsift=0,
                upright=0)
    case.update(kw)
    return case


def listed():
    return [
        # a crop or tile by itself: the smallest call, all latency and launches
        _extract("tile_97x131", "noalloc", 1, (97, 97), (131, 131), pad=5, cap=512),
        # one camera frame at a time (the plain per-image path)
        _extract("vga_480x640", "extract", 1, (480, 480), (640, 640), blobs=651, cap=2048),
        # a fixed-size camera rig: one recorded batch, replayed; fp16 levels
        # after the first octave, descriptors pooled over five domain sizes
        _extract("rig_graph_fp16_dsp5", "graph", 8, (600, 600), (800, 800), upsample=1, fp16=1,
                 dsp=5, rootsift=1, cap=2048),
        # the benchmark's default: a batch with the upsampled octave
        _extract("batch64_768x1024_up", "batch", 64, (768, 768), (1024, 1024), upsample=1),
        # larger photographs, the base octave at full size, for pairwise matching
        _extract("photos32_1066x1600", "batch", 32, (1066, 1066), (1600, 1600), blobs=2345,
                 cap=8192),
        # retrieval indexing: images of mixed sizes, ten pooled domain sizes, RootSIFT
        _extract("index64_dsp10", "batch", 64, (400, 900), (600, 1200), dsp=10, rootsift=1),
        # requests of any size handed to the continuous-batching server together
        _extract("served32_mixed", "server", 32, (320, 2048), (320, 2048), cap=8192),
        # one small pair of descriptor sets (two frames of a tracker)
        dict(name="match_pair_300x263", kind="match", n=1, na=300, nb=263),
        # image pairs of a photo collection
        dict(name="match32_2000x2000", kind="match", n=32, na=2000, nb=2000),
        # two images at the keypoint cap, one of them not quite full
        dict(name="match_pair_8192x7900", kind="match", n=1, na=8192, nb=7900),
        # one pair checked as soon as it is matched
        dict(name="verify_pair_211", kind="verify", n=1, m=211, outliers=0.3),
        # every pair of a photo collection
        dict(name="verify32_1300", kind="verify", n=32, m=1300, outliers=0.4),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    u = rng.random()
    if u < 0.2:
        na, nb = _log_int(rng, 150, 8192), _log_int(rng, 150, 8192)
        most = max(1, min(32, 32 * 2000 * 2000 // (na * nb)))
        return dict(kind="match", n=_log_int(rng, 1, most), na=na, nb=nb)
    if u < 0.35:
        m = _log_int(rng, 40, 4000)
        return dict(kind="verify", n=_log_int(rng, 1, max(1, min(32, 32 * 1300 // m))), m=m,
                    outliers=round(rng.uniform(0.1, 0.6), 3))
    entry = rng.choice(["extract", "noalloc", "batch", "batch", "graph", "server"])
    h, w = _log_int(rng, 97, 2048), _log_int(rng, 97, 2048)
    case = _extract("", entry, 1, (h, h), (w, w), blobs=rng.choice([651, 1272, 2345]),
                    pad=rng.choice([0, 0, rng.randint(1, 67)]), upsample=rng.choice([0, 0, 1]),
                    fp16=rng.choice([0, 0, 1]), dsp=rng.choice([1, 1, 5, 10]),
                    rootsift=rng.choice([0, 1]), upright=int(rng.random() < 0.1))
    del case["name"]
    if entry == "noalloc":   # the static scratch holds images up to about this size
        shrink = min(1.0, math.sqrt((300_000 if case["upsample"] else 1_500_000) / (h * w)))
        case["h0"] = case["h1"] = max(97, int(h * shrink))
        case["w0"] = case["w1"] = max(97, min(int(w * shrink), int(1.5e6) // case["h0"]))
        if case["upsample"]:
            case["w0"] = case["w1"] = max(97, min(case["w0"], 300_000 // case["h0"]))
    elif entry != "extract":
        # the largest listed batch bounds the work: pixels, more per pooled size
        cost = h * w * (4 if case["upsample"] else 1) * (1.0 + 0.3 * (case["dsp"] - 1))
        case["n"] = _log_int(rng, 2, max(2, min(64, int(100e6 / cost))))
        if rng.random() < 0.5:   # images of mixed sizes
            case["h0"], case["w0"] = max(97, int(h * 0.6)), max(97, int(w * 0.6))
    case["cap"] = max(512, min(8192, 256 * math.ceil(h * w * 2.5e-3 / 256)))
    return case


# ---------------------------------------------------------------------------
# Inputs

def _dsp(case):
    if case["dsp"] == 5:
        return [0.5, 2.0 ** -0.5, 1.0, 2.0 ** 0.5, 2.0]
    return [1.0] if case["dsp"] == 1 else [float(v) for v in np.linspace(1 / 6, 4 / 3, case["dsp"])]


def _settings(case):
    return dict(n_octaves=case["octaves"], upsample=case["upsample"], pyramid_fp16=case["fp16"],
                dsp_scales=_dsp(case), rootsift=case["rootsift"], upright=case["upright"],
                max_keypoints=8192)


def _sizes(case):
    rng = np.random.default_rng([case["n"], case["h1"], case["w1"]])
    return [(int(rng.integers(case["h0"], case["h1"] + 1)),
             int(rng.integers(case["w0"], case["w1"] + 1))) for _ in range(case["n"])]


def _image(seed, k, h, w, per_mpix):
    """Gaussian blobs on mid-grey plus low-passed noise, clipped to [0, 1]."""
    rng = np.random.default_rng([seed, k])
    nb = max(20, int(h * w * per_mpix * 1e-6))
    cx, cy = rng.uniform(0, w, nb), rng.uniform(0, h, nb)
    s, a = rng.uniform(1.5, 12.0, nb), rng.uniform(-0.5, 0.5, nb)
    cx, cy, s, a = (torch.from_numpy(v).cuda()[:, None] for v in (cx, cy, s, a))
    ex = torch.exp(-(torch.arange(w, device="cuda") - cx) ** 2 / (2 * s * s))
    ey = a * torch.exp(-(torch.arange(h, device="cuda") - cy) ** 2 / (2 * s * s))
    gen = torch.Generator(device="cuda").manual_seed(int(rng.integers(1 << 62)))
    noise = torch.randn((h + 6, w + 6), generator=gen, device="cuda", dtype=torch.float64) * 0.02
    t = [math.exp(-(i * i) / 0.98) for i in range(-3, 4)]
    noise = sum(g / sum(t) * noise[i:i + h] for i, g in enumerate(t))
    noise = sum(g / sum(t) * noise[:, i:i + w] for i, g in enumerate(t))
    return (0.5 + ey.t().contiguous() @ ex + noise).clamp_(0.0, 1.0).float()


def _images(case, seed):
    out = []
    for k, (h, w) in enumerate(_sizes(case)):
        im = _image(seed, k, h, w, case["blobs"])
        if case["pad"]:
            wide = torch.zeros((h, w + case["pad"]), device="cuda")
            wide[:, :w] = im
            im = wide[:, :w]
        out.append(im)
    return out


def _descriptors(case, seed, pair):
    """Non-negative unit rows; three quarters of the smaller set reappear in
    the other, perturbed and in another order."""
    gen = torch.Generator(device="cuda").manual_seed(1_000_003 * seed + pair)
    na, nb = case["na"], case["nb"]

    def rand(rows):
        return torch.randn((rows, 128), generator=gen, device="cuda")

    a, b = rand(na).abs(), rand(nb).abs()
    a = a / a.norm(dim=1, keepdim=True)
    c = 3 * min(na, nb) // 4
    src = torch.randperm(na, generator=gen, device="cuda")[:c]
    dst = torch.randperm(nb, generator=gen, device="cuda")[:c]
    b[dst] = a[src] + (0.1 * rand(c)).abs()
    return a.contiguous(), (b / b.norm(dim=1, keepdim=True)).contiguous()


def _points(case, seed, pair):
    """Correspondences under a homography near a similarity, in pixels of a
    1600 x 1066 image: noisy inliers and uniform outliers (float32)."""
    rng = np.random.default_rng([seed, pair])
    m, size = case["m"], np.array([1600.0, 1066.0])
    a = rng.uniform(0, 1, (m, 2)) * size
    ang, sc = rng.uniform(0, 2 * math.pi), rng.uniform(0.5, 2.0)
    c, s = math.cos(ang) * sc, math.sin(ang) * sc
    d = a - (size - 1) / 2
    p = rng.uniform(-2e-4, 2e-4, 2)
    b = d @ np.array([[c, s], [-s, c]]) / (1 + d @ p)[:, None] + (size - 1) / 2
    b += rng.normal(0, 0.5, (m, 2))
    out = rng.uniform(size=m) < case["outliers"]
    b[out] = rng.uniform(0, 1, (int(out.sum()), 2)) * size
    return a.astype(np.float32), b.astype(np.float32)


def _samples(case, seed):
    return np.random.default_rng([seed, 77]).random((N_HYP, 4), dtype=np.float32)


# ---------------------------------------------------------------------------
# The state a program keeps, and one pass

def prepare(case, seed):
    n = case["n"]
    if case["kind"] == "match":
        pairs = [(a, None, b, None) for a, b in (_descriptors(case, seed, k) for k in range(n))]
        rec = torch.zeros((n, min(case["na"], case["nb"]), 4), dtype=torch.int32, device="cuda")
        cnt = torch.zeros((n, 2), dtype=torch.int32, device="cuda")
        outs = [sm.Matches(rec[i], cnt[i]) for i in range(n)]
        state = dict(kind="match", pairs=pairs, outs=outs,
                     result=(rec[:, :, :2], rec.view(torch.float32)[:, :, 2:], cnt))
    elif case["kind"] == "verify":
        m = case["m"]
        pairs = []
        for k in range(n):
            kp = np.zeros((2, m, 12), np.float32)
            kp[0, :, :2], b = _points(case, seed, k)
            perm = np.random.default_rng([seed, k, 5]).permutation(m)
            kp[1, perm, :2] = b
            rec = np.zeros((m, 4), np.int32)
            rec[:, 0], rec[:, 1] = np.arange(m), perm
            kp = torch.from_numpy(kp.view(np.int32)).cuda()
            pairs.append((kp[0], kp[1], torch.from_numpy(rec).cuda(), None))
        H = torch.zeros((n, 9), dtype=torch.float64, device="cuda")
        score = torch.zeros((n, 1), dtype=torch.float64, device="cuda")
        ints = torch.zeros((n, 2), dtype=torch.int32, device="cuda")
        wts = torch.zeros((n, m), device="cuda")
        outs = [sm.Verification(H[i], score[i], ints[i], wts[i]) for i in range(n)]
        state = dict(kind="verify", pairs=pairs, outs=outs,
                     samples=torch.from_numpy(_samples(case, seed)).cuda(),
                     result=(H, score, ints, wts))
    else:
        images, cap = _images(case, seed), case["cap"]
        kp = torch.zeros((n, cap, 12), dtype=torch.int32, device="cuda")
        desc = torch.zeros((n, cap, 128), device="cuda")
        cnt = torch.zeros((n, 3), dtype=torch.int32, device="cuda")
        outs = [sm.Features(kp[i], desc[i], cnt[i]) for i in range(n)]
        state = dict(kind=case["entry"], images=images, outs=outs,
                     result=(kp.view(torch.float32)[:, :, :5], kp[:, :, 5:], desc, cnt))
        if case["entry"] == "server":
            need = sm.server_batch_bytes(_settings(case), [tuple(im.shape) for im in images])
            state["server"] = sm.Server(_settings(case), arena_bytes=2 * need + (64 << 20))
        else:
            state["ex"] = ex = sm.Extractor(_settings(case))
            if case["entry"] == "graph":
                state["graph"] = ex.graph(images, outs=outs)
    torch.cuda.synchronize()
    return state


def run(state):
    kind = state["kind"]
    if kind == "match":
        sm.match_batch(state["pairs"], ratio=RATIO, outs=state["outs"])
    elif kind == "verify":
        sm.verify_batch(state["pairs"], state["samples"], sigma_max=SIGMA_MAX, outs=state["outs"])
    elif kind == "extract":
        state["ex"].extract(state["images"][0], out=state["outs"][0])
    elif kind == "noalloc":
        state["ex"].extract_noalloc(state["images"][0], state["outs"][0])
    elif kind == "batch":
        state["ex"].extract_batch(state["images"], outs=state["outs"])
    elif kind == "graph":
        state["graph"].launch()
    else:
        srv = state["server"]
        for ticket in srv.submit_many(state["images"], outs=state["outs"]):
            srv.wait(ticket)
    return state["result"]


def work(case):
    """Inputs read once and outputs written once; operations: the separable
    taps of the pyramid, the similarity products, the residuals."""
    n = case["n"]
    if case["kind"] == "match":
        na, nb = case["na"], case["nb"]
        return {"bytes": n * (512 * (na + nb) + 12 * min(na, nb)), "flops": 256 * n * na * nb}
    if case["kind"] == "verify":
        # 24 operations per residual and weight, every hypothesis and match
        return {"bytes": n * 16 * (case["m"] + 6) + 16 * N_HYP, "flops": 24 * n * N_HYP * case["m"]}
    px = sum(h * w for h, w in _sizes(case))
    rows = 0.9e-6 * case["blobs"] * px            # keypoints, about nine per ten blobs
    first, later = (5, 5, 7, 8, 10, 13), (5, 7, 8, 10, 13)
    taps, area = 0.0, float(px)
    if case["upsample"]:
        area *= 4
    else:
        first = (7,) + first[1:]
    for k in range(case["octaves"] + case["upsample"]):
        taps += area * sum(2 * (2 * r + 1) for r in (later if k else first))
        area /= 4
    return {"bytes": int(4 * px + 560 * rows), "flops": int(2 * taps)}


# ---------------------------------------------------------------------------
# The same results in 64 bits

def exact(case, seed):
    if case["kind"] == "match":
        return _match64(case, seed)
    if case["kind"] == "verify":
        return _verify64(case, seed)
    # fp16 storage rounds levels by design and has no 64-bit value; batches
    # take the arithmetic of single images and would take minutes here
    px = sum(h * w for h, w in _sizes(case)) * (4 if case["upsample"] else 1)
    if case["fp16"] or px * (1 + 0.3 * (case["dsp"] - 1)) > 1_300_000:
        return None
    n, cap = case["n"], case["cap"]
    kp, desc = np.zeros((n, cap, 5)), np.zeros((n, cap, 128))
    for i, im in enumerate(_images(case, seed)):
        k, d = _sift64(im.double().cpu().numpy(), case)
        m = min(len(k), cap)
        kp[i, :m], desc[i, :m] = k[:m], d[:m]
    return (torch.from_numpy(kp), None, torch.from_numpy(desc), None)


def _match64(case, seed):
    """Similarities are defined on descriptors rounded to fp16."""
    na, nb, n = case["na"], case["nb"], case["n"]
    out = torch.zeros((n, min(na, nb), 2), dtype=torch.float64)
    for i in range(n):
        a, b = _descriptors(case, seed, i)
        s = a.half().double() @ b.half().double().t().contiguous()
        (v1, j1), (v2, _) = s.max(dim=1), s.topk(2, dim=1).values.min(dim=1)
        (w1, i1), (w2, _) = s.max(dim=0), s.topk(2, dim=0).values.min(dim=0)

        def passes(best, second):
            return (2 - 2 * best).clamp(min=0) < RATIO * RATIO * (2 - 2 * second).clamp(min=0)

        rows = torch.arange(na, device=s.device)
        keep = (i1[j1] == rows) & passes(v1, v2) & passes(w1, w2)[j1]
        v = v1[keep].cpu()
        out[i, :len(v), 0] = v
        out[i, :len(v), 1] = (2 - 2 * v).clamp(min=0).sqrt()
    return (None, out, None)


def _verify64(case, seed):
    n, m = case["n"], case["m"]
    u = torch.from_numpy(_samples(case, seed)).double()
    tau = math.sqrt(2 * math.log(100.0))
    erf_tau = math.erf(tau / math.sqrt(2))

    def weights(H, a, b):      # H [k, 3, 3] -> [k, m]
        q = torch.cat([a, torch.ones(len(a), 1, dtype=a.dtype, device=a.device)], 1)
        p = q @ H.transpose(1, 2).contiguous()
        r = (p[..., :2] / p[..., 2:] - b).norm(dim=-1)
        w = math.sqrt(math.pi / 2) / SIGMA_MAX * (erf_tau - torch.special.erf(
            r / (math.sqrt(2) * SIGMA_MAX)))
        return torch.where((p[..., 2] > 0) & (r < tau * SIGMA_MAX), w, torch.zeros_like(w))

    def normaliser(p):
        c = p.mean(0)
        s = math.sqrt(2) / (p - c).norm(dim=1).mean()
        T = torch.eye(3, dtype=p.dtype)
        T[0, 0] = T[1, 1] = s
        T[:2, 2] = -s * c
        return T, (p - c) * s

    def rows(a, b):            # [..., 4 or m, 2] -> [..., 2 x points, 9]
        x, y, p, q = a[..., 0], a[..., 1], b[..., 0], b[..., 1]
        o, z = torch.ones_like(x), torch.zeros_like(x)
        r1 = torch.stack([x, y, o, z, z, z, -p * x, -p * y, p], -1)
        r2 = torch.stack([z, z, z, x, y, o, -q * x, -q * y, q], -1)
        return torch.stack([r1, r2], -2).flatten(-3, -2)

    def pixels(h, Ta, Tb):
        M = torch.cat([h, torch.ones_like(h[..., :1])], -1).unflatten(-1, (3, 3))
        M = torch.linalg.inv(Tb) @ M @ Ta
        return M / M[..., 2:, 2:]

    Hs, scores, wts = [], [], []
    for i in range(n):
        a, b = (torch.from_numpy(v).double() for v in _points(case, seed, i))
        (Ta, an), (Tb, bn) = normaliser(a), normaliser(b)
        idx = (u * m).floor().long().clamp(max=m - 1)
        same = torch.zeros(N_HYP, dtype=torch.bool)
        for j in range(4):
            for k in range(j):
                same |= idx[:, j] == idx[:, k]
        A = rows(an[idx], bn[idx])
        A[same, :, :8] = torch.eye(8, dtype=A.dtype)
        h = torch.linalg.solve_ex(A[..., :8], A[..., 8:])[0].squeeze(-1)
        H = pixels(h, Ta, Tb)
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        sc = weights(H.to(dev), a.to(dev), b.to(dev)).sum(1).cpu()
        sc[same | ~torch.isfinite(sc)] = -math.inf
        best = int(sc.argmax())
        H, Q = H[best:best + 1], float(sc[best])
        R = rows(an, bn)
        for _ in range(5):
            w = weights(H, a, b)[0].repeat_interleave(2)[:, None]
            N = R[:, :8].t().contiguous() @ (w * R)
            H2 = pixels(torch.linalg.solve(N[:, :8], N[:, 8:]).t().contiguous(), Ta, Tb)
            Q2 = float(weights(H2, a, b).sum())
            if not Q2 > Q:
                break
            H, Q = H2, Q2
        Hs.append(H.reshape(9))
        scores.append([Q])
        wts.append(weights(H, a, b)[0])
    return (torch.stack(Hs), torch.tensor(scores, dtype=torch.float64), None, torch.stack(wts))


def _mirror(i, n):
    i = np.abs(i) % (2 * (n - 1))
    return np.where(i >= n, 2 * (n - 1) - i, i)


def _blur64(im, sigma):
    r = math.ceil(4 * sigma)
    g = np.exp(-np.arange(-r, r + 1) ** 2 / (2 * sigma * sigma))
    g /= g.sum()
    h, w = im.shape
    im = im[_mirror(np.arange(-r, h + r), h)]
    im = sum(t * im[i:i + h] for i, t in enumerate(g))
    im = im[:, _mirror(np.arange(-r, w + r), w)]
    return sum(t * im[:, i:i + w] for i, t in enumerate(g))


def _sift64(img, case):
    """Keypoints [k, 5] (x, y, sigma, angle, response) and descriptors of one
    image, three scales per octave, in the library's order."""
    up, s, s0, T, border = case["upsample"], 3, 1.6, 0.04 / 3, 5
    base = img
    if up:
        h, w = img.shape
        base = img[np.minimum(np.arange(2 * h + 1) // 2, h - 1)]
        base = ((base[:-1] + base[1:]) / 2)
        base = base[:, np.minimum(np.arange(2 * w + 1) // 2, w - 1)]
        base = ((base[:, :-1] + base[:, 1:]) / 2)
    base = _blur64(base, math.sqrt(s0 * s0 - (0.5 * (2 if up else 1)) ** 2))
    inc = [s0 * math.sqrt(4 ** (i / s) - 4 ** ((i - 1) / s)) for i in range(1, s + 3)]
    kps, descs = [], []
    for o in range(-up, case["octaves"]):
        L = [base]
        for sg in inc:
            L.append(_blur64(L[-1], sg))
        D = np.stack(L[1:]) - np.stack(L[:-1])
        h, w = base.shape
        mid = D[1:-1, border:h - border, border:w - border]
        hi, lo = np.full(mid.shape, -np.inf), np.full(mid.shape, np.inf)
        for a in range(3):
            for r in range(-1, 2):
                for c in range(-1, 2):
                    if (a, r, c) != (1, 0, 0):
                        nb = D[a:a + s, border + r:h - border + r, border + c:w - border + c]
                        hi, lo = np.maximum(hi, nb), np.minimum(lo, nb)
        found = np.argwhere((np.abs(mid) > 0.5 * T) & ((mid > hi) | (mid < lo)))
        for li, r, c in found + [1, border, border]:
            kp = _refine64(D, li, r, c, s, border, T)
            if kp is None:
                continue
            li, r, c, x, resp = kp
            sig = s0 * 2 ** ((li + x[2]) / s)
            gy = np.zeros((h, w))
            gx = np.zeros((h, w))
            gx[1:-1, 1:-1] = (L[li][:, 2:] - L[li][:, :-2])[1:-1]
            gy[1:-1, 1:-1] = (L[li][2:] - L[li][:-2])[:, 1:-1]
            for ang in ([0.0] if case["upright"] else _angles64(gx, gy, r, c, sig)):
                kps.append([(c + x[0]) * 2.0 ** o, (r + x[1]) * 2.0 ** o, sig * 2.0 ** o, ang, resp])
                descs.append(_describe64(gx, gy, r, c, x, sig, ang, case))
        base = L[s][::2, ::2]
    return np.array(kps).reshape(-1, 5), np.array(descs).reshape(-1, 128)


def _refine64(D, li, r, c, s, border, T):
    h, w = D.shape[1:]
    for _ in range(5):
        d = D[li - 1:li + 2, r - 1:r + 2, c - 1:c + 2]
        v = d[1, 1, 1]
        g = 0.5 * np.array([d[1, 1, 2] - d[1, 1, 0], d[1, 2, 1] - d[1, 0, 1],
                            d[2, 1, 1] - d[0, 1, 1]])
        xx, yy = d[1, 1, 2] + d[1, 1, 0] - 2 * v, d[1, 2, 1] + d[1, 0, 1] - 2 * v
        ss = d[2, 1, 1] + d[0, 1, 1] - 2 * v
        xy = 0.25 * (d[1, 2, 2] - d[1, 2, 0] - d[1, 0, 2] + d[1, 0, 0])
        xs = 0.25 * (d[2, 1, 2] - d[2, 1, 0] - d[0, 1, 2] + d[0, 1, 0])
        ys = 0.25 * (d[2, 2, 1] - d[2, 0, 1] - d[0, 2, 1] + d[0, 0, 1])
        try:
            x = np.linalg.solve(np.array([[xx, xy, xs], [xy, yy, ys], [xs, ys, ss]]), -g)
        except np.linalg.LinAlgError:
            return None
        if np.all(np.abs(x) <= 0.5):
            resp = abs(v + 0.5 * g @ x)
            det = xx * yy - xy * xy
            if resp >= T and det > 0 and (xx + yy) ** 2 * 10 < 121 * det:
                return li, r, c, x, resp
            return None
        if np.any(np.abs(x) > 1e6):
            return None
        step = np.where(np.abs(x) > 0.5, np.sign(x) * np.floor(np.abs(x) + 0.5), 0).astype(int)
        c, r, li = c + step[0], r + step[1], li + step[2]
        if not (1 <= li <= s and border <= r < h - border and border <= c < w - border):
            return None
    return None


def _window64(gx, gy, r, c, R):
    h, w = gx.shape
    r0, r1, c0, c1 = max(r - R, 1), min(r + R + 1, h - 1), max(c - R, 1), min(c + R + 1, w - 1)
    dy, dx = np.mgrid[r0 - r:r1 - r, c0 - c:c1 - c]
    a, b = gx[r0:r1, c0:c1], gy[r0:r1, c0:c1]
    return dx.ravel(), dy.ravel(), np.hypot(a, b).ravel(), (np.arctan2(b, a) % (2 * math.pi)).ravel()


def _angles64(gx, gy, r, c, sig):
    sw = 1.5 * sig
    dx, dy, mag, th = _window64(gx, gy, r, c, int(3 * sw + 0.5))
    wgt = mag * np.exp(-(dx * dx + dy * dy) / (2 * sw * sw))
    pos = th * 36 / (2 * math.pi)
    b = np.floor(pos).astype(int)
    f = pos - b
    hist = np.bincount(b % 36, wgt * (1 - f), 36) + np.bincount((b + 1) % 36, wgt * f, 36)
    hist = 0.25 * np.roll(hist, 1) + 0.5 * hist + 0.25 * np.roll(hist, -1)
    left, right = np.roll(hist, 1), np.roll(hist, -1)
    peaks = np.flatnonzero((hist > left) & (hist > right) & (hist >= 0.8 * hist.max()) & (hist > 0))
    return [((p + 0.5 * (left[p] - right[p]) / (left[p] - 2 * hist[p] + right[p])) * 10) % 360
            for p in peaks]


def _describe64(gx, gy, r, c, x, sig, ang, case):
    t = math.radians(ang)
    ct, st = math.cos(t), math.sin(t)
    scales = _dsp(case)
    R = math.ceil(2.5 * 3 * sig * max(scales) * (abs(ct) + abs(st))) + 1
    dx, dy, mag, th = _window64(gx, gy, r, c, R)
    u, v = dx - x[0], dy - x[1]
    xr, yr = ct * u + st * v, ct * v - st * u
    ob = ((th - t) % (2 * math.pi)) * 8 / (2 * math.pi)
    hist = np.zeros(6 * 6 * 8)
    for k in scales:
        a, b = xr / (3 * sig * k), yr / (3 * sig * k)
        ok = (np.abs(a) < 2.5) & (np.abs(b) < 2.5)
        a, b, q = a[ok], b[ok], ob[ok]
        wgt = mag[ok] * np.exp(-(a * a + b * b) / 8)
        a, b = a + 2.5, b + 2.5        # cell (0, 0) of the grid sits at (1, 1)
        ia, ib, iq = np.floor(a).astype(int), np.floor(b).astype(int), np.floor(q).astype(int)
        fa, fb, fq = a - ia, b - ib, q - iq
        for ja, wa in ((0, 1 - fa), (1, fa)):
            for jb, wb in ((0, 1 - fb), (1, fb)):
                for jq, wq in ((0, 1 - fq), (1, fq)):
                    cell = ((ib + jb) * 6 + ia + ja) * 8 + (iq + jq) % 8
                    hist += np.bincount(cell, wgt * wa * wb * wq, 288)
    d = hist.reshape(6, 6, 8)[1:5, 1:5].ravel() / len(scales)

    def unit(q):
        norm = np.linalg.norm(q)
        return q / norm if norm > 0 else q * 0

    d = unit(np.minimum(unit(d), 0.2))
    if case["rootsift"]:
        d = np.sqrt(d / d.sum()) if d.sum() > 0 else d
    return d
