"""Workloads of the detector for timing and comparison, through its public entry points.

A case is a dict of plain values.  `prepare` makes what a program holds before
the call (images on the GPU, the workspace and the result buffers, a recorded
plan), `run` makes one call, `work` counts the bytes and operations that call
cannot do without, and `exact` computes the same results with plain torch in
64-bit integers.

Images are noise with a few drawn top-to-bottom curves: 8-bit ones as a
photograph's gradient image (normal noise, curves of U{120..220}), 16-bit ones
as a sensor image (exponential noise, additive curves).
"""

import math
import random

import numpy as np
import torch

from paper_1912_01884_amd import fhtp

# Shapes of the mixed batch: heights and band counts of its images; the widths
# are uniform in the case's range.
MIXED_HEIGHTS = (128, 256, 512, 1024, 2048)
MIXED_KS = (4, 8, 16)


def _case(name, kind, h, w, k, dtype, bend=-1, gamma=0.0, radius=0, horizontal=False, pin_j=-1,
          pin_pos=0, count=1, layout=0):
    c = dict(kind=kind, h=h, w=w, k=k, dtype=dtype, bend=bend, gamma=gamma, radius=radius,
             horizontal=horizontal, pin_j=pin_j, pin_pos=pin_pos, count=count, layout=layout)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: one thumbnail or one region of interest at a time,
        # where the launch and its latency are the cost.
        _case("detect_64", "detect", 64, 64, 4, "u8", bend=1),
        # One camera frame's gradient image, a call per frame.
        _case("detect_1024", "detect", 1024, 1024, 16, "u8", bend=4),
        # The headline workload: one large 16-bit scan.
        _case("detect_4096", "detect", 4096, 4096, 32, "u16", bend=8),
        # The largest scan: tables of 2.2 GB, 127 steps.
        _case("detect_16384", "detect", 16384, 16384, 128, "u16", bend=8),
        # A frame under the paper's own restriction, an angle of 10 degrees.
        _case("detect_angle_1024", "detect", 1024, 1024, 16, "u8", gamma=0.17),
        # The angle on few tall bands (long straight links).
        _case("detect_angle_tall", "detect", 2048, 2047, 8, "u8", gamma=0.17),
        # No bend limit, odd width: the baseline a user compares the limited curve with.
        _case("detect_unbounded", "detect", 2048, 1501, 16, "u16", bend=1 << 20),
        # A mostly horizontal curve through a marked point of a noisy frame:
        # transpose, smoothing and the pin together.
        _case("detect_ex_2048", "ex", 2048, 2048, 16, "u16", bend=6, radius=2, horizontal=True,
              pin_j=8, pin_pos=1000),
        # A fixed set of 256 images of mixed sizes, recorded once and replayed
        # on fresh pixels: offline processing of a collection.
        _case("plan_mixed_256", "plan", 0, 0, 0, "u8", bend=4, count=256, layout=4),
        # A group of requests as a server admits them, a new call for each group.
        _case("batch_mixed_32", "batch", 0, 0, 0, "u8", bend=4, count=32, layout=5),
        # The Hough tables alone, tall bands and a ragged width.
        _case("fht_tall_u16", "fht", 4096, 3001, 8, "u16"),
        # The dynamic programme alone on tables in hand, swept over the angle
        # (here 10 degrees) without transforming the image again.
        _case("dp_angle_4096", "dp", 4096, 4096, 32, "u16", gamma=math.radians(10)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: images of 48 to 8192 rows, bands of 8
    to 1024 rows, widths of 48 to 8192 columns, both pixel types, every bend form."""
    kind = rng.choice(("detect", "detect", "detect", "ex", "plan", "batch", "fht", "dp"))
    dtype = rng.choice(("u8", "u16"))
    if kind in ("plan", "batch"):
        return _case(None, kind, 0, 0, 0, rng.choice(("u8", "u8", "u16")),
                     bend=rng.randint(0, 8),
                     count=_log_int(rng, 4, 256 if kind == "plan" else 64),
                     layout=rng.randint(6, 1 << 20))
    while True:
        n = 1 << rng.randint(3, 10)
        k = _log_int(rng, 2, 64)
        w = _log_int(rng, 48, 8192)
        if 48 <= n * k <= 8192 and n * k * w <= 1 << 24:
            break
    h = n * k
    bend, gamma = -1, 0.0
    form = rng.choice(("fixed", "fixed", "wide", "angle", "angle", "none"))
    if form == "fixed":
        bend = rng.randint(0, 16)
    elif form == "wide":
        bend = rng.randint(17, 40)
    elif form == "angle":
        gamma = rng.uniform(0.02, 0.6)
    else:
        bend = 1 << 20
    radius, horizontal, pin_j, pin_pos = 0, False, -1, 0
    if kind == "ex":
        radius = rng.randint(0, 7)
        horizontal = rng.random() < 0.5
        if rng.random() < 0.6:
            pin_j, pin_pos = rng.randint(0, k), rng.randint(0, w - 1)
        if horizontal:  # the stored image is the transposed one
            h, w = w, h
    return _case(None, kind, h, w, k, dtype, bend=bend, gamma=gamma, radius=radius,
                 horizontal=horizontal, pin_j=pin_j, pin_pos=pin_pos)


# ---- inputs -------------------------------------------------------------------

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _image(rng, gen, h, w, k, dtype, horizontal=False):
    """Noise and three curves of k links; (h, w) as stored."""
    dev = _device()
    if dtype == "u8":
        img = torch.randn((h, w), generator=gen, device=dev).mul_(15.0).add_(30.0).round_()
        img = img.clamp_(0, 255).to(torch.int32)
    else:
        img = torch.empty((h, w), device=dev).exponential_(1.0 / 500.0, generator=gen).round_()
        img = img.clamp_(0, 65535).to(torch.int32)
    det = img.t() if horizontal else img
    rows, cols = det.shape
    n = rows // k
    reach = max(1, n // 4)
    for _ in range(3):
        d = [rng.randint(-reach, reach)]
        for _ in range(k - 1):
            d.append(max(-reach, min(reach, d[-1] + rng.randint(-2, 2))))
        x = np.concatenate([[0], np.cumsum(d)])
        x = x + rng.randint(0, cols - 1)
        path = np.concatenate([x[i] + (2 * d[i] * np.arange(n) + n) // (2 * n) for i in range(k)])
        path = torch.from_numpy(np.clip(path, 0, cols - 1)).to(dev)
        y = torch.arange(rows, device=dev)
        if dtype == "u8":
            det[y, path] = rng.randint(120, 220)
        else:
            det[y, path] = torch.clamp(det[y, path] + rng.randint(4000, 12000), max=65535)
    if dtype == "u8":
        return img.to(torch.uint8)
    return img.to(torch.uint16)


def _shapes(case):
    """(h, w, k) of every image of the case."""
    if case["kind"] not in ("plan", "batch"):
        return [(case["h"], case["w"], case["k"])]
    rng = random.Random(case["layout"])
    return [(rng.choice(MIXED_HEIGHTS), rng.randint(256, 2048), rng.choice(MIXED_KS))
            for _ in range(case["count"])]


def _images(case, seed):
    rng = random.Random(seed)
    gen = torch.Generator(device=_device()).manual_seed(seed)
    return [_image(rng, gen, h, w, k, case["dtype"], case["horizontal"])
            for h, w, k in _shapes(case)]


def _bend_args(case):
    return dict(gamma=case["gamma"]) if case["bend"] < 0 else dict(bend=case["bend"])


def _pin(case):
    return None if case["pin_j"] < 0 else (case["pin_j"], case["pin_pos"])


def prepare(case, seed):
    dev = _device()
    images = _images(case, seed)
    shapes = _shapes(case)
    state = {"case": case, "images": images}
    kind = case["kind"]
    code = fhtp.FHTP_U8 if case["dtype"] == "u8" else fhtp.FHTP_U16

    def buffer(nbytes):
        return torch.empty(max(1, nbytes), dtype=torch.uint8, device=dev)

    if kind == "fht":
        (h, w, k), = shapes
        state["tables"] = torch.empty(fhtp.table_shape(h, w, k), dtype=torch.int32, device=dev)
        state["ws"] = buffer(fhtp.fht_workspace_bytes(code, h, w, k))
        return state
    if kind in ("plan", "batch"):
        # results side by side in two buffers, as a program collects them
        state["scores"] = torch.zeros(len(shapes), dtype=torch.int32, device=dev)
        state["xs"] = torch.zeros(sum(k + 1 for _, _, k in shapes), dtype=torch.int32, device=dev)
        score_of = [state["scores"][q:q + 1] for q in range(len(shapes))]
        xs_of = list(torch.split(state["xs"], [k + 1 for _, _, k in shapes]))
        ks = [k for _, _, k in shapes]
        bends = [case["bend"]] * len(shapes)
        jobs, _ = fhtp.make_jobs(images, ks, bends=bends, scores=score_of, xss=xs_of)
        ws = buffer(fhtp.batch_workspace_bytes(jobs))
        state.update(ks=ks, bends=bends, score_of=score_of, xs_of=xs_of, ws=ws)
        if kind == "plan":
            state["plan"] = fhtp.Plan(images, ks, bends=bends, ws=ws, scores=score_of, xss=xs_of)
        return state
    (h, w, k), = shapes
    bend = fhtp.make_bend(case["bend"] if case["bend"] >= 0 else None,
                          None if case["bend"] >= 0 else case["gamma"])
    state["score"] = torch.zeros(1, dtype=torch.int32, device=dev)
    state["xs"] = torch.zeros(k + 1, dtype=torch.int32, device=dev)
    if kind == "dp":
        state["tables"] = fhtp.fht_bands(images[0], k)
        state["ws"] = buffer(fhtp.dp_workspace_bytes(h, w, k, bend))
        del state["images"]
    elif kind == "ex":
        opt = fhtp.make_options(case["radius"], case["horizontal"], _pin(case))
        state["ws"] = buffer(fhtp.detect_ex_workspace_bytes(code, h, w, k, bend, opt))
    else:
        state["ws"] = buffer(fhtp.detect_workspace_bytes(code, h, w, k, bend))
    return state


# ---- one pass -----------------------------------------------------------------

def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "detect":
        return fhtp.detect_polyline(state["images"][0], c["k"], ws=state["ws"],
                                    score=state["score"], xs=state["xs"], **_bend_args(c))
    if kind == "ex":
        return fhtp.detect_polyline_ex(state["images"][0], c["k"], smooth_radius=c["radius"],
                                       horizontal=c["horizontal"], pin=_pin(c), ws=state["ws"],
                                       score=state["score"], xs=state["xs"], **_bend_args(c))
    if kind == "dp":
        return fhtp.polyline_dp(state["tables"], c["h"], c["w"], c["k"], ws=state["ws"],
                                score=state["score"], xs=state["xs"], **_bend_args(c))
    if kind == "fht":
        return fhtp.fht_bands(state["images"][0], c["k"], tables=state["tables"], ws=state["ws"])
    if kind == "plan":
        state["plan"].launch()
    else:
        fhtp.detect_batch(state["images"], state["ks"], bends=state["bends"], ws=state["ws"],
                          scores=state["score_of"], xss=state["xs_of"])
    return {"scores": state["scores"], "xs": state["xs"]}


# ---- what a pass cannot do without --------------------------------------------

def work(case):
    """Bytes: inputs read once and outputs written once.  Operations: the
    additions of the transform (log2(n) per cell of both directions) and an
    addition and a comparison per cell of each step of the programme."""
    nbytes = ops = 0
    px = 1 if case["dtype"] == "u8" else 2
    for h, w, k in _shapes(case):
        if case["horizontal"]:
            h, w = w, h
        n = h // k
        W, D = w + n, 2 * n - 1
        tables = 4 * k * D * W
        if case["kind"] == "dp":
            nbytes += 4 * k * D * w + 4 * (k + 2)
        elif case["kind"] == "fht":
            nbytes += h * w * px + tables
        else:
            nbytes += h * w * px + 4 * (k + 2)
        if case["kind"] != "dp":
            ops += 2 * int(math.log2(n)) * n * W * k
        if case["kind"] != "fht":
            ops += 2 * (k - 1) * D * w
        if case["radius"]:
            ops += 2 * (2 * case["radius"] + 1) * h * w
    return {"bytes": nbytes, "flops": ops}


# ---- the same results in 64-bit integers ---------------------------------------

def _direction(band, W):
    """Dyadic line sums [shift][W] of one band [n][W], lines leaning right."""
    t = band.unsqueeze(1)  # [blocks][shifts][W]
    while t.shape[0] > 1:
        top, low = t[0::2], t[1::2]
        half = t.shape[1]
        out = torch.empty((top.shape[0], 2 * half, W), dtype=torch.int64, device=t.device)
        for s in range(2 * half):
            out[:, s] = top[:, s // 2] + torch.roll(low[:, s // 2], -((s + 1) // 2), dims=1)
        t = out
    return t[0]


def _band_table(img, i, n):
    """Band i's sums [2n - 1][w + n] over the zero-extended band."""
    w = img.shape[1]
    W = w + n
    band = torch.zeros((n, W), dtype=torch.int64, device=img.device)
    band[:, :w] = img[i * n:(i + 1) * n]
    right = _direction(band, W)
    left = _direction(band.flip(1), W).flip(1)
    return torch.cat([left[1:].flip(0), right])


def _windows(n, case):
    """Admissible successor rows lo[r] .. hi[r] of each row r = d + n - 1."""
    d = np.arange(-(n - 1), n, dtype=np.float64)
    if case["bend"] >= 0:
        ok = np.abs(d[None, :] - d[:, None]) <= case["bend"]
    else:
        ok = n * np.abs(d[None, :] - d[:, None]) <= math.tan(case["gamma"]) * (
            n * n + d[:, None] * d[None, :])
    return ok.argmax(1), ok.shape[1] - 1 - ok[:, ::-1].argmax(1)


def _best_polyline(img, k, case, pin):
    """(score, vertices) of the best polyline, ties to the smallest (x_0, d_0, ...)."""
    rows, w = img.shape
    n = rows // k
    D = 2 * n - 1
    dev = img.device
    lo, hi = (torch.from_numpy(v).to(dev) for v in _windows(n, case))
    r = torch.arange(D, device=dev)
    x = torch.arange(w, device=dev)
    succ = x[None, :] + (r - (n - 1))[:, None]  # x + d
    inside = (succ >= 0) & (succ < w)
    succ = succ.clamp(0, w - 1)
    reach_lo, reach_hi = int((lo - r).min()), int((hi - r).max())

    def masked(v, i):
        v = torch.where(inside, v, -1)
        if pin and pin[0] == i:
            v[:, x != pin[1]] = -1
        if pin and pin[0] == k and i == k - 1:
            v = torch.where(succ == pin[1], v, -1)
        return v

    v = masked(_band_table(img, k - 1, n)[:, :w], k - 1)
    links = []
    for i in range(k - 2, -1, -1):
        if case["bend"] >= 2 * n - 2:  # every successor: the column's maximum
            best = v.max(0).values.expand(D, w)
            first = torch.where(v == best, r[:, None], D).min(0).values.expand(D, w)
        else:
            best = torch.full((D, w), -2, dtype=torch.int64, device=dev)
            first = torch.zeros((D, w), dtype=torch.int64, device=dev)
            for off in range(reach_lo, reach_hi + 1):  # ascending, a later one only when larger
                q = r + off
                ok = (q >= lo) & (q <= hi) & (q >= 0) & (q < D)
                cand = torch.where(ok[:, None], v[q.clamp(0, D - 1)], -2)
                up = cand > best
                best = torch.where(up, cand, best)
                first = torch.where(up, q[:, None], first)
        links.append(first.to(torch.int16))
        m = best.gather(1, succ)
        h = _band_table(img, i, n)[:, :w]
        v = masked(torch.where(m >= 0, h + m, -1), i)
    links.reverse()  # links[i]: row of d_{i+1} at (d_i, x_{i+1})
    score = int(v.max())
    at = int((v.t().reshape(-1) == score).nonzero()[0])
    x0, row = at // D, at % D
    xs = [x0]
    for i in range(k):
        xs.append(xs[-1] + row - (n - 1))
        if i < k - 1:
            row = int(links[i][row, xs[-1]])
    return (torch.tensor([score], dtype=torch.int64), torch.tensor(xs, dtype=torch.int64))


def _prepared(img, case):
    """The detection image: transposed, its rows smoothed with the binomial kernel."""
    img = img.to(torch.int32).to(torch.int64)
    if case["horizontal"]:
        img = img.t().contiguous()
    rad = case["radius"]
    if rad:
        w = img.shape[1]
        x = torch.arange(w, device=img.device)
        acc = torch.full_like(img, 4 ** rad // 2)
        for i in range(2 * rad + 1):
            acc += math.comb(2 * rad, i) * img[:, (x + i - rad).clamp(0, w - 1)]
        img = acc >> (2 * rad)
    return img


def exact(case, seed):
    images = _images(case, seed)
    shapes = _shapes(case)
    if case["kind"] in ("plan", "batch"):
        if len(shapes) > 40:  # over twenty seconds
            return None
        got = [_best_polyline(_prepared(img, case), k, case, None)
               for img, (_, _, k) in zip(images, shapes)]
        return {"scores": torch.cat([s for s, _ in got]), "xs": torch.cat([x for _, x in got])}
    k = case["k"]
    img = _prepared(images[0], case)
    if case["kind"] == "fht":
        return torch.stack([_band_table(img, i, img.shape[0] // k) for i in range(k)])
    rows, w = img.shape
    lo, hi = _windows(rows // k, case) if case["bend"] < 2 * (rows // k) else (0, 0)
    if np.max(hi - lo + 1) * (2.0 * rows) * w > 3e11:  # over twenty seconds
        return None
    return _best_polyline(img, k, case, _pin(case))
