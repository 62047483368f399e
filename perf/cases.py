"""Performance cases of the framework's public entry points.

Every case is a call (or a short chain of calls) that a program makes with
images already on the GPU: one image at a time from small tiles to a whole
16384 x 16384 slide level, batches of unequal tiles, jobs through the
continuous-batching server, and the segmentation operations alone and chained.
Images are drawn on the GPU in the manner of ``paper_1311_0378_amd.synth``:
uniform noise on [0, 80) blurred with sigma 4, with disks of radius 5..15 and
value 150..250 (some of them rings) painted over it, at 50 or 200 disks per
1024 x 1024 pixels.

Calls that work in place get a fresh copy of their input first, as a program
that keeps its input would make; the copy is part of a pass.
"""
import math
import random

import torch

from paper_1311_0378_amd import mrecon, ops

RECON, FILL = mrecon.MR_OP_RECON, mrecon.MR_OP_FILL
MPX = 1 << 20


def listed():
    return [
        # The smallest calls: one small tile of odd size, where launches and
        # latency count (batches and serving both start near this size).
        dict(name="recon_small", path="recon", H=293, W=421, pad=0, dtype="u8", conn=8, density=200),
        # One ordinary field of view of odd size through the whole
        # segmentation chain, from the colour image to labels and distances.
        dict(name="segment_ragged", path="segment", H=1003, W=1021, conn=4, density=200, rings=0.1),
        # A whole slide level, both pixel types: the largest single images.
        dict(name="recon_slide_u8", path="recon", H=16384, W=16384, pad=0, dtype="u8", conn=8, density=50),
        dict(name="recon_slide_i32", path="recon", H=16384, W=16384, pad=0, dtype="i32", conn=8, density=50),
        # The usual 4096 x 4096 slide tile: holes of a thresholded image.
        dict(name="fill_tile", path="fill", H=4096, W=4096, pad=0, dtype="u8", conn=4, density=50, rings=0.05),
        # The dual reconstruction on such a tile: a flood through the whole
        # background, the longest dependent chain of the reconstructions.
        dict(name="erode_tile", path="erode", H=4096, W=4096, pad=0, dtype="u8", conn=8, density=50),
        # Independent tiles of unequal, mostly odd sizes in one call.
        dict(name="batch_tiles", path="batch", n=40, lo=256, hi=4096, shapes=0, dtype="u8", conn=8,
             fills=0.3, graph=False, density=200),
        # Device jobs through the server, back to back.
        dict(name="serve_jobs", path="serve", n=24, lo=512, hi=4096, shapes=1, dtype="u8", conn=8,
             fills=0.3, density=200),
        # The regular operations on a slide level: colour to gray, opening.
        dict(name="gray_open_slide", path="gray_open", H=16384, W=16384, density=50),
        # Distances inside the objects of a slide level.
        dict(name="distance_slide", path="distance", H=16384, W=16384, conn=8, density=50),
        # Labelling a slide level's objects and keeping those of a size range.
        dict(name="label_slide", path="label", H=16384, W=16384, pad=0, conn=8, density=50,
             lo_area=150, hi_area=500),
        # Domes of a tile with wide pixels (h-dome: seeds of the objects).
        dict(name="dome_tile", path="dome", H=4096, W=4096, kind="hdome", dtype="i32", conn=8, density=50),
    ]


def _side(rng, lo, hi):
    """A side drawn over its logarithm, rounded to a multiple of 64 now and
    then (tile sizes) and otherwise as it falls (odd sizes among them)."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.3:
        v = max(64, (v + 32) // 64 * 64)
    return max(lo, min(hi, v))


def _sides(rng, lo, hi, most):
    while True:
        H, W = _side(rng, lo, hi), _side(rng, lo, hi)
        if H * W <= most:
            return H, W


def draw(rng: random.Random):
    path = rng.choice(["recon", "recon", "recon", "fill", "erode", "batch", "serve", "gray_open",
                       "distance", "label", "dome", "segment"])
    dtype, conn = rng.choice(["u8", "u8", "i32"]), rng.choice([8, 8, 4])
    density = rng.choice([50, 200])
    pad = rng.choice([0, 0, 0, rng.randrange(1, 130)])  # row elements past the image: a window
    if path == "recon":
        H, W = _sides(rng, 200, 16384, 128 * MPX)
        return dict(path=path, H=H, W=W, pad=pad, dtype=dtype, conn=conn, density=density)
    if path == "fill":
        H, W = _sides(rng, 200, 8192, 64 * MPX)
        return dict(path=path, H=H, W=W, pad=pad, dtype=dtype, conn=conn, density=density,
                    rings=rng.choice([0.0, 0.05, 0.5]))
    if path == "erode":
        H, W = _sides(rng, 200, 4096, 16 * MPX)
        return dict(path=path, H=H, W=W, pad=pad, dtype=dtype, conn=conn, density=density)
    if path == "batch":
        return dict(path=path, n=rng.randrange(6, 49), lo=256, hi=rng.choice([1024, 4096]),
                    shapes=rng.randrange(1 << 20), dtype=dtype, conn=conn,
                    fills=rng.choice([0.0, 0.3, 1.0]), graph=rng.random() < 0.5, density=density)
    if path == "serve":
        return dict(path=path, n=rng.randrange(8, 41), lo=512, hi=rng.choice([1024, 4096]),
                    shapes=rng.randrange(1 << 20), dtype=dtype, conn=conn,
                    fills=rng.choice([0.0, 0.3]), density=density)
    if path == "gray_open":
        H, W = _sides(rng, 200, 16384, 128 * MPX)
        return dict(path=path, H=H, W=W, density=density)
    if path == "distance":
        H, W = _sides(rng, 200, 16384, 128 * MPX)
        return dict(path=path, H=H, W=W, conn=conn, density=density)
    if path == "label":
        H, W = _sides(rng, 200, 16384, 128 * MPX)
        return dict(path=path, H=H, W=W, pad=pad, conn=conn, density=density,
                    lo_area=rng.choice([50, 150]), hi_area=rng.choice([300, 500]))
    if path == "dome":
        H, W = _sides(rng, 200, 8192, 32 * MPX)
        return dict(path=path, H=H, W=W, kind=rng.choice(["hdome", "maxima"]), dtype=dtype,
                    conn=conn, density=density)
    H, W = _sides(rng, 200, 4096, 16 * MPX)
    return dict(path=path, H=H, W=W, conn=conn, density=density, rings=rng.choice([0.0, 0.1]))


# ------------------------------------------------------------------- inputs

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _blur(f):
    """Gaussian of sigma 4 (33 taps, mirrored edges) along both axes."""
    k = [math.exp(-0.5 * (t / 4.0) ** 2) for t in range(-16, 17)]
    s = sum(k)
    for axis in (0, 1):
        n = f.shape[axis]
        i = torch.arange(-16, n + 16, device=f.device)
        i = torch.where(i < 0, -1 - i, i)
        i = torch.where(i >= n, 2 * n - 1 - i, i)
        p = f.index_select(axis, i)
        f = torch.zeros_like(f)
        for t in range(33):
            f.add_(p.narrow(axis, t, n), alpha=k[t] / s)
        del p
    return f


def _field(H, W, density, rings, seed):
    """The tissue-like float image of H x W pixels."""
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(int(seed))
    f = _blur(torch.rand((H, W), generator=g, device=dev) * 80.0)
    n = max(1, int(round(density * H * W / MPX)))

    def ints(lo, hi):
        return torch.randint(lo, hi, (n, 1), generator=g, device=dev)

    cy, cx, r, v, w = ints(0, H), ints(0, W), ints(5, 16), ints(150, 251), ints(2, 5)
    ring = torch.rand((n, 1), generator=g, device=dev) < rings
    o = torch.arange(-15, 16, device=dev)
    dy, dx = o.repeat_interleave(31)[None], o.repeat(31)[None]
    d2 = dy * dy + dx * dx
    y, x = cy + dy, cx + dx
    on = (d2 <= r * r) & (~ring | (d2 > (r - w) ** 2)) & (y >= 0) & (y < H) & (x >= 0) & (x < W)
    at, val = (y * W + x)[on], v.expand(-1, 961)[on].to(torch.float32)
    f.view(-1).scatter_reduce_(0, at, val, "amax")  # where disks overlap, the brightest
    return f


def _mask(f, dtype):
    if dtype == "u8":
        return f.round().clamp_(0, 255).to(torch.uint8)
    return (f * 257.0).round().clamp_(0, 65535).to(torch.int32)


def _lowered(mask):
    off = 30 if mask.dtype == torch.uint8 else 7710
    return mask - torch.clamp(mask, max=off)


def _raised(mask):
    off, top = (30, 255) if mask.dtype == torch.uint8 else (7710, 65535)
    return mask + torch.clamp(top - mask, max=off)


def _binary(mask):
    thr, top = (128, 255) if mask.dtype == torch.uint8 else (128 * 257, 65535)
    return (mask >= thr).to(mask.dtype) * top


def _window(t, pad):
    """`t` as a window of rows `pad` elements longer (the tensor itself at 0)."""
    if pad == 0:
        return t.contiguous()
    big = torch.zeros((t.shape[0], t.shape[1] + pad), dtype=t.dtype, device=t.device)
    big[:, :t.shape[1]] = t
    return big[:, :t.shape[1]]


def _rgb(mask):
    """A colour image of stained tissue: the brighter the mask, the darker and bluer."""
    out = torch.empty((*mask.shape, 3), dtype=torch.uint8, device=mask.device)
    for c, (base, weight) in enumerate(((235, 141), (225, 205), (240, 77))):
        out[..., c] = (base - (mask.to(torch.int32) * weight >> 8)).clamp_(0, 255).to(torch.uint8)
    return out


def _shapes(case):
    r = random.Random(case["shapes"])
    lo, hi = math.log(case["lo"]), math.log(case["hi"])
    out = []
    for _ in range(case["n"]):
        H, W = (int(round(math.exp(r.uniform(lo, hi)))) for _ in range(2))
        out.append((H, W, FILL if r.random() < case["fills"] else RECON, r.random(), r.random()))
    return out


def _tiles(case, seed, align):
    """(data, mask or None, op) of the case's tiles: windows of one field."""
    side = case["hi"]
    mask = _mask(_field(side, side, case["density"], 0.05, seed), case["dtype"])
    marker, binary = _lowered(mask), _binary(mask)
    out = []
    for H, W, op, a, b in _shapes(case):
        y, x = int(a * (side - H + 1)), int(b * (side - W + 1)) // align * align
        win = (slice(y, y + H), slice(x, x + W))
        out.append((binary[win], None, op) if op == FILL else (marker[win], mask[win], op))
    return out


def prepare(case, seed):
    path = case["path"]
    s = {"case": case}
    if path in ("recon", "fill", "erode"):
        mask = _mask(_field(case["H"], case["W"], case["density"], case.get("rings", 0.0), seed),
                     case["dtype"])
        if path == "fill":
            s["src"] = _window(_binary(mask), case["pad"])
        else:
            s["mask"] = _window(mask, case["pad"])
            s["src"] = _window(_lowered(mask) if path == "recon" else _raised(mask), case["pad"])
        s["work"] = _window(torch.zeros_like(mask), case["pad"])
        H, W, p, dt = case["H"], case["W"], s["work"].stride(0), mask.dtype
        n = (mrecon.erode_workspace_bytes(H, W, p, dt, case["conn"]) if path == "erode" else
             mrecon.workspace_bytes(FILL if path == "fill" else RECON, H, W, dt, case["conn"]))
        s["ws"] = mrecon.alloc_workspace(n, mask.device)
    elif path == "batch":
        tiles = _tiles(case, seed, 1)
        s["src"] = [d.contiguous() for d, _, _ in tiles]
        s["work"] = [torch.zeros_like(d) for d in s["src"]]
        s["items"] = [(w, m.contiguous() if m is not None else None, op)
                      for w, (_, m, op) in zip(s["work"], tiles)]
        s["ws"] = mrecon.alloc_workspace(mrecon.batch_workspace_bytes(s["items"], case["conn"]),
                                         s["work"][0].device)
        if case["graph"]:
            s["graph"] = mrecon.BatchGraph(s["items"], case["conn"], tune=mrecon.default_tune(),
                                           workspace=s["ws"])
    elif path == "serve":
        s["jobs"] = _tiles(case, seed, 64)
        s["out"] = [torch.empty(d.shape, dtype=d.dtype, device=d.device) for d, _, _ in s["jobs"]]
        s["server"] = mrecon.Server(1 << 30, max_jobs=64, dtype=s["out"][0].dtype,
                                    conn=case["conn"])
    else:
        H, W = case["H"], case["W"]
        mask = _mask(_field(H, W, case["density"], case.get("rings", 0.0), seed),
                     case.get("dtype", "u8"))
        dev = mask.device
        if path in ("gray_open", "segment"):
            s["rgb"] = _rgb(mask)
            if path == "gray_open":
                s["gray"], s["out"] = torch.empty_like(mask), torch.empty_like(mask)
                s["ws"] = mrecon.alloc_workspace((H * W + 255) // 256 * 256, dev)
        elif path == "dome":
            s["src"] = mask
            s["work"] = torch.empty_like(mask)
        else:
            s["img"] = _binary(mask)
            s["out"] = _window(torch.zeros((H, W), dtype=torch.int32, device=dev), case.get("pad", 0))
    return s


def run(s):
    case = s["case"]
    path = case["path"]
    conn = case.get("conn", 8)
    if path == "recon":
        s["work"].copy_(s["src"])
        return mrecon.recon_dilate(s["work"], s["mask"], conn, workspace=s["ws"])
    if path == "fill":
        s["work"].copy_(s["src"])
        return mrecon.fill_holes(s["work"], conn, workspace=s["ws"])
    if path == "erode":
        s["work"].copy_(s["src"])
        return mrecon.recon_erode(s["work"], s["mask"], conn, workspace=s["ws"])
    if path == "batch":
        torch._foreach_copy_(s["work"], s["src"])
        if case["graph"]:
            s["graph"].launch()
        else:
            mrecon.batch(s["items"], conn, workspace=s["ws"])
        return s["work"]
    if path == "serve":
        srv = s["server"]
        for (data, mask, op), out in zip(s["jobs"], s["out"]):
            while srv.submit(data, mask, op, out=out) is None:
                srv.step()
        srv.drain()
        srv.poll()
        return s["out"]
    if path == "gray_open":
        gray = ops.rgb2gray(s["rgb"], out=s["gray"])
        return gray, ops.open_disk13(gray, out=s["out"], workspace=s["ws"])
    if path == "distance":
        return ops.distance_transform(s["img"], conn, out=s["out"])
    if path == "label":
        labels = ops.ccl(s["img"], conn, out=s["out"])
        labels, ws = ops.area_threshold(labels, case["lo_area"], case["hi_area"])
        return labels, ws[:4 * (case["H"] * case["W"] + 1)].view(torch.int32)
    if path == "dome":
        if case["kind"] == "maxima":
            return ops.regional_maxima(s["src"], conn)
        s["work"].copy_(s["src"])
        return ops.hdome(s["work"], 20 if case["dtype"] == "u8" else 20 * 257, conn)
    # segment: colour -> gray -> opening by reconstruction of the inverted
    # gray -> threshold -> holes filled -> labels of a size range, distances
    gray = ops.rgb2gray(s["rgb"])
    inv = torch.bitwise_not(gray)
    rec = mrecon.recon_dilate(ops.open_disk13(inv), inv, 8)
    objects = (rec >= 100).to(torch.uint8).mul_(255)
    mrecon.fill_holes(objects, conn)
    labels, _ = ops.area_threshold(ops.ccl(objects, 8), 100, 2000)
    return {"gray": gray, "rec": rec, "objects": objects, "labels": labels,
            "dist": ops.distance_transform(objects, 8)}


def work(case):
    """Bytes of each input read once and each output written once; the
    operations are comparisons and selections, counted at one per neighbour."""
    path, conn = case["path"], case.get("conn", 8)
    T = 4 if case.get("dtype") == "i32" else 1
    if path in ("batch", "serve"):
        recon = sum(H * W for H, W, op, _, _ in _shapes(case) if op == RECON)
        fill = sum(H * W for H, W, op, _, _ in _shapes(case) if op == FILL)
        return {"bytes": T * (3 * recon + 2 * fill), "flops": (recon + fill) * conn}
    n = case["H"] * case["W"]
    if path in ("recon", "erode"):
        return {"bytes": 3 * T * n, "flops": n * conn}
    if path == "fill":
        return {"bytes": 2 * T * n, "flops": n * conn}
    if path == "gray_open":
        return {"bytes": 5 * n, "flops": 2 * 13 * n}  # rgb read, gray and opening written
    if path == "distance":
        return {"bytes": 5 * n, "flops": n * conn}
    if path == "label":
        return {"bytes": 9 * n, "flops": n * conn}  # image read, labels and areas written
    if path == "dome":
        return {"bytes": (T + (1 if case["kind"] == "maxima" else T)) * n, "flops": n * conn}
    return {"bytes": (3 + 1 + 1 + 1 + 4 + 4) * n, "flops": 5 * n * 8}


# -------------------------------------------------------------------- exact
# The same results from the definitions, with 64-bit integers in plain torch,
# by iterating each operation's local rule to its fixed point.

EXACT_PIXELS = 2 * MPX
LOW, HIGH = -(1 << 40), 1 << 40


def _neighbours(a, conn, fill):
    p = torch.full((a.shape[0] + 2, a.shape[1] + 2), fill, dtype=a.dtype, device=a.device)
    p[1:-1, 1:-1] = a
    H, W = a.shape
    for dy in (-1, 0, 1):
        for dx in (-1, 0, 1):
            if (dy or dx) and (conn == 8 or dy == 0 or dx == 0):
                yield p[1 + dy:1 + dy + H, 1 + dx:1 + dx + W]


def _fixed_point(a, step):
    while True:
        b = a
        for _ in range(32):
            b = step(b)
        if torch.equal(a, b):
            return a
        a = b


def _recon64(marker, mask, conn):
    marker, mask = marker.to(torch.int64), mask.to(torch.int64)

    def step(j):
        m = j
        for q in _neighbours(j, conn, LOW):
            m = torch.maximum(m, q)
        return torch.minimum(m, mask)
    return _fixed_point(torch.minimum(marker, mask), step)


def _fill64(img, conn):
    low, high = (0, 255) if img.dtype == torch.uint8 else (-(1 << 31), (1 << 31) - 1)
    img = img.to(torch.int64)
    inv = (high + low) - img
    j = torch.full_like(inv, low)
    j[0], j[-1], j[:, 0], j[:, -1] = inv[0], inv[-1], inv[:, 0], inv[:, -1]
    return (high + low) - _recon64(j, inv, conn)


def _label64(img, conn):
    H, W = img.shape
    fg = img != 0
    index = torch.arange(1, H * W + 1, device=img.device).reshape(H, W)

    def step(a):
        m = a
        for q in _neighbours(a, conn, HIGH):
            m = torch.minimum(m, q)
        return torch.where(fg, m, HIGH)
    a = _fixed_point(torch.where(fg, index, HIGH), step)
    return torch.where(fg, a, 0)


def _areas64(labels):
    area = torch.bincount(labels.reshape(-1), minlength=labels.numel() + 1)
    area[0] = 0
    return area


def _keep64(labels, area, lo, hi):
    a = area[labels]
    return torch.where((labels > 0) & (a >= lo) & (a <= hi), labels, 0)


def _distance64(img, conn):
    def step(a):
        m = a
        for q in _neighbours(a, conn, HIGH):
            m = torch.minimum(m, q + 1)
        return m
    d = _fixed_point(torch.where(img != 0, HIGH, 0), step)
    return torch.where(d >= HIGH, -1, d)


def _disk64(a, erode):
    worst = HIGH if erode else LOW
    H, W = a.shape
    p = torch.full((H + 12, W + 12), worst, dtype=torch.int64, device=a.device)
    p[6:-6, 6:-6] = a
    out = torch.full_like(a, worst)
    for dy in range(-6, 7):
        for dx in range(-6, 7):
            if dy * dy + dx * dx <= 36:
                q = p[6 + dy:6 + dy + H, 6 + dx:6 + dx + W]
                out = torch.minimum(out, q) if erode else torch.maximum(out, q)
    return out


def _gray64(rgb):
    r, g, b = (rgb[..., c].to(torch.int64) for c in range(3))
    return (4899 * r + 9617 * g + 1868 * b + 8192) >> 14


def exact(case, seed):
    path, conn = case["path"], case.get("conn", 8)
    if path in ("batch", "serve") or case["H"] * case["W"] > EXACT_PIXELS:
        return None  # the fixed points of large images take too long this way
    f = _field(case["H"], case["W"], case["density"], case.get("rings", 0.0), seed)
    mask = _mask(f, case.get("dtype", "u8"))
    if path == "recon":
        return _recon64(_lowered(mask), mask, conn)
    if path == "erode":
        return -_recon64(-_raised(mask).to(torch.int64), -mask.to(torch.int64), conn)
    if path == "fill":
        return _fill64(_binary(mask), conn)
    if path == "distance":
        return _distance64(_binary(mask), conn)
    if path == "label":
        labels = _label64(_binary(mask), conn)
        area = _areas64(labels)
        return _keep64(labels, area, case["lo_area"], case["hi_area"]), area
    if path == "dome":
        img = mask.to(torch.int64)
        if case["kind"] == "maxima":
            return torch.where(img > _recon64(img - 1, img, conn), 255, 0)
        low, h = (0, 20) if case["dtype"] == "u8" else (-(1 << 31), 20 * 257)
        return img - _recon64(torch.clamp(img - h, min=low), img, conn)
    gray = _gray64(_rgb(mask))
    if path == "gray_open":
        return gray, _disk64(_disk64(gray, True), False)
    inv = 255 - gray
    rec = _recon64(_disk64(_disk64(inv, True), False), inv, 8)
    objects = _fill64(((rec >= 100) * 255).to(torch.uint8), conn)
    labels = _label64(objects, 8)
    return {"gray": gray, "rec": rec, "objects": objects,
            "labels": _keep64(labels, _areas64(labels), 100, 2000),
            "dist": _distance64(objects, 8)}
