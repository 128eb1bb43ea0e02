"""The workloads whose speed this repository is measured by, one dict of plain values per case.

``listed()`` gives the standing cases, ``draw(rng)`` one more of the same ranges, ``prepare`` builds
a case's inputs on the GPU from a seed, ``run`` makes one pass through the public entry points and
returns everything it computed, ``work`` states what a pass cannot do without, and ``exact`` gives
the results in plain numpy where that is quick enough.

Every kind stands for one way the framework is used:

* ``carve``     one image to a smaller width (vertical seams), the basic call
* ``hv``        one image to a smaller width and height (``carve_hv``)
* ``batch``     many images of uneven sizes in one planned launch (``BatchCarver``)
* ``forward``   one image with forward-energy seams
* ``fbatch``    many images with forward-energy seams (``ForwardBatch``)
* ``insert``    one image widened by seams
* ``object``    an object under a mask removed and the size restored
* ``steps``     seam by seam through the single-step calls (energy, minimum seam, removal), as an
                interactive program or one with an energy map of its own does
* ``serve``     a burst of requests through the continuous-batching server with teams
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2410_21207_amd import _lib, api, serve


def listed():
    return [
        # the smallest call: a 64x48 image, 16 seams (latency and launches)
        {"name": "carve_64x48", "kind": "carve", "h": 48, "w": 64, "c": 3, "k": 16, "pixels": "uniform"},
        # an ordinary gray photograph or scan of odd size
        {"name": "carve_gray_701x1003", "kind": "carve", "h": 701, "w": 1003, "c": 1, "k": 301, "pixels": "blob"},
        # the single-image workload: 1920x1080 RGB, a quarter of the width
        {"name": "carve_1080p", "kind": "carve", "h": 1080, "w": 1920, "c": 3, "k": 480, "pixels": "blob"},
        # 3840x2160 RGB in both directions: 960 vertical and 540 horizontal seams
        {"name": "carve_4k_hv", "kind": "hv", "h": 2160, "w": 3840, "c": 3, "k": 960, "kh": 540, "pixels": "blob"},
        # the batched workload: 256 images, sides 240..2160, 10-40 % of the width
        {"name": "batch_256", "kind": "batch", "n": 256, "lo": 240, "hi": 2160, "shapes": 3, "c": 3},
        # thumbnails: many small images, where per-seam latency counts and the chip is full
        {"name": "batch_thumbs_512", "kind": "batch", "n": 512, "lo": 64, "hi": 256, "shapes": 5, "c": 3},
        # 1920x1080 with forward energy
        {"name": "forward_1080p", "kind": "forward", "h": 1080, "w": 1920, "c": 3, "k": 480, "pixels": "blob"},
        # a forward-energy batch
        {"name": "forward_batch_64", "kind": "fbatch", "n": 64, "lo": 240, "hi": 2160, "shapes": 3, "c": 3},
        # 1920x1080 widened by a quarter
        {"name": "insert_1080p", "kind": "insert", "h": 1080, "w": 1920, "c": 3, "k": 480, "pixels": "blob"},
        # a 201x401 ellipse taken out of 1920x1080, the size restored
        {"name": "object_1080p", "kind": "object", "h": 1080, "w": 1920, "c": 3, "mh": 401, "mw": 201,
         "restore": True, "pixels": "blob"},
        # eight seams of a 1920x1080 image, step by step
        {"name": "steps_1080p", "kind": "steps", "h": 1080, "w": 1920, "c": 3, "k": 8, "pixels": "blob"},
        # a burst of served requests, sides 128..2048
        {"name": "serve_burst_40", "kind": "serve", "n": 40, "lo": 128, "hi": 2048, "shapes": 4, "c": 3},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["carve", "carve", "carve", "hv", "batch", "forward", "fbatch", "insert", "object", "steps",
                       "serve"])
    c = rng.choice([3, 3, 3, 1, 4, 2])
    if kind in ("batch", "fbatch", "serve"):
        hi = _log(rng, 160, 1200)
        n = {"batch": _log(rng, 24, 384), "fbatch": _log(rng, 8, 64), "serve": rng.randint(8, 48)}[kind]
        return {"kind": kind, "n": n, "lo": max(48, hi // rng.randint(2, 6)), "hi": hi,
                "shapes": rng.randrange(1 << 20), "c": c}
    top = {"carve": 2160, "hv": 1600, "insert": 1800, "forward": 1500, "object": 1200, "steps": 3000}[kind]
    h, w = _log(rng, 48, top), _log(rng, 64, top)
    case = {"kind": kind, "h": h, "w": w, "c": c, "pixels": rng.choice(["blob", "blob", "blob", "uniform"])}
    if kind == "steps":
        case["k"] = rng.randint(1, 8)
    elif kind == "object":
        case.update(mh=max(2, int(h * rng.uniform(0.05, 0.3))), mw=max(2, int(w * rng.uniform(0.05, 0.25))),
                    restore=rng.random() < 0.7)
    else:
        case["k"] = max(1, int(w * rng.uniform(0.05, 0.45)))
        if kind == "hv":
            case["kh"] = max(1, int(h * rng.uniform(0.05, 0.4)))
    return case


# ------------------------------------------------------------------------------------------ inputs
def _shapes(case):
    """(h, w, target width) of every image of a batch or burst: from the case alone."""
    rng = np.random.default_rng(case["shapes"])
    n, lo, hi = case["n"], case["lo"], case["hi"]
    if case["kind"] == "serve":  # log-uniform sides, 50-90 % of the width kept
        side = np.exp(rng.uniform(math.log(lo), math.log(hi), (n, 2))).round().astype(int)
        keep = rng.uniform(0.5, 0.9, n)
    else:                        # uniform sides, 60-90 % of the width kept
        side = rng.integers(lo, hi + 1, (n, 2))
        keep = 1.0 - rng.uniform(0.1, 0.4, n)
    return [(int(h), int(w), max(1, int(w * f))) for (h, w), f in zip(side, keep)]


def _pixels(h, w, c, gen, kind="blob"):
    """uint8 [h, w, c]: uniform bytes, or 32 smooth blobs plus small noise (soft edges in large
    low-energy regions, like a photograph)."""
    dev = gen.device
    if kind == "uniform":
        return torch.randint(0, 256, (h, w, c), generator=gen, device=dev, dtype=torch.uint8)
    u = torch.rand((32, 3 + c), generator=gen, device=dev)
    sg = 20.0 + 180.0 * u[:, 2:3]
    gx = torch.exp(-((torch.arange(w, device=dev) - u[:, 0:1] * w) ** 2) / (2.0 * sg * sg))
    gy = torch.exp(-((torch.arange(h, device=dev) - u[:, 1:2] * h) ** 2) / (2.0 * sg * sg))
    out = torch.empty((h, w, c), dtype=torch.uint8, device=dev)
    noise = torch.randint(-8, 9, (c, h, w), generator=gen, device=dev, dtype=torch.int8)
    for ch in range(c):
        v = 128.0 + gy.t().contiguous() @ ((192.0 * u[:, 3 + ch:4 + ch] - 96.0) * gx)
        out[:, :, ch] = (v + noise[ch]).round_().clamp_(0, 255).to(torch.uint8)
    return out


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind, c = case["kind"], case["c"]
    lib = _lib.load()
    if kind in ("batch", "fbatch"):
        shapes = _shapes(case)
        srcs = [_pixels(h, w, c, gen) for h, w, _ in shapes]
        # the results lie one behind the other in one buffer
        flat = torch.zeros(sum(h * w * c for h, w, _ in shapes), dtype=torch.uint8, device="cuda")
        imgs, at = [], 0
        for h, w, _ in shapes:
            imgs.append(flat[at:at + h * w * c].view(h, w, c))
            at += h * w * c
        make = api.BatchCarver if kind == "batch" else api.ForwardBatch
        return {"kind": kind, "flat": flat,
                "batch": make(imgs, [t for _, _, t in shapes], srcs=srcs, record=False)}
    if kind == "serve":
        shapes = _shapes(case)
        return {"kind": kind, "ex": serve.GPUExecutor(64), "c": c,
                "requests": [(h, w, t, _pixels(h, w, c, gen)) for h, w, t in shapes]}
    h, w = case["h"], case["w"]
    src = _pixels(h, w, c, gen, case["pixels"])
    st = {"kind": kind, "src": src, "k": case.get("k", 0), "w": w, "h": h}
    if kind == "carve":
        st.update(img=torch.zeros_like(src), ws=api.workspace(lib.sc_workspace_bytes(h, w, c), src.device))
    elif kind == "forward":
        st.update(img=torch.zeros_like(src), ws=api.workspace(lib.sc_forward_workspace_bytes(h, w, c), src.device))
    elif kind == "hv":
        st.update(kh=case["kh"], img=torch.zeros_like(src))
    elif kind == "insert":
        st.update(ws=api.workspace(lib.sc_insert_workspace_bytes(h, w, c, w * c, case["k"]), src.device))
    elif kind == "object":
        y = (torch.arange(h, device="cuda") - h // 2).double() / (case["mh"] / 2.0)
        x = (torch.arange(w, device="cuda") - w // 2).double() / (case["mw"] / 2.0)
        st.update(mask=((y * y)[:, None] + (x * x)[None, :] <= 1.0).to(torch.uint8), restore=case["restore"],
                  ws=api.workspace(lib.sc_object_workspace_bytes(h, w, c, int(case["restore"])), src.device))
    elif kind == "steps":
        st.update(img=torch.zeros_like(src), ws=api.workspace(lib.sc_workspace_bytes(h, w, 1), src.device))
    return st


# -------------------------------------------------------------------------------------------- runs
def run(st):
    kind = st["kind"]
    if kind == "carve":
        return api.carve(st["img"], st["w"] - st["k"], src=st["src"], ws=st["ws"])
    if kind == "hv":
        st["img"].copy_(st["src"])
        return api.carve_hv(st["img"], st["w"] - st["k"], st["h"] - st["kh"])
    if kind in ("batch", "fbatch"):
        st["batch"].launch()
        return st["flat"]
    if kind == "forward":
        return api.carve_forward(st["img"], st["w"] - st["k"], src=st["src"], ws=st["ws"])
    if kind == "insert":
        return api.insert_seams(st["src"], st["k"], ws=st["ws"])
    if kind == "object":
        out, info, seams, costs = api.remove_object(st["src"], st["mask"], restore=st["restore"], ws=st["ws"])
        return out, info["k"], info["left"], seams, costs
    if kind == "steps":
        img = st["img"].copy_(st["src"])
        found = []
        for _ in range(st["k"]):
            seam, cost = api.dp_seam(api.energy(img), ws=st["ws"])
            img = api.remove_seam(img, seam)
            found.append((seam, cost))
        return img, found
    srv = serve.Server(st["ex"], max_slots=64, seams_per_step=1 << 20, step_budget_us=20000,
                       team_policy=serve.team_by_work())
    for h, w, t, px in st["requests"]:
        srv.submit(h, w, st["c"], t, px)
    while not srv.idle():
        srv.step()
    return [t.result[0] for t in srv.tickets]


# -------------------------------------------------------------------------------------------- work
def work(case):
    """Input pixels read once, results written once, and the arithmetic of the recurrence: two
    comparisons and one addition per pixel of every image a seam is taken from (six more operations
    per channel for the forward costs), and the energy of every source pixel."""
    kind, c = case["kind"], case["c"]

    def carve(h, w, k, record=True):
        out = h * (w - k) * c + (k * h * 4 + k * 8 if record else 0)
        return h * w * c + out, 3 * h * (k * w - k * (k - 1) // 2) + 6 * c * h * w

    if kind in ("batch", "fbatch", "serve"):
        each = [carve(h, w, w - t, kind == "serve") for h, w, t in _shapes(case)]
        b, f = sum(x for x, _ in each), sum(y for _, y in each)
        return {"bytes": b, "flops": f * (1 + 2 * c) if kind == "fbatch" else f}
    h, w = case["h"], case["w"]
    if kind == "object":
        # the seams run along the mask's longer side
        vert = case["mw"] <= case["mh"]
        fh, fw, k = (h, w, case["mw"]) if vert else (w, h, case["mh"])
        b, f = carve(fh, fw, k)
        return {"bytes": b + h * w, "flops": f * (2 if case["restore"] else 1)}
    if kind == "steps":
        k = case["k"]
        b = sum(h * (w - i) * c + h * (w - i - 1) * c + h * 4 + 8 for i in range(k))
        return {"bytes": b, "flops": (3 + 6 * c) * h * (k * w - k * (k - 1) // 2)}
    b, f = carve(h, w, case["k"])
    if kind == "hv":
        b2, f2 = carve(w - case["k"], h, case["kh"])
        return {"bytes": b + b2, "flops": f + f2}
    if kind == "insert":
        b += 2 * h * case["k"] * c
    return {"bytes": b, "flops": f * (1 + 2 * c) if kind == "forward" else f}


# ------------------------------------------------------------------------------------------- exact
def _np_seam(img):
    """(seam, cost) of the minimum e1 seam, ties to the left, in 64-bit integers."""
    p = img.astype(np.int64)
    x = np.pad(p, ((0, 0), (1, 1), (0, 0)), mode="edge")
    y = np.pad(p, ((1, 1), (0, 0), (0, 0)), mode="edge")
    e = (np.abs(x[:, 2:] - x[:, :-2]) + np.abs(y[2:] - y[:-2])).sum(2)
    h, w = e.shape
    back = np.ones((h, w), np.int8)
    m, far = e[0], np.int64(1) << 60
    for i in range(1, h):
        c = np.stack([np.concatenate(([far], m[:-1])), m, np.concatenate((m[1:], [far]))])
        back[i] = c.argmin(0)
        m = c.min(0) + e[i]
    s = np.empty(h, np.int64)
    s[-1] = int(m.argmin())
    for i in range(h - 1, 0, -1):
        s[i - 1] = s[i] + back[i, s[i]] - 1
    return s, int(m.min())


def exact(case, seed):
    if case["kind"] not in ("carve", "steps"):
        return None
    h, w, k = case["h"], case["w"], case["k"]
    if k * h * (40e-6 + 60e-9 * w) > 8.0:  # seconds, about
        return None
    img = prepare(case, seed)["src"].cpu().numpy()
    seams, costs = [], []
    for _ in range(k):
        s, m = _np_seam(img)
        keep = np.ones(img.shape[:2], bool)
        keep[np.arange(h), s] = False
        img = img[keep].reshape(h, img.shape[1] - 1, -1)
        seams.append(s)
        costs.append(m)
    if case["kind"] == "steps":
        return img.copy(), [(s, np.array([m])) for s, m in zip(seams, costs)]
    return img.copy(), np.stack(seams), np.array(costs)
