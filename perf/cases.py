"""Performance cases: the calls a user of this package makes, at the sizes it is used at.

listed()   the cases themselves; draw(rng) gives further ones of the same ranges.
prepare    what a program holds before the call: inputs on the GPU and the buffers it keeps.
run        one pass through the public entry points; its outputs, whole.
work       bytes one pass cannot do without (the path holds no arithmetic worth counting).
exact      pair values and gradient in 64 bits by a plain sequential algorithm (small
           V-filtration cases; None elsewhere: every output is a copy of an input value, a whole
           number or a sum of a few such differences).

Inputs are of two kinds, as in the tests and the benchmark: smooth random fields (sigma in
pixels), standing for natural images and volumes, and i.i.d. uniform noise, the paper's
synthetic workload and the worst case for pruning.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2606_04801_amd as fc

DTYPES = {"f32": torch.float32, "u8": torch.uint8, "u16": torch.uint16}


def listed():
    return [
        # a serving loop over small patches: no allocation, latency alone counts
        dict(name="patch_64", call="noalloc", h=64, w=64, sigma=2.0, dtype="f32"),
        # the paper's smallest synthetic image, one image into buffers that are kept
        dict(name="noise_316", call="batch", n2=1, h=316, w=316, sigma2=0.0, dtype="f32"),
        # one large float32 image under autograd (topological loss on a single picture)
        dict(name="image_2048_grad", call="autograd", h=2048, w=2048, sigma=8.0, dtype="f32"),
        # one large 8-bit picture, heavy ties, plain call; the diagram padded to a fixed length, as
        # programs that stack diagrams do
        dict(name="image_2048_u8", call="single", h=2048, w=2048, sigma=8.0, dtype="u8"),
        # one volume into buffers that are kept
        dict(name="volume_256", call="batch", n3=1, d3=256, h3=256, w3=256, sigma3=4.0, dtype="f32"),
        # a minibatch of small patches in a training step, forward and backward
        dict(name="patches_train", call="train", n2=64, h=64, w=64, sigma2=2.0),
        # a data set of 512 images of uneven sizes, forward
        dict(name="ragged_512", call="batch", n2=512, lo=64, hi=512, sigma2=4.0, ragged=999, dtype="f32"),
        # the training step of the benchmark: volumes and images in one batch
        dict(name="mixed_train", call="train", n3=64, d3=96, h3=96, w3=96, sigma3=3.0, n2=64, h=512, w=512, sigma2=6.0),
        # pixels as top cells (T-filtration), odd extents, forward and backward with a gradient by hand
        dict(name="mixed_tfilt", call="batch", n3=16, d3=90, h3=97, w3=103, sigma3=3.0, n2=16, h=509, w=510, sigma2=6.0,
             dtype="f32", filtration="T", grad=True),
        # every dimension of volumes (H0, H1, H2), forward
        dict(name="volumes_h1", call="batch", n3=32, d3=96, h3=96, w3=96, sigma3=3.0, dtype="f32", h1=True),
        # the paper's larger noise workloads, with the flag documented for them
        dict(name="noise_1024", call="batch", n2=1, h=1024, w=1024, sigma2=0.0, dtype="f32", wide=True),
        dict(name="noise_volume_128", call="batch", n3=1, d3=128, h3=128, w3=128, sigma3=0.0, dtype="f32", wide=True),
    ]


def draw(rng: random.Random):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["patch", "noise", "image", "volume", "patches", "ragged", "mixed", "tfilt", "h1", "wide2", "wide3"])
    sigma = round(rng.uniform(2.0, 6.0), 1)
    if kind == "patch":
        return dict(call="noalloc", h=log(24, 200), w=log(24, 200), sigma=sigma, dtype=rng.choice(["f32", "u8"]))
    if kind == "noise":
        return dict(call="batch", n2=1, h=log(64, 400), w=log(64, 400), sigma2=0.0, dtype="f32")
    if kind == "image":
        call = rng.choice(["autograd", "single"])
        return dict(call=call, h=log(300, 2048), w=log(300, 2048), sigma=sigma + 2.0,
                    dtype="f32" if call == "autograd" else rng.choice(["f32", "u8", "u16"]))
    if kind == "volume":
        return dict(call="batch", n3=1, d3=log(40, 256), h3=log(40, 256), w3=log(40, 256), sigma3=sigma, dtype="f32")
    if kind == "patches":
        return dict(call="train", n2=log(8, 128), h=log(24, 160), w=log(24, 160), sigma2=sigma)
    if kind == "ragged":
        lo = rng.randint(32, 128)
        return dict(call="batch", n2=log(32, 512), lo=lo, hi=rng.randint(lo + 64, 512), sigma2=sigma,
                    ragged=rng.randint(0, 10 ** 6), dtype=rng.choice(["f32", "u8"]))
    if kind == "mixed":
        return dict(call="train", n3=log(4, 64), d3=log(32, 96), h3=log(32, 96), w3=log(32, 96), sigma3=3.0,
                    n2=log(4, 64), h=log(100, 512), w=log(100, 512), sigma2=sigma)
    if kind == "tfilt":
        return dict(call="batch", n3=log(2, 16), d3=log(32, 104), h3=log(32, 104), w3=log(32, 104), sigma3=3.0,
                    n2=log(2, 16), h=log(100, 512), w=log(100, 512), sigma2=sigma, dtype="f32", filtration="T", grad=True)
    if kind == "h1":
        return dict(call="batch", n3=log(2, 32), d3=log(24, 96), h3=log(24, 96), w3=log(24, 96), sigma3=3.0,
                    dtype=rng.choice(["f32", "u8"]), h1=True)
    if kind == "wide2":
        return dict(call="batch", n2=1, h=rng.randint(1024, 1200), w=rng.randint(1024, 1200), sigma2=0.0, dtype="f32", wide=True)
    return dict(call="batch", n3=1, d3=rng.randint(102, 128), h3=rng.randint(102, 128), w3=rng.randint(102, 128), sigma3=0.0,
                dtype="f32", wide=True)


# ---------------------------------------------------------------------------- inputs --

def shapes_of(case):
    if "n2" not in case and "n3" not in case:
        return [(case["d"], case["h"], case["w"]) if "d" in case else (case["h"], case["w"])]
    shapes = [(case["d3"], case["h3"], case["w3"])] * case["n3"] if case.get("n3") else []
    if "ragged" in case:
        r = random.Random(case["ragged"])
        shapes += [(r.randint(case["lo"], case["hi"]), r.randint(case["lo"], case["hi"])) for _ in range(case["n2"])]
    elif case.get("n2"):
        shapes += [(case["h"], case["w"])] * case["n2"]
    return shapes


def field(n, shape, sigma, gen):
    """n smooth fields (sigma 0: uniform noise) of one shape in [0, 1), float32, on the GPU."""
    x = torch.rand((n,) + tuple(shape), generator=gen, device="cuda")
    if not sigma:
        return x
    r = int(math.ceil(3 * sigma))
    w = [math.exp(-0.5 * (t / sigma) ** 2) for t in range(-r, r + 1)]
    for axis in range(1, x.dim()):
        acc = torch.zeros_like(x)
        for t in range(-r, r + 1):
            acc.add_(torch.roll(x, t, axis), alpha=w[t + r])       # periodic
        x = acc
    dims = tuple(range(1, x.dim()))
    lo, hi = x.amin(dims, keepdim=True), x.amax(dims, keepdim=True)
    return (x - lo) / (hi - lo) * (1.0 - 2.0 ** -24)


def as_type(x, dtype):
    if dtype == "f32":
        return x
    levels = 256 if dtype == "u8" else 65536
    return (x * levels).floor_().clamp_(max=levels - 1).to(torch.int32).to(DTYPES[dtype])


def images_of(case, seed):
    """The instances, in the order of shapes_of."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dtype = case.get("dtype", "f32")
    shapes = shapes_of(case)
    if "n2" not in case and "n3" not in case:
        return [as_type(field(1, shapes[0], case["sigma"], gen)[0], dtype)]
    out = []
    if case.get("n3"):
        out += list(as_type(field(case["n3"], shapes[0], case["sigma3"], gen), dtype))
    if case.get("n2"):
        flat = shapes[case.get("n3", 0):]
        top = (max(h for h, _ in flat), max(w for _, w in flat))
        for x, (h, w) in zip(as_type(field(case["n2"], top, case["sigma2"], gen), dtype), flat):
            out.append(x[:h, :w])
    return out


def pair_room(case, shape):
    """Pair slots a program keeps for one instance: noise has a pair on up to a third of its
    pixels, a smooth field on well under one in fifty."""
    n = math.prod(shape)
    noise = case.get("sigma3" if len(shape) == 3 else "sigma2", case.get("sigma")) == 0.0
    return n // 2 + 64 if noise else n // 24 + 256


def prepare(case, seed):
    imgs = images_of(case, seed)
    s = {"case": case}
    if case["call"] in ("single", "autograd"):
        s["img"] = imgs[0].contiguous()
        if case["call"] == "autograd":
            s["img"].requires_grad_(True)
        return s
    if case["call"] == "noalloc":
        if fc.lib().ph_init_device() != fc.PH_OK:
            raise RuntimeError("ph_init_device")
        s["img"] = imgs[0].contiguous()
        s["bufs"] = fc.PairBuffers(pair_room(case, imgs[0].shape), "cuda")
        clear(s["bufs"])
        s["count"] = torch.zeros(1, dtype=torch.int64, device="cuda")
        s["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        return s
    shapes = shapes_of(case)
    flags = fc.PH_H0 | fc.PH_HTOP | (fc.PH_H1 if case.get("h1") else 0) | (fc.PH_WIDE if case.get("wide") else 0)
    b = fc.Batch(shapes, flags=flags, capacities=[pair_room(case, x) for x in shapes], dtype=DTYPES[case.get("dtype", "f32")],
                 filtration=case.get("filtration", "V"))
    clear(b.pairs)
    for i, x in enumerate(imgs):
        b.image(i).copy_(x)
    s["batch"] = b
    if case["call"] == "train":
        b.images.requires_grad_(True)
        b.valid_mask()
    elif case.get("grad"):
        s["gb"] = torch.full((b.pairs.cap,), -1.0, device="cuda")      # total persistence: dL/dbirth, dL/ddeath
        s["gd"] = torch.ones(b.pairs.cap, device="cuda")
    return s


FIELDS = ("dim", "birth", "death", "birth_cell", "death_cell", "birth_vertex", "death_vertex")


def clear(bufs):
    for f in FIELDS:
        getattr(bufs, f).zero_()


# ------------------------------------------------------------------------------- run --

def whole(bufs, count, status):
    out = {f: getattr(bufs, f) for f in FIELDS}
    out["counts"], out["status"] = count, status
    return out


def run(s):
    case = s["case"]
    call = case["call"]
    if call == "noalloc":
        rc = fc.ph_diagram_noalloc(s["img"], s["bufs"], s["count"], s["status"])
        if rc != fc.PH_OK:
            raise fc.PHError(rc, "ph_diagram_noalloc")
        return whole(s["bufs"], s["count"], s["status"])
    if call == "single":
        d = fc.ph_diagram(s["img"])
        n = d.check()
        pad = (0, pair_room(case, d.shape) - n)
        return {f: torch.nn.functional.pad(getattr(d.bufs, f)[:n], pad) for f in FIELDS}
    if call == "autograd":
        birth, death, _ = fc.PHDiagramFn.apply(s["img"])
        fin = torch.isfinite(death)
        pers = torch.where(fin, death - birth, torch.zeros_like(birth))
        loss = (pers * pers).sum()
        (grad,) = torch.autograd.grad(loss, s["img"])
        return {"loss": loss.detach(), "grad": grad}
    b = s["batch"]
    if call == "train":
        birth, death = fc.BatchDiagramFn.apply(b.images, b)
        fin = b.valid_mask() & (b.pairs.death_cell >= 0)
        pers = torch.where(fin, death - birth, torch.zeros_like(birth))
        (grad,) = torch.autograd.grad((pers * pers).sum(), b.images)
        out = whole(b.pairs, b.counts, b.status)
        out["grad"] = grad
        return out
    if case.get("grad"):
        b.ph_diagram_batch(grad=b.grad)
        b.ph_backward(s["gb"], s["gd"], zeroed=True)
        out = whole(b.pairs, b.counts, b.status)
        out["grad"] = b.grad
        return out
    b.ph_diagram_batch()
    return whole(b.pairs, b.counts, b.status)


def work(case):
    """Pixels read once; the gradient, where there is one, written once; and of the outputs the
    34 bytes of each pair, which only noise has enough of to count (0.31 pairs a pixel of an
    image, 0.17 a voxel: every local minimum and every critical top cell)."""
    size = {"f32": 4, "u8": 1, "u16": 2}[case.get("dtype", "f32")]
    total = 0
    for s in shapes_of(case):
        n = math.prod(s)
        noise = case.get("sigma3" if len(s) == 3 else "sigma2", case.get("sigma")) == 0.0
        total += n * size
        if case["call"] in ("autograd", "train") or case.get("grad"):
            total += 4 * n
        if noise:
            total += int(n * (0.31 if len(s) == 2 else 0.17) * 34)
    return {"bytes": total, "flops": 0}


# ----------------------------------------------------------------------------- exact --

def pairs_of(img):
    """(birth value, death value, birth pixel, death pixel) of the pairs of one image or volume
    under the V-filtration, H0 then the top dimension, in birth order: sequential union-find on
    the pixels, and on the top cells and a cell at infinity with the facets taken backwards."""
    shape, nd, n = img.shape, img.ndim, img.size
    flat = img.reshape(-1)
    rank = np.empty(n, np.int64)
    rank[np.argsort(flat, kind="stable")] = np.arange(n)
    order = np.argsort(flat, kind="stable")
    grid = rank.reshape(shape)
    dbl = tuple(2 * e - 1 for e in shape)

    def cells(axes):
        """Every cell spanning `axes`: rank of its last vertex and its doubled-grid index."""
        r = grid
        for a in axes:
            r = np.maximum(np.take(r, range(shape[a] - 1), a), np.take(r, range(1, shape[a]), a))
        at = np.meshgrid(*[2 * np.arange(e) + (1 if a in axes else 0) for a, e in enumerate(r.shape)], indexing="ij")
        return r, np.ravel_multi_index(at, dbl)

    def find(par, x):
        while par[x] != x:
            par[x] = par[par[x]]
            x = par[x]
        return x

    out = []
    # H0: the edges in order
    rs, cs, us, vs = [], [], [], []
    index = np.arange(n).reshape(shape)
    for a in range(nd):
        r, c = cells([a])
        rs.append(r.ravel()); cs.append(c.ravel())
        us.append(np.take(index, range(shape[a] - 1), a).ravel()); vs.append(np.take(index, range(1, shape[a]), a).ravel())
    rs, cs, us, vs = (np.concatenate(x) for x in (rs, cs, us, vs))
    par, rk, h0 = list(range(n)), rank.tolist(), [(int(rank.min()), -1)]
    go = np.lexsort((cs, rs))
    for r, u, v in zip(rs[go].tolist(), us[go].tolist(), vs[go].tolist()):
        x, y = find(par, u), find(par, v)
        if x != y:
            if rk[x] < rk[y]:
                x, y = y, x
            par[x] = y
            h0.append((rk[x], r))
    h0.sort()
    out += [(b, d) for b, d in h0 if d < 0 or flat[order[b]] != flat[order[d]]]
    # top dimension: the facets backwards; node 0 is the cell at infinity
    r, c = cells(list(range(nd)))
    if r.size:
        trank, tcell = [1 << 62] + r.ravel().tolist(), [1 << 62] + c.ravel().tolist()
        num = np.pad(np.arange(1, r.size + 1).reshape(r.shape), 1)
        rs, cs, us, vs = [], [], [], []
        for a in range(nd):
            fr, fcell = cells([k for k in range(nd) if k != a])
            inner = tuple(slice(None) if k == a else slice(1, -1) for k in range(nd))
            m = num[inner]
            us.append(np.take(m, range(m.shape[a] - 1), a).ravel()); vs.append(np.take(m, range(1, m.shape[a]), a).ravel())
            rs.append(fr.ravel()); cs.append(fcell.ravel())
        rs, cs, us, vs = (np.concatenate(x) for x in (rs, cs, us, vs))
        go = np.lexsort((cs, rs))[::-1]
        par, top = list(range(len(trank))), []
        for fr, fcell, u, v in zip(rs[go].tolist(), cs[go].tolist(), us[go].tolist(), vs[go].tolist()):
            x, y = find(par, u), find(par, v)
            if x != y:
                if (trank[x], tcell[x]) > (trank[y], tcell[y]):
                    x, y = y, x
                par[x] = y
                top.append((fr, fcell, trank[x]))
        top.sort()
        out += [(b, d) for b, _, d in top if flat[order[b]] != flat[order[d]]]
    b = np.array([p for p, _ in out])
    d = np.array([q for _, q in out])
    fin = d >= 0
    bv, dv = order[b], np.where(fin, order[d], -1)
    return flat[bv].astype(np.float64), np.where(fin, flat[dv].astype(np.float64), np.inf), bv, dv


def exact(case, seed):
    shapes = shapes_of(case)
    if sum(math.prod(s) for s in shapes) > 300_000 or case.get("filtration") == "T" or case.get("h1"):
        return None
    births, deaths, grads, loss = [], [], [], 0.0
    for img in images_of(case, seed):
        img = img.cpu().numpy()
        b, d, bv, dv = pairs_of(img)
        fin = dv >= 0
        g = np.zeros(img.size)
        pers = np.where(fin, d, 0.0) - np.where(fin, b, 0.0)
        np.add.at(g, bv, -2 * pers)
        np.add.at(g, dv[fin], 2 * pers[fin])
        loss += float((pers * pers).sum())
        full = np.zeros((2, pair_room(case, img.shape)))
        full[0, :len(b)], full[1, :len(b)] = b, d
        births.append(full[0]); deaths.append(full[1]); grads.append(g)
    if case["call"] == "autograd":
        return {"loss": loss, "grad": grads[0].reshape(shapes[0])}
    out = {"birth": np.concatenate(births), "death": np.concatenate(deaths)}
    if case["call"] == "train":
        out["grad"] = np.concatenate(grads)
    return out
