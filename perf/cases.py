"""Performance cases: the work a user of this framework has it do, through its
public entry points, with a 64-bit reference of every result.

Site sets are the two families the repository's workloads use, made on the GPU:

  pen      polylines one pixel wide on a 2-D grid (about 400 pixels of 64^2);
  surface  unions of shells one voxel thick (spheres, rotated ellipsoids and,
           up to 256^3, planes) on a 3-D grid.

Rows are in lexicographic order of the sites, as numpy.argwhere gives them, or
in random order (`shuffled`), as a point cloud's voxels come.

Kinds of a case, by what a program does per pass:

  layer   new sites arrive: build the rule book, run one VSC or SC layer on it,
          give the book back (inference on a stream of samples; the benchmark's
          step is one of these);
  infer   the book is kept: one layer with batch norm, residual and ReLU fused;
  train   the book is kept: forward, input gradient, weight and bias gradient of
          one VSC, SC or DC layer;
  updown  new sites arrive at a U-Net level: build the SC book with its
          transpose, max-pool the shortcut, SC down, DC up;
  pool    the book is kept: max and average pooling;
  stack   new sites arrive at a whole network: per level two VSC 3^d with batch
          norm and ReLU fused (the second with the block's residual where the
          widths allow), levels joined by SC 2^d stride 2, each level's book
          built on the one above.
"""
import functools
import math

import numpy as np
import torch

import paper_1706_01307_amd as spc

DEV = "cuda"

# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
BASE = dict(kind="layer", op="vsc", d=3, size=64, batch=1, sites=400, f=3, s=1, c_in=32,
            c_out=32, dtype="f32", shuffled=False, widths="")


def _case(**kw):
    return dict(BASE, **kw)


def listed():
    return [
        # the smallest call: one handwritten character, first layer of a network, one at a
        # time (pen64_vsc3_c1x16): latency and launches
        _case(name="pen1_layer_f32", d=2, size=64, batch=1, sites=461, c_in=1, c_out=16),
        # a batch of CAD models at the related-work size (32^3, 423 sites each), a strided
        # 3^3 layer of a ResNet with widths that are no power of two, voxels in no order
        _case(name="cad32_strided_f32", op="sc", f=3, s=2, size=32, batch=64, sites=423, c_in=24,
              c_out=40, shuffled=True),
        # a batch of characters through a small network (pen64x64_vsc3x3_sc2's widths)
        _case(name="pen64_stack_f32", kind="stack", d=2, size=64, batch=64, sites=465,
              widths="1,32|32,32"),
        # the same batch in training: one 3x3 layer forward and backward, fp32
        _case(name="pen64_train_f32", kind="train", d=2, size=64, batch=64, sites=465),
        # fp32 training on surfaces (surf64x16_vsc3_c32)
        _case(name="surf64_train_f32", kind="train", size=64, batch=16, sites=21763),
        # the benchmark's step: book and forward, bf16 (surf128x8_vsc3_c64_bf16)
        _case(name="surf128_layer_bf16", size=128, batch=8, sites=112813, c_in=64, c_out=64,
              dtype="bf16"),
        # the same layer in training
        _case(name="surf128_train_bf16", kind="train", size=128, batch=8, sites=112813, c_in=64,
              c_out=64, dtype="bf16"),
        # the strided layer between the first two levels of the 256^3 encoder, in training
        _case(name="surf256_down_train_bf16", kind="train", op="sc", f=2, s=2, size=256, batch=4,
              sites=425801, c_in=32, c_out=64, dtype="bf16"),
        # the same level of a U-Net at inference on new sites: book with its transpose,
        # pooled shortcut, down and up again
        _case(name="surf256_updown_bf16", kind="updown", f=2, s=2, size=256, batch=4,
              sites=425801, c_in=32, c_out=64, dtype="bf16"),
        # a U-Net decoder's block after the skip connection is concatenated (96 + 96 planes
        # of the encoder's third width), batch norm and ReLU fused
        _case(name="surf64_concat_bf16", kind="infer", size=64, batch=4, sites=21763, c_in=192,
              c_out=96, dtype="bf16"),
        # one large scan, far too sparse for a dense index of its grid, points in no order
        _case(name="scene1024_layer_bf16", size=1024, batch=1, sites=412345, c_in=32, c_out=32,
              dtype="bf16", shuffled=True),
        # the largest: four samples through the four-level encoder (surf256x4_unet_enc_bf16)
        _case(name="surf256_encoder_bf16", kind="stack", size=256, batch=4, sites=425801,
              dtype="bf16", widths="32,32|64,64|96,96|128,128"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng):
    """Plane counts: mostly the networks' multiples of 16, some of 8, a few odd ones."""
    u = rng.random()
    if u < 0.6:
        return 16 * rng.randint(1, 12)
    if u < 0.85:
        return 8 * rng.randint(1, 24)
    return rng.randint(1, 130)


def draw(rng):
    """One more case of the same kinds: any kind on pens or surfaces, from one sample of 16^d to
    the listed ones' sizes, widths 1 to 192 (odd ones among them), both types, either row order.
    The work stays within the encoder's."""
    while True:
        d = rng.choice([2, 3, 3])
        dtype = rng.choice(["f32", "bf16"])
        kind = rng.choice(["layer", "layer", "infer", "train", "train", "updown", "pool", "stack"])
        op = "vsc"
        if d == 2:
            size, batch = _log_int(rng, 24, 128), _log_int(rng, 1, 256)
            sites = int(6.2 * size)
        else:
            size = _log_int(rng, 16, 256) if rng.random() < 0.85 else _log_int(rng, 512, 1024)
            batch = _log_int(rng, 1, max(1, min(64, 2 ** 26 // size ** 3))) if size <= 256 else 1
            sites = int(min(400000, rng.uniform(0.4, 6.0) * size ** 2))
        c_in, c_out = _width(rng), _width(rng)
        if kind == "layer" and rng.random() < 0.15:
            c_in = rng.randint(1, 4)                      # a network's first layer
        f, s = rng.choice([3, 3, 3, 3, 1, 5] if d == 2 else [3, 3, 3, 3, 1]), 1
        widths = ""
        if kind == "train":
            op = rng.choice(["vsc", "vsc", "sc", "dc"])
        elif kind == "layer":
            op = rng.choice(["vsc", "vsc", "sc"])
        if kind in ("updown", "pool") or op in ("sc", "dc"):
            op = "vsc" if kind in ("updown", "pool") else op
            f, s = rng.choice([(2, 2), (2, 2), (3, 2)])
        if kind == "stack":
            w = 16 * rng.randint(1, 4)
            widths = "%d,%d|%d,%d" % (rng.choice([1, 3, w]), w, 2 * w, 2 * w)
            if size > 256:
                continue
            c_in, c_out, f = 32, 32, 3                    # (the layers' own are in widths)
        c = _case(kind=kind, op=op, d=d, size=size, batch=batch, sites=sites, f=f, s=s, c_in=c_in,
                  c_out=c_out, dtype=dtype, shuffled=rng.random() < 0.3, widths=widths)
        n = batch * sites
        if 100 <= n <= 1_000_000 and n * f ** d * c_in * c_out <= 6e10:
            return c


# ---------------------------------------------------------------------------
# Sites
# ---------------------------------------------------------------------------
def _shell(rng, size, planes):
    """Keys (x, y, z flattened) of one shell, as the repository's surfaces draw it."""
    r_lo, r_hi = 0.125 * min(size, 256), 0.47 * min(size, 256)
    kind = int(rng.integers(0, 3 if planes else 2))
    if kind == 2:
        nrm, q = rng.standard_normal(3), rng.uniform(0, size, size=3)
        nrm /= np.linalg.norm(nrm)
        lo, hi, off = [0] * 3, [size] * 3, float(nrm @ q)
    else:
        c = rng.uniform(0, size, size=3)
        a = np.full(3, rng.uniform(r_lo, r_hi)) if kind == 0 else rng.uniform(r_lo, r_hi, size=3)
        rot = np.linalg.qr(rng.standard_normal((3, 3)))[0] if kind else np.eye(3)
        ext = float(a.max()) + 2.0
        lo = [int(max(0, math.floor(v - ext))) for v in c]
        hi = [int(min(size, math.ceil(v + ext) + 1)) for v in c]
    ax = [torch.arange(lo[k], hi[k], device=DEV, dtype=torch.float32) + 0.5 for k in range(3)]
    x, y, z = ax[0][:, None, None], ax[1][None, :, None], ax[2][None, None, :]
    if kind == 2:
        hit = (x * float(nrm[0]) + y * float(nrm[1]) + z * float(nrm[2]) - off).abs() <= 0.5
    else:
        x, y, z = x - float(c[0]), y - float(c[1]), z - float(c[2])
        rad = sum((float(rot[0, k]) / float(a[k]) * x + float(rot[1, k]) / float(a[k]) * y +
                   float(rot[2, k]) / float(a[k]) * z) ** 2 for k in range(3)).sqrt()
        hit = (rad - 1.0).abs() * float(a.min()) <= 0.5
    p = hit.nonzero()
    return ((p[:, 0] + lo[0]) * size + p[:, 1] + lo[1]) * size + p[:, 2] + lo[2]


def _strokes(rng, size, sites):
    """Keys (x, y flattened) of polylines of 3 to 6 segments, until there are `sites`."""
    got = set()
    while len(got) < sites:
        v = rng.integers(0, size, size=(int(rng.integers(4, 8)), 2))
        for p, q in zip(v[:-1], v[1:]):
            n = max(1, int(np.abs(q - p).max()))
            t = np.arange(n + 1)[:, None]
            pts = p + (2 * t * (q - p) + n) // (2 * n)
            got.update((pts[:, 0] * size + pts[:, 1]).tolist())
    return torch.tensor(sorted(got), device=DEV)


def _sites(case, seed):
    """int32 [N, 1 + d] on the GPU."""
    d, size = case["d"], case["size"]
    keys = []
    for b in range(case["batch"]):
        rng = np.random.default_rng([seed, b, 17])
        if d == 2:
            k = _strokes(rng, size, case["sites"])
        else:
            k = torch.zeros(0, dtype=torch.int64, device=DEV)
            for _ in range(256):
                k = torch.cat([k, _shell(rng, size, size <= 256)])
                if k.numel() >= case["sites"]:
                    k = torch.unique(k)
                    if k.numel() >= case["sites"]:
                        break
            k = torch.unique(k)
        # exactly the stated count, so that every seed's tensors have the same shapes: the
        # sample ends at a plane across it
        assert k.numel() >= case["sites"]
        keys.append(k[:case["sites"]] + b * size ** d)
    k = torch.cat(keys)
    cols = []
    for _ in range(d):
        cols.append(k % size)
        k = k // size
    c = torch.stack([k] + cols[::-1], 1).to(torch.int32).contiguous()
    if case["shuffled"]:
        g = torch.Generator(device="cpu").manual_seed(seed + 5)
        c = c[torch.randperm(len(c), generator=g).to(DEV)].contiguous()
    return c


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


class _Rand:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV).manual_seed(int(seed) * 7 + 3)

    def __call__(self, shape, std=1.0, dtype=torch.float32):
        return (torch.randn(shape, generator=self.g, device=DEV) * std).to(dtype)


def _fsz(case):
    d = case["d"]
    return [case["batch"]] + [case["size"]] * d, [1] + [case["f"]] * d, [1] + [case["s"]] * d


def _levels(case):
    return [tuple(int(v) for v in p.split(",")) for p in case["widths"].split("|")]


# ---------------------------------------------------------------------------
# A pass
# ---------------------------------------------------------------------------
def _inputs(case, seed):
    """Every tensor of a pass.  The rows of an SC layer's output are the book's to count: they
    live in buffers of a bound (_rows), as a program that does not wait for the count has it."""
    d, dt, r = case["d"], _dtype(case), _Rand(seed)
    c = _sites(case, seed)
    n, t = len(c), dict(coords=c)
    K, ci, co = case["f"] ** d, case["c_in"], case["c_out"]

    def weights(k, m, o):
        return r((k, m, o), 1.0 / math.sqrt(k * m), dt)

    if case["kind"] == "stack":
        lv = _levels(case)
        t["x"] = r((n, lv[0][0]), 1.0, dt)
        t["layers"] = []
        m = lv[0][0]
        for j, (a, b) in enumerate(lv):
            if j:
                t["layers"].append((weights(2 ** d, m, a), 1.7 + r(a, 0.1), r(a, 0.1)))
                m = a
            for _ in range(2):
                # the scale keeps the planes' size from layer to layer (about half of the
                # neighbours are active, and ReLU halves the square)
                t["layers"].append((weights(3 ** d, m, b), 1.7 + r(b, 0.1), r(b, 0.1)))
                m = b
        return t
    if case["kind"] == "pool":
        t["x"] = r((n, ci), 1.0, dt)
        return t
    n_out = _rows(case)
    rows_in, rows_out = (n_out, n) if case["op"] == "dc" else (n, n_out)
    t["x"] = r((rows_in, ci), 1.0, dt)
    t["w"] = weights(K, ci, co)
    t["b"] = r(co, 0.1)
    if case["kind"] == "infer":
        t["scale"], t["res"] = 1.0 + r(co, 0.1), r((n, co), 1.0, dt)
    if case["kind"] == "train":
        t["dy"] = r((rows_out, co), 1.0, dt)
    if case["kind"] == "updown":
        t["xu"], t["wu"], t["bu"] = r((n_out, co), 1.0, dt), weights(K, co, ci), r(ci, 0.1)
    return t


def _is_sc(case):
    return case["op"] != "vsc" or case["kind"] in ("updown", "pool")


def _rows(case):
    """Rows of the layer's output buffers: the sites' for VSC; for SC a bound on the output sites
    (every input site reaches one where f = s; where they overlap, surfaces and strokes share
    most of theirs, which prepare checks)."""
    n = case["batch"] * case["sites"]
    return n if not _is_sc(case) or case["f"] == case["s"] else 2 * n + 64


def prepare(case, seed):
    t = _inputs(case, seed)
    size, f, s = _fsz(case)
    t["case"], t["size"], t["f"], t["s"] = case, size, f, s
    kind, dt, n, ci, co = case["kind"], _dtype(case), len(t["coords"]), case["c_in"], case["c_out"]

    def buf(rows, c):
        return torch.zeros((rows, c), dtype=dt, device=DEV)

    if _is_sc(case):
        assert len(_sc_sites(case, t["coords"])[0]) <= _rows(case)
    if kind == "stack":
        # per level: the strided layer's output and the two blocks'
        t["y"] = [[buf(n, a), buf(n, b), buf(n, b)] for a, b in _levels(case)]
        return t
    if kind == "layer":
        t["y"] = buf(_rows(case), co)
    elif kind == "updown":
        t["y"] = {"mp": buf(_rows(case), ci), "down": buf(_rows(case), co), "up": buf(n, ci)}
    elif kind == "pool":
        t["y"] = {"mp": buf(_rows(case), ci), "ap": buf(_rows(case), ci)}
    elif kind == "train":
        back = case["op"] == "dc"
        t["y"] = {"y": buf(n if back else _rows(case), co),
                  "dx": buf(_rows(case) if back else n, ci)}
    if kind == "infer" or (kind == "train" and case["op"] == "vsc"):
        t["rb"] = spc.build_rulebook(spc.VSC, t["coords"], size, f)
    elif kind in ("train", "pool"):
        t["rb"] = spc.build_rulebook(spc.SC, t["coords"], size, f, s, transpose=kind == "train")
    return t


def _run_layer(t, c):
    sc = c["op"] == "sc"
    rb = spc.build_rulebook(spc.SC if sc else spc.VSC, t["coords"], t["size"], t["f"], t["s"],
                            sync=False)
    y = (spc.sc_forward if sc else spc.vsc_forward)(rb, t["x"], t["w"], t["b"], out=t["y"])
    rb.close()
    return y


def _run_infer(t, c):
    return spc.forward_fused(t["rb"], t["x"], t["w"], scale=t["scale"], shift=t["b"],
                             residual=t["res"], relu=True)


def _run_train(t, c):
    op = {"vsc": spc.OP_VSC, "sc": spc.OP_SC, "dc": spc.OP_DC}[c["op"]]
    fwd = {"vsc": spc.vsc_forward, "sc": spc.sc_forward, "dc": spc.dc_forward}[c["op"]]
    y = fwd(t["rb"], t["x"], t["w"], t["b"], out=t["y"]["y"])
    dx = spc.backward_data(t["rb"], op, t["dy"], t["w"], out=t["y"]["dx"])
    dw, db = spc.backward_weight(t["rb"], op, t["x"], t["dy"], c["c_in"], c["c_out"])
    return {"y": y, "dx": dx, "dw": dw, "db": db}


def _run_updown(t, c):
    rb = spc.build_rulebook(spc.SC, t["coords"], t["size"], t["f"], t["s"], transpose=True,
                            sync=False)
    y = t["y"]
    spc.pool_forward(rb, t["x"], spc.POOL_MAX, out=y["mp"])
    spc.sc_forward(rb, t["x"], t["w"], t["b"], out=y["down"])
    spc.dc_forward(rb, t["xu"], t["wu"], t["bu"], out=y["up"])
    rb.close()
    return y


def _run_pool(t, c):
    spc.pool_forward(t["rb"], t["x"], spc.POOL_MAX, out=t["y"]["mp"])
    spc.pool_forward(t["rb"], t["x"], spc.POOL_AVG, out=t["y"]["ap"])
    return t["y"]


def _run_stack(t, c):
    d = c["d"]
    f3, f2 = [1] + [3] * d, [1] + [2] * d
    layers, books = iter(t["layers"]), []
    x = t["x"]
    rb = spc.build_rulebook(spc.VSC, t["coords"], t["size"], f3, sync=False)
    books.append(rb)
    down = None
    for j, y in enumerate(t["y"]):
        if j:
            down = (spc.build_rulebook(spc.SC, t["coords"], t["size"], f2, f2, sync=False)
                    if down is None else
                    spc.build_rulebook_on(down, spc.SC, f2, f2, sync=False))
            rb = spc.build_rulebook_on(down, spc.VSC, f3, sync=False)
            books += [down, rb]
            w, a, b = next(layers)
            x = spc.forward_fused(down, x, w, scale=a, shift=b, relu=True, out=y[0])
        w, a, b = next(layers)
        x = spc.forward_fused(rb, x, w, scale=a, shift=b, relu=True, out=y[1])
        w, a, b = next(layers)
        x = spc.forward_fused(rb, x, w, scale=a, shift=b, relu=True, out=y[2],
                              residual=x if w.shape[1] == w.shape[2] else None)
    for rb in books[::-1]:
        rb.close()
    return [y[2] for y in t["y"]]                        # the skip connections of a decoder


RUN = dict(layer=_run_layer, infer=_run_infer, train=_run_train, updown=_run_updown,
           pool=_run_pool, stack=_run_stack)


def run(state):
    return RUN[state["case"]["kind"]](state, state["case"])


# ---------------------------------------------------------------------------
# The same in 64 bits with plain torch
# ---------------------------------------------------------------------------
def _keys(c, size):
    k = c[:, 0].long()
    for j, e in enumerate(size[1:]):
        k = k * e + c[:, j + 1].long()
    return k


def _offsets(f, d):
    return [tuple((i // f ** (d - 1 - j)) % f for j in range(d)) for i in range(f ** d)]


def _lookup(keys, order, want, ok):
    """Rows whose key is `want` (keys sorted, order the rows they came from), -1 for none."""
    at = torch.searchsorted(keys, want).clamp_(max=len(keys) - 1)
    return torch.where(ok & (keys[at] == want), order[at], -1)


def _vsc_pairs(c, size, f):
    """Per offset (input rows, output rows)."""
    d = c.shape[1] - 1
    keys, order = torch.sort(_keys(c, size))
    got = []
    for o in _offsets(f, d):
        n = c.long().clone()
        ok = torch.ones(len(c), dtype=torch.bool, device=c.device)
        for j in range(d):
            n[:, j + 1] += o[j] - (f - 1) // 2
            ok &= (n[:, j + 1] >= 0) & (n[:, j + 1] < size[j + 1])
        a = _lookup(keys, order, _keys(n, size), ok)
        b = (a >= 0).nonzero()[:, 0]
        got.append((a[b], b))
    return got


def _sc_reach(c, size, f, s):
    """Per offset (input rows that reach an output site through it, those sites)."""
    d = c.shape[1] - 1
    out = [size[0]] + [(e - f) // s + 1 if e >= f else 0 for e in size[1:]]
    got = []
    for o in _offsets(f, d):
        n = c.long().clone()
        ok = torch.ones(len(c), dtype=torch.bool, device=c.device)
        for j in range(d):
            v = n[:, j + 1] - o[j]
            q = torch.div(v, s, rounding_mode="floor")
            ok &= (v >= 0) & (q * s == v) & (q < out[j + 1])
            n[:, j + 1] = q
        r = ok.nonzero()[:, 0]
        got.append((r, n[r]))
    return got, out


def _sc_sites(case, c, size=None, f=None, s=None):
    """(output sites, pairs, output extent) of the case's SC layer."""
    size, f, s = size or _fsz(case)[0], f or case["f"], s or case["s"]
    reach, out = _sc_reach(c, size, f, s)
    keys = torch.unique(torch.cat([_keys(n, out) for _, n in reach]))
    pairs = [(r, torch.searchsorted(keys, _keys(n, out))) for r, n in reach]
    k, cols = keys, []
    for e in out[:0:-1]:
        cols.append(k % e)
        k = k // e
    return torch.stack([k] + cols[::-1], 1).to(torch.int32), pairs, out


def _conv(pairs, x, w, rows, back=False):
    y = torch.zeros((rows, w.shape[2]), dtype=torch.float64, device=x.device)
    for (a, b), wi in zip(pairs, w.double()):
        src, dst = (b, a) if back else (a, b)
        for at in range(0, len(src), 1 << 18):
            y.index_add_(0, dst[at:at + (1 << 18)], x[src[at:at + (1 << 18)]].double() @ wi)
    return y


def _weight_grad(pairs, x, dy):
    """x by the pairs' first rows, dy by their second."""
    dw = torch.zeros((len(pairs), x.shape[1], dy.shape[1]), dtype=torch.float64, device=x.device)
    for i, (a, b) in enumerate(pairs):
        for at in range(0, len(a), 1 << 18):
            dw[i] += x[a[at:at + (1 << 18)]].double().T @ dy[b[at:at + (1 << 18)]].double()
    return dw


def _pool(pairs, x, rows, mode, K):
    y = torch.zeros((rows, x.shape[1]), dtype=torch.float64, device=x.device)
    for a, b in pairs:                                    # each output row at most once
        y[b] = torch.maximum(y[b], x[a].double()) if mode == "max" else y[b] + x[a].double()
    return y if mode == "max" else y / K


def _padded(y, rows):
    """y, and zeros up to the rows of the buffer it lives in."""
    return torch.cat([y, y.new_zeros((rows - len(y), y.shape[1]))])


def exact(case, seed):
    t = _inputs(case, seed)
    c, size, K = t["coords"], _fsz(case)[0], case["f"] ** case["d"]
    if case["kind"] == "stack":
        return _exact_stack(case, t)
    if _is_sc(case):
        co, pairs, _ = _sc_sites(case, c)
        n_out = len(co)
    else:
        pairs, n_out = _vsc_pairs(c, size, case["f"]), len(c)
    rows = _rows(case)
    if case["kind"] == "pool":
        return {"mp": _pool(pairs, t["x"], rows, "max", K),
                "ap": _pool(pairs, t["x"], rows, "avg", K)}
    back = case["op"] == "dc"
    y = _conv(pairs, t["x"], t["w"], len(c) if back else n_out, back)
    if case["kind"] == "infer":
        return (y * t["scale"].double() + t["b"].double() + t["res"].double()).clamp_(min=0)
    y = _padded(y + t["b"].double(), len(c) if back else rows)
    if case["kind"] == "layer":
        return y
    if case["kind"] == "updown":
        up = _conv(pairs, t["xu"], t["wu"], len(c), True) + t["bu"].double()
        return {"mp": _pool(pairs, t["x"], rows, "max", K), "down": y, "up": up}
    dx = _conv(pairs, t["dy"], t["w"].transpose(1, 2), rows if back else len(c), not back)
    pw = [(b, a) for a, b in pairs] if back else pairs
    dy = t["dy"] if back else t["dy"][:n_out]
    return {"y": y, "dx": dx, "dw": _weight_grad(pw, t["x"], dy), "db": dy.double().sum(0)}


def _exact_stack(case, t):
    x, c, size, outs = t["x"].double(), t["coords"], _fsz(case)[0], []
    n = len(c)
    layers = iter(t["layers"])

    def block(pairs, x, rows, res):
        w, a, b = next(layers)
        y = _conv(pairs, x, w, rows) * a.double() + b.double()
        return (y + x if res and w.shape[1] == w.shape[2] else y).clamp_(min=0)

    for j in range(len(_levels(case))):
        if j:
            c, pairs, size = _sc_sites(case, c, size, 2, 2)
            x = block(pairs, x, len(c), False)
        pairs = _vsc_pairs(c, size, 3)
        x = block(pairs, x, len(c), False)
        x = block(pairs, x, len(c), True)
        outs.append(_padded(x, n))
    return outs


# ---------------------------------------------------------------------------
# Work and tolerance
# ---------------------------------------------------------------------------
@functools.lru_cache(maxsize=None)
def _counts(key):
    """Rows and pairs of the case's layers, on the sites of one seed (they vary by a few per
    cent with the seed): [(rows in, rows out, pairs)]."""
    case = dict(key)
    c, size = _sites(case, 1), _fsz(case)[0]
    if case["kind"] == "stack":
        got = []
        for j in range(len(_levels(case))):
            if j:
                n = len(c)
                c, p, size = _sc_sites(case, c, size, 2, 2)
                got.append((n, len(c), sum(len(a) for a, _ in p)))
            got.append((len(c), len(c), sum(len(a) for a, _ in _vsc_pairs(c, size, 3))))
        return got
    if _is_sc(case):
        o, p, _ = _sc_sites(case, c)
        return [(len(c), len(o), sum(len(a) for a, _ in p))]
    return [(len(c), len(c), sum(len(a) for a, _ in _vsc_pairs(c, size, case["f"])))]


def work(case):
    """Inputs read once, outputs written once; 2 operations per multiply-add of the active pairs.
    The sites are read where the book is built in the pass; nothing is counted for the book."""
    n = _counts(tuple(sorted((k, v) for k, v in case.items() if k != "name")))
    e, d = (2 if case["dtype"] == "bf16" else 4), case["d"]
    sites = 4 * (d + 1) * n[0][0]
    if case["kind"] == "stack":
        lv, m, by, fl, at = _levels(case), _levels(case)[0][0], 0, 0, 0
        by = sites + n[0][0] * m * e
        for j, (a, b) in enumerate(lv):
            if j:
                by, fl, m, at = by + 2 ** d * m * a * e, fl + 2 * n[at][2] * m * a, a, at + 1
            for _ in range(2):
                by, fl, m = by + 3 ** d * m * b * e, fl + 2 * n[at][2] * m * b, b
            by, at = by + n[at][1] * b * e, at + 1
        return {"bytes": by, "flops": fl}
    (ri, ro, p), ci, co, K = n[0], case["c_in"], case["c_out"], case["f"] ** d
    if case["kind"] == "pool":
        return {"bytes": e * ci * (ri + 2 * ro), "flops": 2 * p * ci}
    if case["op"] == "dc":
        ri, ro = ro, ri
    layer, fl = e * (ri * ci + ro * co + K * ci * co) + 4 * co, 2 * p * ci * co
    if case["kind"] == "layer":
        return {"bytes": sites + layer, "flops": fl}
    if case["kind"] == "infer":
        return {"bytes": layer + e * ro * co + 4 * co, "flops": fl}
    if case["kind"] == "updown":
        return {"bytes": sites + e * ro * ci + 2 * layer, "flops": 2 * fl + p * ci}
    return {"bytes": layer + e * (ro * co + ri * ci) + 4 * (K * ci * co + co), "flops": 3 * fl}


def tolerance(case):
    """Measured against exact(): fp32 results are 1e-7 to 8e-7 off, bf16 ones 1.7e-3 (one rounding
    of the output) and through the bf16 stack's layers 2e-3 to 5e-3; about four times that.
    The largest single difference is a rounding step or two of an element."""
    if case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 1e-4}
    if case["kind"] == "stack":
        return {"rel": 1.6e-2, "max": 0.2}
    return {"rel": 7e-3, "max": 0.03}
