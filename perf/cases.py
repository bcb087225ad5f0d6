"""The work that a user of this package has it do, as cases that can be timed and compared.

A user's program holds a network (``SparseDeepCNet``: plan and workspace), weights and a batch of sparse
inputs on the GPU, and per batch calls ``rulebook_build`` -> ``forward`` (classification) or
``rulebook_build`` -> ``forward`` -> ``backward`` (training), with ``StrokeEncoder.encode`` before and
``sgd_step`` behind where it trains from raw pen paths.  Those calls are the package's units: one forward or
backward call runs every layer, and a new batch has a new set of active sites, so no shorter sequence is
anything that a program does.  The shallow networks among the drawn cases (ell = 2, 3) stand closest to a
single layer.

``listed`` holds the networks of the repository's own workloads; ``draw`` spreads the same kinds of
work over depth, width, input features, classes, batch size, storage type and options.
"""

import math

import numpy as np
import torch

from paper_1409_6070_amd.sscn import SparseDeepCNet, StrokeEncoder

# ---------------------------------------------------------------------------------------------------------
# the cases


def _case(name, mode, arch, ell, k, c_in, classes, batch, dtype, inputs, dropout=False, dfeats=False):
    return {"name": name, "mode": mode, "arch": arch, "ell": ell, "k": k, "c_in": c_in, "classes": classes,
            "batch": batch, "dtype": dtype, "inputs": inputs, "dropout": dropout, "dfeats": dfeats}


def listed():
    return [
        # one character written on a tablet, classified as soon as it is drawn: a call of latencies
        _case("classify_one_digit", "infer", "deepcnet", 5, 10, 1, 10, 1, "bf16", "digits"),
        # the network and input that the paper times: digit pictures classified in large batches
        _case("classify_digits_b1000", "infer", "deepcnet", 5, 10, 1, 10, 1000, "f32", "digits"),
        # a small network on a small batch, as in a first experiment or a test set of a few classes
        _case("train_4_20_b8_f32", "train", "deepcnet", 4, 20, 1, 10, 8, "f32", "pen"),
        # the package's headline: handwriting with 3755 classes, the ordinary training batch
        _case("train_5_50_b100", "train", "deepcnet", 5, 50, 1, 3755, 100, "bf16", "pen"),
        # the same in float32
        _case("train_5_50_b100_f32", "train", "deepcnet", 5, 50, 1, 3755, 100, "f32", "pen"),
        # eight features per pen pixel: a first layer on the matrix cores
        _case("train_5_50_m8_b100", "train", "deepcnet", 5, 50, 8, 3755, 100, "bf16", "pen_normal"),
        # small colour pictures padded into the grid: dense inside, sites listed in any order
        _case("train_5_100_rgb_b128", "train", "deepcnet", 5, 100, 3, 10, 128, "bf16", "patch"),
        # the deep and wide network on fine pen strokes, the largest grid: a handwriting recogniser at work
        _case("classify_6_100_b64", "infer", "deepcnet", 6, 100, 1, 3755, 64, "bf16", "pen_fine"),
        # network-in-network layers and the leaky rectifier
        _case("train_nin_5_50_b100", "train", "deepcnin", 5, 50, 1, 3755, 100, "bf16", "pen"),
        # dropout in the upper levels
        _case("train_5_50_dropout", "train", "deepcnet", 5, 50, 1, 3755, 100, "bf16", "pen", dropout=True),
        # a whole training step from raw pen paths: encoding on the device, gradients, update
        _case("step_4_20_paths_b100", "step", "deepcnet", 4, 20, 9, 10, 100, "bf16", "paths"),
        # the headline network where the batch fills the chip
        _case("train_5_50_b1600", "train", "deepcnet", 5, 50, 1, 3755, 1600, "bf16", "pen"),
    ]


def draw(rng):
    """Another case of the same ranges: depth 2-6, width 5-110, batch 1-1600 (over its logarithm)."""
    while True:
        mode = rng.choice(["infer", "train", "train", "train", "step"])
        inputs = "paths" if mode == "step" else rng.choice(["pen", "pen", "pen_normal", "pen_fine", "patch", "digits"])
        ell = rng.choice([2, 3, 4, 5, 5, 6])
        if inputs in ("patch", "digits") and ell < 4:
            continue  # these pictures are up to 40 squares wide and do not fit
        dtype = rng.choice(["bf16", "bf16", "f32"])
        batch = int(math.exp(rng.uniform(0.0, math.log(1601))))
        if dtype == "bf16" and mode != "infer":  # see tolerance(): other 16-bit gradients cannot be compared
            ell = min(ell, 5)
            batch = max(batch, 4 ** (ell - 2))
        case = _case("", mode, rng.choice(["deepcnet", "deepcnet", "deepcnet", "deepcnin"]), ell,
                     int(math.exp(rng.uniform(math.log(5), math.log(111)))),
                     9 if inputs == "paths" else 3 if inputs == "patch" else rng.choice([2, 4, 8, 9]) if inputs == "pen_normal" else 1,
                     rng.choice([10, 26, rng.randrange(2, 200), rng.randrange(1000, 4000), 3755]),
                     batch, dtype, inputs,
                     dropout=mode == "train" and rng.random() < 0.15, dfeats=mode == "train" and inputs == "patch" and dtype == "f32")
        del case["name"]
        # a drawn case costs no more than the largest listed one: float32 products cost about 16 times as much
        grid = 9.0 * 4 ** ell
        cost = case["batch"] * grid * case["k"] ** 2 * ell ** 2 * (1.0 if mode == "infer" else 3.0)
        if cost * (8.0 if case["dtype"] == "f32" else 1.0) <= 1600 * 9216 * 2500.0 * 25 * 3 / 1.2 and case["batch"] * grid < 1.6e7:
            return case


# ---------------------------------------------------------------------------------------------------------
# inputs

_PEN = {"pen": ((1, 20), (10, 60), 2 / 3, 2.0), "pen_normal": ((1, 20), (10, 60), 2 / 3, 2.0),
        "pen_fine": ((1, 30), (10, 120), 2 / 3, 1.0), "paths": ((1, 3), (10, 30), 2 / 3, 2.0),
        "digits": ((2, 4), (10, 18), 20, 2.5)}


def _grid(case):
    return 3 * 2 ** case["ell"]


def _walks(rng, kind, batch, N):
    """Pen strokes as point sequences: random walks of rounded normal steps, kept inside a centred box."""
    strokes, points, box, sigma = _PEN[kind]
    box = box if isinstance(box, int) else int(N * box)
    lo = (N - box) // 2
    sample = np.repeat(np.arange(batch), rng.integers(strokes[0], strokes[1] + 1, size=batch))
    length = rng.integers(points[0], points[1] + 1, size=sample.size)
    at = rng.integers(lo, lo + box, size=(sample.size, 2))
    step = np.rint(rng.normal(0.0, sigma, size=(points[1], sample.size, 2))).astype(np.int64)
    path = np.empty((points[1], sample.size, 2), np.int64)
    for i in range(points[1]):
        path[i] = at
        at = np.clip(at + step[i], lo, lo + box - 1)
    path = path.transpose(1, 0, 2)
    pts = path[np.arange(points[1])[None, :] < length[:, None]]
    return pts, np.concatenate([[0], np.cumsum(length)]), sample


def _raster(pts, begin, sample):
    """The pixels of the lines that join consecutive points: (sample, pixel, last pixel before it or itself)."""
    start = np.zeros(len(pts), bool)
    start[begin[:-1]] = True
    prev = np.where(start[:, None], pts, np.concatenate([pts[:1], pts[:-1]]))
    d = pts - prev
    L = np.abs(d).max(axis=1)
    n = np.maximum(L, 1)
    seg = np.repeat(np.arange(len(pts)), n)
    i = np.arange(seg.size) - np.repeat(np.cumsum(n) - n, n) + 1

    def pixel(i):
        den = n[seg][:, None]
        return prev[seg] + (2 * i[:, None] * d[seg] + den) // (2 * den)

    point = np.repeat(sample, np.diff(begin))
    return point[seg], pixel(i), pixel(i - 1)


def _sites(case, rng):
    """coords [n, 3] (b, y, x), each site once, and the per-sample offsets (None where they are in any order)."""
    N, B, kind = _grid(case), case["batch"], case["inputs"]
    if kind == "patch":
        lo = (N - 40) // 2
        at = lo + rng.integers(0, 9, size=(B, 2))
        yx = np.stack(np.meshgrid(np.arange(32), np.arange(32), indexing="ij"), -1).reshape(1, -1, 2) + at[:, None]
        c = np.concatenate([np.repeat(np.arange(B), 1024)[:, None], yx.reshape(-1, 2)], axis=1)
        return rng.permutation(c), None
    b, p, _ = _raster(*_walks(rng, kind, B, N))
    if kind == "digits":  # a brush two squares wide
        brush = np.array([(0, 0), (0, 1), (1, 0), (1, 1)])
        b, p = np.repeat(b, 4), (p[:, None] + brush).reshape(-1, 2)
    key = (b * N + p[:, 0]) * N + p[:, 1]
    first = np.sort(np.unique(key, return_index=True)[1])  # in the order of drawing, sample by sample
    c = np.stack([b[first], p[first, 0], p[first, 1]], axis=1)
    return c, np.searchsorted(c[:, 0], np.arange(B + 1))


def _inputs(case, seed):
    rng = np.random.default_rng(seed)
    got = {}
    if case["inputs"] == "paths":
        pts, begin, sample = _walks(rng, "paths", case["batch"], _grid(case))
        got.update(points=pts, begin=begin, sample=sample, most=_raster(pts, begin, sample)[0].size)
    else:
        got["coords"], got["offsets"] = _sites(case, rng)
        n, c = got["most"], _ = len(got["coords"]), case["c_in"]
        got["feats"] = (rng.normal(size=(n, c)) if case["inputs"] == "pen_normal" else 1 - rng.random((n, c))
                        if case["inputs"] in ("patch", "digits") else np.ones((n, c)))
    got["labels"] = rng.integers(0, case["classes"], size=case["batch"])
    got["W"], got["b"] = [], []
    shapes = _shapes(case)
    for i, (rows, cols) in enumerate(shapes):
        var = 2.0 / rows if i + 1 < len(shapes) else 2.0 / (rows + cols)
        got["W"].append(rng.standard_normal((rows, cols), dtype=np.float32) * np.float32(math.sqrt(var)))
        got["b"].append(rng.uniform(-0.1, 0.1, size=cols).astype(np.float32))
    return got


def _convs(case):
    """(window side, input channels, output channels) of the convolutions, None for a pooling layer."""
    k, nin, out = case["k"], case["arch"] == "deepcnin", [(3, case["c_in"], case["k"])]
    for n in range(1, case["ell"] + 1):
        out += [None] + ([(1, n * k, n * k)] if nin else []) + [(2, n * k, (n + 1) * k)]
    top = (case["ell"] + 1) * k
    return out + ([(1, top, top)] if nin else [])


def _shapes(case):
    return [(F * F * ci, co) for F, ci, co in filter(None, _convs(case))] + [((case["ell"] + 1) * case["k"], case["classes"])]


def _rates(case):
    """No dropout on the lower half of the levels, one half on the upper ones and the softmax layer's input."""
    return [0.0] * ((case["ell"] + 1) // 2) + [0.5] * (case["ell"] + 2 - (case["ell"] + 1) // 2)


_DROPOUT_SEED, _LR, _MOMENTUM, _DECAY = 1234567890123, 0.01, 0.9, 1e-4


# ---------------------------------------------------------------------------------------------------------
# the calls


def prepare(case, seed):
    x = _inputs(case, seed)
    storage = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def dev(a, dtype):
        return torch.as_tensor(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype)

    s = {"case": case, "labels": dev(x["labels"], torch.int32), "W": [dev(w, storage) for w in x["W"]],
         "b": [dev(b, torch.float32) for b in x["b"]]}
    # a program sizes its buffers for the batches to come: a quarter above this one
    most = int(x["most"] * 1.25) + 16
    s["net"] = SparseDeepCNet(case["ell"], case["k"], case["c_in"], case["classes"], case["batch"], most,
                              case["dtype"], arch=case["arch"], dropout=case["dropout"])
    if case["dropout"]:
        s["net"].set_dropout(_rates(case), _DROPOUT_SEED)
    if case["mode"] == "step":
        s["paths"] = [dev(x[n], torch.int32) for n in ("points", "begin", "sample")]
        s["encoder"] = StrokeEncoder(_grid(case), case["batch"], most, case["dtype"])
        s["W32"] = [dev(w, torch.float32) for w in x["W"]] if case["dtype"] == "bf16" else s["W"]
        s["vW"], s["vb"] = [torch.zeros_like(w) for w in s["W32"]], [torch.zeros_like(b) for b in s["b"]]
    else:
        s["coords"], s["feats"] = dev(x["coords"], torch.int32), dev(x["feats"], storage)
        s["offsets"] = dev(x["offsets"], torch.int32) if x["offsets"] is not None else None
    return s


def run(s):
    case, net = s["case"], s["net"]
    if case["mode"] == "step":
        coords, feats = s["encoder"].encode(*s["paths"], case["batch"])
        net.rulebook_build(coords, case["batch"])
        logits, loss = net.forward(feats, s["W"], s["b"], s["labels"])
        net.backward()
        net.sgd_step(s["W32"], s["W"], s["b"], s["vW"], s["vb"], _LR, _MOMENTUM, _DECAY)
        return {"logits": logits, "loss": loss, "W": s["W32"], "b": s["b"],
                "vW": s["vW"], "vb": s["vb"]}  # the velocities hold the gradients
    net.rulebook_build(s["coords"], case["batch"], s["offsets"])
    if case["mode"] == "infer":
        return {"logits": net.forward(s["feats"], s["W"], s["b"], None)[0]}
    logits, loss = net.forward(s["feats"], s["W"], s["b"], s["labels"])
    dW, db, dfeats = net.backward(want_dfeats=case["dfeats"])
    out = {"logits": logits, "loss": loss, "dW": dW, "db": db}
    if case["dfeats"]:
        out["dfeats"] = dfeats
    return out


# ---------------------------------------------------------------------------------------------------------
# what the path cannot do without


def _active(case, a):
    """The active sites of every layer above the boolean input grid a [B, N, N], as a list of grids."""
    out = []
    for conv in _convs(case):
        if conv is None:
            a = a[:, 0::2, 0::2] | a[:, 0::2, 1::2] | a[:, 1::2, 0::2] | a[:, 1::2, 1::2]
        else:
            S = a.shape[1] - conv[0] + 1
            got = a[:, :S, :S]
            for f in range(1, conv[0] ** 2):
                got = got | a[:, f // conv[0]: f // conv[0] + S, f % conv[0]: f % conv[0] + S]
            a = got
        out.append(a)
    return out


def work(case):
    """Products: 2 x window x channels x sites of each convolution, for the output and, in training, for both
    gradients (none for the input's unless it is asked for).  Bytes: the call's inputs and parameters read
    once and its outputs written once; what the layers hold in between is not counted."""
    part = dict(case, batch=min(case["batch"], 64))  # the sites of a part of one batch, scaled
    x = _inputs(part, 1)
    N, B = _grid(case), part["batch"]
    if "coords" in x:
        b, p = x["coords"][:, 0], x["coords"][:, 1:]
    else:
        b, p, _ = _raster(x["points"], x["begin"], x["sample"])
    a = np.zeros((B, N, N), bool)
    a[b, p[:, 0], p[:, 1]] = True
    up = case["batch"] / B
    n0, flops, train = a.sum() * up, 0.0, case["mode"] != "infer"
    for i, (conv, grid) in enumerate(zip(_convs(case), _active(case, a))):
        if conv is not None:
            one = 2.0 * (grid.sum() * up + 1) * conv[0] ** 2 * conv[1] * conv[2]
            flops += one * (1 if not train else 3 if i or case["dfeats"] else 2)
    weights = sum(r * c for r, c in _shapes(case))
    biases = sum(c for _, c in _shapes(case))
    rows, cols = _shapes(case)[-1]
    flops += 2.0 * case["batch"] * rows * cols * (3 if train else 1)
    e = 2 if case["dtype"] == "bf16" else 4
    size = n0 * (12 + e * case["c_in"]) + e * weights + 4 * biases + 4 * case["batch"] * case["classes"]
    if train:
        size += 4 * (weights + biases) + 4 * case["batch"]
    if case["dfeats"]:
        size += n0 * e * case["c_in"]
    if case["mode"] == "step":  # paths read, sites written; weights, biases and velocities read and written
        size += 8 * len(x["points"]) * up + (12 + e * case["c_in"]) * n0 + (16 + (e if e == 2 else 0)) * weights + 16 * biases
    return {"bytes": float(size), "flops": float(flops)}


def tolerance(case):
    """Against another correct implementation at the same precision, measured with every hidden layer's
    channels in another order (the sums of all products in another order, the results permuted back).
    Logits: float32 4e-7, bf16 2e-3.  A gradient has passed ell max-pooling layers, each of which sends a
    value to another place where rounding makes another of a window's near values the largest.  float32:
    mostly 5e-7, but 2e-3 where that happens once.  bf16: 0.006 to 0.02 at five pooling layers and
    batches of 64 and more, 0.4 to 0.7 at single elements; over 0.03 at six layers or a few samples."""
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 2e-5} if case["mode"] == "infer" else {"rel": 4e-3, "max": 0.5}
    return {"rel": 8e-3, "max": 5e-2} if case["mode"] == "infer" else {"rel": 3e-2, "max": 0.99}


# ---------------------------------------------------------------------------------------------------------
# the same in 64 bits


def _philox(counter, key):
    """Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC 2011): four arrays of output words."""
    c = [np.asarray(v, np.uint64) for v in counter]
    k0, k1 = key
    m = np.uint64(0xFFFFFFFF)
    for _ in range(10):
        p0, p1 = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & m, (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & m]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _factors(rate, level, keys, channels):
    """Dropout factors [len(keys), channels] of the elements of one level."""
    q = np.asarray(keys, np.uint64)[:, None]
    g = np.arange((channels + 3) // 4, dtype=np.uint64)[None, :]
    zero = np.zeros(np.broadcast_shapes(q.shape, g.shape), np.uint64)
    words = _philox((q + zero, g + zero, zero + np.uint64(level), zero), (_DROPOUT_SEED & 0xFFFFFFFF, _DROPOUT_SEED >> 32))
    w = np.stack(words, -1).reshape(len(keys), -1)[:, :channels]
    return np.where(w >= np.uint64(int(rate * 2 ** 32)), 1.0 / (1.0 - rate), 0.0)


def _encode(x, case):
    """Picture and 8-direction histogram of every touched square: sites in ascending order, features."""
    N = _grid(case)
    b, p, q = _raster(x["points"], x["begin"], x["sample"])
    here, there = (b * N + p[:, 0]) * N + p[:, 1], (b * N + q[:, 0]) * N + q[:, 1]
    keys, at = np.unique(here, return_inverse=True)
    d = p - q
    moved = (d != 0).any(axis=1)
    dirs = np.array([[3, 2, 1], [4, -1, 0], [5, 6, 7]])[d[:, 0] + 1, d[:, 1] + 1]
    half = np.where((d != 0).all(axis=1), math.sqrt(2.0), 1.0) / 2
    feats = np.zeros((keys.size, 9))
    feats[:, 0] = 1.0
    np.add.at(feats, (at[moved], 1 + dirs[moved]), half[moved])
    np.add.at(feats, (np.searchsorted(keys, there[moved]), 1 + dirs[moved]), half[moved])
    return np.stack([keys // (N * N), keys // N % N, keys % N], axis=1), feats


def exact(case, seed):
    """The dense network on the whole grid, in 64 bits with torch's autograd, some samples at a time.

    16-bit gradients below a max-pooling layer have no such value: 64 bits choose another one of a window's
    four values where 16 bits leave them nearly equal, which puts these gradients 0.02 to 0.25 apart at any
    precision of the sums.  The gradients above the last pooling layer are compared."""
    x = _inputs(case, seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    if case["mode"] == "step":
        x["coords"], x["feats"] = _encode(x, case)

    def stored(a):  # weights and features are given in the storage type
        t = torch.as_tensor(np.ascontiguousarray(a))
        return (t.to(torch.bfloat16) if case["dtype"] == "bf16" else t.float()).to(dev, torch.float64)

    W = [stored(w).requires_grad_(True) for w in x["W"]]
    bias = [torch.as_tensor(b).to(dev, torch.float64).requires_grad_(True) for b in x["b"]]
    feats = stored(x["feats"]).requires_grad_(case["dfeats"])
    labels = torch.as_tensor(x["labels"]).to(dev)
    coords = torch.as_tensor(x["coords"]).to(dev)
    N, B, nin, train = _grid(case), case["batch"], case["arch"] == "deepcnin", case["mode"] != "infer"
    rates = _rates(case) if case["dropout"] else [0.0] * (case["ell"] + 2)
    logits, loss = torch.empty(B, case["classes"], dtype=torch.float64, device=dev), 0.0
    per = max(1, min(B, int(64 * 9216 * 50 / (N * N * case["k"]))))
    for lo in range(0, B, per):
        hi = min(B, lo + per)
        mine = (coords[:, 0] >= lo) & (coords[:, 0] < hi)
        c = coords[mine]
        h = torch.zeros(hi - lo, N, N, case["c_in"], dtype=torch.float64, device=dev)
        h = h.index_put((c[:, 0] - lo, c[:, 1], c[:, 2]), feats[mine])
        if case["dropout"]:
            active = np.zeros((hi - lo, N, N), bool)
            cc = c.cpu().numpy()
            active[cc[:, 0] - lo, cc[:, 1], cc[:, 2]] = True
            below = [active] + _active(case, active)
        n = level = 0
        for stage, conv in enumerate(_convs(case)):
            if conv is None:
                h = torch.nn.functional.max_pool2d(h.permute(0, 3, 1, 2).contiguous(), 2).permute(0, 2, 3, 1)
                continue
            F, ci = conv[:2]
            if F > 1:
                if rates[level] and train:
                    b, y, xx = np.nonzero(below[stage])
                    S = below[stage].shape[1]
                    f = torch.ones_like(h)
                    f[b, y, xx] = torch.as_tensor(_factors(rates[level], level, ((b + lo) * S + y) * S + xx, ci)).to(dev)
                    h = h * f
                level += 1
            S = h.shape[1] - F + 1
            G = torch.cat([h[:, f // F: f // F + S, f % F: f % F + S, :] for f in range(F * F)], 3).reshape(hi - lo, S * S, -1)
            z = torch.bmm(G, W[n].expand(hi - lo, -1, -1)).reshape(hi - lo, S, S, -1) + bias[n]
            h = torch.where(z >= 0, z, z / 3) if nin else torch.relu(z)
            n += 1
        h = h.reshape(hi - lo, -1)
        if rates[level] and train:
            h = h * torch.as_tensor(_factors(rates[level], level, np.arange(lo, hi), h.shape[1])).to(dev)
        out = h @ W[n] + bias[n]
        logits[lo:hi] = out.detach()
        if train:
            part = torch.nn.functional.cross_entropy(out, labels[lo:hi], reduction="sum") / B
            part.backward()
            loss += float(part.detach())
    if not train:
        return {"logits": logits}
    dW, db = [w.grad for w in W], [b.grad for b in bias]
    top = 0 if case["dtype"] == "f32" else len(W) - (3 if nin else 2)  # the first matrix with an exact value

    got = {"logits": logits, "loss": torch.tensor([loss], dtype=torch.float64)}
    if case["mode"] != "step":
        got.update(dW=[None] * top + dW[top:], db=[None] * top + db[top:])
        if case["dfeats"]:
            got["dfeats"] = feats.grad
        return got
    W32 = [torch.as_tensor(w).to(dev, torch.float64) for w in x["W"]]  # the first update: no velocity yet
    vW = [g + _DECAY * w for w, g in zip(W32, dW)]
    got.update(vW=[None] * top + vW[top:], vb=[None] * top + db[top:], W=[w - _LR * v for w, v in zip(W32, vW)],
               b=[b.detach() - _LR * g for b, g in zip(bias, db)])
    return got
