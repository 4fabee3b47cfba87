"""The workloads that this library's speed is measured on.

`listed()` names them, `draw()` gives more of the same ranges, `prepare()` makes what a program holds
before the call (inputs from a seed, plans, packed weights, rulebooks), `run()` is one pass through
the public entry points, `work()` the bytes and operations that the pass cannot do without, and
`exact()` what it returns, computed in 64 bits with torch and numpy alone.

Kinds of case:
  pvs     triangles -> PVS and logits through a captured plan (one call per frame of a server)
  train   one captured training step: froxelize to Adam, with gradients, weights and statistics
  front   froxelize, sites and rulebook with pair lists, input and label gather
  layer   one 3^3 submanifold layer, forward, over the rulebook of a batch of grids
  bwd     the backward of one such layer: data, weight and bias gradient
  cull    the triangles and objects of a scene tested against a PVS
Grids are "x x y x z" froxel extents joined by commas; `fill` is the share of a layer's blocks that
are active, in per cent.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2509_24677_amd as npvs
from paper_2509_24677_amd import train as npvs_train

DTYPES = {"bf16": npvs.NPVS_BF16, "f32": npvs.NPVS_F32}
TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}
FRAME = "256x256x128"  # one viewcell frame at the paper's resolution
PAIRS_PER_SITE = 14.0  # neighbours of a site, itself among them, on scenes of walls and boxes
# sixteen uneven grids, as a server batches viewcells of different extents
BATCH = ",".join(["64x64x64", "128x128x64", "128x128x128", "192x192x128", "256x256x128"] * 3 + ["64x64x64"])


def listed():
    return [
        # the smallest call: a 32^3 viewcell of 200 triangles through a three-layer net (latency)
        dict(name="pvs_small", kind="pvs", grids="32x32x32", tris=200, boxes=20, d=2, hidden=16, layers=3, dtype="bf16"),
        # the ordinary inference call: one city frame, six 64-channel layers
        dict(name="pvs_city", kind="pvs", grids=FRAME, tris=50000, boxes=840, d=4, hidden=64, layers=6, dtype="bf16"),
        # the training step of the same frame
        dict(name="train_city", kind="train", grids=FRAME, tris=50000, boxes=840, d=4, hidden=64, layers=6, dtype="bf16"),
        # what a server does for a batch of uneven grids before its network runs
        dict(name="front_batch", kind="front", grids=BATCH, tris=16000, boxes=420, d=4, dtype="bf16"),
        # a hidden layer over such a batch (the throughput case)
        dict(name="layer_batch", kind="layer", grids=BATCH, d=4, fill=18.0, cin=64, cout=64, dtype="bf16"),
        # the same layer in float32 on one frame: the reference precision of the library
        dict(name="layer_f32", kind="layer", grids=FRAME, d=4, fill=7.4, cin=64, cout=64, dtype="f32"),
        # a layer without much interleave: a fine grid (d = 2), few channels in
        dict(name="layer_fine", kind="layer", grids=FRAME, d=2, fill=4.7, cin=8, cout=64, dtype="bf16"),
        # the first layer at interleave factor 16 (d^3 = 4096 inputs on few sites)
        dict(name="layer_d16", kind="layer", grids=FRAME, d=16, fill=19.4, cin=4096, cout=64, dtype="bf16"),
        # the first decoder layer of the U-Net (160 inputs: upsampled and skip channels)
        dict(name="layer_decoder", kind="layer", grids=FRAME, d=4, fill=7.4, cin=160, cout=96, dtype="bf16"),
        # backward of a hidden layer over four 128^3 training grids
        dict(name="bwd_batch4", kind="bwd", grids=",".join(["128x128x128"] * 4), d=4, fill=16.0, cin=64, cout=64,
             dtype="bf16"),
        # the same in float32 on one frame
        dict(name="bwd_f32", kind="bwd", grids=FRAME, d=4, fill=7.4, cin=64, cout=64, dtype="f32"),
        # culling the scene's triangles and its objects against the PVS
        dict(name="cull_city", kind="cull", grids=FRAME, tris=50000, boxes=840, objects=2048),
    ]


def draw(rng):
    def log(lo, hi):
        return lo * (hi / lo) ** rng.random()

    def grids(d, most, n_most):
        # extents that are multiples of 8 and of d, ragged against 32 half of the time
        n = rng.choice([1, 1, 1, 2, 3, 4, 8, 16][:n_most])
        out = []
        for _ in range(n):
            g = [max(1, round(log(32, 256) / max(8, d))) * max(8, d) for _ in range(3)]
            if rng.random() < 0.5:
                g[0] = max(32, g[0] // 32 * 32)
            while g[0] * g[1] * g[2] > most // n:
                a = g.index(max(g))
                g[a] = max(max(8, d), (g[a] // 2) // max(8, d) * max(8, d))
            out.append("%dx%dx%d" % tuple(g))
        return ",".join(out)

    kind = rng.choice(["pvs", "train", "front", "layer", "layer", "layer", "bwd", "bwd", "cull"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    if kind in ("layer", "bwd"):
        d = rng.choice([2, 4, 4, 8])
        wide = rng.random() < 0.25
        small = [8, 16, 24, 32, 40, 64, 64, 64, 96, 160]
        cin, cout = rng.choice(small), rng.choice(small)
        if dtype == "f32" and rng.random() < 0.3:
            cin, cout = rng.choice([1, 3, 10, 27, 50]), rng.choice([1, 5, 16, 33, 64])
        g = grids(d, 1 << 23, 8)
        if wide:  # the outer layers of a network at d = 8 or 16
            d = rng.choice([8, 16])
            g = grids(d, 1 << 23, 3)
            cin, cout = (d ** 3, rng.choice([32, 64])) if rng.random() < 0.5 else (rng.choice([32, 64]), d ** 3)
            if dtype == "f32":
                d, cin, cout = 8, min(cin, 512), min(cout, 512)
                g = grids(d, 1 << 21, 3)
        blocks = sum(np.prod([int(v) // d for v in s.split("x")]) for s in g.split(","))
        # no drawn layer costs more than the listed ones: sites limited by the channel product
        most = (140000 if dtype == "bf16" else 14000) * 4096 / (cin * cout)
        most = min(most, 140000) / (4 if kind == "bwd" else 1)
        fill = min(log(1.0, 30.0), 100.0 * most / blocks)
        return dict(kind=kind, grids=g, d=d, fill=round(max(fill, 0.5), 2), cin=cin, cout=cout, dtype=dtype)
    if kind == "cull":
        t = int(log(200, 50000))
        return dict(kind="cull", grids=grids(8, 1 << 23, 3), tris=t, boxes=max(4, t // 60), objects=int(log(16, 2048)))
    if kind == "front":
        t = int(log(200, 16000))
        return dict(kind="front", grids=grids(rng.choice([2, 4, 8]), 1 << 23, 8), tris=t, boxes=max(4, t // 40),
                    d=rng.choice([2, 4, 4, 8]), dtype=dtype)
    d = rng.choice([2, 4, 4, 8]) if dtype == "bf16" else rng.choice([2, 4])
    t = int(log(200, 50000))
    return dict(kind=kind, grids=grids(d, (1 << 23) if dtype == "bf16" and d > 2 else 1 << 20, 6), tris=t,
                boxes=max(4, t // 60), d=d, hidden=rng.choice([16, 32, 64]), layers=rng.randint(2, 6), dtype=dtype)


# ------------------------------------------------------------------------------------ inputs
def _dims(case):
    return [tuple(int(v) for v in g.split("x")) for g in case["grids"].split(",")]


def _rng(seed, i=0):
    return np.random.Generator(np.random.PCG64([int(seed) & 0xFFFFFFFF, i]))


def _device():
    return torch.device("cuda") if torch.cuda.is_available() else torch.device("cpu")


def _scene(rng, dims, n_tris, n_boxes):
    """float32 [n_tris][3][3]: boxes (five faces each) on a ground plane, the faces cut into quads of
    one edge length; the ground's quads make up the exact count."""
    nx, ny, nz = dims
    n_boxes = max(1, min(n_boxes, (n_tris - 2) // 12))
    side = np.stack([rng.uniform(2.0, max(3.0, min(24.0, 0.3 * e)), n_boxes) for e in dims], 1)
    if nx >= 128:  # buildings: small footprints, log-normal heights
        side[:, 0] = rng.uniform(3.0, 10.0, n_boxes)
        side[:, 2] = rng.uniform(3.0, 10.0, n_boxes)
        side[:, 1] = np.clip(np.exp(rng.normal(math.log(12.0), 0.6, n_boxes)), 1.0, 0.8 * ny)
    ground = float(rng.uniform(0.02, 0.04)) * ny + 0.37
    lo = rng.random((n_boxes, 3)) * np.maximum(np.array(dims) - side - 1.0, 0.5)
    if nx >= 128:
        lo[:, 1] = ground
    hi = np.minimum(lo + side, np.array(dims) - 0.01)
    x0, y0, z0 = lo.T
    w, h, l = (hi - lo).T
    o = np.zeros(n_boxes)
    V = lambda a, b, c: np.stack([a, b, c], 1)  # noqa: E731
    P = np.concatenate([V(x0, y0 + h, z0), V(x0, y0, z0), V(x0, y0, z0 + l), V(x0, y0, z0), V(x0 + w, y0, z0)])
    A = np.concatenate([V(w, o, o), V(w, o, o), V(w, o, o), V(o, o, l), V(o, o, l)])
    B = np.concatenate([V(o, o, l), V(o, h, o), V(o, h, o), V(o, h, o), V(o, h, o)])
    la, lb = np.linalg.norm(A, axis=1), np.linalg.norm(B, axis=1)

    def cuts(s):
        return np.maximum(1, np.round(la / s)).astype(int), np.maximum(1, np.round(lb / s)).astype(int)

    budget, s_lo, s_hi = int(0.9 * n_tris), 0.05, 1e3
    for _ in range(40):
        s = math.sqrt(s_lo * s_hi)
        a, b = cuts(s)
        s_lo, s_hi = (s, s_hi) if 2 * (a * b).sum() > budget else (s_lo, s)
    a, b = cuts(s_hi)
    f = np.repeat(np.arange(len(a)), a * b)  # face of each quad
    q = np.arange(len(f)) - np.repeat(np.cumsum(a * b) - a * b, a * b)
    i, j = q // b[f], q % b[f]
    k = max(1, -(-(n_tris - 2 * len(f)) // 2))  # ground quads
    kx = max(1, min(k, int(round(math.sqrt(k * nx / nz)))))
    kz = -(-k // kx)
    gi, gj = np.divmod(np.arange(kx * kz), kz)
    P = np.concatenate([P[f] + A[f] * (i / a[f])[:, None] + B[f] * (j / b[f])[:, None],
                        np.stack([gi * (nx / kx), np.full(kx * kz, ground), gj * (nz / kz)], 1)])
    dA = np.concatenate([A[f] / a[f][:, None], np.tile([nx / kx, 0.0, 0.0], (kx * kz, 1))])
    dB = np.concatenate([B[f] / b[f][:, None], np.tile([0.0, 0.0, nz / kz], (kx * kz, 1))])
    t = np.stack([np.stack([P, P + dA, P + dA + dB], 1), np.stack([P, P + dA + dB, P + dB], 1)], 1)
    return t.reshape(-1, 3, 3)[:n_tris].astype(np.float32)


def _tris(case, seed):
    """(triangles of all grids, triangles per grid): the count is shared out by the grids' volumes."""
    dims = _dims(case)
    vol = np.array([np.prod(g) for g in dims], float)
    n = np.maximum(24, np.floor(case["tris"] * vol / vol.sum())).astype(int)
    boxes = np.maximum(1, np.round(case["boxes"] * vol / vol.sum())).astype(int)
    return np.concatenate([_scene(_rng(seed, i), g, int(n[i]), int(boxes[i])) for i, g in enumerate(dims)]), n.tolist()


def _weights(seed, channels):
    """He-normal weights and small biases, float32, per layer."""
    rng = _rng(seed, 1000)
    return [(rng.normal(0.0, math.sqrt(2.0 / (27 * i)), (27, i, o)).astype(np.float32),
             rng.normal(0.0, 0.05, o).astype(np.float32)) for i, o in zip(channels[:-1], channels[1:])]


def _channels(case):
    c = case["d"] ** 3
    return [c] + [case["hidden"]] * (case["layers"] - 1) + [c]


def _label_mask(seed, n_bytes):
    return np.packbits(_rng(seed, 2000).random((n_bytes, 8)) < 0.35, axis=-1, bitorder="little").reshape(-1)


def _site_counts(case):
    b = [np.prod([v // case["d"] for v in g]) for g in _dims(case)]
    return [int(max(1, min(v, v * case["fill"] / 100.0))) for v in b]


def _blocks(case, seed):
    """bool [Bz][By][Bx] per grid: shells of boxes and columns over a ground layer, exactly as many
    active blocks as the fill gives (those of the nearest depth slices)."""
    out = []
    for gi, (g, want) in enumerate(zip(_dims(case), _site_counts(case))):
        B = np.array(g) // case["d"]
        rng, m = _rng(seed, gi), np.zeros(B[::-1], bool)
        m[:, min(1, B[1] - 1), :] = True
        n = int(m.sum())
        while n < min(want * 1.05 + 1, m.size):
            for _ in range(32):
                column = rng.random() < 0.7  # a building on the ground, else a box anywhere
                s = np.minimum(rng.integers((1, 1, 1), (4, 7, 4)) if column else rng.integers(1, 7, 3), B)
                p = (rng.random(3) * (B - s + 1)).astype(int)
                p[1] = 0 if column else p[1]
                x, y, z = (slice(p[a], p[a] + s[a]) for a in range(3))
                m[z, y, p[0]] = m[z, y, p[0] + s[0] - 1] = True
                m[z, p[1] + s[1] - 1, x] = True
                m[p[2], y, x] = m[p[2] + s[2] - 1, y, x] = True
            n = int(m.sum())
        flat = m.reshape(-1)
        flat[np.flatnonzero(flat)[want:]] = False
        out.append(m)
    return out


def _block_bits(case, masks, seed):
    """Packed occupancy with the first froxel row of every active block set."""
    d, out = case["d"], []
    for g, m in zip(_dims(case), masks):
        v = np.zeros((g[2], g[1], g[0]), bool)
        v[::d, ::d, :] = np.repeat(m, d, axis=2)
        out.append(np.packbits(v, axis=-1, bitorder="little").reshape(-1))
    return np.concatenate(out)


def _layer_data(case, seed, dev):
    """X, W, b (and for the backward the saved output Y and its gradient dY) of one layer."""
    n, cin, cout = sum(_site_counts(case)), case["cin"], case["cout"]
    g = torch.Generator(device=dev).manual_seed(int(seed) * 7919 + 17)
    dt = TORCH[case["dtype"]]

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev)

    if cin in (8, 512, 4096):  # a network's input: the froxels of a block, about a fifth occupied
        X = (torch.rand((n, cin), generator=g, device=dev) < 0.2).to(dt)
    else:  # activations after a ReLU
        X = normal(n, cin).clamp_min_(0).to(dt)
    W = normal(27, cin, cout) * math.sqrt(2.0 / (27 * cin))
    b = normal(cout) * 0.05
    if case["kind"] == "layer":
        return X, W, b, None, None
    return X, W, b, normal(n, cout).clamp_min_(0).to(dt), normal(n, cout) * 1e-3


# ------------------------------------------------------------------------------------ passes
def prepare(case, seed):
    kind, dev = case["kind"], torch.device("cuda")
    if kind in ("layer", "bwd"):
        dims, dt = _dims(case), DTYPES[case["dtype"]]
        bits = torch.from_numpy(_block_bits(case, _blocks(case, seed), seed)).to(dev)
        X, W, b, Y, dY = _layer_data(case, seed, dev)
        rb = npvs.build_rulebook(bits, dims, case["d"], csr=kind == "bwd")

        def rows(t):  # rows up to the rulebook's capacity, as the library hands layers on
            out = torch.zeros((rb.cap, t.shape[1]), dtype=t.dtype, device=dev)
            out[:t.shape[0]] = t
            return out

        s = dict(case=case, dt=dt, rb=rb, n=X.shape[0], X=rows(X))
        if kind == "layer":
            return dict(s, Wp=npvs.pack_weights(W, dt), b=b)
        return dict(s, Wt=npvs.pack_weights(W, dt, flip_transpose=True), Y=rows(Y), dY=rows(dY))
    dims = _dims(case)
    tris_np, n_tris = _tris(case, seed)
    tris = torch.from_numpy(tris_np).to(dev)
    if kind == "cull":
        occ = npvs.froxelize(tris, n_tris, dims)
        keep = torch.from_numpy(_label_mask(seed, occ.numel())).to(dev)
        off = np.sort(_rng(seed, 3000).integers(0, len(tris_np) + 1, case["objects"] - 1))
        off = np.concatenate([[0], off, [len(tris_np)]]).astype(np.int64)
        return dict(case=case, tris=tris, n_tris=n_tris, dims=dims, pvs=occ & keep, off=torch.from_numpy(off).to(dev))
    if kind == "front":
        occ = npvs.froxelize(tris, n_tris, dims)
        rb = npvs.build_rulebook(occ, dims, case["d"], csr=True)
        for t in (rb.site_keys, rb.nbr, rb.rb_pairs):
            t.fill_(-1)  # entries past the counts are not written
        X = torch.zeros((rb.cap, case["d"] ** 3), dtype=TORCH[case["dtype"]], device=dev)
        return dict(case=case, tris=tris, n_tris=n_tris, dims=dims, rb=rb, occ=occ, X=X)
    layers, dt = _weights(seed, _channels(case)), DTYPES[case["dtype"]]
    if kind == "pvs":
        plan = npvs.Plan(dims, n_tris, case["d"], _channels(case), dt)
        for i, (W, b) in enumerate(layers):
            plan.set_weights(i, torch.from_numpy(W).to(dev), torch.from_numpy(b).to(dev))
        torch.cuda.synchronize()
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            pvs, logits = plan.capture(tris, want_logits=True)
        torch.cuda.current_stream().wait_stream(side)
        return dict(case=case, plan=plan, pvs=pvs, logits=logits)
    # train: a program that resumes at step 1000 with its optimizer state, the step captured once
    occ = npvs.froxelize(tris, n_tris, dims)
    labels = occ & torch.from_numpy(_label_mask(seed, occ.numel())).to(dev)
    net = npvs_train.Network(layers, case["d"], dt)
    tr = npvs_train.Trainer(net, dims, n_tris, checkpoint=False)
    m0, v0 = (torch.from_numpy(a).to(dev) for a in _adam_state(seed, net.flat.numel()))
    p0 = net.flat.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        tr.step(tris, labels)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        stats, pvs = tr.step(tris, labels)
    net.flat.copy_(p0)
    tr.m.copy_(m0)
    tr.v.copy_(v0)
    tr.adam_step.view(torch.int64)[0] = 1000
    net.repack()
    torch.cuda.synchronize()
    return dict(case=case, graph=graph, net=net, trainer=tr, tris=tris, labels=labels, stats=stats, pvs=pvs)


def _adam_state(seed, n):
    rng = _rng(seed, 4000)
    return (rng.normal(0.0, 1e-3, n)).astype(np.float32), (1e-6 * (0.5 + rng.random(n))).astype(np.float32)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "layer":
        y = npvs.sparse_conv_fwd(state["X"], state["Wp"], state["b"], case["cin"], case["cout"], state["rb"],
                                 state["dt"], True)
        return {"y": y[:state["n"]]}
    if kind == "bwd":
        dx, dw, db = npvs.sparse_conv_bwd(state["X"], state["Wt"], case["cin"], case["cout"], state["Y"], state["dY"],
                                          state["rb"], state["dt"], True)
        return {"dx": dx[:state["n"]], "dw": dw, "db": db}
    if kind == "pvs":
        state["plan"].replay()
        return {"logits": state["logits"], "pvs": state["pvs"]}
    if kind == "train":
        state["graph"].replay()
        return {"grads": state["net"].gflat, "weights": state["net"].flat, "stats": state["stats"],
                "pvs": state["pvs"]}
    if kind == "front":
        d, dt = case["d"], DTYPES[case["dtype"]]
        occ = npvs.froxelize(state["tris"], state["n_tris"], state["dims"], occ=state["occ"])
        rb = npvs.build_rulebook(occ, state["dims"], d, csr=True, out=state["rb"])
        X = npvs.gather_input(occ, rb, dt, out=state["X"])
        return {"occ": occ, "counts": rb.counts[:3], "keys": rb.site_keys, "rows": rb.block_row,
                "grid_rows": rb.grid_rows, "nbr": rb.nbr, "off": rb.rb_off, "pairs": rb.rb_pairs, "x": X}
    vis = npvs.visible_triangles(state["tris"], state["n_tris"], state["dims"], state["pvs"])
    return {"triangles": vis, "objects": npvs.visible_objects(vis, state["off"])}


# ------------------------------------------------------------------------------------ work
def work(case):
    kind, dims = case["kind"], _dims(case)
    froxels = float(sum(np.prod(g) for g in dims))
    if kind in ("layer", "bwd"):
        n, cin, cout = sum(_site_counts(case)), case["cin"], case["cout"]
        es = 2 if case["dtype"] == "bf16" else 4
        flops = 2.0 * PAIRS_PER_SITE * n * cin * cout
        if kind == "layer":  # X and the map in, Y out, the weights
            return {"bytes": es * n * (cin + cout) + 4 * 27 * n + es * 27 * cin * cout, "flops": flops}
        return {"bytes": n * (es * (cin + cout) + 4 * (cin + cout) + 4 * 27 + 8 * PAIRS_PER_SITE)
                + 27 * cin * cout * (es + 4), "flops": 2 * flops}
    if kind == "cull":
        return {"bytes": 36.0 * case["tris"] + froxels / 8 + case["tris"] + 9 * case["objects"], "flops": 0.0}
    sites = 0.07 * froxels / case["d"] ** 3  # active blocks of such scenes
    blocks = froxels / case["d"] ** 3
    if kind == "front":
        es = 2 if case["dtype"] == "bf16" else 4
        return {"bytes": 36.0 * case["tris"] + froxels / 8 + 4 * blocks
                + sites * (4 + 4 * 27 + 8 * PAIRS_PER_SITE + es * case["d"] ** 3), "flops": 0.0}
    ch = _channels(case)
    params = sum(27 * a * b for a, b in zip(ch[:-1], ch[1:]))
    flops = 2.0 * PAIRS_PER_SITE * sites * params / 27
    if kind == "pvs":
        return {"bytes": 36.0 * case["tris"] + froxels / 8 + 4 * froxels + 2.0 * params, "flops": flops}
    return {"bytes": 36.0 * case["tris"] + froxels / 4 + 4.0 * params * 7, "flops": 3 * flops}


# ------------------------------------------------------------------------------------ 64 bits
def _exact_occ(tris, dims):
    """bool [nz][ny][nx]: the froxels that closed triangles meet, by the separating-axis test in
    integers on vertices rounded to 1/256 froxel (half to even)."""
    dev = _device()
    q = torch.round(torch.from_numpy(tris).to(dev).double() * 256).long()  # [T][3][3]
    N = torch.tensor(dims, device=dev)
    mn, mx = q.amin(1), q.amax(1)
    lo = torch.div(mn - 1, 256, rounding_mode="floor").clamp_min(0)
    hi = torch.minimum(torch.div(mx, 256, rounding_mode="floor"), N - 1)
    ext = (hi - lo + 1).clamp_min(0)
    cnt = ext.prod(1)
    occ = torch.zeros(dims[2] * dims[1] * dims[0], dtype=torch.bool, device=dev)
    ends = torch.cumsum(cnt, 0)
    first, total = 0, int(cnt.sum())
    while first < total:  # candidates in blocks of at most 4 million
        c = torch.arange(first, min(total, first + 4_000_000), device=dev)
        first += len(c)
        t = torch.searchsorted(ends, c, right=True)
        k = c - (ends[t] - cnt[t])
        ex, ey = ext[t, 0], ext[t, 1]
        I = torch.stack([lo[t, 0] + k % ex, lo[t, 1] + (k // ex) % ey, lo[t, 2] + k // (ex * ey)], 1) * 256
        v = q[t]
        e = [v[:, (i + 1) % 3] - v[:, i] for i in range(3)]
        zero = torch.zeros_like(e[0][:, 0])
        axes = [torch.linalg.cross(e[0], e[1])]
        for w in e:
            axes += [torch.stack([zero, w[:, 2], -w[:, 1]], 1), torch.stack([-w[:, 2], zero, w[:, 0]], 1),
                     torch.stack([w[:, 1], -w[:, 0], zero], 1)]
        hit = torch.ones(len(c), dtype=torch.bool, device=dev)
        for a in axes:
            p = (v * a[:, None, :]).sum(-1)
            base = (I * a).sum(-1)
            up, down = 256 * a.clamp_min(0).sum(-1), 256 * a.clamp_max(0).sum(-1)
            hit &= (p.amin(1) <= base + up) & (p.amax(1) >= base + down)
        I = I[hit] // 256
        occ[(I[:, 2] * dims[1] + I[:, 1]) * dims[0] + I[:, 0]] = True
    return occ.view(dims[2], dims[1], dims[0])


def _exact_nbr(masks):
    """int64 [27][n]: the row of each site's neighbour, n (a zero row) where there is none."""
    dev, n, out = _device(), sum(int(m.sum()) for m in masks), []
    base = 0
    for m in masks:
        m = torch.as_tensor(m, device=dev)
        rows = torch.full([s + 2 for s in m.shape], n, dtype=torch.long, device=dev)
        z, y, x = torch.nonzero(m, as_tuple=True)
        rows[z + 1, y + 1, x + 1] = base + torch.arange(len(z), device=dev)
        base += len(z)
        out.append(torch.stack([rows[z + dz, y + dy, x + dx] for dz in range(3) for dy in range(3) for dx in range(3)]))
    return torch.cat(out, 1)


def _exact_conv(X, W, b, nbr):
    Xz = torch.cat([X, X.new_zeros(1, X.shape[1])])
    y = b.expand(nbr.shape[1], -1).clone()
    for k in range(27):
        y = y + Xz[nbr[k]] @ W[k]
    return y


def _to_blocks(v, d):
    """[nz][ny][nx] -> [blocks][d^3], z outermost within a block as among the blocks."""
    nz, ny, nx = v.shape
    return v.view(nz // d, d, ny // d, d, nx // d, d).permute(0, 2, 4, 1, 3, 5).reshape(-1, d ** 3)


def _from_blocks(v, dims, d):
    nx, ny, nz = dims
    return v.view(nz // d, ny // d, nx // d, d, d, d).permute(0, 3, 1, 4, 2, 5).reshape(nz, ny, nx)


def _exact_network(case, seed):
    dims, d, dev = _dims(case), case["d"], _device()
    tris, n_tris = _tris(case, seed)
    occ, at = [], 0
    for g, t in zip(dims, n_tris):
        occ.append(_exact_occ(tris[at:at + t], g))
        at += t
    blocks = [_to_blocks(o, d) for o in occ]
    active = [b.any(1) for b in blocks]
    nbr = _exact_nbr([a.view(g[2] // d, g[1] // d, g[0] // d) for a, g in zip(active, dims)])
    X = torch.cat([b[a] for a, b in zip(active, blocks)]).double()
    layers = [(torch.from_numpy(W).to(dev).double().requires_grad_(), torch.from_numpy(b).to(dev).double().requires_grad_())
              for W, b in _weights(seed, _channels(case))]
    h = X
    for i, (W, b) in enumerate(layers):
        h = _exact_conv(h, W, b, nbr)
        h = h.clamp_min(0) if i + 1 < len(layers) else h
    return dims, occ, active, layers, h


def _exact_pvs(case, seed):
    with torch.no_grad():
        dims, _, active, _, logits = _exact_network(case, seed)
        out, at = [], 0
        for a, g in zip(active, dims):
            v = torch.full((len(a), logits.shape[1]), -math.inf, dtype=torch.float64, device=a.device)
            k = int(a.sum())
            v[a] = logits[at:at + k]
            at += k
            out.append(_from_blocks(v, g, case["d"]).reshape(-1))
        return {"logits": torch.cat(out), "pvs": None}


def _exact_train(case, seed):
    dims, occ, active, layers, logits = _exact_network(case, seed)
    mask = np.unpackbits(_label_mask(seed, sum(o.numel() for o in occ) // 8), bitorder="little").astype(bool)
    mask, at, r, lam = torch.from_numpy(mask).to(logits.device), 0, 0, 0.99
    rows = []
    for o, a in zip(occ, active):
        lab = _to_blocks(o & mask[at:at + o.numel()].view(o.shape), case["d"])[a].double()
        at += o.numel()
        l = logits[r:r + len(lab)]
        r += len(lab)
        p = torch.sigmoid(l)
        bce = (torch.nn.functional.softplus(l) - lab * l).mean()
        tp, fn, fp, gtp = (lab * p).sum(), (lab * (1 - p)).sum(), ((1 - lab) * p).sum(), lab.sum()
        lrv = (fn + fp) / gtp.clamp_min(1.0)
        rows.append(torch.stack([lam * bce + (1 - lam) * lrv, bce, lrv, tp, fn, fp, gtp,
                                 torch.tensor(float(l.numel()), dtype=torch.float64, device=l.device)]))
    stats = torch.stack(rows + [torch.stack(rows).mean(0)])
    stats[-1, 0].backward()
    flat = lambda ts: torch.cat([t.reshape(-1) for t in ts])  # noqa: E731
    p0 = flat([W.detach() for W, _ in layers] + [b.detach() for _, b in layers])
    g0 = flat([W.grad for W, _ in layers] + [b.grad for _, b in layers])
    m, v = (torch.from_numpy(a).to(p0.device).double() for a in _adam_state(seed, p0.numel()))
    g = g0 + 1e-10 * p0
    m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
    w = p0 - 1e-3 * (m / (1 - 0.9 ** 1001)) / (torch.sqrt(v / (1 - 0.999 ** 1001)) + 1e-8)
    return {"grads": g0, "weights": w, "stats": stats.detach(), "pvs": None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "pvs":
        return _exact_pvs(case, seed)
    if kind == "train":
        return _exact_train(case, seed)
    if kind not in ("layer", "bwd"):
        return None  # whole numbers only
    dev = _device()
    nbr = _exact_nbr(_blocks(case, seed))
    X, W, b, Y, dY = _layer_data(case, seed, dev)
    X, W, b = X.double(), W.double(), b.double()
    if kind == "layer":
        return {"y": _exact_conv(X, W, b, nbr).clamp_min(0)}
    dZ = torch.where(Y > 0, dY, torch.zeros_like(dY)).double()
    Xz = torch.cat([X, X.new_zeros(1, X.shape[1])])
    dX, dW = torch.zeros_like(Xz), torch.empty_like(W)
    for k in range(27):
        dW[k] = Xz[nbr[k]].T @ dZ
        dX.index_add_(0, nbr[k], dZ @ W[k].T)
    return {"dx": dX[:-1], "dw": dW, "db": dZ.sum(0)}
