"""What a user of this library has it do, as cases that can be timed.

A case names a path through the public entry points and its sizes:

  infer     flexconv_fwd: a layer in a serving network
  train     flexconv_fwd, then flexconv_bwd for all three gradients over prebuilt in-edge lists
  layer     train, then flex-max-pooling forward and backward over the same neighbourhoods
  pool      flex-max-pooling forward and backward alone, through the gather plans where they apply
  resample  the change of resolution between two stages: pooling onto a kept quarter of the points and upsampling
            from it, each forward and backward
  block     1x1 convolution composed into a flex-convolution: compose, forward, backward (features, parameters and
            point locations), gradients mapped back
  prepare   a new cloud: neighbour search, transposed lists, importance sub-sampling to a quarter

Neighbourhoods are static per cloud, so everything that depends on them alone (neighbour tensor, in-edge lists, gather
plans, selection) is built in prepare(), except where building it is the case.  Clouds, features and parameters follow
the recipes of the benchmark configurations (furnished rooms, jittered box surfaces, the unit cube; points along a
Z-order curve unless the case says otherwise), drawn on the GPU from the seed.
"""
import math

import numpy as np
import torch

import paper_1803_07289_amd as fx

PATHS = ("infer", "train", "layer", "pool", "resample", "block", "prepare")


def _case(path, cloud, order, layout, B, N, K, Din, Dout, name=None):
    c = dict(path=path, cloud=cloud, order=order, layout=layout, B=B, N=N, K=K, Din=Din, Dout=Dout)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one small scan through a network's first layer: nothing but latency
        _case("infer", "cube", "generator", "bnc", 1, 1024, 8, 9, 64, "infer_1k_9x64"),
        # the smallest training configuration, in the paper's channel-major form (the binding's default layout)
        _case("train", "cube", "generator", "bcn", 1, 4096, 8, 32, 32, "train_4k_32x32_bcn"),
        # a batch of object scans with wider neighbourhoods: convolution and pooling, forward and backward
        _case("layer", "box", "generator", "bnc", 8, 4096, 16, 64, 64, "layer_8x4k_k16_64x64"),
        # a scanned room through the first layer (xyz, rgb, normalised xyz)
        _case("infer", "room", "morton", "bnc", 1, 1_000_000, 8, 9, 64, "infer_room1m_9x64"),
        # a deep layer at a room's full resolution
        _case("train", "room", "morton", "bnc", 1, 1_000_000, 8, 128, 128, "train_room1m_128x128"),
        # the headline workload: a 7M-point hall, convolution and pooling
        _case("train", "hall", "morton", "bnc", 1, 7_000_000, 8, 64, 64, "train_hall7m_64x64"),
        _case("pool", "hall", "morton", "bnc", 1, 7_000_000, 8, 64, 64, "pool_hall7m_64"),
        # a low-resolution, wide stage: width doubles while the point count drops by four from stage to stage
        _case("train", "room", "morton", "bnc", 1, 109_375, 8, 512, 512, "train_109k_512x512"),
        # class scores: a width no kernel is written for, ragged point count, K off the multiples, channel-major
        _case("train", "room", "morton", "bcn", 2, 50_021, 9, 64, 13, "train_2x50k_k9_64x13_bcn"),
        # between two stages: down to a quarter of the points and up again, with gradients
        _case("resample", "room", "morton", "bnc", 1, 437_500, 8, 128, 128, "resample_437k_128"),
        # a block with a 1x1 convolution, gradients down to the point locations, odd point count
        _case("block", "room", "morton", "bnc", 1, 250_007, 8, 64, 64, "block_250k_64x64"),
        # a new scan, points as the sensor gave them
        _case("prepare", "room", "generator", "bnc", 1, 1_000_000, 8, 1, 1, "prepare_room1m_k8"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# widths as networks of this kind chain them (input features, equal stages, doublings, class scores)
_WIDTHS = ((9, 64), (9, 64), (32, 32), (64, 64), (64, 64), (64, 64), (32, 64), (64, 32), (64, 128), (128, 64), (128, 128),
           (128, 128), (256, 256), (256, 512), (512, 512), (64, 9), (64, 13), (6, 64), (3, 32))


def draw(rng):
    """One more case of the same ranges."""
    path = rng.choice(("infer", "infer", "train", "train", "train", "layer", "pool", "resample", "block", "prepare"))
    K = rng.choice((4, 6, 8, 8, 8, 8, 9, 10, 12, 16))
    B = rng.choice((1, 1, 1, 2, 3, 8))
    layout = rng.choice(("bnc", "bnc", "bcn"))
    order = rng.choice(("morton", "morton", "morton", "generator"))
    points = _log_int(rng, 1024, 2_000_000)
    if path in ("infer", "train", "layer", "block"):
        Din, Dout = rng.choice(_WIDTHS) if rng.random() < 0.7 else (rng.randint(3, 160), rng.randint(3, 160))
        if path == "layer":
            Dout = Din                               # the pooling step's upstream gradient has the features' shape
        if path == "block":
            Din, Dout = min(Din, 128), min(Dout, 128)
        up = lambda w: w if w <= 64 else -(-w // 128) * 128
        points = min(points, int((4e9 if path in ("layer", "block") else 8e9) / (up(Din) * up(Dout))))
    elif path in ("pool", "resample"):
        Din = rng.choice((32, 64, 64, 128, 128, 256, rng.randint(3, 160)))
        Dout = Din
        points = min(points, int(128e6 / Din))
    else:
        Din = Dout = 1
        points = min(points, 1_500_000)
    if order == "generator":
        points = min(points, 500_000)                # an unsorted cloud's neighbours are anywhere in memory
    N = max(256, points // B)
    cloud = rng.choice(("cube", "box")) if N < 20_000 else rng.choice(("room", "hall"))
    return _case(path, cloud, order, layout, B, N, K, Din, Dout)


# ---- inputs, on the GPU ---------------------------------------------------------------------------------------------
def _box_faces(lo, hi):
    """Origins and edge vectors of the six faces of an axis-aligned box."""
    ext, faces = hi - lo, []
    for ax in range(3):
        a, b = [i for i in range(3) if i != ax]
        for side in (lo[ax], hi[ax]):
            o, u, v = lo.copy(), np.zeros(3), np.zeros(3)
            o[ax], u[a], v[b] = side, ext[a], ext[b]
            faces.append((o, u, v))
    return faces


def _on_faces(faces, n, sigma, gen):
    """n points on the faces, in runs per face in proportion to area, with Gaussian jitter."""
    o, u, v = (torch.tensor(np.array([f[i] for f in faces]), dtype=torch.float32, device="cuda") for i in range(3))
    area = u.norm(dim=1) * v.norm(dim=1)
    at = (torch.arange(n, device="cuda", dtype=torch.float64) + 0.5) / n
    face = torch.searchsorted((area.double().cumsum(0) / area.double().sum()), at).clamp_(max=len(faces) - 1)
    s = torch.rand((n, 2), device="cuda", generator=gen)
    p = o[face] + s[:, :1] * u[face] + s[:, 1:] * v[face]
    return p + sigma * torch.randn((n, 3), device="cuda", generator=gen)


def _cloud(kind, n, seed, gen):
    rng = np.random.default_rng(seed)
    if kind == "cube":
        return torch.rand((n, 3), device="cuda", generator=gen)
    if kind == "box":
        side = rng.uniform(0.5, 1.5, size=3)
        inside = n // 5
        p = torch.cat([_on_faces(_box_faces(np.zeros(3), side), n - inside, 0.005, gen),
                       torch.rand((inside, 3), device="cuda", generator=gen) *
                       torch.tensor(side, dtype=torch.float32, device="cuda")])
        return p[torch.randperm(n, device="cuda", generator=gen)]
    size, boxes, sigma = (((25.0, 25.0, 4.0), 200, 0.003) if kind == "hall" else ((10.0, 10.0, 3.0), 30, 0.005))
    size = np.asarray(size)
    faces = _box_faces(np.zeros(3), size)
    for _ in range(boxes):
        ext = rng.uniform(0.3, 2.0, size=3)
        lo = rng.random(3) * (size - ext)
        lo[2] = 0.0 if rng.random() < 0.7 else lo[2]
        faces += _box_faces(lo, lo + ext)
    return _on_faces(faces, n, sigma, gen)


def _morton(p):
    lo = p.min(dim=0).values
    q = ((p - lo) / (p.max(dim=0).values - lo).clamp_min(1e-30) * 1024).clamp_(max=1023).long()

    def spread(x):
        for shift, mask in ((16, 0x030000FF), (8, 0x0300F00F), (4, 0x030C30C3), (2, 0x09249249)):
            x = (x | (x << shift)) & mask
        return x
    return torch.argsort(spread(q[:, 0]) | spread(q[:, 1]) << 1 | spread(q[:, 2]) << 2, stable=True)


def prepare(case, seed):
    path, B, N, K, Din, Dout = (case[k] for k in ("path", "B", "N", "K", "Din", "Dout"))
    gen = torch.Generator("cuda").manual_seed(int(seed))
    pos = torch.empty((B, 3, N), device="cuda")
    for b in range(B):
        p = _cloud(case["cloud"], N, [int(seed), b], gen)
        pos[b] = (p[_morton(p)] if case["order"] == "morton" else p).t()
    layout = fx.BNC if case["layout"] == "bnc" else fx.BCN
    s = dict(path=path, layout=layout, pos=pos, N=N, K=K, B=B)
    randn = lambda *shape: torch.randn(shape, device="cuda", generator=gen)
    rows = lambda n, c: randn(B, n, c) if layout == fx.BNC else randn(B, c, n)
    Ns = max(1, N // 4)
    words = lambda: torch.randint(-2 ** 31, 2 ** 31, (B, Ns), device="cuda", generator=gen, dtype=torch.int64).int()
    if path == "prepare":
        s["words"] = words()
        return s
    nbr = s["nbr"] = fx.flex_knn(pos, K)
    s["feat"] = rows(N, Din)
    if path in ("infer", "train", "layer", "block"):
        Dmid = Dout if path == "block" else Din
        std = (4.0 * Dmid * K) ** -0.5
        s["theta"], s["bias"] = randn(3, Dmid, Dout) * std, randn(Dmid, Dout) * std
        if path == "block":
            s["W"] = randn(Dmid, Din) * Din ** -0.5
    if path in ("train", "layer", "block"):
        s["grad"] = rows(N, Dout)
    if path in ("pool", "layer"):
        s["pool_grad"] = rows(N, Din)
    if path != "infer":
        s["edges"] = fx.flex_inedges_build(nbr)
    if path in ("pool", "layer") and layout == fx.BNC:
        s["fwd_plan"] = fx.flexpool_fwd_plan_build(nbr)
        s["bwd_plan"] = fx.flexpool_plan_build(s["edges"], B, N)
    if path == "resample":
        s["sel"] = fx.flex_selection_make_distinct(fx.flex_idiss_sample(fx.flex_idiss_phi(pos, nbr), words()), N)
        s["sub_edges"] = fx.flex_inedges_build_sub(nbr, s["sel"])
        s["small"], s["small_grad"] = rows(Ns, Din), rows(Ns, Din)
        s["grad"] = rows(N, Din)
    return s


# ---- one pass -------------------------------------------------------------------------------------------------------
def _conv(s):
    out = fx.flexconv_fwd(s["feat"], s["pos"], s["nbr"], s["theta"], s["bias"], layout=s["layout"])
    return (out,) + fx.flexconv_bwd(s["feat"], s["pos"], s["nbr"], s["theta"], s["bias"], s["grad"], layout=s["layout"],
                                    in_edges=s["edges"])


def _pool(s):
    if s["layout"] == fx.BNC:
        out, arg = fx.flexpool_fwd_planned(s["feat"], s["nbr"], s["fwd_plan"], layout=s["layout"])
        return out, arg, fx.flexpool_bwd_planned(s["pool_grad"], arg, s["edges"], s["bwd_plan"], layout=s["layout"])
    out, arg = fx.flexpool_fwd(s["feat"], s["nbr"], layout=s["layout"])
    return out, arg, fx.flexpool_bwd(s["pool_grad"], arg, layout=s["layout"], in_edges=s["edges"])


def run(s):
    path, layout = s["path"], s["layout"]
    if path == "infer":
        return fx.flexconv_fwd(s["feat"], s["pos"], s["nbr"], s["theta"], s["bias"], layout=layout)
    if path == "train":
        return _conv(s)
    if path == "layer":
        return _conv(s) + _pool(s)
    if path == "pool":
        return _pool(s)
    if path == "resample":
        down, down_arg = fx.flexpool_sub_fwd(s["feat"], s["nbr"], s["sel"], layout=layout)
        up, up_arg = fx.flexupsample_fwd(s["small"], s["sel"], s["nbr"], layout=layout)
        up_grad = fx.flexupsample_bwd(s["grad"], up_arg, s["sel"], s["edges"], layout=layout)
        down_grad = fx.flexpool_sub_bwd(s["small_grad"], down_arg, s["N"], layout=layout, in_edges=s["sub_edges"])
        return down, down_arg, up, up_arg, up_grad, down_grad
    if path == "block":
        tc, bc = fx.flexconv_compose_1x1(s["W"], s["theta"], s["bias"])
        out = fx.flexconv_fwd(s["feat"], s["pos"], s["nbr"], tc, bc, layout=layout)
        gf, gtc, gbc = fx.flexconv_bwd(s["feat"], s["pos"], s["nbr"], tc, bc, s["grad"], layout=layout, in_edges=s["edges"])
        gp = fx.flexconv_bwd_pos(s["feat"], s["nbr"], tc, s["grad"], layout=layout, in_edges=s["edges"])
        return (out, gf, gp) + fx.flexconv_compose_1x1_bwd(s["W"], s["theta"], s["bias"], gtc, gbc)
    nbr = fx.flex_knn(s["pos"], s["K"])
    off, src = fx.flex_inedges_build(nbr)
    phi = fx.flex_idiss_phi(s["pos"], nbr)
    sel = fx.flex_selection_make_distinct(fx.flex_idiss_sample(phi, s["words"]), s["N"])
    return nbr, off, src, phi, sel


# ---- what a pass cannot do without ----------------------------------------------------------------------------------
def work(case):
    """Every entry point's arrays touched once each, summed over the calls of the pass (in a network other layers run
    between them); flops of the factored form (aggregate of 4 Din values per point, then a (4 Din) x Dout product)."""
    path, B, N, K, Di, Do = (case[k] for k in ("path", "B", "N", "K", "Din", "Dout"))
    P, params = B * N, 4 * Di * Do
    ids, lists, pos = K, K + 1, 3                    # 4-byte words per point
    fwd = P * (Di + Do + pos + ids) + params
    bwd = P * (2 * Di + Do + pos + lists) + 2 * params
    pool = P * (3 * Di + ids) + P * (3 * Di + lists)
    agg, gemm = 8.0 * K * P, 2.0 * params * P
    if path == "infer":
        return {"bytes": 4.0 * fwd, "flops": agg * Di + gemm}
    if path == "train":
        return {"bytes": 4.0 * (fwd + bwd), "flops": agg * (Di + Do) + 3 * gemm}
    if path == "layer":
        return {"bytes": 4.0 * (fwd + bwd + pool), "flops": agg * (Di + Do) + 3 * gemm}
    if path == "pool":
        return {"bytes": 4.0 * pool, "flops": 2.0 * K * P * Di}
    if path == "resample":
        S = B * max(1, N // 4)
        words = (P * Di + S * (K + 1 + 2 * Di)) + (S * (Di + 1) + P * (K + 2 * Di)) + \
                (P * (2 * Di + lists) + S * (Di + 1)) + (S * (2 * Di + K) + P * (1 + Di))
        return {"bytes": 4.0 * words, "flops": 2.0 * K * (P + S) * Di}
    if path == "block":
        loc = P * (Di + Do + ids + lists + pos) + 3 * Di * Do
        compose = 4 * (Do * Di + 2 * Do * Do + 2 * Di * Do)
        return {"bytes": 4.0 * (fwd + bwd + loc + compose),
                "flops": agg * (Di + Do) + 3 * gemm + 2.0 * K * P * (Di + Do) + 12.0 * Di * Do * P + 24.0 * Di * Do * Do}
    S = B * max(1, N // 4)
    return {"bytes": 4.0 * (P * (pos + ids) + P * (ids + lists) + P * (pos + ids + 1) + P + 2 * S + 2 * S),
            "flops": 8.0 * K * P}


def tolerance(case):
    """32-bit sums throughout (the split contractions keep 22 bits and accumulate in 32); winners, neighbours and lists
    are whole numbers and exact, the draw follows the importances, whose last bit may move a threshold."""
    if case["path"] == "prepare":
        return {"rel": 1e-6, "max": 1e-5, "differ": 1e-5}
    return {"rel": 1e-5, "max": 1e-4, "differ": 0.0}
