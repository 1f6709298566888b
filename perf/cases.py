"""The workloads that the performance of the NSA layer is judged by.

A case is one pass of the layer through its public entry points (`paper_2604_05182_amd.binding`) on inputs that
already sit in GPU memory, as a program that calls the layer would have them:

  forward  routing, block pooling with the repacking of K and V, fused attention (what an inference step does)
  train    the same with the saved results (log-sum-exp, branch outputs), then the gradients of q, k and v
  tokens   the four-rule routing per query token (a table of its own; attention shares one list per block)

Sizes, heads, budgets and windows are those of the repository's configurations (`inputs.CONFIGS`), of its tests, or in
between.  Values are N(0, 1) in bf16, gates sigmoid(N(0, 1)), positions and cameras from the seeded generators of
`inputs`.  Buffers and workspaces are allocated once per state, which is how the C boundary is meant to be used.
"""
import random

import numpy as np
import torch

from paper_2604_05182_amd import binding as B
from paper_2604_05182_amd import inputs as I

KIND = ("forward", "train", "tokens")


def _case(name, kind, n_obj, n_views, grid, heads, d, topk, window, points="uniform", near_views=0, h_kv=0,
          gate_channels=False, k_vol=0, window_mode=0, ragged=False, two_pass=False):
    """k_vol: 0 routes by projected centroids; else by the four geometric rules with k_vol volume blocks and
    topk - k_vol image blocks per query.  ragged: spatial blocks of several 64-slot blocks with partly filled last
    blocks.  two_pass: pooling on its own and a forward that repacks K and V itself."""
    return {"name": name, "kind": kind, "n_obj": n_obj, "n_views": n_views, "grid": grid, "heads": heads,
            "h_kv": h_kv or heads, "d": d, "topk": topk, "window": window, "points": points, "near_views": near_views,
            "gate_channels": gate_channels, "k_vol": k_vol, "window_mode": window_mode, "ragged": ragged,
            "two_pass": two_pass}


def _of_config(name, kind, number, **more):
    c = I.CONFIGS[number]
    k_vol = I.ROUTE3D[number]["k_v2v"] if number in I.ROUTE3D else 0
    return _case(name, kind, c.n_obj, c.n_views, c.grid, c.heads, c.d, c.topk, c.window, c.points, c.near_views,
                 c.kv_heads, c.gate_channels, k_vol, **more)


def listed():
    return [
        # an interactive preview of a small object: two views, 6 K tokens; latency and launches count
        _of_config("tiny forward", "forward", 1),
        # the same in a training loop (unit-sized models, debugging runs): forward, saved results, backward
        _of_config("tiny train", "train", 1),
        # a small odd problem at d = 128 through the separate pooling call: 3 heads, 43 blocks (no multiple of four),
        # 9 routed blocks, as the parity tests use
        _case("small odd d128", "forward", 25 * 64, 2, 24, 3, 128, 9, 192, two_pass=True),
        # ordinary reconstruction: six views, 57 K tokens
        _of_config("mid forward", "forward", 2),
        # its training step
        _of_config("mid train", "train", 5),
        # volume blocks with a variable number of active tokens (up to 8 x 64), the window over the query's own
        # spatial block, grouped heads: training on active voxels only, 21 K token slots
        _case("ragged blocks train", "train", 237 * 64, 4, 40, 8, 64, 20, 512, "ellipsoids", h_kv=2, k_vol=8,
              window_mode=1, ragged=True),
        # twelve views and a dense surface, 180 K tokens: clustered routing
        _of_config("large forward", "forward", 3),
        # the largest inference on one GPU: 428 K tokens, d = 128, near and far views
        _of_config("extreme forward", "forward", 4),
        # one layer of a training step at that size
        _of_config("extreme train", "train", 4),
        # the paper's head shape (32 heads of 32 channels on 2 key/value heads, gates per channel, rows of 80 blocks)
        _of_config("paper heads forward", "forward", 6),
        # the same in training
        _of_config("paper heads train", "train", 6),
        # the paper's routing rules evaluated for every token of a mid-sized scene, e.g. to vote on block lists
        _case("routing per token", "tokens", 32768, 6, 64, 1, 64, 32, 512, "ellipsoids", k_vol=8),
    ]


def _config(case, seed):
    return I.NSAConfig("case", case["n_obj"], case["n_views"], case["grid"], case["heads"], case["d"], case["topk"],
                       case["window"], case["points"], case["near_views"], seed, case["h_kv"], case["gate_channels"])


def _pairs(case):
    """Attended (query, key) pairs of one head; with ragged blocks about a tenth of the slots are padding, which this
    counts, as the kernels' callers cannot leave their rows out either."""
    c = _config(case, 0)
    n_tiles, nb_obj = c.n_tiles, c.nb_obj
    if case["k_vol"]:
        k_img = min(case["topk"] - case["k_vol"], n_tiles, c.n_views * min(4, c.tiles_per_view))
        entries = c.nb * (min(case["k_vol"], nb_obj) + k_img)
    else:
        entries = nb_obj * min(c.topk, n_tiles) + n_tiles * min(c.topk, nb_obj)
    # ragged: spatial blocks of 1 .. 8 object blocks; otherwise one pooled pair per block
    n_pool = (nb_obj * 2 / 9 + n_tiles) if case["ragged"] else c.nb
    if case["window_mode"] == 0:
        win = c.window_pairs()
    elif case["ragged"]:
        win = c.n_obj * 64 * (17 / 3) + c.n_img * 64   # E[size^2] / E[size] of 1 .. 8
    else:
        win = c.n * 64
    return c.n * n_pool + 64 * 64 * entries + win


def _cost(case):
    """Rough relative time: below d = 128 the softmax arithmetic, not the contractions, sets the pace."""
    if case["kind"] == "tokens":
        return 0
    return _pairs(case) * case["heads"] * (32 + case["d"]) * (4.5 if case["kind"] == "train" else 1.0)


def _memory(case):
    c = _config(case, 0)
    rows = 2 * c.n * c.d * (c.heads + c.kv_heads)
    gates = 12 * c.n * c.heads * (c.d if c.gate_channels else 1)
    return rows * (12 if case["kind"] == "train" else 4) + gates * (2 if case["kind"] == "train" else 1)


def draw(rng: random.Random):
    largest = max(listed(), key=_cost)
    while True:
        kind = rng.choices(KIND, (9, 9, 2))[0]
        n_obj = 64 * max(8, round(8 * 2 ** rng.uniform(0, 9)))           # 512 .. 262144
        n_views = max(1, round(2 ** rng.uniform(0, 4.17)))                # 1 .. 18
        grid = 8 * rng.randint(2, 12)                                     # 16 .. 96
        d = rng.choice((32, 64, 128))
        heads = rng.choice((1, 2, 3, 4, 6, 8, 12, 16, 32))
        h_kv = heads if rng.random() < 0.6 else rng.choice([h for h in range(1, heads + 1) if heads % h == 0])
        topk = rng.choice((rng.randint(3, 16), rng.randint(9, 40), rng.randint(33, 80)))
        four_rule = kind == "tokens" or rng.random() < 0.35
        ragged = kind != "tokens" and rng.random() < 0.2
        window_mode = 1 if rng.random() < (0.6 if ragged else 0.1) else 0
        case = _case("", kind, n_obj, n_views, grid, heads, d, topk, 2 * round(2 ** rng.uniform(5, 9)),
                     rng.choice(("uniform", "ellipsoids")), rng.choice((0, 0, 1)), h_kv, rng.random() < 0.25,
                     max(1, topk // 4) if four_rule else 0, window_mode, ragged, rng.random() < 0.2)
        del case["name"]
        if kind == "tokens" and n_obj + n_views * grid * grid > 80000:
            continue
        if _cost(case) <= 0.5 * _cost(largest) and _memory(case) <= 20e9:
            return case


def _ragged_blocks(cfg, seed):
    """Spatial blocks of 1 .. 8 consecutive object blocks, each with a partly filled last block; an image tile is a
    spatial block of its own.  The sizes of the spatial blocks belong to the case, their fill to the seed.
    (active tokens per 64-slot block, group offsets)"""
    layout, rng = np.random.default_rng(cfg.nb_obj), np.random.default_rng(seed)
    sizes = []
    while sum(sizes) < cfg.nb_obj:
        sizes.append(int(min(layout.integers(1, 9), cfg.nb_obj - sum(sizes))))
    ends = np.concatenate([np.cumsum(sizes), cfg.nb_obj + 1 + np.arange(cfg.n_tiles)])
    counts = np.full(cfg.nb, 64, dtype=np.int32)
    counts[ends[:len(sizes)] - 1] = rng.integers(8, 65, size=len(sizes))
    return counts, np.concatenate([[0], ends]).astype(np.int32)


def prepare(case, seed):
    cfg = _config(case, 1000 + seed)
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    train = case["kind"] == "train"

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=dev, dtype=torch.bfloat16)

    def like(t):
        return torch.empty_like(t)

    cams = I.make_cameras(cfg)
    s = {"case": case, "pos": torch.from_numpy(I.make_points(cfg)).to(dev), "cams": torch.from_numpy(cams).to(dev)}
    counts = groups = None
    if case["ragged"]:
        counts, groups = (torch.from_numpy(a).to(dev) for a in _ragged_blocks(cfg, seed))
    p = B.make_params(cfg.n_obj, cfg.n_views, cfg.grid, cfg.heads, cfg.d, cfg.topk, cfg.window, h_kv=cfg.kv_heads,
                      gate_channels=cfg.gate_channels, window_mode=case["window_mode"], block_count=counts,
                      group_offsets=groups)
    p.kv_packed = 0 if case["two_pass"] else 1
    s["p"] = p
    rows = cfg.n if case["kind"] == "tokens" else cfg.nb
    s["idx"] = torch.empty((rows, cfg.topk), dtype=torch.int32, device=dev)
    if case["k_vol"]:
        k_vol, k_img = case["k_vol"], case["topk"] - case["k_vol"]
        s["rules"] = B.lsrm_route3d_params(4, k_vol, k_img, k_vol, k_img, 1 if case["kind"] == "tokens" else 0)
        s["pos_img"] = torch.from_numpy(I.make_points_img(cfg, cams)).to(dev)
        s["ws_route"] = B.alloc_workspace(p, B.LSRM_WS_ROUTE_3D)
    else:
        s["ws_route"] = B.alloc_workspace(p, B.LSRM_WS_ROUTE)
    if case["kind"] == "tokens":
        s["dist2"] = torch.empty((rows, cfg.topk), dtype=torch.float32, device=dev)
        return s
    s["q"] = normal(cfg.n, cfg.heads, cfg.d)
    s["k"], s["v"] = normal(cfg.n, cfg.kv_heads, cfg.d), normal(cfg.n, cfg.kv_heads, cfg.d)
    g_shape = (cfg.n, 3, cfg.heads, cfg.d) if cfg.gate_channels else (cfg.n, cfg.heads, 3)
    s["gates"] = torch.randn(g_shape, generator=gen, device=dev).sigmoid_()
    pairs = cfg.nb if groups is None else groups.numel() - 1
    s["kc"] = torch.empty((pairs, cfg.kv_heads, cfg.d), dtype=torch.bfloat16, device=dev)
    s["vc"] = like(s["kc"])
    s["out"] = like(s["q"])
    s["ws"] = B.alloc_workspace(p, B.LSRM_WS_FORWARD)
    s["lse"] = s["branches"] = None
    if train:
        s["lse"] = torch.empty((3, cfg.n, cfg.heads), dtype=torch.float32, device=dev)
        s["branches"] = torch.empty((3, cfg.n, cfg.heads, cfg.d), dtype=torch.bfloat16, device=dev)
        s["dout"] = normal(cfg.n, cfg.heads, cfg.d)
        s["dq"], s["dk"], s["dv"] = like(s["q"]), like(s["k"]), like(s["v"])
        s["ws_back"] = B.alloc_workspace(p, B.LSRM_WS_BACKWARD)
    return s


def run(s):
    p, case = s["p"], s["case"]
    if case["k_vol"]:
        B.lsrm_route_blocks_3d(p, s["rules"], s["pos"], s["pos_img"], s["cams"], s["idx"], s.get("dist2"), s["ws_route"])
    else:
        B.lsrm_route_blocks(p, s["pos"], s["cams"], s["idx"], None, s["ws_route"])
    if case["kind"] == "tokens":
        return s["idx"], s["dist2"]
    if case["two_pass"]:
        B.lsrm_nsa_compress(p, s["k"], s["v"], s["kc"], s["vc"])
    else:
        B.lsrm_nsa_compress_pack(p, s["k"], s["v"], s["kc"], s["vc"], s["ws"])
    B.lsrm_nsa_forward(p, s["q"], s["k"], s["v"], s["kc"], s["vc"], s["idx"], s["gates"], s["out"], s["lse"],
                       s["branches"], s["ws"])
    if case["kind"] == "forward":
        return s["idx"], s["kc"], s["vc"], s["out"]
    B.lsrm_nsa_backward(p, s["q"], s["k"], s["v"], s["kc"], s["vc"], s["idx"], s["gates"], s["lse"], s["branches"],
                        s["dout"], s["dq"], s["dk"], s["dv"], s["ws_back"])
    return s["idx"], s["kc"], s["vc"], s["out"], s["lse"], s["branches"], s["dq"], s["dk"], s["dv"]


def work(case):
    """Inputs read once, outputs written once; floating-point operations of the attended pairs (two contractions
    forward, five backward) or, for the routing, of the distances that have to be looked at."""
    c = _config(case, 0)
    geometry = 12 * c.n_obj + 64 * c.n_views + (12 * c.n_img if case["k_vol"] else 0)
    if case["kind"] == "tokens":
        # a volume query and an image query alike: every volume centre, every tile centre, the points of 4 tiles a view
        per_row = 8 * c.nb_obj + 5 * c.n_tiles + 8 * 64 * c.n_views * min(4, c.tiles_per_view)
        return {"bytes": geometry + 8 * c.n * c.topk, "flops": float(c.n) * per_row}
    q_bytes, kv_bytes = 2 * c.n * c.heads * c.d, 2 * c.n * c.kv_heads * c.d
    pool = 2 * 2 * c.nb * c.kv_heads * c.d
    gates = 12 * c.n * c.heads * (c.d if c.gate_channels else 1)
    total = geometry + 4 * c.nb * c.topk + 2 * q_bytes + 2 * kv_bytes + gates + pool
    flops = 4.0 * c.d * c.heads * _pairs(case)
    if case["kind"] == "train":
        # the saved results, the incoming gradient and the three gradients
        total += 12 * c.n * c.heads + 3 * q_bytes + 2 * q_bytes + 2 * kv_bytes
        flops *= 3.5
    return {"bytes": float(total), "flops": flops}


def tolerance(case):
    """Routing tables are whole numbers and the same bit for bit, squared distances too.  Attention and its gradients
    are bf16 with bf16 probabilities between the contractions: measured against the float64 formulation of the layer
    they are 2.3e-3 to 2.6e-3 off in the 2-norm and up to about 0.03 of the root mean square in a single element."""
    if case["kind"] == "tokens":
        return "exact"
    return {"rel": 1e-2, "max": 0.15}
