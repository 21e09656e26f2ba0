"""The merge path as users of this library call it: workloads for timing and for comparing two builds.

Every case is one pass through the ctypes binding (`Sttm`), in one of three forms:

* "budget":  statistics -> threshold from a token budget -> quadtree -> temporal statistics -> threshold from the
             budget -> edges and roots -> gather / average (the paper's setting, thresholds found automatically);
* "fixed":   the same with thresholds the caller has (two calls, then the gather);
* "reduce":  the gather / average alone on cluster ids the caller already has, without a workspace
             (`sttm_reduce_noalloc`: serving loops, code under graph capture).

The videos follow the recipe of the package's own generator (`workloads.py`): each frame is a random quadtree of
blocks, a block has a vector of its own, a token is its block's vector plus noise that is fresh per token and frame, and
a block stays as it is from one frame to the next with some probability. Every block has a noise level of its own,
spread over a range: still background and busy regions side by side, so that the similarities spread over an interval
as they do in real videos and a budget's threshold falls between values that are well apart.
"""
import math

import numpy as np
import torch

from paper_2507_07990_amd import binding as lib
from paper_2507_07990_amd import workloads as wl

DEVICE = "cuda:0"
TYPES = {"f32": (lib.STTM_F32, torch.float32), "bf16": (lib.STTM_BF16, torch.bfloat16),
         "f16": (lib.STTM_F16, torch.float16)}

# What a case says unless it says something else. noise_lo / noise_hi: noise per channel relative to the block's own
# vector; persist (.. persist_hi, one draw per video): how likely a block stays as it is from frame to frame; cut_gap /
# cut_prob: scene cuts; kept: share of the tokens that remain (the budget, or about what fixed thresholds leave);
# values: the caller asks for the thresholds and the number of rows (and so waits for them); nodes: the gather gets the
# stage-1 partition.
DEFAULTS = dict(form="budget", B=1, root_grid=1, dtype="bf16", out="", noise_lo=0.1, noise_hi=1.0, persist=0.9,
                persist_hi=0.0, cut_gap=0.0, cut_prob=0.0, kept=0.5, tau_s=0.0, tau_t=0.0, cell_dots=1, match=0, order=0,
                positions=False, values=False, nodes=True)


def _case(name, **over):
    c = dict(DEFAULTS, **over)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest calls: a preview clip of small descriptors, and one image; launches and host work are all there is
        _case("tiny_clip_f32", form="fixed", T=8, H=8, W=8, D=64, dtype="f32", noise_lo=0.03, noise_hi=0.08, persist=0.7,
              tau_s=0.8, tau_t=0.8, kept=0.11),
        _case("one_image_f16", T=1, H=24, W=24, D=1152, dtype="f16", kept=0.4, order=1, values=True),
        # a minute at one frame per second into a 7B model, half of the tokens kept
        _case("short_clip", T=64, H=13, W=13, D=3584, persist=0.8),
        # the same at a vision encoder's own width, many scene cuts, 30 % kept
        _case("encoder_width", T=64, H=16, W=16, D=1152, persist=0.6, cut_prob=0.1, kept=0.3, cell_dots=2),
        # the headline workload: a long video at both budgets
        _case("long_video_half", T=512, H=13, W=13, D=3584, cut_gap=64.0),
        _case("long_video_third", T=512, H=13, W=13, D=3584, cut_gap=64.0, kept=0.3, cell_dots=2),
        # many videos at once, unpooled grids, thresholds set by hand
        _case("batched_unpooled", form="fixed", B=32, T=32, H=27, W=27, D=1152, noise_lo=0.05, noise_hi=0.3, persist=0.3,
              persist_hi=0.95, tau_s=0.9, tau_t=0.85, kept=0.24),
        # the paper's set-up (180 frames of 14 x 14 tokens, 4 x 4 roots) with everything a host model needs for its
        # position encoding: rows in the Z-shaped scan, position indices
        _case("paper_grid_positions", T=180, H=14, W=14, D=3584, cut_gap=64.0, root_grid=4, order=1, positions=True),
        # a 72B model's width on a dynamic-resolution encoder's non-square grid: the largest rows
        _case("wide_nonsquare", T=180, H=18, W=24, D=8192, cut_gap=64.0, kept=0.3, cell_dots=2),
        # full precision with odd sizes, every value handed back to the host
        _case("ragged_f32", T=96, H=11, W=19, D=1000, dtype="f32", cut_gap=32.0, values=True),
        # a batch of half-precision clips, fp32 rows out, most similar destination, gather without the partition
        _case("clip_batch_f16", form="fixed", B=6, T=25, H=15, W=20, D=1280, dtype="f16", out="f32", noise_lo=0.05,
              noise_hi=0.3, persist=0.6, tau_s=0.9, tau_t=0.8, match=2, kept=0.1, nodes=False),
        # the gather alone for a caller that may not allocate
        _case("gather_noalloc", form="reduce", T=64, H=13, W=13, D=3584, persist=0.8, kept=0.5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: from a handful of small frames to a gigabyte, odd sizes among them."""
    form = rng.choice(["budget", "budget", "budget", "fixed", "fixed", "reduce"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f16", "f32"])
    width = 4 if dtype == "f32" else 2
    B = rng.choice([1, 1, 1, 2, 3, 5, 8, 16])
    T = _log_int(rng, 1, 512)
    H, W = rng.randint(4, 32), rng.randint(4, 32)
    if rng.random() < 0.4:
        W = H
    D = 8 * _log_int(rng, 8, 1024)
    if rng.random() < 0.5:  # widths that models have
        D = max(64, D // 128 * 128)
    while B * T * H * W * D * width > 1.1e9 or (form == "reduce" and
                                                lib.sttm_reduce_noalloc_bytes(B, T, H, W, D, TYPES[dtype][0])
                                                > lib.sttm_reduce_noalloc_max_bytes()):
        if B > 1:
            B -= 1
        elif T > 2:
            T = (T + 1) // 2
        else:
            D = max(64, D // 16 * 8)
    c = dict(form=form, B=B, T=T, H=H, W=W, D=D, dtype=dtype, persist=round(rng.uniform(0.5, 0.95), 2),
             cut_gap=rng.choice([0.0, 24.0, 64.0]), order=rng.randint(0, 1), nodes=rng.random() < 0.8)
    c["out"] = rng.choice(["", "", "", "f32"])
    if form == "fixed":
        c.update(noise_lo=0.05, noise_hi=0.3, tau_s=rng.choice([0.85, 0.9]), tau_t=rng.choice([0.8, 0.85]), kept=0.1)
    else:
        c["kept"] = round(rng.uniform(0.1, 0.8), 2)
    if form != "reduce":
        c.update(root_grid=rng.choice([1, 1, 2, 4]), match=rng.choice([0, 0, 0, 1, 2]), values=rng.random() < 0.3,
                 positions=rng.random() < 0.3, cell_dots=2 if c["kept"] <= 0.35 else 1)
    return _case("", **c)


def _blocks(case, seed):
    """Which block every token belongs to, [B, T, H, W] numbers from 0 on: the generator's recipe, all videos at once."""
    B, T, H, W = (case[k] for k in ("B", "T", "H", "W"))
    rng = np.random.default_rng(seed)
    P = wl.pow2_ceil(max(H, W))
    top = P.bit_length() - 1
    persist = np.full((B, 1, 1), case["persist"])
    if case["persist_hi"]:
        persist = rng.uniform(case["persist"], case["persist_hi"], (B, 1, 1))
    cut = rng.random((B, T)) < case["cut_prob"]
    if case["cut_gap"]:
        cut |= rng.random((B, T)) < 1.0 / case["cut_gap"]
    cut[:, 0] = True
    rows, cols = np.arange(P)[:, None], np.arange(P)[None, :]
    video = np.arange(B)[:, None, None]
    level = np.full((B, P, P), top)                        # of the block that covers the cell
    number = np.zeros((B, P, P), dtype=np.int64)
    out = np.empty((B, T, H, W), dtype=np.int64)
    for t in range(T):
        chance = rng.random((B, P, P))                     # a block's own: the one at its top-left cell
        anew = chance[video, rows >> level << level, cols >> level << level] >= persist
        anew |= cut[:, t, None, None]
        grown = np.where(cut[:, t, None, None], top, level)
        for l in range(1, top + 1):                        # four siblings replaced at once: their parent is
            s = 1 << l
            all_new = anew.reshape(B, P // s, s, P // s, s).all(axis=(2, 4)).repeat(s, 1).repeat(s, 2)
            grown = np.where(all_new, np.maximum(grown, l), grown)
        for l in range(top, 0, -1):                        # a new block splits with probability one half, level by level
            split = (rng.random((B, P >> l, P >> l)) < 0.5).repeat(1 << l, 1).repeat(1 << l, 2)
            grown = np.where(anew & (grown == l) & split, l - 1, grown)
        level = np.where(anew, grown, level)
        own = ((t * B + video) * P + (rows >> level << level)) * P + (cols >> level << level)
        number = np.where(anew, own, number)
        out[:, t] = number[:, :H, :W]
    return out


def _features(case, seed):
    """[B, T, H, W, D] on the GPU, from the seed alone."""
    B, T, H, W, D = (case[k] for k in ("B", "T", "H", "W", "D"))
    ids = torch.from_numpy(_blocks(case, seed)).to(DEVICE).view(-1)
    names, ids = torch.unique(ids, return_inverse=True)
    blocks = names.numel()
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    base = torch.randn(blocks, D, device=DEVICE, generator=gen)
    lo, hi = case["noise_lo"], case["noise_hi"]
    noise = lo * (hi / lo) ** torch.rand(blocks, 1, device=DEVICE, generator=gen)
    x = torch.empty(B, T, H, W, D, dtype=TYPES[case["dtype"]][1], device=DEVICE)
    rows, step = x.view(-1, D), max(1, (1 << 24) // D)
    for i in range(0, rows.shape[0], step):
        at = ids[i:i + step]
        rows[i:i + step] = base[at] + noise[at] * torch.randn(at.numel(), D, device=DEVICE, generator=gen)
    return x


def prepare(case, seed):
    B, T, H, W, D = (case[k] for k in ("B", "T", "H", "W", "D"))
    N = B * T * H * W
    out = case["out"] or case["dtype"]
    if case["dtype"] == "f32" and not case["out"]:
        out = "f32"
    torch.cuda.set_device(0)
    s = {"case": case, "x": _features(case, seed), "dtype": TYPES[case["dtype"]][0], "out_dtype": TYPES[out][0]}
    ctx = lib.Sttm(0)
    ctx.sttm_set_match_mode(case["match"])
    ctx.sttm_set_output_order(case["order"])
    ctx.sttm_set_cell_dots(case["cell_dots"])
    ctx.ensure_workspace(B, T, H, W, D, s["dtype"], case["root_grid"])

    def ints(*shape, dtype=torch.int32):
        return torch.zeros(*shape, dtype=dtype, device=DEVICE)

    s.update(ctx=ctx, node_map=ints(N), node_level=ints(N, dtype=torch.uint8), cluster=ints(N),
             merged=torch.zeros(N, D, dtype=TYPES[out][1], device=DEVICE), counts=ints(N), out_ids=ints(N),
             offsets=ints(B + 1, dtype=torch.int64))
    if case["positions"]:
        s.update(survived=ints(N), reassigned=ints(N), root=ints(N, 4),
                 merged_pos=torch.zeros(N, dtype=torch.float32, device=DEVICE))
    if case["form"] == "reduce":                           # the caller's cluster ids: those of a budget pass
        _budget(s)
    return s


def _budget(s):
    case, ctx, x = s["case"], s["ctx"], s["x"]
    shape = (s["dtype"],) + tuple(case[k] for k in ("B", "T", "H", "W", "D", "root_grid"))
    ctx.sttm_spatial_stats(x, *shape)
    a = ctx.sttm_budget_threshold(lib.STTM_STAGE_SPATIAL, case["kept"], want_tau=case["values"])
    ctx.sttm_spatial_quadtree(x, *shape, None, s["node_map"], s["node_level"])
    ctx.sttm_temporal_stats(x, s["node_map"], s["node_level"])
    b = ctx.sttm_budget_threshold(lib.STTM_STAGE_TEMPORAL, case["kept"], want_tau=case["values"])
    ctx.sttm_temporal_merge(x, s["node_map"], s["node_level"], None, s["cluster"])
    return a, b


def run(s):
    case, ctx, x = s["case"], s["ctx"], s["x"]
    B, T, H, W, D = (case[k] for k in ("B", "T", "H", "W", "D"))
    N = B * T * H * W
    rows = {"merged": s["merged"], "counts": s["counts"], "out_ids": s["out_ids"], "offsets": s["offsets"]}
    if case["form"] == "reduce":
        ctx.sttm_reduce_noalloc(x, s["dtype"], B, T, H, W, D, s["cluster"], s["out_dtype"], N, s["merged"], s["counts"],
                                s["out_ids"], s["offsets"])
        return rows
    taus = (None, None)
    if case["form"] == "budget":
        taus = _budget(s)
    else:
        ctx.sttm_spatial_quadtree(x, s["dtype"], B, T, H, W, D, case["root_grid"], [case["tau_s"]], s["node_map"],
                                  s["node_level"])
        ctx.sttm_temporal_merge(x, s["node_map"], s["node_level"], [case["tau_t"]], s["cluster"])
    node_map, node_level = (s["node_map"], s["node_level"]) if case["nodes"] else (None, None)
    n = ctx.sttm_reduce(x, s["cluster"], node_map, node_level, s["out_dtype"], N, s["merged"], s["counts"], s["out_ids"],
                        s["offsets"], want_n=case["values"])
    if case["positions"]:
        ctx.sttm_positions(s["cluster"], s["node_map"], s["node_level"], s["offsets"], N, s["survived"], s["reassigned"],
                           s["merged_pos"], s["root"])
        rows.update({k: s[k] for k in ("survived", "reassigned", "merged_pos", "root")})
    rows.update(node_map=s["node_map"], node_level=s["node_level"], cluster=s["cluster"])
    if case["values"]:
        rows.update(n=n, tau_s=taus[0], tau_t=taus[1])
    return rows


def work(case):
    """Every feature read once, every kept row written once, the cell tables written once; per channel of a token a
    squared norm, a product with its parent and one with the next frame, and the addition into its mean."""
    N = case["B"] * case["T"] * case["H"] * case["W"]
    width = {"f32": 4, "bf16": 2, "f16": 2}
    out = case["out"] or case["dtype"]
    kept = N * case["kept"]
    nbytes = N * case["D"] * width[case["dtype"]] + kept * (case["D"] * width[out] + 8)
    if case["form"] == "reduce":
        return {"bytes": nbytes + 4 * N, "flops": N * case["D"]}
    return {"bytes": nbytes + 9 * N, "flops": 7 * N * case["D"]}


def tolerance(case):
    """Whole numbers (maps, ids, counts, positions) are the same as long as no similarity changes sides of a
    threshold; what differs between correct implementations is the order of the fp32 sums, then the rounding of the
    rows to their type."""
    out = case["out"] or case["dtype"]
    return {"f32": {"rel": 1e-6, "max": 1e-5}, "bf16": {"rel": 2e-3, "max": 2e-2}, "f16": {"rel": 2e-4, "max": 2e-3}}[out]
