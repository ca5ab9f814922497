"""Performance cases of the mask feature extraction library and its consumers.

Every case is one call sequence that a mapping or serving program makes,
through the public functions of ``paper_2603_03935_amd``:

* ``embed``     masks of one frame or of a (ragged) batch -> unit embeddings
* ``pack``      boolean masks as a segmenter returns them -> packed mask bits
* ``query``     open-vocabulary retrieval over the instance embeddings
* ``heatmap``   dense similarity of text queries over one frame's patches
* ``geometry``  one RGB-D frame's segments: points, denoising, voxel sets and
                their overlap with the map's instances
* ``map``       view quality of a batch of observations and their fusion

``listed()`` names fixed sizes (those of the repository's workloads and of its
benchmark), ``draw(rng)`` gives other sizes of the same ranges.  Inputs are
synthetic and depend on the seed alone: overlapping objects rasterised on the
GPU, region-structured patch tokens with noise and a few outlier tokens, unit
embeddings, depth with range-scaled noise, outliers and missing readings.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2603_03935_amd as disc

DEV = "cuda"


def listed():
    return [
        # one small frame, a handful of masks: the latency of a single call
        {"name": "embed_f32_336x336_m8", "kind": "embed", "dtype": "f32", "frames": 1, "h": 336, "w": 336, "patch": 14,
         "masks": 8, "c": 1024, "e": 768, "ragged": False, "quality": False, "area": False, "distinct": True},
        # a live camera frame with its instance masks
        {"name": "embed_f32_480x640_m128", "kind": "embed", "dtype": "f32", "frames": 1, "h": 480, "w": 640, "patch": 16,
         "masks": 128, "c": 1024, "e": 768, "ragged": False, "quality": False, "area": False, "distinct": True},
        # three odd-sized camera frames with everything the mapping stage asks for (pooled features, mean
        # distinctiveness, area)
        {"name": "embed_bf16_ragged_quality", "kind": "embed", "dtype": "bf16", "frames": 3, "h": 719, "w": 1283,
         "patch": 14, "masks": 80, "c": 1024, "e": 768, "ragged": True, "quality": True, "area": False, "distinct": True},
        # offline processing of a recorded sequence, 64 frames a call
        {"name": "embed_bf16_64x480x640_m60", "kind": "embed", "dtype": "bf16", "frames": 64, "h": 480, "w": 640,
         "patch": 16, "masks": 60, "c": 1024, "e": 768, "ragged": False, "quality": False, "area": False,
         "distinct": True},
        # the largest batch: full-HD frames with everything the segmenter finds, quantised tokens
        {"name": "embed_f8_16x1080x1920_m500", "kind": "embed", "dtype": "f8", "frames": 16, "h": 1080, "w": 1920,
         "patch": 16, "masks": 500, "c": 1280, "e": 1024, "ragged": False, "quality": False, "area": False,
         "distinct": True},
        # a segmenter's boolean masks of one camera frame, packed before the embedding call
        {"name": "pack_bool_720x1280_m80", "kind": "pack", "bool": True, "m": 80, "h": 720, "w": 1280},
        # someone types a few queries over a whole map
        {"name": "query_bf16_5x20011", "kind": "query", "q": 5, "m": 20011, "e": 768, "k": 10, "text": "bf16"},
        # an evaluation's vocabulary against every instance
        {"name": "query_f32_1024x8000", "kind": "query", "q": 1024, "m": 8000, "e": 1024, "k": 10, "text": "f32"},
        # where in this frame do the queries light up
        {"name": "heatmap_bf16_480x640_q8", "kind": "heatmap", "dtype": "bf16", "gh": 30, "gw": 40, "patch": 16,
         "c": 1024, "e": 768, "q": 8, "text": "bf16"},
        # a subsampled small depth frame with few segments
        {"name": "geometry_240x320_s2", "kind": "geometry", "h": 240, "w": 320, "objects": 14, "stride": 2,
         "eps": 0.05, "min_pts": 6, "voxel": 0.05},
        # every pixel of a camera frame's segments
        {"name": "geometry_480x640_s1", "kind": "geometry", "h": 480, "w": 640, "objects": 40, "stride": 1,
         "eps": 0.03, "min_pts": 8, "voxel": 0.02},
        # a keyframe batch's observations scored and fused into the map
        {"name": "map_100k_into_20k", "kind": "map", "m": 100_000, "e": 768, "n_map": 20_000, "voxels": 4_000_000},
    ]


def _log_int(rng: random.Random, lo: int, hi: int) -> int:
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    kind = rng.choice(["embed", "embed", "embed", "pack", "query", "heatmap", "geometry", "map"])
    if kind == "embed":
        h, w = rng.randint(240, 1080), rng.randint(320, 1920)
        frames = _log_int(rng, 1, 16)
        masks = _log_int(rng, 1, 500)
        while frames * masks * h * w > 2_000_000_000:  # well below the largest listed batch
            masks = max(1, masks // 2)
        return {"kind": "embed", "dtype": rng.choice(["f32", "bf16", "f8"]), "frames": frames, "h": h, "w": w,
                "patch": rng.choice([14, 16]), "masks": masks, "c": rng.choice([768, 1024, 1280]),
                "e": rng.choice([512, 768, 1024]), "ragged": rng.random() < 0.5, "quality": rng.random() < 0.3,
                "area": rng.random() < 0.15, "distinct": rng.random() < 0.85}
    if kind == "pack":
        return {"kind": "pack", "bool": rng.random() < 0.5, "m": _log_int(rng, 1, 200), "h": rng.randint(240, 1080),
                "w": rng.randint(320, 1920)}
    if kind == "query":
        q, m = _log_int(rng, 1, 1024), _log_int(rng, 50, 20_000)
        while q * m > 8_000_000:
            q //= 2
        return {"kind": "query", "q": q, "m": m, "e": rng.choice([512, 768, 1024]), "k": _log_int(rng, 1, 50),
                "text": rng.choice(["f32", "bf16"])}
    if kind == "heatmap":
        patch = rng.choice([14, 16])
        return {"kind": "heatmap", "dtype": rng.choice(["f32", "bf16", "f8"]), "gh": -(-rng.randint(240, 1080) // patch),
                "gw": -(-rng.randint(320, 1920) // patch), "patch": patch, "c": rng.choice([768, 1024, 1280]),
                "e": rng.choice([512, 768, 1024]), "q": _log_int(rng, 1, 64), "text": rng.choice(["f32", "bf16"])}
    if kind == "geometry":
        h = rng.randint(240, 720)
        return {"kind": "geometry", "h": h, "w": rng.randint(h, h * 16 // 9), "objects": _log_int(rng, 4, 60),
                "stride": rng.choice([1, 2, 3]), "eps": rng.choice([0.03, 0.05]), "min_pts": rng.choice([4, 8, 12]),
                "voxel": rng.choice([0.02, 0.05])}
    return {"kind": "map", "m": _log_int(rng, 1000, 100_000), "e": rng.choice([512, 768, 1024]),
            "n_map": _log_int(rng, 500, 20_000), "voxels": _log_int(rng, 40_000, 4_000_000)}


# ---------------------------------------------------------------- inputs

def _gen(seed: int) -> torch.Generator:
    return torch.Generator(device=DEV).manual_seed(seed)


def _uniform(g, n, lo, hi):
    return lo + (hi - lo) * torch.rand(n, generator=g, device=DEV)


def _frame_shapes(case):
    """(h, w, masks) of every frame; a ragged batch varies all three."""
    rs = np.random.RandomState(case["masks"] * 1009 + case["frames"])
    shapes = []
    for i in range(case["frames"]):
        h, w, m = case["h"], case["w"], case["masks"]
        if case["ragged"]:
            h, w = h - (53 * i) % (h // 3), w - (97 * i) % (w // 3)
        if case["frames"] > 1:
            m = int(np.clip(rs.poisson(m), 1, 500))
        shapes.append((h, w, m))
    return shapes


def _masks_u8(g, m, h, w, chunk_px=120_000_000):
    """Bool [m][h][w], in chunks of masks: instance-like objects (half ellipses of aspect up to 4, half star-shaped
    outlines), their area log-uniform between 0.05 % and 25 % of the frame, centred anywhere in it."""
    area = torch.exp(_uniform(g, m, math.log(5e-4), math.log(0.25))) * (h * w)
    cy, cx, th = _uniform(g, m, 0.0, h), _uniform(g, m, 0.0, w), _uniform(g, m, 0.0, math.pi)
    aspect = _uniform(g, m, 1.0, 4.0)
    star = torch.arange(m, device=DEV) % 2 == 1
    aspect = torch.where(star, 1.0 + 0.25 * (aspect - 1.0), aspect)
    amp = torch.where(star, _uniform(g, m, 0.1, 0.45), torch.zeros(m, device=DEV))
    lobes = torch.floor(_uniform(g, m, 3.0, 9.0))
    a = torch.sqrt(area * aspect / math.pi) + 1.0
    b = a / aspect
    yy = torch.arange(h, device=DEV, dtype=torch.float32) + 0.5
    xx = torch.arange(w, device=DEV, dtype=torch.float32) + 0.5
    step = max(1, chunk_px // (h * w))
    for i in range(0, m, step):
        s = slice(i, min(i + step, m))
        col = lambda t: t[s, None, None]  # noqa: E731
        dy, dx = yy[None, :, None] - col(cy), xx[None, None, :] - col(cx)
        c, sn = torch.cos(col(th)), torch.sin(col(th))
        u, v = (dx * c + dy * sn) / col(a), (dy * c - dx * sn) / col(b)
        rim = 1.0 + col(amp) * torch.cos(col(lobes) * torch.atan2(v, u))
        yield u * u + v * v <= rim * rim


def _pack(u8):
    """Bool [m][h][w] -> int64 [m][h][ceil(w / 64)], bit i of word k = pixel 64 k + i."""
    m, h, w = u8.shape
    wq = (w + 63) // 64
    by = torch.nn.functional.pad(u8.to(torch.uint8), (0, wq * 64 - w)).view(m, h, wq * 8, 8)
    bit = torch.tensor([1, 2, 4, 8, 16, 32, 64, 128], dtype=torch.uint8, device=DEV)
    return (by * bit).sum(dim=-1, dtype=torch.uint8).view(torch.int64).contiguous()


def _token_values(g, gh, gw, c):
    """float32 [gh * gw][c]: the regions of an image share a feature, plus noise, plus a few high-norm outliers."""
    G = gh * gw
    y = torch.arange(G, device=DEV) // gw
    x = torch.arange(G, device=DEV) % gw
    regions = 12
    ry, rx = _uniform(g, regions, 0.0, gh), _uniform(g, regions, 0.0, gw)
    region = ((y[:, None] - ry) ** 2 + (x[:, None] - rx) ** 2).argmin(dim=1)
    phi = torch.randn(regions, c, generator=g, device=DEV)
    v = phi[region] + 0.5 * torch.randn(G, c, generator=g, device=DEV)
    out = torch.randint(0, G, (max(1, G // 100),), generator=g, device=DEV)
    v[out] *= 4.0
    return v


def _tokens(g, gh, gw, c, dtype):
    """(tokens [gh][gw][c] as the library takes them, per-token scales of FP8 tokens)."""
    v = _token_values(g, gh, gw, c)
    if dtype == "f32":
        return v.view(gh, gw, c), None
    if dtype == "bf16":
        return v.to(torch.bfloat16).view(gh, gw, c), None
    scale = v.abs().amax(dim=1) / 448.0
    codes = (v / scale[:, None]).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
    return codes.view(gh, gw, c), scale


def _projection(g, c, e, dtype):
    p = torch.randn(c, e, generator=g, device=DEV) / math.sqrt(c)
    return p if dtype == "f32" else p.to(torch.bfloat16)


def _unit(g, n, e):
    return torch.nn.functional.normalize(torch.randn(n, e, generator=g, device=DEV), dim=1)


def _texts(g, emb, q, dtype):
    """Unit text embeddings, each leaning towards some instance."""
    near = emb[torch.randint(0, emb.shape[0], (q,), generator=g, device=DEV)]
    t = torch.nn.functional.normalize(0.3 * near + _unit(g, q, emb.shape[1]), dim=1)
    return t if dtype == "f32" else t.to(torch.bfloat16)


def _depth_scene(case, seed):
    """Overlapping dome-shaped objects in front of a tilted plane: (depth [h][w], bool masks of the visible pixels
    [m][h][w], camera).  The image layout (outlines and missing readings) belongs to the case, the depths, their
    noise and the outliers to the seed."""
    h, w = case["h"], case["w"]
    g = _gen(seed)
    fixed = h * 4099 + w * 61 + case["objects"]
    r, rz = random.Random(fixed), random.Random(seed)
    yy = (torch.arange(h, device=DEV, dtype=torch.float32) + 0.5)[:, None]
    xx = (torch.arange(w, device=DEV, dtype=torch.float32) + 0.5)[None, :]
    depth = (4.5 + 0.5 * yy / h).expand(h, w).clone()
    label = torch.zeros(h, w, dtype=torch.int32, device=DEV)
    f = 525.0 * w / 640.0
    for k in range(1, case["objects"] + 1):
        cy, cx, th = r.uniform(0, h), r.uniform(0, w), r.uniform(0, math.pi)
        a = math.exp(r.uniform(math.log(0.02 * w), math.log(0.22 * w)))
        b, z0, bulge = a * r.uniform(0.35, 1.0), rz.uniform(0.8, 4.0), rz.uniform(0.0, 0.3)
        dy, dx = yy - cy, xx - cx
        u, v = dx * math.cos(th) + dy * math.sin(th), dy * math.cos(th) - dx * math.sin(th)
        r2 = (u / a) ** 2 + (v / b) ** 2
        inside = r2 <= 1.0
        label = torch.where(inside, torch.full_like(label, k), label)
        depth = torch.where(inside, z0 - bulge * (z0 * a / f) * (1.0 - r2), depth)
    depth = depth + 0.002 * depth ** 2 * torch.randn(h, w, generator=g, device=DEV)
    stray = torch.rand(h, w, generator=g, device=DEV) < 0.003
    depth = torch.where(stray, 0.3 + 5.7 * torch.rand(h, w, generator=g, device=DEV), depth)
    missing = torch.rand(h, w, generator=_gen(fixed), device=DEV) < 0.01
    depth = torch.where(missing, torch.zeros_like(depth), depth)
    seen = torch.bincount(label.view(-1), minlength=case["objects"] + 1)[1:]
    keep = (torch.nonzero(seen >= 64).view(-1) + 1).to(torch.int32)
    masks = label[None] == keep[:, None, None]
    c, s = math.cos(0.3), math.sin(0.3)
    cam = {"fx": f, "fy": f, "cx": w / 2.0 - 0.5, "cy": h / 2.0 - 0.5,
           "R": [[1.0, 0.0, 0.0], [0.0, c, -s], [0.0, s, c]], "t": [1.5, -0.4, 1.2], "depth_min": 0.1,
           "depth_max": 10.0}
    return depth.contiguous(), masks, cam


# ---------------------------------------------------------------- prepare and run

def _embed_inputs(case, seed):
    """Per frame (tokens, scale, bool mask chunks, h, w), then the projection."""
    for i, (h, w, m) in enumerate(_frame_shapes(case)):
        g = _gen(seed * 1000 + i)
        gh, gw = -(-h // case["patch"]), -(-w // case["patch"])
        tok, scale = _tokens(g, gh, gw, case["c"], case["dtype"])
        yield tok, scale, _masks_u8(g, m, h, w), h, w
    yield _projection(_gen(seed * 1000 + 999), case["c"], case["e"], case["dtype"])


def prepare(case, seed):
    kind = case["kind"]
    if kind == "embed":
        frames = []
        *inputs, proj = _embed_inputs(case, seed)
        for tok, scale, chunks, h, w in inputs:
            bits = torch.cat([_pack(c) for c in chunks])
            frames.append(disc.FrameInput(tok, bits, h, w, case["patch"], scale))
        opts = disc.make_options(spatial=disc.SPATIAL_AREA if case["area"] else disc.SPATIAL_EDT,
                                 distinct=int(case["distinct"]))
        # one buffer per output over the batch, a slice of it for every frame
        M = sum(f.m for f in frames)
        whole = {"out": torch.empty(M, case["e"], device=DEV), "status": torch.empty(M, dtype=torch.int32, device=DEV)}
        if case["quality"]:
            whole["pooled"] = torch.empty(M, case["c"], device=DEV)
            whole["dbar"] = torch.empty(M, device=DEV)
            whole["area"] = torch.empty(M, dtype=torch.int32, device=DEV)
        outs, at = [], 0
        for f in frames:
            outs.append(disc.FrameOutput(**{k: v[at:at + f.m] for k, v in whole.items()}))
            at += f.m
        return {"kind": kind, "frames": frames, "proj": proj, "outs": outs, "whole": whole, "opts": opts}
    if kind == "pack":
        u8 = torch.cat(list(_masks_u8(_gen(seed), case["m"], case["h"], case["w"])))
        return {"kind": kind, "u8": u8 if case["bool"] else u8.to(torch.uint8)}
    if kind == "query":
        g = _gen(seed)
        emb = _unit(g, case["m"], case["e"])
        return {"kind": kind, "emb": emb, "text": _texts(g, emb, case["q"], case["text"]), "k": case["k"]}
    if kind == "heatmap":
        g = _gen(seed)
        tok, scale = _tokens(g, case["gh"], case["gw"], case["c"], case["dtype"])
        proj = _projection(g, case["c"], case["e"], case["dtype"])
        text = _texts(g, _unit(g, 64, case["e"]), case["q"], case["text"])
        return {"kind": kind, "tok": tok, "scale": scale, "proj": proj, "text": text, "patch": case["patch"]}
    if kind == "geometry":
        depth, masks, cam = _depth_scene(case, seed)
        bits = _pack(masks)
        # the map: the instances as an earlier frame of the same scene (camera 3 cm away) left them
        cam0 = dict(cam, t=[1.53, -0.4, 1.18])
        pts, off = disc.backproject(depth, bits, case["h"], case["w"], cam0, 1)
        vox, voff, _ = disc.voxelize(pts, off, case["voxel"])
        m = bits.shape[0]
        i = torch.arange(m, device=DEV, dtype=torch.int32)
        pairs = torch.stack([i.repeat_interleave(m), i.repeat(m)], dim=1).contiguous()
        # where the program keeps the voxel lists of the frame's segments
        store = torch.zeros(case["h"] * case["w"], 3, dtype=torch.int32, device=DEV)
        return {"kind": kind, "case": case, "depth": depth, "bits": bits, "cam": cam, "map": (vox, voff), "pairs": pairs,
                "store": store}
    g = _gen(seed)
    m, n_map, nv = case["m"], case["n_map"], case["voxels"]
    emb = _unit(g, m, case["e"])
    cuts = torch.sort(torch.randint(0, nv + 1, (m - 1,), generator=g, device=DEV)).values.to(torch.int32)
    off = torch.cat([cuts.new_zeros(1), cuts, cuts.new_full((1,), nv)])
    return {"kind": kind, "emb": emb, "off": off, "rays": _unit(g, nv, 3), "normals": _unit(g, nv, 3),
            "g": torch.nn.functional.normalize(emb[: min(m, 64)].sum(dim=0), dim=0),
            "area": torch.randint(1, 480 * 640 // 4, (m,), generator=g, device=DEV).to(torch.int32),
            "dbar": _uniform(g, m, 0.2, 2.0), "ids": torch.randint(0, n_map, (m,), generator=g, device=DEV).to(torch.int32),
            "map_q0": _uniform(g, n_map, 0.0, 0.02), "map_q": torch.empty(n_map, device=DEV),
            "map_emb": torch.zeros(n_map, case["e"], device=DEV), "won": torch.empty(m, dtype=torch.int32, device=DEV)}


def run(state):
    kind = state["kind"]
    if kind == "embed":
        disc.embed_frames(state["frames"], state["proj"], outputs=state["outs"], options=state["opts"])
        return state["whole"]
    if kind == "pack":
        return disc.pack_masks(state["u8"])
    if kind == "query":
        return disc.query_topk(state["emb"], state["text"], state["k"])
    if kind == "heatmap":
        return disc.query_heatmap(state["tok"], state["proj"], state["text"], state["patch"], scale=state["scale"])
    if kind == "geometry":
        case = state["case"]
        pts, off = disc.backproject(state["depth"], state["bits"], case["h"], case["w"], state["cam"], case["stride"])
        keep = disc.dbscan_denoise(pts, off, case["eps"], case["min_pts"])
        vox, voff, status = disc.voxelize(pts, off, case["voxel"], keep=keep)
        shared = disc.voxel_overlap(vox, voff, *state["map"], state["pairs"])
        state["store"][: vox.shape[0]].copy_(vox)
        return {"points": pts, "offsets": off, "keep": keep, "voxels": state["store"], "voxel_offsets": voff,
                "status": status, "shared": shared}
    # the map a program holds before this batch (its qualities; the batch overwrites the rows it wins)
    state["map_q"].copy_(state["map_q0"])
    angle = disc.angle_score(state["rays"], state["normals"], state["off"])
    q, comp = disc.view_quality(state["area"], state["dbar"], state["emb"], state["g"], 480, 640, angle)
    won = disc.fuse(state["ids"], q, state["emb"], state["map_q"], state["map_emb"], won=state["won"])
    return {"angle": angle, "q": q, "comp": comp, "won": won, "map_q": state["map_q"], "map_emb": state["map_emb"]}


def work(case):
    kind = case["kind"]
    if kind == "embed":
        size = {"f32": 4, "bf16": 2, "f8": 1}[case["dtype"]]
        c, e = case["c"], case["e"]
        nbytes = c * e * (4 if case["dtype"] == "f32" else 2)
        flops = 0
        for h, w, m in _frame_shapes(case):
            G = -(-h // case["patch"]) * -(-w // case["patch"])
            nbytes += m * h * -(-w // 64) * 8 + G * c * size + m * e * 4
            flops += 2 * m * c * e + 2 * int(0.05 * m * G) * c
        return {"bytes": nbytes, "flops": flops}
    if kind == "pack":
        return {"bytes": case["m"] * case["h"] * (case["w"] + -(-case["w"] // 64) * 8), "flops": 0}
    if kind == "query":
        q, m, e = case["q"], case["m"], case["e"]
        return {"bytes": 4 * m * e + (4 if case["text"] == "f32" else 2) * q * e + 4 * q * m + 8 * q * case["k"],
                "flops": 2 * q * m * e}
    if kind == "heatmap":
        G, c, e, q = case["gh"] * case["gw"], case["c"], case["e"], case["q"]
        size = {"f32": 4, "bf16": 2, "f8": 1}[case["dtype"]]
        return {"bytes": G * c * size + c * e * (4 if case["dtype"] == "f32" else 2) + 4 * q * (e + G),
                "flops": 2 * G * e * (c + q)}
    if kind == "geometry":
        h, w, m = case["h"], case["w"], case["objects"]
        n = int(0.65 * h * w / case["stride"] ** 2)  # the objects cover about two thirds of the frame
        return {"bytes": 4 * h * w + m * h * -(-w // 64) * 8 + 16 * n + 12 * n // 4 + 12 * m * m, "flops": 30 * n}
    m, e = case["m"], case["e"]
    won = min(m, case["n_map"])
    return {"bytes": 24 * case["voxels"] + 4 * m * e + 44 * m + 8 * won * e + 12 * case["n_map"],
            "flops": 6 * case["voxels"] + 6 * m * e}


# ---------------------------------------------------------------- 64-bit values

def _edt_sq(mask):
    """Exact squared distance of every set pixel of bool [m][h][w] to the nearest unset one (the outside of the
    frame is unset), int32."""
    m, h, w = mask.shape
    x = torch.arange(w, device=DEV, dtype=torch.int32)
    left = x - torch.cummax(torch.where(mask, -1, x), dim=2).values
    right = torch.flip(torch.cummin(torch.flip(torch.where(mask, w, x), [2]), dim=2).values, [2]) - x
    g2 = torch.minimum(left, right).to(torch.int32) ** 2
    y = torch.arange(h, device=DEV, dtype=torch.int32)
    edge = torch.minimum(y + 1, h - y) ** 2
    e = torch.minimum(g2, edge[None, :, None])
    d = 1
    while d < h and d * d < int(e.max()):
        for _ in range(8):
            if d >= h:
                break
            e[:, d:] = torch.minimum(e[:, d:], g2[:, :-d] + d * d)
            e[:, :-d] = torch.minimum(e[:, :-d], g2[:, d:] + d * d)
            d += 1
    return e


def _patch_sums(v, patch):
    """float64 [m][h][w] -> [m][gh * gw], the sum over each patch."""
    m, h, w = v.shape
    gh, gw = -(-h // patch), -(-w // patch)
    v = torch.nn.functional.pad(v, (0, gw * patch - w, 0, gh * patch - h))
    return v.view(m, gh, patch, gw, patch).sum(dim=(2, 4)).view(m, gh * gw)


def _tokens64(tok, scale):
    G = tok.shape[0] * tok.shape[1]
    if scale is None:
        return tok.reshape(G, -1).double()
    return tok.view(torch.float8_e4m3fn).reshape(G, -1).float().double() * scale.double()[:, None]


def _residual_norm(f):
    return torch.linalg.vector_norm(f - f.mean(dim=0), dim=1)


def _exact_embed(case, seed):
    if sum(h * w * m for h, w, m in _frame_shapes(case)) > 1_300_000_000:
        return None
    *inputs, proj = _embed_inputs(case, seed)
    proj = proj.double()
    out, pooled, dbar = [], [], []
    for tok, scale, chunks, h, w in inputs:
        f = _tokens64(tok, scale)
        r = _residual_norm(f)
        D = r / (r.mean() + 1e-6)
        for mask in chunks:
            for part in mask.split(max(1, 20_000_000 // (h * w))):
                count = _patch_sums(part.double(), case["patch"])
                s = count if case["area"] else _patch_sums(_edt_sq(part).double().sqrt(), case["patch"])
                wt = s * r if case["distinct"] else s
                wt = torch.where(wt.sum(dim=1, keepdim=True) > 0, wt, s)
                F = (wt @ f) / wt.sum(dim=1, keepdim=True).clamp_min(1e-300)
                out.append(torch.nn.functional.normalize(F @ proj, dim=1))
                pooled.append(F)
                dbar.append((count @ D) / count.sum(dim=1).clamp_min(1.0))
    want = {"out": torch.cat(out), "status": None}
    if case["quality"]:
        want.update(pooled=torch.cat(pooled), dbar=torch.cat(dbar), area=None)
    return want


def exact(case, seed):
    kind = case["kind"]
    if kind == "embed":
        return _exact_embed(case, seed)
    if kind == "pack":
        return None
    if kind == "geometry":
        depth, masks, cam = _depth_scene(case, seed)
        # the camera's floats as the library receives them
        k = {n: float(np.float32(cam[n])) for n in ("fx", "fy", "cx", "cy")}
        ok = torch.isfinite(depth) & (depth >= cam["depth_min"]) & (depth <= cam["depth_max"])
        grid = torch.zeros_like(ok)
        grid[:: case["stride"], :: case["stride"]] = True
        at = torch.nonzero(masks & (ok & grid)[None])
        y, x = at[:, 1], at[:, 2]
        z = depth[y, x].double()
        p = torch.stack([(x - k["cx"]) * z / k["fx"], (y - k["cy"]) * z / k["fy"], z], dim=1)
        R = torch.tensor(cam["R"], device=DEV, dtype=torch.float32).double()
        t = torch.tensor(cam["t"], device=DEV, dtype=torch.float32).double()
        return {"points": p @ R.T + t, "offsets": None, "keep": None, "voxels": None, "voxel_offsets": None,
                "status": None, "shared": None}
    s = prepare(case, seed)
    if kind == "query":
        sim = (torch.nn.functional.normalize(s["text"].double(), dim=1)
               @ torch.nn.functional.normalize(s["emb"].double(), dim=1).T)
        return torch.topk(sim, min(case["k"], case["m"]), dim=1).values, None, sim
    if kind == "heatmap":
        f = _tokens64(s["tok"], s["scale"])
        r = _residual_norm(f)
        D = r / (r.mean() + 1e-6)
        y = torch.nn.functional.normalize(f @ s["proj"].double(), dim=1)
        heat = torch.nn.functional.normalize(s["text"].double(), dim=1) @ y.T * D
        return heat.view(-1, case["gh"], case["gw"])
    off = s["off"].long()
    score = (-(s["rays"].double() * s["normals"].double()).sum(dim=1)).clamp_min(0.0)
    total = torch.cat([score.new_zeros(1), score.cumsum(0)])
    n = off[1:] - off[:-1]
    angle = (total[off[1:]] - total[off[:-1]]) / n.clamp_min(1)
    size = (3.3 * s["area"].double() / (480 * 640)).clamp_max(1.0)
    e = s["emb"].double()
    sem = (torch.nn.functional.normalize(e, dim=1) @ torch.nn.functional.normalize(s["g"].double(), dim=0)).clamp(0.0, 1.0)
    dist = 0.5 + 0.5 * s["dbar"].double()
    return {"angle": angle, "q": size * angle * sem * dist, "comp": torch.stack([size, angle, sem, dist], dim=1),
            "won": None, "map_q": None, "map_emb": None}
