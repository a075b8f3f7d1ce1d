"""The work a user of this library has it do, as cases that can be timed.

A case is one attention layer of a video diffusion transformer (or one of the passes around it),
called through the package's public entry points with everything resident on the GPU.  The shapes
are those of `workloads.CONFIGS`, one head shard of the largest of them, and one odd generic size.

`call` says which pipeline a case runs:
  layer      svg_profile_heads -> svg_layout_kv_temporal -> svg_sparse_attn_fwd_kv2
  in_place   svg_profile_heads -> svg_sparse_attn_fwd_ex with q, k, v, o all left in token order
  four_pass  svg_profile_heads -> svg_layout_fwd of q, k, v -> svg_sparse_attn_fwd -> svg_layout_inv
  fp8        svg_profile_heads -> svg_fp8_quantize -> svg_sparse_attn_fp8_fwd
  dense      svg_dense_attn_fwd (the warm-up steps of the method run dense)
  rope       svg_qk_norm_rope of q and of k, in front of the attention
"""
from __future__ import annotations

import math

import torch

import paper_2502_01776_amd as S
from workloads import CONFIGS, make_qkv, sample_rows

_GEOMETRY = ("B", "H", "F", "P", "T", "D", "text_first", "w_s", "w_t", "block_m", "block_n", "t")


def _named(name, config, call, **options):
    """A case of one of the named workloads; `spatial` is the share of heads planted spatial."""
    cfg = CONFIGS[config]
    case = {"name": name, "call": call, **{k: cfg[k] for k in _GEOMETRY}, "sigma": cfg["sigma"], "sink": 0,
            "exact": False, "norm": "none", "pairing": "interleaved",
            "spatial": len(cfg["spatial_heads"]) / cfg["H"]}
    case.update(options)
    return case


def listed():
    return [
        # the smallest layer: 272 tokens, 4 heads, 32 x 32 tiles; launches and latency are what counts
        _named("tiny_layer", "tiny", "layer"),
        # small ragged layers: a batch of two guidance branches at head dimension 64 ...
        _named("mid64_layer", "mid64", "layer"),
        # ... and the FP8 pipeline on a short clip at head dimension 128
        _named("mid128_fp8", "mid128", "fp8"),
        # an odd, ragged, mid-sized layer under the exact element masks with the first-frame sink
        {"name": "odd_exact_sink", "call": "layer", "B": 1, "H": 16, "F": 9, "P": 1001, "T": 77, "D": 128,
         "text_first": 1, "w_s": 1, "w_t": 33, "block_m": 128, "block_n": 64, "t": 91, "sigma": 1.0, "sink": 1,
         "exact": True, "norm": "none", "pairing": "interleaved", "spatial": 0.5},
        # one layer of the models the benchmark names, each in the pipeline it would run
        _named("cogvideox_v1_layer", "cogvideox_v1", "layer"),
        _named("wan21_14b_layer", "wan21_14b", "layer"),
        # the four separate layout passes, for callers that want whole permuted tensors
        _named("cogvideox_v15_four_pass", "cogvideox_v15", "four_pass"),
        # three of the 24 heads: what one GPU of eight holds, no second copy of k and v
        _named("hunyuan_shard_in_place", "hunyuan_skip85", "in_place", H=3, spatial=0.67),
        # the default workload of bench.py, in bf16 and with the sparse pass in FP8
        _named("hunyuan_skip85_layer", "hunyuan_skip85", "layer"),
        _named("hunyuan_skip85_fp8", "hunyuan_skip85", "fp8"),
        # a dense warm-up step
        _named("wan21_14b_dense", "wan21_14b", "dense"),
        # QK-norm + rotary embedding of q and k
        _named("hunyuan_qk_norm_rope", "hunyuan_skip85", "rope", norm="rms"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same pipelines with sizes of its own."""
    call = rng.choice(["layer", "layer", "layer", "in_place", "four_pass", "fp8", "dense", "rope"])
    D = 128 if call == "fp8" else rng.choice([64, 128])
    F = rng.randint(5, 33)
    P = _log_int(rng, 48, 3600)
    T = rng.choice([0, _log_int(rng, 8, 256)])
    H = _log_int(rng, 2, 48)
    # no more work than the largest listed case
    limit = 1.2e13 if call == "dense" else 2.0e13
    while 4.0 * (F * P + T) ** 2 * D * H * (1.0 if call == "dense" else 0.2) > limit:
        P = max(48, int(P * 0.85))
        H = max(2, H - 1)
    N = F * P + T
    B = 2 if N < 20000 and H <= 24 and rng.random() < 0.25 else 1
    small_tiles = N < 1500 and call in ("layer", "four_pass", "dense") and rng.random() < 0.5
    return {"call": call, "B": B, "H": H, "F": F, "P": P, "T": T, "D": D, "text_first": rng.randint(0, 1),
            "w_s": rng.randint(1, max(1, (F - 3) // 5)), "w_t": max(2, int(P * rng.uniform(0.01, 0.12))),
            "block_m": 32 if small_tiles else 128, "block_n": 32 if small_tiles else 64,
            "t": max(16, -(-N // 100)), "sigma": 1.0,
            "sink": 1 if call == "layer" and rng.random() < 0.25 else 0,
            "exact": call == "layer" and rng.random() < 0.25,
            "norm": rng.choice(["rms", "layer"]) if call == "rope" else "none",
            "pairing": rng.choice(["interleaved", "half"]) if call == "rope" else "interleaved",
            "spatial": rng.choice([0.4, 0.5, 0.6])}


def _spatial_heads(case):
    """The planted spatial heads of a batch entry, spread evenly over the heads."""
    s = case["spatial"]
    return [h for h in range(case["H"]) if math.floor((h + 1) * s + 1e-9) > math.floor(h * s + 1e-9)]


def _config(case):
    cfg = {k: case[k] for k in _GEOMETRY}
    cfg.update(N=case["F"] * case["P"] + case["T"], sigma=case["sigma"], sink_first_frame=case["sink"],
               spatial_heads=_spatial_heads(case))
    return cfg


def prepare(case, seed):
    """Activations of the layer in HBM, and what a program keeps per shape: tile lists, workspace, buffers."""
    cfg = _config(case)
    sh = S.shape_from_config(cfg)
    call = case["call"]
    q, k, v = make_qkv(cfg, seed=seed, device="cuda")
    st = {"call": call, "sh": sh, "q": q, "k": k, "v": v}
    if call == "rope":
        gen = torch.Generator(device="cuda").manual_seed(seed + 1)
        D, nv = case["D"], case["F"] * case["P"]
        st["weight"] = 1.0 + 0.1 * torch.randn(D, generator=gen, device="cuda")
        st["bias"] = 0.1 * torch.randn(D, generator=gen, device="cuda")
        freq = 1.0 / 10000.0 ** (torch.arange(D // 2, device="cuda", dtype=torch.float32) / (D // 2))
        theta = torch.arange(nv, device="cuda", dtype=torch.float32)[:, None] * freq[None, :]
        st["cos"], st["sin"] = torch.cos(theta).contiguous(), torch.sin(theta).contiguous()
        st["norm"] = S.SVG_NORM_RMS if case["norm"] == "rms" else S.SVG_NORM_LAYER
        st["pairing"] = S.SVG_ROPE_HALF if case["pairing"] == "half" else S.SVG_ROPE_INTERLEAVED
        st["yq"], st["yk"] = torch.empty_like(q), torch.empty_like(k)
        return st
    st["o"] = torch.empty_like(q)
    if call == "dense":
        return st
    rows = sample_rows(cfg, seed=seed)
    st["t"], st["rows"] = len(rows), torch.from_numpy(rows).cuda()
    st["lists"] = []
    for pattern in (S.SVG_HEAD_SPATIAL, S.SVG_HEAD_TEMPORAL):
        for a in S.svg_tile_list_build(sh, pattern):
            st["lists"].append(torch.from_numpy(a).cuda())
    st["ws_bytes"] = S.svg_workspace_bytes(sh, st["t"])
    st["ws"] = torch.empty(st["ws_bytes"], dtype=torch.uint8, device="cuda")
    st["labels"] = torch.zeros(sh.B * sh.H, dtype=torch.uint8, device="cuda")
    st["mse"] = torch.zeros(sh.B * sh.H, 2, dtype=torch.float32, device="cuda")
    st["flags"] = S.SVG_ATTN_ELEMENT_MASK if case["exact"] else 0
    if call in ("layer", "four_pass"):
        st["kt"], st["vt"] = torch.empty_like(k), torch.empty_like(v)
    if call == "four_pass":
        st["qt"], st["ot"] = torch.empty_like(q), torch.empty_like(q)
    if call == "fp8":
        st["f8"] = [torch.empty(S.svg_fp8_buffer_bytes(sh, w), dtype=torch.uint8, device="cuda")
                    for w in (S.SVG_FP8_Q, S.SVG_FP8_K, S.SVG_FP8_VT)]
        st["scales"] = torch.zeros(S.svg_fp8_buffer_bytes(sh, S.SVG_FP8_SCALES) // 4, dtype=torch.float32, device="cuda")
    return st


def run(st):
    sh, q, k, v, call = st["sh"], st["q"], st["k"], st["v"], st["call"]
    if call == "rope":
        for x, y in ((q, st["yq"]), (k, st["yk"])):
            S.svg_qk_norm_rope(sh, x, y, st["norm"], st["weight"], st["bias"], 1e-6, st["cos"], st["sin"], st["pairing"])
        return {"q": st["yq"], "k": st["yk"]}
    o = st["o"]
    if call == "dense":
        S.svg_dense_attn_fwd(sh, q, k, v, o)
        return {"o": o}
    labels, lists = st["labels"], st["lists"]
    S.svg_profile_heads(sh, q, k, v, st["rows"], st["t"], labels, st["mse"], st["ws"], st["ws_bytes"])
    if call == "layer":
        S.svg_layout_kv_temporal(sh, k, v, st["kt"], st["vt"], labels)
        S.svg_sparse_attn_fwd_kv2(sh, q, k, v, st["kt"], st["vt"], o, labels, *lists, flags=st["flags"])
    elif call == "in_place":
        S.svg_sparse_attn_fwd_ex(sh, q, k, v, o, labels, *lists,
                                 flags=S.SVG_ATTN_QO_TOKEN_ORDER | S.SVG_ATTN_KV_TOKEN_ORDER,
                                 workspace=st["ws"], workspace_bytes=st["ws_bytes"])
    elif call == "four_pass":
        for x, y in ((q, st["qt"]), (k, st["kt"]), (v, st["vt"])):
            S.svg_layout_fwd(sh, x, y, labels)
        S.svg_sparse_attn_fwd(sh, st["qt"], st["kt"], st["vt"], st["ot"], labels, *lists)
        S.svg_layout_inv(sh, st["ot"], o, labels)
    else:
        S.svg_fp8_quantize(sh, q, k, v, labels, *st["f8"], st["scales"])
        S.svg_sparse_attn_fp8_fwd(sh, *st["f8"], st["scales"], o, labels, *lists)
    return {"o": o, "labels": labels, "mse": st["mse"]}


def work(case):
    """Bytes: q, k, v read once, o written once (rope: q and k read and written, the tables once).
    Operations: both products over every element of the kept tiles, and of the sampled rows against all
    keys once (the two masked outputs of profiling are sums over parts of the same products)."""
    B, H, D = case["B"], case["H"], case["D"]
    N = case["F"] * case["P"] + case["T"]
    tensor = 2.0 * B * H * N * D
    if case["call"] == "rope":
        return {"bytes": 4 * tensor + 4.0 * case["F"] * case["P"] * D, "flops": 2.0 * B * H * N * D * 8}
    if case["call"] == "dense":
        return {"bytes": 4 * tensor, "flops": 4.0 * B * H * N * N * D}
    sh = S.shape_from_config(_config(case))
    n_spatial = len(_spatial_heads(case))
    tiles = 0.0
    for pattern, heads in ((S.SVG_HEAD_SPATIAL, n_spatial), (S.SVG_HEAD_TEMPORAL, H - n_spatial)):
        row_ptr, _ = S.svg_tile_list_build(sh, pattern)
        tiles += float(row_ptr[-1]) * heads * B
    # tiles at the ragged end count in full: at most one row and one column of them
    return {"bytes": 4 * tensor + 4.0 * case["t"],
            "flops": 4.0 * D * (tiles * case["block_m"] * case["block_n"] + float(B * H) * case["t"] * N)}


def tolerance(case):
    """Four times the distance of each path from the fp64 oracle over the same inputs (relative 2-norm
    0.0019-0.0022 for the attention outputs and below 0.0006 for the errors of profiling, largest 0.013;
    FP8, against the oracle over the same quantised tensors: 0.013 and 0.13).  QK-norm + rotation is
    fp32 arithmetic rounded once, so two orders of its sums differ by single roundings of the output."""
    if case["call"] == "rope":
        return {"rel": 0.001, "max": 0.01}
    if case["call"] == "fp8":
        return {"rel": 0.03, "max": 0.5}
    return {"rel": 0.008, "max": 0.05}
