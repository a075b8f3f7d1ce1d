"""The attention passes of calls with few rows, whose keys are split over the wavefronts of a workgroup: at the ends of
its groups of 32 rows and units of 32 keys, against the oracle, and against the general kernel, which takes
the same heads once there are many of them."""
import numpy as np
import pytest
import torch

import paper_2502_01776_amd as S
from oracle import svg_oracle as O
from workloads import get_config, make_plain_qkv
from helpers import (f64, gpu_fp8_quantize, gpu_profile, gpu_layer, gpu_layer_in_place, gpu_layer_kv2, assert_attn_close, assert_fp8_attn_close,
                     device_tile_lists, labels_match,
                     takes_split_form, DENSE, GATHER, SPARSE)

pytestmark = pytest.mark.gpu


def setup(H, D, F, P, T, **kw):
    cfg = dict(get_config("mid64"), B=1, H=H, D=D, F=F, P=P, T=T, w_s=1, w_t=max(1, P // 5), spatial_heads=[0], **kw)
    cfg["N"] = F * P + T
    return cfg, S.shape_from_config(cfg), O.Geometry.from_config(cfg)


def run(form, sh, q, k, v, lab):
    if form == "dense":
        o = torch.full_like(q, float("nan"))
        S.svg_dense_attn_fwd(sh, q, k, v, o)
        torch.cuda.synchronize()
        return o
    if form == "fp8":
        bufs, o = gpu_fp8_quantize(sh, q, k, v, lab), torch.full_like(q, float("nan"))
        S.svg_sparse_attn_fp8_fwd(sh, *bufs, o, lab, *device_tile_lists(sh))
        torch.cuda.synchronize()
        return o
    if form == "gather":
        return gpu_layer_in_place(sh, q, k, v, lab)[0]
    return gpu_layer_kv2(sh, q, k, v, lab, flags=S.SVG_ATTN_ELEMENT_MASK if form == "exact" else 0)[0]


@pytest.mark.parametrize("F, P, T, sink", [(1, 1, 0, 0), (1, 31, 0, 1), (3, 11, 0, 0), (2, 15, 3, 1), (5, 25, 3, 0), (4, 37, 45, 1)])
@pytest.mark.parametrize("form, blocks", [("dense", (128, 64)), ("sparse", (128, 64)), ("sparse", (32, 32)), ("exact", (128, 64)),
                                          ("exact", (32, 32)), ("gather", (128, 64))])
@pytest.mark.parametrize("D", [64, 128])
def test_few_rows_against_the_oracle_and_the_general_kernel(form, blocks, D, F, P, T, sink):
    cfg, sh, g = setup(2, D, F, P, T, sink_first_frame=sink, text_first=P % 2, block_m=blocks[0], block_n=blocks[1])
    groups = -(-g.N // 32)
    many = (1024 // groups + 2) // 2 * 2      # more workgroups than the split form takes
    assert 2 * groups <= 416 and many * groups > 640
    q, k, v = make_plain_qkv(1, 2, g.N, D, seed=P)
    k = (k.float() * torch.linspace(0.2, 3.0, g.N)[None, None, :, None]).bfloat16()
    lab = torch.tensor([0, 1], dtype=torch.uint8)
    few = run(form, sh, q.cuda(), k.cuda(), v.cuda(), lab.cuda())
    rep = lambda x: x.repeat(1, many // 2, 1, 1).cuda()
    general = run(form, setup(many, D, F, P, T, sink_first_frame=sink, text_first=P % 2, block_m=blocks[0], block_n=blocks[1])[1],
                  rep(q), rep(k), rep(v), lab.repeat(many // 2).cuda())
    for h in (0, 1):
        qh, kh, vh = f64(q)[0, h], f64(k)[0, h], f64(v)[0, h]
        if form == "dense":
            ref = O.dense_attention_head(qh, kh, vh, g)
        elif form == "exact":
            ref = O.masked_attention(qh, kh, vh, (O.temporal_mask if h else O.spatial_mask)(g), g.scale)
        else:
            ref = O.svg_attention_layer(f64(q), f64(k), f64(v), np.array([[0, 1]]), g)[0, h]
        assert_attn_close(few[0, h], ref, f"{form} head {h}")
        assert_attn_close(general[0, many - 2 + h], ref, f"{form} head {h}, general kernel")


@pytest.mark.parametrize("F, P, t", [(5, 9, 1), (5, 9, 32), (5, 40, 33), (3, 100, 256), (3, 100, 257), (61, 3, 40), (62, 3, 40), (1, 1, 5)])
@pytest.mark.parametrize("D, blocks", [(64, (128, 64)), (128, (128, 64)), (64, (32, 32))])
def test_profiling_with_few_rows(F, P, t, D, blocks):
    """t: groups of rows with and without an order, sorted by the workgroups or before them; F: one run of keys per frame in a
    lane's hand, and one frame more than there are lanes for (the general kernel)."""
    cfg, sh, g = setup(2, D, F, P, 7, sink_first_frame=F % 2, text_first=P % 2, block_m=blocks[0], block_n=blocks[1])
    q, k, v = make_plain_qkv(1, 2, g.N, D, seed=t)
    rows = np.random.default_rng(t).integers(0, g.N, t).astype(np.int32)
    labels, mse = gpu_profile(sh, q.cuda(), k.cuda(), v.cuda(), rows)
    omse, olab = O.profile_heads(f64(q), f64(k), f64(v), rows, g)
    # the bounds of the other profiling tests: bf16 rounding of the weights under every measured error
    assert np.allclose(mse.cpu().numpy().reshape(omse.shape), omse, rtol=0.05, atol=2e-5)
    assert labels_match(labels, omse, olab)


@pytest.mark.parametrize("F, P, T, sink", [(1, 1, 0, 0), (1, 31, 0, 1), (3, 43, 0, 0), (2, 15, 3, 1), (9, 75, 30, 0), (7, 97, 45, 1)])
def test_fp8_with_few_rows(F, P, T, sink):
    """Lists of one to twelve tiles over four wavefronts, a row of the general kernel beside it."""
    cfg, sh, g = setup(2, 128, F, P, T, sink_first_frame=sink, text_first=P % 2, block_m=128, block_n=64)
    groups = -(-g.N // 32)
    many = (1024 // groups + 2) // 2 * 2
    assert 2 * groups <= 600 < many * groups
    q, k, v = make_plain_qkv(1, 2, g.N, 128, seed=P)
    k = (k.float() * torch.linspace(0.2, 3.0, g.N)[None, None, :, None]).bfloat16()
    lab = torch.tensor([0, 1], dtype=torch.uint8)

    def layer(H):
        shape = setup(H, 128, F, P, T, sink_first_frame=sink, text_first=P % 2, block_m=128, block_n=64)[1]
        x = [t.repeat(1, H // 2, 1, 1).cuda() for t in (q, k, v)]
        labels = lab.repeat(H // 2).cuda()
        bufs = gpu_fp8_quantize(shape, *x, labels)
        o = torch.full_like(x[0], float("nan"))
        S.svg_sparse_attn_fp8_fwd(shape, *bufs, o, labels, *device_tile_lists(shape))
        torch.cuda.synchronize()
        return o[0, -2:]

    deq = [np.stack([O.fp8_dequantize(*O.fp8_quantize_head(f64(x)[0, h])) for h in (0, 1)])[None] for x in (q, k, v)]
    ref = O.svg_attention_layer(*deq, np.array([[0, 1]]), g)
    few, general = layer(2), layer(many)
    for h in (0, 1):
        for o, what in ((few, "few rows"), (general, "general kernel")):
            assert_fp8_attn_close(o[h], ref[0, h], float(np.abs(deq[2][0, h]).max()), f"{what}, head {h}")


@pytest.mark.parametrize("text_first, T, heads", [(0, 90, 2), (1, 90, 2), (1, 257, 2), (0, 90, 40)])
@pytest.mark.parametrize("form, D", [("sparse", 64), ("exact", 64), ("gather", 64), ("sparse", 128), ("exact", 128), ("gather", 128), ("fp8", 128)])
def test_text_rows_split_in_the_general_kernel(form, D, text_first, T, heads):
    """Query tiles with text rows, whose lists are many times longer than the others': taken in four parts of 32 rows where
    they would be the whole time of the pass (two heads), whole where they would not (forty)."""
    F, P = 5, 2100
    cfg, sh, g = setup(heads, D, F, P, T, text_first=text_first, block_m=128, block_n=64)
    cfg.update(w_s=0, w_t=40)
    sh, g = S.shape_from_config(cfg), O.Geometry.from_config(cfg)
    nq, nk = S.svg_tile_counts(sh)
    csr = [S.svg_tile_list_build(sh, p) for p in (0, 1)]
    heavy = [a for a in range(nq) if min(g.N, (a + 1) * 128) > g.off + F * P or a * 128 < g.off]
    light = sum(heads // 2 * (int(rp[-1]) - len(heavy) * nk) for rp, _ in csr)
    slots = 768 if D == 64 else 512
    assert heads * -(-g.N // 32) > 640 and (12 * nk * slots > 25 * (light + 4 * heads * len(heavy) * nk)) == (heads == 2)
    q, k, v = make_plain_qkv(1, 2, g.N, D, seed=T)
    k = (k.float() * torch.linspace(0.2, 3.0, g.N)[None, None, :, None]).bfloat16()
    rep = lambda x: x.repeat(1, heads // 2, 1, 1).cuda()
    o = run(form, sh, rep(q), rep(k), rep(v), torch.tensor([0, 1] * (heads // 2), dtype=torch.uint8).cuda())
    in_order = np.empty(g.N, np.int64)
    in_order[O.layout_perm(g)] = np.arange(g.N)
    fp8 = lambda x: O.fp8_dequantize(*O.fp8_quantize_head(x)) if form == "fp8" else x      # the products' own inputs
    for h in (0, 1):
        qh, kh, vh = (fp8(f64(x)[0, h]) for x in (q, k, v))
        token = in_order if h else np.arange(g.N)
        rp, ci = csr[h]
        for a in heavy + [heavy[-1] - 1 if heavy[-1] == nq - 1 else heavy[-1] + 1, nq // 2]:
            rows = slice(a * 128, min(g.N, (a + 1) * 128))
            cols = np.concatenate([np.arange(b * 64, min(g.N, (b + 1) * 64)) for b in ci[rp[a]:rp[a + 1]]])
            qr, kr, vr = qh[token[rows]], kh[token[cols]], vh[token[cols]]
            keep = np.ones((len(qr), len(cols)), bool)
            if form == "exact":
                keep = (O.temporal_mask if h else O.spatial_mask)(g, token[rows])[:, token[cols]]
            ref = O.masked_attention(qr, kr, vr, keep, g.scale)
            got, what = o[0, heads - 2 + h][torch.from_numpy(token[rows]).cuda()], f"{form} head {h}, tile {a}"
            if form == "fp8":
                assert_fp8_attn_close(got, ref, float(np.abs(vh).max()), what)
            else:
                assert_attn_close(got, ref, what)


def test_more_text_tiles_than_a_launch_has_parts_for():
    """2^22 heads of one video and one text token: one workgroup per query tile fits a launch, four do not."""
    heads = 2 ** 22
    cfg, sh, g = setup(heads, 64, 1, 1, 1, block_m=128, block_n=64)
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn(1, heads, 2, 64, generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    lab = torch.zeros(heads, dtype=torch.uint8, device="cuda")
    o = torch.full_like(q, float("nan"))
    S.svg_sparse_attn_fwd(sh, q, k, v, o, lab, *device_tile_lists(sh))
    torch.cuda.synchronize()
    assert bool(torch.isfinite(o).all())
    for h in (0, 1, heads // 2 - 1, heads // 2, heads - 1):
        assert_attn_close(o[0, h], O.dense_attention_head(*[f64(x[0, h]) for x in (q, k, v)], g), f"head {h}")


@pytest.mark.parametrize("D, heads, F, P, T, w_t, parts", [(64, 52, 4, 108, 10, 10, False), (128, 36, 4, 146, 10, 20, False), (64, 26, 4, 336, 104, 30, False),
                                                           (128, 18, 4, 348, 42, 40, False), (64, 26, 9, 200, 30, 8, True), (128, 2, 5, 2100, 90, 40, True)])
def test_text_rows_of_short_sequences_are_taken_whole(D, heads, F, P, T, w_t, parts):
    """Below the line of the parts a text row has the bits of the dense kernel, which walks the same key tiles in the same
    order; taken in parts it has not."""
    cfg, sh, g = setup(heads, D, F, P, T, text_first=0, block_m=128, block_n=64)
    cfg.update(w_s=1, w_t=w_t)
    sh = S.shape_from_config(cfg)
    assert not takes_split_form(sh, SPARSE) and not takes_split_form(sh, DENSE)
    gen = torch.Generator(device="cuda").manual_seed(P)
    q, k, v = (torch.randn(1, heads, g.N, D, generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    lab = torch.tensor([0, 1] * (heads // 2), dtype=torch.uint8, device="cuda")
    o, d = run("sparse", sh, q, k, v, lab), run("dense", sh, q, k, v, lab)
    text = slice(F * P, g.N)
    assert torch.equal(o[0, ::2, text].view(torch.int16), d[0, ::2, text].view(torch.int16)) == (not parts)
    assert float((o[0, ::2, text].float() - d[0, ::2, text].float()).abs().max()) <= 2e-2


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("heads, P, T, w_t, split", [(2, 300, 40, 30, True), (2, 2100, 90, 40, False), (40, 300, 40, 30, False)])
def test_pipelines_agree_bit_for_bit(D, heads, P, T, w_t, split):
    """Layout passes, copies of the temporal heads' k and v, and gathering in place: in the split form, with text-row tiles taken
    in parts and with all tiles taken whole."""
    cfg, sh, g = setup(heads, D, 5, P, T, text_first=1, block_m=128, block_n=64)
    cfg["w_t"] = w_t
    sh = S.shape_from_config(cfg)
    assert takes_split_form(sh, SPARSE) == takes_split_form(sh, GATHER) == split
    gen = torch.Generator(device="cuda").manual_seed(P)
    q, k, v = (torch.randn(1, heads, g.N, D, generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    lab = torch.tensor([0, 1] * (heads // 2), dtype=torch.uint8, device="cuda")
    four = gpu_layer(sh, q, k, v, lab).view(torch.int16)
    assert torch.equal(four, gpu_layer_kv2(sh, q, k, v, lab)[0].view(torch.int16))
    assert torch.equal(four, gpu_layer_in_place(sh, q, k, v, lab)[0].view(torch.int16))
