"""Kept-tile lists of every length at which the attention kernels change what they do: none, one and two
tiles, odd and even numbers, and the ends of the 64 entries that are fetched at a time; with and without a
ragged last key tile in them; in the form for few rows and, with more heads, in the general kernels."""
import numpy as np
import pytest
import torch

import paper_2502_01776_amd as S
from oracle import svg_oracle as O
from workloads import get_config, make_plain_qkv
from helpers import (f64, dev_i32, gpu_fp8_quantize, gpu_layer, gpu_layer_in_place, gpu_layer_kv2, assert_attn_close,
                     assert_fp8_attn_close, takes_split_form, takes_fp8_split_form, SPARSE, EXACT, GATHER)

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 2, 3, 4, 5, 62, 63, 64, 65, 66, 126, 127, 128, 129, 130, 131, 132]


def random_lists(nq, nk, last_tile, seed):
    """One list of every length for the first query tiles, empty ones for the others."""
    rng = np.random.default_rng(seed)
    lists = [np.zeros(0, np.int32)] * nq
    for i, n in enumerate(LENGTHS):
        cols = np.sort(rng.choice(nk, n, replace=False)).astype(np.int32)
        if last_tile and n:
            cols[-1] = nk - 1
        elif n and n < nk:
            cols = np.sort(rng.choice(nk - 1, n, replace=False)).astype(np.int32)
        lists[i] = cols
    return np.concatenate([[0], np.cumsum([len(c) for c in lists])]).astype(np.int32), np.concatenate(lists)


@pytest.mark.parametrize("last_tile", [False, True])
@pytest.mark.parametrize("D, fp8", [(64, False), (128, False), (128, True)])
@pytest.mark.parametrize("heads", [1, 3])
def test_list_lengths(D, fp8, last_tile, heads):
    cfg = dict(get_config("mid128"), B=1, H=heads, F=3, P=2812, T=0, D=D, spatial_heads=[0])
    cfg["N"] = cfg["F"] * cfg["P"]                      # 8436 = 131 * 64 + 52
    sh, g = S.shape_from_config(cfg), O.Geometry.from_config(cfg)
    nq, nk = S.svg_tile_counts(sh)
    assert nk == 132 and nq >= len(LENGTHS)
    assert (takes_fp8_split_form(sh) if fp8 else takes_split_form(sh, SPARSE)) == (heads == 1)
    rp, ci = random_lists(nq, nk, last_tile, D + last_tile)
    csr = [dev_i32(rp), dev_i32(ci), dev_i32(rp), dev_i32(ci)]
    # logits that grow along the sequence, so that the reference maximum of the softmax has to follow
    q, k, v = make_plain_qkv(1, 1, g.N, D, seed=D)
    k = (k.float() * torch.linspace(0.2, 3.0, g.N)[None, None, :, None]).bfloat16()
    qc, kc, vc = (x.repeat(1, heads, 1, 1).cuda() for x in (q, k, v))
    lab = torch.zeros(heads, dtype=torch.uint8, device="cuda")
    o = torch.full_like(qc, float("nan"))
    if fp8:
        bufs = gpu_fp8_quantize(sh, qc, kc, vc, lab)
        S.svg_sparse_attn_fp8_fwd(sh, *bufs, o, lab, *csr)
        qh, kh, vh = (O.fp8_dequantize(*O.fp8_quantize_head(f64(x)[0, 0])) for x in (q, k, v))
    else:
        S.svg_sparse_attn_fwd_ex(sh, qc, kc, vc, o, lab, *csr)
        qh, kh, vh = (f64(x)[0, 0] for x in (q, k, v))
    torch.cuda.synchronize()
    tiles = list(range(len(LENGTHS)))
    ref = O.sparse_attention_head(qh, kh, vh, rp.astype(np.int64), ci, g, q_tiles=[a for a in tiles if LENGTHS[a]])
    for a in tiles:
        rows = slice(a * g.block_m, min(g.N, (a + 1) * g.block_m))
        if LENGTHS[a] == 0:
            assert (o[0, :, rows] == 0).all()
        elif fp8:
            assert_fp8_attn_close(o[0, heads - 1, rows], ref[rows], float(np.abs(vh).max()), f"{LENGTHS[a]} tiles")
        else:
            assert_attn_close(o[0, heads - 1, rows], ref[rows], f"{LENGTHS[a]} tiles")


@pytest.mark.parametrize("last_tile", [False, True])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("form, blocks", [("gather", (128, 64)), ("exact", (128, 64)), ("exact", (32, 32)), ("plain", (32, 32))])
@pytest.mark.parametrize("copies", [1, 3])
def test_list_lengths_of_the_other_forms(form, blocks, D, last_tile, copies):
    """The forms with loops of their own: the gathering one (row numbers fetched a tile ahead of their rows), the one
    under element masks (one tile after the other) and the 32-row ones; a spatial and a temporal head."""
    P = 2812 if blocks[1] == 64 else 1404
    cfg = dict(get_config("mid128"), B=1, H=2 * copies, F=3, P=P, T=0, D=D, w_s=1, w_t=P // 3, spatial_heads=[0],
               block_m=blocks[0], block_n=blocks[1])
    cfg["N"] = cfg["F"] * cfg["P"]                      # 131 full key tiles and a part of one
    sh, g = S.shape_from_config(cfg), O.Geometry.from_config(cfg)
    nq, nk = S.svg_tile_counts(sh)
    assert nk == 132 and nq >= len(LENGTHS) and g.N % blocks[1]
    # one copy of the two heads is few rows, but for two of the forms with 128-row tiles; three are not
    split = takes_split_form(sh, {"gather": GATHER, "exact": EXACT, "plain": SPARSE}[form])
    assert split == (copies == 1 and (blocks[0] == 32 or (form, D) == ("exact", 64)))
    csr = [random_lists(nq, nk, last_tile, 2 * D + 10 * h + last_tile) for h in (0, 1)]
    lists = [dev_i32(x) for rp_ci in csr for x in rp_ci]
    q, k, v = make_plain_qkv(1, 2, g.N, D, seed=D)
    k = (k.float() * torch.linspace(0.2, 3.0, g.N)[None, None, :, None]).bfloat16()
    qc, kc, vc = (x.repeat(1, copies, 1, 1).cuda() for x in (q, k, v))
    lab = torch.tensor([0, 1] * copies, dtype=torch.uint8, device="cuda")
    if form == "gather":
        o, guard_ok = gpu_layer_in_place(sh, qc, kc, vc, lab, lists)
        assert guard_ok
    elif form == "exact":
        o, _, _ = gpu_layer_kv2(sh, qc, kc, vc, lab, lists, flags=S.SVG_ATTN_ELEMENT_MASK)
    else:
        o = gpu_layer(sh, qc, kc, vc, lab, lists)
    in_order = np.empty(g.N, np.int64)
    in_order[O.layout_perm(g)] = np.arange(g.N)
    for h in (0, 1):
        token = in_order if h else np.arange(g.N)       # token of each row of the order the lists refer to
        rp, ci = csr[h]
        got = f64(o[0, 2 * copies - 2 + h])[token]
        for a, n in enumerate(LENGTHS):
            rows = slice(a * g.block_m, min(g.N, (a + 1) * g.block_m))
            cols = np.concatenate([np.arange(b * g.block_n, min(g.N, (b + 1) * g.block_n)) for b in ci[rp[a]:rp[a + 1]]] or
                                  [np.zeros(0, np.int64)])
            qr, kr, vr = f64(q)[0, h][token[rows]], f64(k)[0, h][token[cols]], f64(v)[0, h][token[cols]]
            keep = np.ones((len(qr), len(cols)), bool)
            if form == "exact":
                keep = (O.temporal_mask if h else O.spatial_mask)(g, token[rows])[:, token[cols]]
            some = keep.any(1)
            assert (got[rows][~some] == 0).all(), f"{form} head {h}, {n} tiles: rows without keys"
            if some.any():
                ref = O.masked_attention(qr[some], kr, vr, keep[some], g.scale)
                assert_attn_close(torch.from_numpy(got[rows][some]), ref, f"{form} head {h}, {n} tiles")


@pytest.mark.parametrize("P", [1, 7, 1023, 1024, 1025, 1027])
def test_fp8_scales_of_heads_around_one_block(P):
    """The largest magnitude of a head, wherever it stands, for heads of one block of rows and of several."""
    cfg = dict(get_config("mid128"), B=1, H=2, F=1, P=P, T=0, spatial_heads=[0])
    cfg["N"] = P
    sh = S.shape_from_config(cfg)
    for at in sorted({0, P // 2, P - 1}):
        q, k, v = make_plain_qkv(1, 2, P, 128, seed=P + at)
        for x, peak in ((q, 31.0), (k, -47.0), (v, 63.0)):
            x[0, 1, at, 127 if at else 0] = peak
        scales = gpu_fp8_quantize(sh, q.cuda(), k.cuda(), v.cuda(), torch.zeros(2, dtype=torch.uint8, device="cuda"))[3]
        want = np.array([[np.abs(f64(x)[0, h]).max() for h in range(2)] for x in (q, k, v)], np.float32) / np.float32(448)
        assert np.array_equal(scales[:6].cpu().numpy().reshape(3, 2), want)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("heads", [21, 63, 64, 65, 127, 129])
def test_every_dense_query_tile_is_computed(D, heads):
    """Eight query tiles a head, dealt to the XCDs in blocks of equal size: 512 tiles and fewer in one block each, more in
    two or three, with and without tiles left over.  All heads hold the same rows, so all outputs have the same bits."""
    cfg = dict(get_config("mid128"), B=1, H=heads, F=1, P=1000, T=0, D=D, spatial_heads=[0])
    cfg["N"] = 1000
    sh, g = S.shape_from_config(cfg), O.Geometry.from_config(cfg)
    q, k, v = make_plain_qkv(1, 1, g.N, D, seed=D)
    o = torch.full((1, heads, g.N, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    S.svg_dense_attn_fwd(sh, *(x.repeat(1, heads, 1, 1).cuda() for x in (q, k, v)), o)
    torch.cuda.synchronize()
    assert_attn_close(o[0, 0], O.dense_attention_head(*(f64(x)[0, 0] for x in (q, k, v)), g), "head 0")
    assert torch.equal(o.view(torch.int16), o[:, :1].expand_as(o).contiguous().view(torch.int16))


@pytest.mark.parametrize("tiles", [1, 3, 25])
@pytest.mark.parametrize("text", [0, 1])
@pytest.mark.parametrize("heads, temporal", [(5, [1]), (8, [0, 3, 7]), (11, [0, 2, 4, 6, 8]), (9, []), (10, list(range(10))), (70, list(range(0, 70, 3)))])
def test_every_sparse_query_tile_is_computed(heads, temporal, text, tiles):
    """Every mixture of labels is dealt to the XCDs in shares that take each tile once.  All heads hold the same rows and keep every key, so all
    outputs have the bits of the dense pass."""
    cfg = dict(get_config("mid128"), B=1, H=heads, F=1, P=128 * tiles - 5, T=text, D=64, w_s=1, w_t=128 * tiles, spatial_heads=[0])
    cfg["N"] = cfg["P"] + text
    sh = S.shape_from_config(cfg)
    x = [t.repeat(1, heads, 1, 1).cuda() for t in make_plain_qkv(1, 1, cfg["N"], 64, seed=tiles)]
    lab = torch.zeros(heads, dtype=torch.uint8, device="cuda")
    lab[temporal] = 1
    lists = [dev_i32(a) for p in (S.SVG_HEAD_SPATIAL, S.SVG_HEAD_TEMPORAL) for a in S.svg_tile_list_build(sh, p)]
    o, want = torch.full_like(x[0], float("nan")), torch.full_like(x[0], float("nan"))
    S.svg_sparse_attn_fwd_ex(sh, *x, o, lab, *lists, flags=S.SVG_ATTN_QO_TOKEN_ORDER)
    S.svg_dense_attn_fwd(sh, *x, want)
    torch.cuda.synchronize()
    assert torch.allclose(o.float(), want[:, :1].float(), atol=2e-2, rtol=0) and torch.isfinite(o).all()
    if not text:
        assert torch.equal(o.view(torch.int16), want.view(torch.int16))
