"""The form in which two teams of wavefronts take the key tiles of a query tile in turn: odd and even numbers of tiles, a last
key tile of one key, text rows taken in parts beside it, against the oracle; and lists of every length."""
import numpy as np
import pytest
import torch

import paper_2502_01776_amd as S
from oracle import svg_oracle as O
from workloads import get_config, make_plain_qkv
from helpers import (f64, dev_i32, gpu_layer_in_place, gpu_layer_kv2, assert_attn_close, takes_split_form, takes_two_teams, DENSE, SPARSE, EXACT, GATHER)
from test_gpu_lists import LENGTHS, random_lists, test_list_lengths as list_lengths, test_list_lengths_of_the_other_forms as list_lengths_of_the_other_forms

MODES = {"dense": DENSE, "sparse": SPARSE, "exact": EXACT, "gather": GATHER}


def setup(H, D, F, P, T, **kw):
    cfg = dict(get_config("mid64"), B=1, H=H, D=D, F=F, P=P, T=T, w_s=1, w_t=max(1, P // 5), spatial_heads=[0], text_first=P % 2,
               block_m=128, block_n=64, **kw)
    cfg["N"] = F * P + T
    return S.shape_from_config(cfg), O.Geometry.from_config(dict(cfg, H=2))


@pytest.mark.gpu
@pytest.mark.parametrize("H, F, P, T, sink", [(20, 3, 512, 0, 0), (20, 3, 491, 0, 1), (18, 3, 534, 0, 0), (16, 3, 533, 1, 0), (14, 5, 310, 90, 1)])
@pytest.mark.parametrize("form", list(MODES))
@pytest.mark.parametrize("D", [64, 128])
def test_against_the_oracle(D, form, H, F, P, T, sink):
    sh, g = setup(H, D, F, P, T, sink_first_frame=sink)
    assert takes_two_teams(sh) and not takes_split_form(sh, MODES[form])
    q, k, v = make_plain_qkv(1, 2, g.N, D, seed=P)
    k = (k.float() * torch.linspace(0.2, 3.0, g.N)[None, None, :, None]).bfloat16()
    x = [t.repeat(1, H // 2, 1, 1).cuda() for t in (q, k, v)]
    lab = torch.tensor([0, 1] * (H // 2), dtype=torch.uint8, device="cuda")
    if form == "dense":
        o = torch.full_like(x[0], float("nan"))
        S.svg_dense_attn_fwd(sh, *x, o)
        torch.cuda.synchronize()
    elif form == "gather":
        o = gpu_layer_in_place(sh, *x, lab)[0]
    else:
        o = gpu_layer_kv2(sh, *x, lab, flags=S.SVG_ATTN_ELEMENT_MASK if form == "exact" else 0)[0]
    for h in (0, 1):
        qh, kh, vh = (f64(t)[0, h] for t in (q, k, v))
        if form == "dense":
            ref = O.dense_attention_head(qh, kh, vh, g)
        elif form == "exact":
            ref = O.masked_attention(qh, kh, vh, (O.temporal_mask if h else O.spatial_mask)(g), g.scale)
        else:
            ref = O.svg_attention_layer(f64(q), f64(k), f64(v), np.array([[0, 1]]), g)[0, h]
        assert_attn_close(o[0, h], ref, f"{form} head {h}")
        assert torch.equal(o[0, h::2].view(torch.int16), o[0, h:h + 1].expand(H // 2, -1, -1).contiguous().view(torch.int16))


@pytest.mark.gpu
@pytest.mark.parametrize("last_tile", [False, True])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("form, heads, two", [("plain", 3, True), ("plain", 4, False), ("gather", 2, True), ("gather", 4, False), ("exact", 4, False)])
def test_list_lengths(form, heads, two, D, last_tile):
    """As in test_gpu_lists, on both sides of the line; empty lists and lists of one tile leave a team without any."""
    assert takes_two_teams(setup(heads, D, 3, 2812, 0)[0]) == two
    if form == "plain":
        list_lengths(D, False, last_tile, heads)
    else:
        list_lengths_of_the_other_forms(form, (128, 64), D, last_tile, heads // 2)


@pytest.mark.gpu
@pytest.mark.parametrize("last_tile", [False, True])
@pytest.mark.parametrize("D", [64, 128])
def test_list_lengths_under_element_masks(D, last_tile):
    """Three heads: two are few rows at head dimension 64, four more than 256 query tiles."""
    sh, g = setup(3, D, 3, 2812, 0)
    assert takes_two_teams(sh) and not takes_split_form(sh, EXACT)
    rp, ci = random_lists(*S.svg_tile_counts(sh), last_tile, 3 * D + last_tile)
    q, k, v = make_plain_qkv(1, 1, g.N, D, seed=D)
    k = (k.float() * torch.linspace(0.2, 3.0, g.N)[None, None, :, None]).bfloat16()
    o = gpu_layer_kv2(sh, *(x.repeat(1, 3, 1, 1).cuda() for x in (q, k, v)), torch.zeros(3, dtype=torch.uint8, device="cuda"),
                      [dev_i32(x) for x in (rp, ci, rp, ci)], flags=S.SVG_ATTN_ELEMENT_MASK)[0]
    got, (qh, kh, vh) = f64(o[0, 2]), (f64(x)[0, 0] for x in (q, k, v))
    for a, n in enumerate(LENGTHS):
        rows = np.arange(a * g.block_m, min(g.N, (a + 1) * g.block_m))
        cols = np.concatenate([np.arange(b * g.block_n, min(g.N, (b + 1) * g.block_n)) for b in ci[rp[a]:rp[a + 1]]] or [np.zeros(0, np.int64)])
        keep = O.spatial_mask(g, rows)[:, cols]
        some = keep.any(1) if n else np.zeros(len(rows), bool)
        assert (got[rows][~some] == 0).all(), f"{n} tiles: rows without keys"
        if some.any():
            assert_attn_close(torch.from_numpy(got[rows][some]), O.masked_attention(qh[rows[some]], kh[cols], vh[cols], keep[some], g.scale), f"{n} tiles")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("F, P, T, most", [(3, 512, 0, 21), (3, 490, 0, 0), (3, 491, 0, 21), (3, 533, 1, 16), (1, 32768, 0, 1), (1, 32769, 0, 0)])
def test_numbers_of_query_tiles(D, F, P, T, most):
    """One workgroup to a compute unit, four for a tile with text rows; 24 key tiles and more."""
    for H in range(1, 24):
        assert takes_two_teams(setup(H, D, F, P, T)[0]) == (H <= most), H
