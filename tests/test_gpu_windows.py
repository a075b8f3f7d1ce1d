"""The window bits of the masked passes and the staging of ragged tiles at the sizes where they can go wrong:
frames shorter than, as long as and just longer than a key tile (a tile then touches many frames, one, or
two), windows of one position and of nearly all, and memory behind the last key that must never be read; with few heads in the
form for few rows, with many in the general kernels."""
import numpy as np
import pytest
import torch

import paper_2502_01776_amd as S
from oracle import svg_oracle as O
from workloads import get_config, make_plain_qkv
from helpers import (f64, gpu_profile, gpu_layer_in_place, gpu_layer_kv2, assert_attn_close, takes_split_form, DENSE, EXACT, GATHER, PROFILE)

pytestmark = pytest.mark.gpu


def setup(H=2, **kw):
    cfg = dict(get_config("mid64"), B=1, H=H, spatial_heads=[0], **kw)
    cfg["N"] = cfg["F"] * cfg["P"] + cfg["T"]
    return cfg, S.shape_from_config(cfg), O.Geometry.from_config(cfg)


@pytest.mark.parametrize("P, F, w_t", [(1, 70, 0), (7, 19, 1), (31, 9, 3), (32, 9, 14), (33, 9, 2), (63, 5, 5), (64, 5, 0),
                                       (65, 5, 60), (127, 3, 9), (129, 3, 1)])
@pytest.mark.parametrize("blocks, D", [((128, 64), 64), ((128, 64), 128), ((32, 32), 64)])
@pytest.mark.parametrize("general", [False, True])
def test_profile_and_element_masks_where_frames_and_tiles_meet(P, F, w_t, blocks, D, general):
    groups = -(-(F * P + 5) // 32)
    H = 2 * (641 // (2 * groups) + 1) if general else 2
    cfg, sh, g = setup(H=H, F=F, P=P, T=5, D=D, text_first=P % 2, w_s=1, w_t=w_t, block_m=blocks[0], block_n=blocks[1],
                       sink_first_frame=int(P % 3 == 0))
    q, k, v = make_plain_qkv(1, 2, g.N, g.D, seed=P)
    qc, kc, vc = (x.repeat(1, H // 2, 1, 1).cuda() for x in (q, k, v))
    rows = np.arange(0, g.N, 3, dtype=np.int32)
    assert takes_split_form(sh, EXACT) == (not general) and takes_split_form(sh, PROFILE, len(rows)) == (not general and F <= 61)
    _, mse = gpu_profile(sh, qc, kc, vc, rows)
    mse = mse[-2:]
    omse, _ = O.profile_heads(f64(q), f64(k), f64(v), rows, O.Geometry.from_config(dict(cfg, H=2)))
    # the bounds of the other profiling tests: bf16 rounding of the weights under every measured error
    assert np.allclose(mse.cpu().numpy().reshape(omse.shape), omse, rtol=0.05, atol=2e-5)
    lab = torch.tensor([0, 1] * (H // 2), dtype=torch.uint8, device="cuda")
    o, _, _ = gpu_layer_kv2(sh, qc, kc, vc, lab, flags=S.SVG_ATTN_ELEMENT_MASK)
    for h, mask in ((0, O.spatial_mask(g)), (1, O.temporal_mask(g))):
        ref = O.masked_attention(f64(q)[0, h], f64(k)[0, h], f64(v)[0, h], mask, g.scale)
        assert_attn_close(o[0, H - 2 + h], ref, f"P={P} head {h}")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("tail", [1, 63])
@pytest.mark.parametrize("H", [2, 162])
def test_rows_behind_the_last_key_are_never_read(D, tail, H):
    """k and v of the last head end where their allocation's NaN filling starts; a head's ragged last tile
    must not see it, nor, as weights times NaN, let it through."""
    cfg, sh, g = setup(H=H, F=2, P=64 + tail // 2, T=tail - 2 * (tail // 2), D=D, text_first=1, w_s=1, w_t=3,
                       block_m=128, block_n=64)
    assert g.N % 64 == tail and takes_split_form(sh, DENSE) == takes_split_form(sh, GATHER) == (H == 2)
    q, k, v = (x.repeat(1, H // 2, 1, 1) for x in make_plain_qkv(1, 2, g.N, D, seed=tail))
    def in_nan(x):
        buf = torch.full((x.numel() + 64 * D,), float("nan"), dtype=torch.bfloat16, device="cuda")
        buf[:x.numel()] = x.cuda().flatten()
        return buf[:x.numel()].view(x.shape)
    qc, kc, vc = q.cuda(), in_nan(k), in_nan(v)
    od = torch.empty_like(qc)
    S.svg_dense_attn_fwd(sh, qc, kc, vc, od)
    lab = torch.tensor([1, 0] * (H // 2), dtype=torch.uint8, device="cuda")
    og, _ = gpu_layer_in_place(sh, qc, kc, vc, lab)
    torch.cuda.synchronize()
    ref = O.svg_attention_layer(*[f64(x[:, :2]) for x in (q, k, v)], np.array([[1, 0]]), O.Geometry.from_config(dict(cfg, H=2)))
    for h in range(2):
        last = H - 2 + h
        assert_attn_close(od[0, last], O.dense_attention_head(f64(q)[0, h], f64(k)[0, h], f64(v)[0, h], g))
        assert_attn_close(og[0, last], ref[0, h])


@pytest.mark.parametrize("w_s, w_t", [(2 ** 31 - 1, 3), (2 ** 31 - 4, 3), (1, 2 ** 31 - 1), (1, 2 ** 31 - 20)])
@pytest.mark.parametrize("P, heads", [(40, 2), (41, 2), (40, 80)])
@pytest.mark.parametrize("blocks, D", [((128, 64), 64), ((128, 64), 128), ((32, 32), 64)])
def test_windows_as_wide_as_the_type(w_s, w_t, P, heads, blocks, D):
    """Half-windows at the end of their type keep every key: no error under that mask.  Few heads and many: both forms
    of the profiling passes."""
    cfg, sh, g = setup(F=9, P=P, T=5, D=D, text_first=1, w_s=w_s, w_t=w_t, block_m=blocks[0], block_n=blocks[1], sink_first_frame=0)
    q, k, v = make_plain_qkv(1, 2, g.N, D, seed=P)
    rows = np.arange(0, g.N, 4, dtype=np.int32)
    omse, olab = O.profile_heads(f64(q), f64(k), f64(v), rows, g)
    wide = 0 if w_s > w_t else 1
    assert (omse[..., wide] == 0).all() and (omse[..., 1 - wide] > 1e-4).all() and (olab == wide).all()
    many = S.shape_from_config(dict(cfg, H=heads))
    assert takes_split_form(many, PROFILE, len(rows)) == (heads == 2)
    labels, mse = gpu_profile(many, *[x.repeat(1, heads // 2, 1, 1).cuda() for x in (q, k, v)], rows)
    mse = mse.cpu().numpy().reshape(heads // 2, 2, 2)
    # the bounds of the other profiling tests: bf16 rounding of the weights under every measured error
    for pair in (0, -1):
        assert np.allclose(mse[pair], omse[0], rtol=0.05, atol=2e-5)
    assert (labels.cpu().numpy() == wide).all()
