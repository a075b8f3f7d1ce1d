"""The attention weights of the FP8 pass: what becomes of them at the ends of the scales' range."""
import numpy as np
import pytest
import torch

import paper_2502_01776_amd as S
from oracle import svg_oracle as O
from workloads import get_config, make_plain_qkv
from helpers import f64, dev_i32, gpu_fp8_quantize, assert_fp8_attn_close

pytestmark = pytest.mark.gpu


def one_head(P, frames=1):
    """One head without text, frames short enough that every query tile walks its list from the first entry."""
    cfg = dict(get_config("mid128"), B=1, H=1, F=frames, P=P, T=0, w_s=0, sink_first_frame=0, spatial_heads=[0])
    cfg["N"] = frames * P
    return S.shape_from_config(cfg), O.Geometry.from_config(cfg)


def run_lists(sh, q, k, v, lists):
    """lists: kept key tiles of each query tile.  Returns the output and the quantised tensors (codes, scale)."""
    rp = np.concatenate([[0], np.cumsum([len(c) for c in lists])]).astype(np.int32)
    ci = np.concatenate(lists).astype(np.int32)
    csr = [dev_i32(rp), dev_i32(ci), dev_i32(rp), dev_i32(ci)]
    qc, kc, vc = q.cuda(), k.cuda(), v.cuda()
    lab = torch.zeros(1, dtype=torch.uint8, device="cuda")
    o = torch.full_like(qc, float("nan"))
    S.svg_sparse_attn_fp8_fwd(sh, *gpu_fp8_quantize(sh, qc, kc, vc, lab), o, lab, *csr)
    torch.cuda.synchronize()
    return o, rp, ci


@pytest.mark.parametrize("N", [512, 500])
def test_product_of_the_scales_underflows(N):
    """q and k so small that softmax scale * q scale * k scale is zero in float32: all logits are zero and the
    output is the mean of the kept rows of v, also where keys are masked (a ragged last tile, a list of odd length)."""
    sh, g = one_head(N)
    q, k, v = make_plain_qkv(1, 1, N, 128, seed=9)
    q, k = q * 2.0 ** -90, k * 2.0 ** -90
    lists = [[0], [1, 2, 7], [0, 3, 4, 5, 6], [2, 7]]
    o, rp, ci = run_lists(sh, q, k, v, lists)
    vh = O.fp8_dequantize(*O.fp8_quantize_head(f64(v)[0, 0]))
    zero = np.zeros_like(vh)
    ref = O.sparse_attention_head(zero, zero, vh, rp.astype(np.int64), ci, g)
    assert_fp8_attn_close(o[0, 0], ref, float(np.abs(vh).max()), "zero logits")
