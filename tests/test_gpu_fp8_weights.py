"""The attention weights of the FP8 pass: which maximum they are rounded against, and what becomes of them at the
end of the scales' range."""
import numpy as np
import pytest
import torch

import paper_2502_01776_amd as S
from oracle import svg_oracle as O
from workloads import get_config, make_plain_qkv
from helpers import f64, dev_i32, gpu_fp8_quantize, v8t_rows, assert_fp8_attn_close, takes_fp8_split_form

pytestmark = pytest.mark.gpu


def one_head(P, frames=1, heads=1):
    """Heads without text, frames short enough that every query tile walks its list from the first entry; one head or few run in the
    form for few rows, many in the general kernel."""
    cfg = dict(get_config("mid128"), B=1, H=heads, F=frames, P=P, T=0, w_s=0, sink_first_frame=0, spatial_heads=[0])
    cfg["N"] = frames * P
    return S.shape_from_config(cfg), O.Geometry.from_config(cfg)


def run_lists(sh, q, k, v, lists):
    """lists: kept key tiles of each query tile.  Returns the output, the lists as CSR and the quantised q, k, v the
    pass was given (the device's codes: on a rounding boundary they may differ from the oracle's)."""
    rp = np.concatenate([[0], np.cumsum([len(c) for c in lists])]).astype(np.int32)
    ci = np.concatenate(lists).astype(np.int32)
    csr = [dev_i32(rp), dev_i32(ci), dev_i32(rp), dev_i32(ci)]
    assert takes_fp8_split_form(sh) == (sh.H == 1)
    qc, kc, vc = (x.repeat(1, sh.H, 1, 1).cuda() for x in (q, k, v))      # the same head over again
    lab = torch.zeros(sh.H, dtype=torch.uint8, device="cuda")
    o = torch.full_like(qc, float("nan"))
    q8, k8, v8t, scales = gpu_fp8_quantize(sh, qc, kc, vc, lab)
    S.svg_sparse_attn_fp8_fwd(sh, q8, k8, v8t, scales, o, lab, *csr)
    torch.cuda.synchronize()
    N, nk = q.shape[2], len(v8t) // (8192 * sh.H)
    codes = (q8.cpu().numpy().reshape(-1, 128)[:N], k8.cpu().numpy().reshape(-1, 128)[:N], v8t_rows(v8t.cpu().numpy()[:nk * 8192], nk)[:N])
    return o[:, -1:], rp, ci, [O.fp8_dequantize(c, s) for c, s in zip(codes, scales.cpu().numpy()[::sh.H])]


@pytest.mark.parametrize("heads", [1, 40])
@pytest.mark.parametrize("N", [512, 500])
def test_product_of_the_scales_underflows(N, heads):
    """q and k so small that softmax scale * q scale * k scale is zero in float32: all logits are zero and the
    output is the mean of the kept rows of v, also where keys are masked (a ragged last tile, a list of odd length)."""
    sh, g = one_head(N, heads=heads)
    q, k, v = make_plain_qkv(1, 1, N, 128, seed=9)
    q, k = q * 2.0 ** -90, k * 2.0 ** -90
    lists = [[0], [1, 2, 7], [0, 3, 4, 5, 6], [2, 7]]
    o, rp, ci, (_, _, vh) = run_lists(sh, q, k, v, lists)
    zero = np.zeros_like(vh)
    ref = O.sparse_attention_head(zero, zero, vh, rp.astype(np.int64), ci, g)
    assert_fp8_attn_close(o[0, 0], ref, float(np.abs(vh).max()), "zero logits")


def walk(q, k, v, lists, g):
    """The FP8 pass in float64 but for its one rounding: tile after tile, every weight is rounded to E4M3 against the
    row's maximum up to and including its own 64-key tile, and earlier sums are rescaled when that rises."""
    out = np.zeros((g.N, g.D))
    for a, tiles in enumerate(lists):
        rows = slice(a * g.block_m, min(g.N, (a + 1) * g.block_m))
        m, l, o = -np.inf, 0.0, 0.0
        for b in tiles:
            cols = slice(b * g.block_n, min(g.N, (b + 1) * g.block_n))
            s = (q[rows] @ k[cols].T) * g.scale
            m_new = np.maximum(m, s.max(1, keepdims=True))
            alpha, m = np.exp(m - m_new), m_new
            w = O.fp8_round_weights(np.exp(s - m))
            l, o = l * alpha + w.sum(1, keepdims=True), o * alpha + w @ v[cols]
        out[rows] = o / l
    return out


@pytest.mark.parametrize("growth", [0.0, 1.0])
@pytest.mark.parametrize("seed", [1, 2])
@pytest.mark.parametrize("heads", [1, 14])
def test_weights_are_rounded_against_the_maximum_of_their_own_tile(growth, seed, heads):
    """Lists of 1 to 12 tiles, logits that stay alike or grow along the list, so that the maximum rises at odd places
    of the list, at even ones, at both or at neither.  A row differs from the model by its rounding to bf16,
    at most 2^-9 of a value, except where the float32 arithmetic lets a weight on a rounding boundary take the other of
    its two codes (up to 4 of 128 rows here).  With one maximum for two tiles together 20 to 80 rows differ by more."""
    sh, g = one_head(64, frames=24, heads=heads)
    q, k, v = make_plain_qkv(1, 1, g.N, 128, seed=seed)
    q = q * 1.5
    k = (k.float() * torch.linspace(1.0, 1.0 + growth, g.N)[None, None, :, None]).bfloat16()
    rng = np.random.default_rng(seed)
    lists = [np.sort(rng.choice(24, n, replace=False)) for n in range(1, 13)]
    o, _, _, (qh, kh, vh) = run_lists(sh, q, k, v, lists)
    ref = walk(qh, kh, vh, lists, g)
    for a in range(len(lists)):
        rows = slice(a * 128, (a + 1) * 128)
        rel = np.linalg.norm(f64(o)[0, 0, rows] - ref[rows], axis=1) / np.linalg.norm(ref[rows], axis=1)
        assert (rel > 2.0 ** -8).sum() <= 6 and rel.max() <= 2.0 ** -3, f"{len(lists[a])} tiles: {np.sort(rel)[-8:]}"
