"""Profiling at the numbers of sampled rows where its route changes: one group of rows (which sorts them
itself) or several, one error block per head (which writes the label itself) or several, and every number
of parts the unmasked pass is cut into."""
import numpy as np
import pytest
import torch

import paper_2502_01776_amd as S
from oracle import svg_oracle as O
from workloads import get_config, make_qkv
from helpers import f64, gpu_profile, labels_match

pytestmark = pytest.mark.gpu


def check(cfg, t):
    cfg["N"] = cfg["F"] * cfg["P"] + cfg["T"]
    sh, g = S.shape_from_config(cfg), O.Geometry.from_config(cfg)
    q, k, v = make_qkv(cfg)
    # unsorted, with text rows and repetitions among them
    rows = np.random.default_rng(t).integers(0, g.N, t).astype(np.int32)
    qc, kc, vc = q.cuda(), k.cuda(), v.cuda()
    labels, mse = gpu_profile(sh, qc, kc, vc, rows)
    omse, olab = O.profile_heads(f64(q), f64(k), f64(v), rows, g)
    # the bounds of the other profiling tests: bf16 rounding of the weights under every measured error
    assert np.allclose(mse.cpu().numpy().reshape(omse.shape), omse, rtol=0.05, atol=2e-5)
    assert labels_match(labels, omse, olab)
    again, mse2 = gpu_profile(sh, qc, kc, vc, rows)
    assert torch.equal(labels, again) and torch.equal(mse, mse2)
    return S.svg_profile_plan(sh, t)


@pytest.mark.parametrize("t", [1, 31, 32, 33, 127, 128, 129, 255, 256, 257])
@pytest.mark.parametrize("blocks, D", [((128, 64), 64), ((128, 64), 128), ((32, 32), 64), ((32, 32), 128)])
def test_numbers_of_sampled_rows(t, blocks, D):
    check(dict(get_config("mid64"), D=D, B=1, H=3, spatial_heads=[0, 2], block_m=blocks[0], block_n=blocks[1]), t)


@pytest.mark.parametrize("H, F, P, t, n_full, D", [(2, 5, 150, 24, 1, 64), (2, 9, 190, 130, 4, 64), (2, 9, 700, 70, 6, 64),
                                                   (64, 5, 200, 1024, 3, 64), (2, 1, 250, 24, 1, 128), (2, 1, 300, 24, 1, 128),
                                                   (2, 5, 158, 24, 3, 128), (2, 5, 158, 65, 1, 128),
                                                   (2, 9, 150, 24, 3, 128), (64, 5, 150, 140, 1, 128)])
def test_parts_of_the_unmasked_pass(H, F, P, t, n_full, D):
    b = (32, 32) if t == 1024 else (128, 64)
    plan = check(dict(get_config("mid64"), D=D, B=1, H=H, F=F, P=P, spatial_heads=[0], block_m=b[0], block_n=b[1]), t)
    assert plan[0] == n_full


@pytest.mark.parametrize("H, F, P, t, D", [(6, 5, 1300, 90, 128), (8, 9, 400, 60, 64), (2, 9, 160, 700, 128), (8, 9, 160, 700, 64), (12, 5, 330, 256, 64)])
def test_cuts_of_the_launch(H, F, P, t, D):
    """Numbers of groups of rows around which the split form cuts its passes otherwise than the plan says."""
    check(dict(get_config("mid64"), D=D, B=1, H=H, F=F, P=P, spatial_heads=[0]), t)
