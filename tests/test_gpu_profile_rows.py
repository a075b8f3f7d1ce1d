"""Profiling at the numbers of sampled rows where its route changes: one group of rows (which sorts them
itself) or several, one error block per head (which writes the label itself) or several, and every number
of parts the unmasked pass is cut into; in the form for few rows and in the general one."""
import numpy as np
import pytest
import torch

import paper_2502_01776_amd as S
from oracle import svg_oracle as O
from workloads import get_config, make_qkv
from helpers import f64, error_blocks, gpu_profile, labels_match, profile_cuts, profile_pieces, takes_split_form, PROFILE

pytestmark = pytest.mark.gpu


def check(cfg, t, copies=1, qkv=None):
    """copies: the heads over again, to make them many."""
    cfg["N"] = cfg["F"] * cfg["P"] + cfg["T"]
    sh, g = S.shape_from_config(dict(cfg, H=cfg["H"] * copies)), O.Geometry.from_config(cfg)
    q, k, v = qkv or make_qkv(cfg)
    # unsorted, with text rows and repetitions among them
    rows = np.random.default_rng(t).integers(0, g.N, t).astype(np.int32)
    qc, kc, vc = (x.repeat(1, copies, 1, 1).cuda() for x in (q, k, v))
    labels, mse = gpu_profile(sh, qc, kc, vc, rows)
    omse, olab = O.profile_heads(f64(q), f64(k), f64(v), rows, g)
    # the bounds of the other profiling tests: bf16 rounding of the weights under every measured error
    last = slice(-cfg["B"] * cfg["H"], None)
    assert np.allclose(mse[last].cpu().numpy().reshape(omse.shape), omse, rtol=0.05, atol=2e-5)
    assert labels_match(labels[last], omse, olab)
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


@pytest.mark.parametrize("t", [1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257])
@pytest.mark.parametrize("blocks, D", [((128, 64), 64), ((128, 64), 128), ((32, 32), 64), ((32, 32), 128)])
def test_numbers_of_sampled_rows_in_the_general_form(t, blocks, D):
    """Rows that a workgroup sorts itself (up to two groups) and rows sorted before it."""
    cfg = dict(get_config("mid64"), D=D, B=1, H=3, spatial_heads=[0, 2], block_m=blocks[0], block_n=blocks[1])
    copies = 130 // (3 * -(-t // 32)) + 1
    assert not takes_split_form(S.shape_from_config(dict(cfg, H=3 * copies)), PROFILE, t)
    check(cfg, t, copies)


@pytest.mark.parametrize("H, copies, F, P, t, D, split, cut", [
    # the split form: the plan's cut, four parts and three, four and two, three and three
    (8, 1, 9, 400, 60, 64, True, (4, 4)), (6, 1, 5, 1300, 90, 128, True, (4, 3)), (2, 1, 9, 160, 700, 128, True, (4, 3)),
    (12, 1, 5, 330, 256, 64, True, (4, 2)), (3, 1, 5, 100, 40, 128, True, (3, 3)), (2, 1, 9, 700, 70, 64, True, (6, 4)),
    # the general form: every number of parts of the unmasked pass, with masked passes whole and cut
    (2, 2, 70, 20, 40, 64, False, (1, 4)), (2, 2, 70, 14, 40, 128, False, (3, 3)), (2, 80, 5, 140, 40, 128, False, (1, 1)), (2, 2, 70, 30, 150, 128, False, (4, 4)),
    (2, 80, 5, 330, 40, 64, False, (4, 2)), (4, 1, 9, 700, 700, 128, False, (6, 4)), (2, 260, 5, 330, 40, 64, False, (4, 1)),
    (2, 100, 9, 700, 40, 64, False, (6, 1))])
def test_forms_and_cuts(H, copies, F, P, t, D, split, cut):
    cfg = dict(get_config("mid64"), D=D, B=1, H=H, F=F, P=P, spatial_heads=[0])
    sh = S.shape_from_config(dict(cfg, H=H * copies))
    assert takes_split_form(sh, PROFILE, t) == split
    got = profile_cuts(sh, t)[1]
    assert (got.n_full, got.n_masked) == cut
    check(cfg, t, copies)


PIECES = dict(get_config("mid64"), B=1, H=2, spatial_heads=[0])


@pytest.mark.parametrize("F, P, T, text_first, sink, w_s", [
    (6, 256, 0, 0, 0, 1), (6, 257, 37, 1, 0, 0), (6, 320, 64, 0, 0, 1), (5, 333, 50, 0, 1, 1), (5, 320, 64, 1, 1, 9),
    (1, 1600, 0, 0, 0, 0), (1, 1600, 20, 1, 1, 0), (2, 800, 0, 0, 1, 0), (4, 300, 900, 1, 0, 1), (4, 300, 900, 0, 0, 1)])
@pytest.mark.parametrize("blocks, D, t, copies", [((128, 64), 64, 70, 50), ((128, 64), 128, 129, 20), ((32, 32), 64, 33, 60), ((32, 32), 128, 40, 300)])
def test_unmasked_pass_in_pieces(F, P, T, text_first, sink, w_s, blocks, D, t, copies):
    """Windows that end inside key tiles, at their edges, at the ends of the video and of the parts; parts without a video key."""
    cfg = dict(PIECES, D=D, F=F, P=P, T=T, text_first=text_first, sink_first_frame=sink, w_s=w_s, block_m=blocks[0], block_n=blocks[1])
    cfg["N"] = F * P + T
    assert profile_pieces(S.shape_from_config(dict(cfg, H=2 * copies)), t)[0] > 0
    check(cfg, t, copies)


@pytest.mark.parametrize("D", [64, 128])
def test_a_window_far_below_the_rest_of_its_row(D):
    """Every other row's window holds logits 200 below those outside it: its output must not depend on them."""
    cfg = dict(PIECES, D=D, F=6, P=300, T=0, w_s=0, N=1800)
    q, k, v = make_qkv(cfg, boost_nats=3.0)
    sign = torch.where(torch.arange(1800) // 300 % 2 == 0, 1.0, -1.0)[:, None]
    q[..., :1] = (100 * D ** 0.5) ** 0.5
    k[..., :1] = ((100 * D ** 0.5) ** 0.5 * sign).to(k.dtype)
    assert profile_pieces(S.shape_from_config(dict(cfg, H=80)), 60)[0] > 0
    check(cfg, 60, 40, (q, k, v))


@pytest.mark.parametrize("H, t", [(2, 33), (2, 200), (32, 129), (80, 33), (80, 65), (80, 129)])
def test_error_blocks_of_a_head_meet_in_a_graph(H, t):
    """Several error blocks per head (32 rows each): the last one finds its ticket in a workspace of any content, replay after replay; with many
    blocks a launch of its own adds their sums up."""
    replay(dict(PIECES, D=128, H=H, F=6, P=300, T=20, N=1820, spatial_heads=list(range(0, H, 2))), t)


@pytest.mark.parametrize("H, F, P, T, D, t, pieces, blocks", [
    (20, 62, 30, 0, 128, 60, False, 2), (12, 62, 30, 20, 64, 130, False, 3), (4, 62, 256, 0, 64, 120, True, 2), (2, 62, 256, 20, 128, 97, True, 4)])
def test_tickets_of_the_general_form_in_a_graph(H, F, P, T, D, t, pieces, blocks):
    """As above; the general form is the one that clears the tickets, in three passes and with the unmasked one in pieces."""
    cfg = dict(PIECES, D=D, H=H, F=F, P=P, T=T, N=F * P + T, spatial_heads=list(range(0, H, 2)))
    sh = S.shape_from_config(cfg)
    assert not takes_split_form(sh, PROFILE, t) and (profile_pieces(sh, t)[0] > 0) == pieces
    assert error_blocks(sh, t) == blocks and H * blocks <= 64
    replay(cfg, t)


def replay(cfg, t):
    H = cfg["H"]
    sh = S.shape_from_config(cfg)
    q, k, v = make_qkv(cfg, device="cuda")
    rows = torch.from_numpy(np.random.default_rng(t).integers(0, cfg["N"], t).astype(np.int32)).cuda()
    ws = torch.full((S.svg_workspace_bytes(sh, t),), 255, dtype=torch.uint8, device="cuda")
    labels, mse = torch.zeros(H, dtype=torch.uint8, device="cuda"), torch.zeros(H, 2, device="cuda")
    want = gpu_profile(sh, q, k, v, rows.cpu().numpy())
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        S.svg_profile_heads(sh, q, k, v, rows, t, labels, mse, ws, ws.numel())
    for fill in (255, 0, 1):
        ws.fill_(fill)
        labels.fill_(7)
        mse.fill_(-1.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(labels, want[0]) and torch.equal(mse, want[1])
