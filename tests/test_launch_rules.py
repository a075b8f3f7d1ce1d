"""The rules by which the library chooses the form of a kernel and the cut of a profiling call (host side, no GPU)."""
import pytest

import paper_2502_01776_amd as S
from workloads import get_config
from helpers import DENSE, EXACT, GATHER, PROFILE, SPARSE, profile_cuts, profile_pieces, error_blocks, takes_fp8_split_form, takes_split_form, dense_cohort


def shape(H, N, D=128, blocks=(128, 64), F=1, T=0, **kw):
    assert (N - T) % F == 0
    cfg = dict(get_config("mid128"), B=1, H=H, D=D, F=F, P=(N - T) // F, T=T, block_m=blocks[0], block_n=blocks[1], **kw)
    return S.shape_from_config(cfg)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("blocks", [(128, 64), (32, 32)])
def test_a_cut_fits_the_workspace_and_covers_every_key_tile(D, blocks):
    for N in (1, 33, 800, 1536, 1537, 6144, 40000, 200000):
        for H in (1, 3, 12, 24, 41, 96, 150, 400, 3000):
            for t in (1, 32, 33, 64, 65, 200, 700, 3000):
                sh = shape(H, N, D, blocks)
                plan, cut = profile_cuts(sh, t)
                nf, nm, bound = S.svg_profile_plan(sh, t)
                nk = S.svg_tile_counts(sh)[1]
                assert (plan.n_full, plan.n_masked, list(plan.full_bound)[:nf + 1]) == (nf, nm, bound)
                assert cut.slots() <= plan.slots() and cut.n_full in (1, 3, 4, 6) and 1 <= cut.n_masked <= 4
                b = list(cut.full_bound)[:cut.n_full + 1]
                assert b[0] == 0 and b[-1] == nk and b == sorted(b)
                if not takes_split_form(sh, PROFILE, t):
                    assert bytes(cut) == bytes(plan)      # the general form runs the plan


@pytest.mark.parametrize("mode, D, blocks, N, T, most", [
    (DENSE, 64, (128, 64), 320, 0, 640), (EXACT, 64, (128, 64), 320, 0, 640), (DENSE, 128, (128, 64), 416, 0, 416), (EXACT, 128, (128, 64), 416, 0, 416),
    (SPARSE, 64, (128, 64), 512, 0, 512), (SPARSE, 128, (128, 64), 960, 0, 256), (SPARSE, 128, (128, 64), 1000, 0, 416),
    (SPARSE, 64, (32, 32), 256, 0, 256), (SPARSE, 64, (32, 32), 512, 0, 512),
    (DENSE, 64, (32, 32), 256, 0, 512), (SPARSE, 64, (32, 32), 1600, 0, 600), (SPARSE, 64, (32, 32), 256, 9, 600), (SPARSE, 128, (32, 32), 1024, 0, 256),
    (SPARSE, 128, (32, 32), 1664, 0, 416), (SPARSE, 128, (32, 32), 416, 9, 416), (DENSE, 128, (32, 32), 256, 0, 256), (DENSE, 128, (32, 32), 832, 0, 416),
    (EXACT, 128, (32, 32), 416, 0, 416), (EXACT, 64, (32, 32), 320, 0, 640)])
def test_numbers_of_workgroups_the_split_form_takes(mode, D, blocks, N, T, most):
    """Beyond them it measured slower than the general kernel on some calls, by up to 13 %."""
    per_head = -(-N // 32)
    for H in range(max(1, most // per_head - 2), most // per_head + 3):
        assert takes_split_form(shape(H, N, D, blocks, T=T), mode) == (H * per_head <= most), H


@pytest.mark.parametrize("D", [64, 128])
def test_gathering_in_place_has_the_line_of_the_passes_it_replaces(D):
    """Their outputs are the same bit for bit, so the same form has to take them."""
    for N in (32, 200, 959, 960, 961, 1000, 5000, 20000):
        for H in range(1, 90):
            sh = shape(H, N, D)
            assert takes_split_form(sh, GATHER) == takes_split_form(sh, SPARSE), (N, H)


@pytest.mark.parametrize("N, most", [(500, 512), (4095, 512), (4096, 600), (19000, 600)])
def test_numbers_of_workgroups_the_fp8_split_form_takes(N, most):
    per_head = -(-N // 32)
    for H in range(max(1, most // per_head - 2), most // per_head + 3):
        assert takes_fp8_split_form(shape(H, N)) == (H * per_head <= most), H


@pytest.mark.parametrize("D, H, t, N, cut", [
    (128, 16, 32, 7000, None), (128, 17, 32, 7000, (4, 3)), (128, 24, 32, 7000, (4, 3)), (128, 25, 32, 7000, None), (128, 40, 32, 7000, None),
    (128, 41, 32, 7000, (4, 3)), (128, 48, 32, 7000, (4, 3)), (128, 49, 32, 7000, None), (64, 24, 32, 7000, None), (64, 56, 32, 7000, None),
    (64, 57, 32, 7000, (4, 3)), (64, 72, 32, 7000, (4, 3)), (64, 73, 32, 7000, None), (64, 88, 32, 7000, None), (64, 44, 64, 7000, None),
    (64, 45, 64, 7000, (4, 2)), (64, 48, 64, 7000, (4, 2)), (64, 49, 64, 7000, None), (128, 9, 32, 700, (3, 3))])
def test_cuts_of_the_split_form(D, H, t, N, cut):
    """Fewer parts than the plan where those find a place at once and the plan's do not."""
    plan, got = profile_cuts(shape(H, N, D), t)
    assert takes_split_form(shape(H, N, D), PROFILE, t) and plan.n_masked == 4
    assert (got.n_full, got.n_masked) == (cut or (plan.n_full, plan.n_masked))
    if cut is None:
        assert bytes(got) == bytes(plan)


@pytest.mark.parametrize("D, free, most, keys", [(64, 64, 128, 2400000), (128, 48, 72, 1600000)])
def test_groups_of_rows_the_split_form_profiles(D, free, most, keys):
    for N in (1000, 15000, 18751, 22000, 33334, 200000):
        for H in range(1, most + 3):
            assert takes_split_form(shape(H, N, D), PROFILE, 20) == (H <= free or (H <= most and H * N <= keys)), (H, N)
    assert takes_split_form(shape(2, 6100, D, F=61), PROFILE, 20) and not takes_split_form(shape(2, 6200, D, F=62), PROFILE, 20)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("blocks", [(128, 64), (32, 32)])
def test_pieces_of_the_unmasked_pass_fit_the_workspace(D, blocks):
    """From 24 key tiles and frames of four on, with as many slots as the plan and the error pass hold."""
    taken = 0
    for F, P in ((1, 1600), (3, 1000), (13, 1350), (33, 3600), (40, 255), (40, 256), (80, 127), (80, 128)):
        for T, sink in ((0, 0), (0, 1), (226, 0)):
            for H in (1, 3, 12, 24, 40, 48, 96, 400, 3000):
                for t in (1, 40, 178, 328, 1191, 5000):
                    sh = shape(H, F * P + T, D, blocks, F=F, T=T, sink_first_frame=sink)
                    plan = profile_cuts(sh, t)[0]
                    n, cut = profile_pieces(sh, t)
                    if not n:
                        continue
                    taken += 1
                    assert P >= 4 * blocks[1] and n == cut.n_full + 2 + (T > 0 or sink) and n <= 11
                    assert n + cut.n_masked <= plan.slots() and cut.n_full >= 1 and 1 <= cut.n_masked <= 4
                    b = list(cut.full_bound)[:cut.n_full + 1]
                    assert b[0] == 0 and b[-1] == S.svg_tile_counts(sh)[1] and b == sorted(b)
    assert taken > 200


@pytest.mark.parametrize("D", [64, 128])
def test_error_blocks_of_a_head(D):
    """One to a pass over its rows; two passes in one block where that is less than what brings two blocks together: few parts, a second pass of
    at most three eighths, or blocks too many for tickets."""
    rows = 4096 // D
    few, four, many = shape(20, 1200, D), shape(20, 1680, D), shape(33, 2400, D, F=10)
    pieces = shape(200, 4914, D, F=6)
    assert [error_blocks(s, rows) for s in (few, four, many, pieces)] == [1, 1, 1, 1]
    for t in (rows + 1, rows * 11 // 8, rows * 11 // 8 + 1, 2 * rows):
        assert profile_cuts(few, t)[1].n_full <= 3 and profile_cuts(four, t)[1].n_full == 4 and profile_pieces(pieces, t)[0]
        two = 1 if t <= rows * 11 // 8 else 2
        assert [error_blocks(s, t) for s in (few, four, many, pieces)] == [1, two, 1, 2]
        assert [error_blocks(shape(H, 2400, D, F=10), t) for H in (31, 32)] == [two, two]
    assert [error_blocks(s, 2 * rows + 1) for s in (few, four, many, pieces)] == [3, 3, 3, 3]


@pytest.mark.parametrize("H, F, P, T, D, t, blocks, w_s, w_t, cut", [
    # up to 9 groups of rows to an XCD the temporal pass is the longest chain unless it has as many parts as there can be
    (30, 9, 1024, 0, 128, 92, (128, 64), 1, 68, (8, 4)), (14, 37, 3387, 0, 128, 112, (128, 64), 4, 338, (8, 4)), (25, 8, 982, 226, 128, 78, (128, 64), 1, 77, (7, 4)),
    (30, 34, 676, 0, 128, 229, (128, 64), 3, 92, (7, 3)), (47, 3, 2066, 0, 128, 121, (32, 32), 1, 90, (4, 2)),
    # where the windows are narrow it is not
    (8, 25, 3223, 0, 128, 805, (128, 64), 2, 40, (8, 2)), (40, 25, 834, 0, 128, 987, (128, 64), 2, 47, (5, 1)),
    # on both sides of one and two parts in the plan
    (37, 21, 1560, 0, 128, 328, (128, 64), 2, 156, (6, 2)), (40, 21, 1560, 0, 128, 328, (128, 64), 2, 156, (4, 2)), (46, 21, 1560, 0, 128, 328, (128, 64), 2, 156, (4, 2)),
    # three passes: the workspace leaves the unmasked pass three parts
    (14, 12, 491, 77, 128, 663, (128, 64), 1, 33, None)])
def test_temporal_parts_beside_the_pieces(H, F, P, T, D, t, blocks, w_s, w_t, cut):
    n, got = profile_pieces(shape(H, F * P + T, D, blocks, F=F, T=T, w_s=w_s, w_t=w_t), t)
    assert (got.n_full, got.n_masked) == cut if cut else n == 0


@pytest.mark.parametrize("most", [64, 32])
def test_blocks_of_dense_tiles(most):
    """Equal ones, but whole ones where they leave one XCD a tile to each of its 32 compute units at the most; every tile in one of them."""
    for tiles in list(range(1, 40 * most)) + [10 ** 6, 10 ** 6 + 77]:
        n, got = -(-tiles // (8 * most)), dense_cohort(tiles, most)
        left = tiles - (n - 1) * 8 * most
        assert got == (most if n > 1 and left <= 32 else -(-tiles // (8 * n))) and 1 <= got <= most and 8 * n * got >= tiles
