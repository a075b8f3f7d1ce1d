"""The rules by which the library chooses the form of a kernel and the cut of a profiling call (host side, no GPU)."""
import pytest

import paper_2502_01776_amd as S
from workloads import get_config
from helpers import PROFILE, profile_cuts, takes_split_form


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
