"""The checks of test_isa_waits on the kernels with two teams of wavefronts (CPU only)."""
import os
import re
import subprocess

import pytest

from paper_2502_01776_amd import build as B
from test_isa_waits import WAIT_STATES, parse

pytestmark = pytest.mark.skipif(not os.path.exists(B.hipcc_path()), reason="needs hipcc")


def test_direct_loads_of_both_teams(tmp_path):
    """Settled scalar registers, m0 for the loads only, the tiles of two teams alone in LDS, nothing spilled."""
    out = str(tmp_path / "kernels.s")
    subprocess.run([B.hipcc_path(), *B.compile_flags(), "--offload-device-only", "-S", os.path.join(B.CSRC, "svg_teams.hip"), "-o", out],
                   check=True, capture_output=True)
    text = open(out).read()
    size = dict(re.findall(r"\.amdhsa_kernel (\w+)\n\s*\.amdhsa_group_segment_fixed_size (\d+)", text))
    kernels = parse(text)
    assert len(kernels) == 8      # four passes, two head dimensions; never more than 64 heads
    for k in kernels:
        pred = k.predecessors()
        assert k.direct_loads() and min(k.nearest_vector_write(at, pred) for at in k.direct_loads()) >= WAIT_STATES, k.name
        assert not [i for i in k.ins if (not i[2] and "m0" in i[1]) or i[0].startswith(("v_accvgpr", "scratch_"))], k.name
        D = int(re.search(r"11attn_kernelILi(\d+)E", k.name).group(1))
        assert int(size[k.name]) == 2 * 2 * 2 * 64 * D * 2, k.name
