"""The several-token kernels keep their values in registers: no instance spills (a spill's
memory traffic would also run into the waits that count loads)."""
import os
import re

import pytest

from paper_2608_08910_amd import build


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")
def test_several_token_kernels_do_not_spill():
    asm = build.device_asm(os.path.join(build.CSRC, "tq_gemv_mfma.hip"))
    spills = dict(zip(re.findall(r"^    \.name: +(\S+)", asm, re.M), map(int, re.findall(r"\.vgpr_spill_count: +(\d+)", asm))))
    assert len(spills) >= 24 and all("k_gemv_mfma" in n for n in spills)
    assert not {n: v for n, v in spills.items() if v}
