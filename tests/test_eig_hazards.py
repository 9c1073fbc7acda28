"""The generated-code check of test_isa_hazards on the direct rotation's kernels."""
import os
import re
import shutil

import pytest

from paper_1703_00387_amd import build as B
from test_isa_hazards import _compile, short_reads, short_vgpr_reads


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not installed")
def test_no_mfma_result_read_inside_its_latency(tmp_path):
    text = open(_compile(os.path.join(B.CSRC, "eig.hip"), str(tmp_path))).read()
    kernels = [m.group(0) for m in re.finditer(r"^(_Z\w+):.*?s_endpgm", text, re.M | re.S)]
    assert sum(k.count("v_mfma") for k in kernels) > 100
    found = [x for k in kernels for x in short_reads(k) + short_vgpr_reads(k)]
    assert not found, found[:5]
