"""The generated-code check of test_isa_hazards on every source with matrix
instructions that it and test_eig_hazards do not list."""
import os
import re
import shutil

import pytest

from paper_1703_00387_amd import build as B
from test_isa_hazards import MFMA_SOURCES, _compile, short_reads, short_vgpr_reads


def _others():
    names = []
    for path in B.sources():
        name = os.path.basename(path)
        if name not in MFMA_SOURCES + ["eig.hip"] and re.search(r'"mfma_\w+\.h"|amdgcn_mfma', open(path).read()):
            names.append(name)
    return names


def test_the_expectation_values_are_among_them():
    assert "observe.hip" in _others()


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not installed")
@pytest.mark.parametrize("name", _others())
def test_no_mfma_result_read_inside_its_latency(tmp_path, name):
    text = open(_compile(os.path.join(B.CSRC, name), str(tmp_path))).read()
    kernels = [m.group(0) for m in re.finditer(r"^(_Z\w+):.*?s_endpgm", text, re.M | re.S)]
    assert name != "observe.hip" or sum(k.count("v_mfma") for k in kernels) > 0
    found = [x for k in kernels for x in short_reads(k) + short_vgpr_reads(k)]
    assert not found, found[:5]
