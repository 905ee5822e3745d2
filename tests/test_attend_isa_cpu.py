"""The check of the kernels' assembly for early reads of MFMA results, over the source it does not list elsewhere."""
import os
import subprocess

import pytest

from paper_2502_06766_amd import build as hip_build
from paper_2502_06766_amd import isa_check


@pytest.mark.skipif(not os.path.exists(hip_build.HIPCC), reason="hipcc not installed")
def test_no_mfma_result_is_read_early_in_the_rescoring_of_an_unusable_list(tmp_path):
    out = str(tmp_path / "attend.s")
    subprocess.check_call([hip_build.HIPCC, *hip_build.FLAGS, "--offload-device-only", "-S",
                           os.path.join(hip_build.CSRC, "attend.hip"), "-o", out], stderr=subprocess.DEVNULL)
    assert open(out).read().count("v_mfma") > 20
    assert not isa_check.check(out)
