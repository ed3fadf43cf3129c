"""The few-token kernels hand their sums over in LDS by stores in pairs: single ones, each with an address computation of its own, are what the compiler makes of offsets that it
cannot see to be positive, in some instances or in all."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2603_05232_amd import build


def test_sums_are_stored_in_pairs(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if shutil.which(hipcc) is None:
        pytest.skip("no hipcc")
    target = tmp_path / "gemm_skinny.s"
    subprocess.run([hipcc, *build.FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, "gemm_skinny.hip"), "-o", str(target)], check=True, stderr=subprocess.DEVNULL)
    kernels = re.findall(r"^(_ZN2ss1\dk_(?:sparse|dense)_skinny\w+):(.*?)\.Lfunc_end", target.read_text(), re.M | re.S)
    assert len(kernels) == 32
    for name, body in kernels:
        assert "ds_write2st64_b32" in body and "ds_write_b32" not in body, name
