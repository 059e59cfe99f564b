"""Registers of kernels whose speed depends on how many waves share a SIMD, as the compiler reports them (no GPU needed)."""
import os
import re
import subprocess

import pytest

from paper_2504_18082_amd import build

pytestmark = pytest.mark.skipif(not os.path.exists(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")), reason="needs hipcc")


def test_weight_gradient_leaves_room_for_three_waves(tmp_path):
    """The weight gradient of four waves, alone and next to the input gradient's product: both are bound by memory round trips."""
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + build.FLAGS + ["-Rpass-analysis=kernel-resource-usage", "--cuda-device-only", "-c",
           os.path.join(build.CSRC, "linear.hip"), "-o", str(tmp_path / "linear.o")]
    run = subprocess.run(cmd, capture_output=True, text=True)
    assert run.returncode == 0, run.stderr
    waves = dict(re.findall(r"Function Name: \w*?(gemm_\w+_kernel)E?N.*?Occupancy \[waves/SIMD\]: (\d+)", run.stderr, re.S))
    assert int(waves["gemm_tn_kernel"]) >= 3 and int(waves["gemm_tn_nt_kernel"]) >= 3, waves
