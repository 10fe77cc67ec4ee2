"""The compiled resources of the step kernel's form for tables of both
precisions (CPU: a compile with the compiler's resource remarks), as for the
single ones: no scratch memory, no VGPR spills, at most 128 VGPRs and 4
wavefronts per SIMD for every instantiation, and LDS for two blocks on a CU."""
import os
import re
import shutil
import subprocess

import pytest


def test_step_kernel_of_both_precisions(tmp_path):
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    from paper_1309_5796_amd import build as B
    cmd = [hipcc if os.path.exists(hipcc) else "hipcc", *B.FLAGS, "-c",
           os.path.join(B.CSRC, "kernels.hip"), "-o", str(tmp_path / "k.o"),
           "-Rpass-analysis=kernel-resource-usage"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    blocks = re.split(r"remark: Function Name: ", r.stderr)[1:]
    both = [b for b in blocks if b.startswith("_ZN4mmsd12_GLOBAL__N_16k_both")]
    assert len(both) == 3, len(both)   # 4, 8 and 16 lanes per magnet row
    for b in both:
        name = b.split()[0]
        field = lambda key: int(re.search(key + r": (\d+)", b).group(1))
        assert field(r"ScratchSize \[bytes/lane\]") == 0, name
        assert field(r"VGPRs Spill") == 0, name
        assert field(r"VGPRs") <= 128, name
        assert field(r"Occupancy \[waves/SIMD\]") >= 4, name
        assert 2 * field(r"LDS Size \[bytes/block\]") <= 160 * 1024, name
