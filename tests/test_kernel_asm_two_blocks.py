"""The kernels over pairs of query or key blocks hold 240 to 256 registers a lane: neither registers nor scalars may be spilled (36 bytes of private
memory in the loop over the lists cost a tenth of the time)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2506_19852_amd import build as hip_build
from test_kernel_asm import instructions, kernels


@pytest.mark.parametrize("source, kernel", [("radial_attn_fwd.hip", "radial_fwd_two_kernel"), ("radial_attn_fwd_fp8.hip", "radial_fwd_fp8_two_kernel"), ("radial_attn_bwd.hip", "radial_bwd_two_keys_kernel")])
def test_nothing_is_spilled(source, kernel, tmp_path):
    if not os.path.exists(hip_build.HIPCC) and shutil.which(hip_build.HIPCC) is None:
        pytest.skip("hipcc not available")
    out = tmp_path / "kernels.s"
    cmd = [hip_build.HIPCC, *hip_build.FLAGS, "--cuda-device-only", "-S", os.path.join(hip_build.CSRC, source), "-o", str(out)]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-3000:]
    text = out.read_text()
    sizes = re.findall(r"\.amdhsa_kernel (\S*" + kernel + r"\S*).*?\.amdhsa_private_segment_fixed_size (\d+)", text, re.S)
    assert len(sizes) == 1 and sizes[0][1] == "0", sizes
    bodies = [list(instructions(body)) for _, body in kernels(text.split("\n"), kernel)]
    assert len(bodies) == 1 and not [ins for ins in bodies[0] if ins.startswith(("v_writelane_b32", "scratch_"))]
