"""What the compiler makes of the fp32 SDPA kernels: no register spilled to scratch memory (a reload
inside a tile loop waits for the tile prefetch issued before it), and a build of seconds."""
import os
import re
import subprocess

import pytest

from paper_2605_06554_amd import build


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="hipcc not installed")
def test_fp32_sdpa_kernels_do_not_spill(tmp_path):
    src = os.path.join(build.CSRC, "k_sdpa_f32.hip")
    cmd = [build.HIPCC, *build.FLAGS, "-Rpass-analysis=kernel-resource-usage", "--cuda-device-only", "-x", "hip", "-c",
           src, "-o", str(tmp_path / "f32.o")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-3000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    spills = [int(x) for x in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)]
    assert sum("bwd_f32" in n for n in names) == 3 and len(names) == len(spills) == len(scratch)
    bad = [(n, v, b) for n, v, b in zip(names, spills, scratch) if v or b]
    assert not bad, f"(kernel, spilled VGPRs, scratch bytes): {bad}"
