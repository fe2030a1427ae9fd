"""Compiler's resource report of the one-kernel step's kernels: no instance keeps
anything in scratch memory (a private array indexed at run time goes there, and every
access to it to global memory).  CPU only: the device code is compiled, not run."""
from __future__ import annotations

import re
import subprocess

from paper_2512_01032_amd import build


def test_no_scratch_memory(tmp_path):
    # (FP32 stands for the three storage modes: the same templates, 45 s each)
    src = "k_fp32.hip"
    cmd = [build.hipcc()] + build.FLAGS + ["--cuda-device-only", "-Rpass-analysis=kernel-resource-usage",
                                           "-c", "%s/%s" % (build.CSRC, src), "-o", str(tmp_path / "k.o")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    sizes = dict(re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+)", r.stderr, re.S))
    fused = {k: int(v) for k, v in sizes.items() if "step_kernel" in k or "fused_" in k}
    assert len(fused) >= 20
    assert not {k: v for k, v in fused.items() if v}
