"""What the compiler makes of the kernels of the cosine similarity, by its own resource report (CPU only: it cross-compiles).
A register spilled inside their streaming loops is read back behind the loads that should overlap with the arithmetic, and the
wait for it drains them."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2501_18512_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")
def test_cosine_kernels_use_no_scratch(tmp_path):
    src = next(s for s in build.SOURCES if s.endswith("sdl_cosine.hip"))
    flags = [f for f in build.FLAGS if f != "-shared"]
    out = subprocess.run([HIPCC, *flags, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", src, "-o",
                          str(tmp_path / "cosine.o")], check=True, capture_output=True, text=True).stderr
    scratch = dict(re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+)", out, re.S))
    kernels = [k for k in scratch if "sdl_gram" in k]
    assert len(kernels) >= 12 and any("mfma" in k for k in kernels)
    assert {k: int(scratch[k]) for k in kernels if int(scratch[k])} == {}
