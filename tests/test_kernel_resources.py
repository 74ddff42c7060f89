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
    kernels = {re.sub(r"^_Z\D*\d+\w+?_N_1\d+", "", k): int(x) for k, x in scratch.items() if "sdl_gram" in k}
    names = [f"sdl_gram_kernelILi{M}E" for M in range(1, 9)] + [f"sdl_gram_pair_kernelILi{H}E" for H in range(5, 9)] + ["sdl_gram_finalizeE"]
    assert sorted(n for n in names for k in kernels if k.startswith(n)) == sorted(names) and len(kernels) == len(names)
    assert {k: x for k, x in kernels.items() if x} == {}
