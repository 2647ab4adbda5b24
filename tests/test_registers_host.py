"""The kernels that hold their operands in registers by design spill none of them: in the grouped GEMM a spill is
reloaded once per tile, and the wait for it empties the loads that run ahead.  Checked on what the compiler reports,
without a GPU."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2310_18859_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs the HIP compiler")
@pytest.mark.parametrize("source,kernels", [
    ("grouped_ffn.hip", ("grouped_gemm_nt", "stream_gemm_nt")),
    ("hash_fn.hip", ("hash_recurrence", "hash_lstm", "hash_dense", "hash_attention", "hash_heads")),
])
def test_no_spills(source, kernels):
    out = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-x", "hip", "-Xclang", "-target-feature",
                          "-Xclang", "-packed-fp32-ops", "-I" + os.path.join(build.ROOT, "include"), "-I" + build.CSRC,
                          "--cuda-device-only", "-c", "-Rpass-analysis=kernel-resource-usage", "-o", os.devnull,
                          os.path.join(build.CSRC, source)], capture_output=True, text=True, check=True).stderr
    scratch = {}
    for name, rest in re.findall(r"Function Name: (\S+)(.*?)(?=Function Name:|\Z)", out, re.S):
        scratch[name] = int(re.search(r"ScratchSize \[bytes/lane\]: (\d+)", rest).group(1))
    for kernel in kernels:
        mine = {n: s for n, s in scratch.items() if kernel in n}
        assert mine, f"{kernel} is not among {sorted(scratch)}"
        assert not any(mine.values()), {n: s for n, s in mine.items() if s}
