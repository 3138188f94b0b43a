"""The other HIP sources too: no register spills and no scratch (which is device memory the runtime may have to
allocate during a launch, also in the entry point that promises to allocate none)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2603_02207_amd.build import CSRC, HIPCC_FLAGS, ROOT, SOURCES, hipcc


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                    reason="hipcc not available")
@pytest.mark.parametrize("source", [s for s in SOURCES if s.endswith(".hip") and s not in ("kernels.hip", "api.hip")])
def test_kernels_of_every_source_use_no_scratch(source, tmp_path):
    cmd = [hipcc()] + HIPCC_FLAGS + ["-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "hip", "-c",
                                     os.path.join(CSRC, source), "-o", str(tmp_path / "k.o"),
                                     "-Rpass-analysis=kernel-resource-usage"]
    out = subprocess.run(cmd, capture_output=True, text=True)
    assert out.returncode == 0, out.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", out.stderr)
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", out.stderr)]
    spills = [int(x) for x in re.findall(r"VGPRs Spill: (\d+)", out.stderr)]
    assert names and len(names) == len(scratch) == len(spills)
    bad = [(n, s, p) for n, s, p in zip(names, scratch, spills) if s or p]
    assert not bad, bad
