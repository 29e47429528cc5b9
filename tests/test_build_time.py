"""Every source compiles in minutes: whoever builds the library waits for the slowest of them."""
import glob
import os
import subprocess

import pytest

from paper_2505_21467_amd import build

LIMIT_S = 240  # the slowest takes 47 s on one core, and took 1000 and more with its loops written as recursive templates


@pytest.mark.parametrize("src", [os.path.basename(p) for p in sorted(glob.glob(os.path.join(build.CSRC, "*.hip")))])
def test_source_compiles_in_minutes(src, tmp_path):
    cmd = [build.HIPCC, *build.FLAGS, "-c", os.path.join(build.CSRC, src), "-o", str(tmp_path / "out.o")]
    subprocess.run(cmd, check=True, capture_output=True, timeout=LIMIT_S)
