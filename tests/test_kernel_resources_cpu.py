"""Registers of the score kernels, from the compiler's resource report."""

import os
import re
import subprocess

import pytest

from paper_2608_08794_amd import build


@pytest.fixture(scope="module")
def prune_kernels(tmp_path_factory):
    """{mangled name: scratch bytes a lane} of the kernels of prune.hip."""
    out = tmp_path_factory.mktemp("resources") / "prune.o"
    r = subprocess.run([build.HIPCC, *build.FLAGS, "-Rpass-analysis=kernel-resource-usage", "--cuda-device-only", "-c",
                        os.path.join(build.CSRC, "prune.hip"), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    found = re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+)", r.stderr, re.S)
    return {name: int(scratch) for name, scratch in found}


@pytest.mark.parametrize("kernel", ["k_rowstats", "k_few_logits"])
def test_the_first_score_kernels_hold_no_scratch(prune_kernels, kernel):
    # Two descriptor sources in one kernel had cost k_rowstats 28 bytes a lane.
    mine = {n: s for n, s in prune_kernels.items() if kernel in n}
    assert mine
    assert not {n: s for n, s in mine.items() if s}
