"""Host-and-device helpers of the kernels, compiled for the host and checked
on the CPU at the ends of their ranges."""

import os
import subprocess

import pytest

from paper_2608_08794_amd import build as B


def _run(tmp_path, name, body):
    """stdout of a host program built from the kernels' own headers."""
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")
    src, exe = tmp_path / f"{name}.hip", tmp_path / name
    src.write_text(body)
    r = subprocess.run([B.HIPCC, *B.FLAGS, "-O1", "--offload-host-only", str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def test_row_starts_past_2_to_the_31_elements(tmp_path):
    """The largest clips that the scorer accepts pass 2^31 elements: a gate
    GEMM tile that starts there must not wrap."""
    cases = [(0, 8), (131071, 16384), (131072, 16384), (131328, 16384), (599187, 3584), (2**31 - 256, 16384)]
    rows = ", ".join(f"{{{r}, {d}}}" for r, d in cases)
    out = _run(tmp_path, "row_start", f"""
#include <cstdio>
#include "dynamics_plan.hpp"
int main() {{
  const int c[][2] = {{{rows}}};
  for (auto& x : c) {{
    apack::GemmTileDev t{{0, x[0], x[0], 0}};
    printf("%lld %lld\\n", (long long)apack::row_start(t.m0, x[1]), (long long)apack::row_start(t.n0, x[1]));
  }}
}}
""")
    want = [[r * d] * 2 for r, d in cases]
    assert [[int(v) for v in line.split()] for line in out.splitlines()] == want
