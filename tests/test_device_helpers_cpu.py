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


def test_pick_keys_have_the_order_of_doubles(tmp_path):
    """DA-FPS picks by the high words of the values and, among equal ones, by
    the low words: together they must order as the doubles do, negative values
    (every cosine above 1 by rounding) among them, and a value that underflows
    is a zero."""
    _run(tmp_path, "pick_key", r"""
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "pick_key.hpp"
using namespace apack;
int main() {
  const double eps = 0x1p-52;
  std::vector<double> v = {0.0, 5e-324, eps, 1.0, 1.0 + eps, 2.0, 12.0, INFINITY};
  // Neighbours whose magnitudes share a high word, and across a carry of the
  // low word.
  for (double w : {12.0, 0.75, 1.0, 4294967295.0, 3.0e300, 1.0e-300, 5.0})
    for (double x = w, i = 0; i < 3; ++i, x = std::nextafter(x, INFINITY)) v.push_back(pick_value(-eps, x));
  std::srand(1);
  for (int i = 0; i < 400; ++i) {
    const double x = std::ldexp(1.0 + std::rand() / (double)RAND_MAX, std::rand() % 40 - 20);
    for (double y : {x, std::nextafter(x, 0.0), x + std::ldexp(x, -31), -x}) v.push_back(y);
  }
  const size_t n = v.size();
  for (size_t i = 0; i < n; ++i) v.push_back(-v[i] == 0.0 ? 0.0 : -v[i]);
  for (double a : v)
    for (double b : v) {
      const int ha = pick_key_high(a), hb = pick_key_high(b);
      const bool less = ha != hb ? ha < hb : pick_key_low(a) < pick_key_low(b);
      if (less != (a < b)) return printf("%.17g %.17g\n", a, b), 1;
    }
  for (double z : {pick_value(-0.0, 1.0), pick_value(-eps, 0.0), pick_value(-eps, 5e-324)})
    if (z != 0.0 || std::signbit(z)) return printf("zero %g\n", z), 1;
  return 0;
}
""")
