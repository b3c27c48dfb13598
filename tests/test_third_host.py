"""The SSP-RK3 update's third (third_of, shared by host and device code) against
the division by 3, bit for bit: zeros of either sign, subnormals, the largest and
non-finite values, and random ones.  Compiled for the host; no GPU needed."""
import os
import shutil
import subprocess

import pytest

from paper_2404_03399_amd import build

PROGRAM = r"""
#include <math.h>
#include <stdio.h>
#include <string.h>
#include "adg_common.hpp"
static long bad = 0;
static void check(uint64_t u) {
  double x, y, t;
  memcpy(&x, &u, 8);
  y = adg::third_of(x);
  t = x / 3.0;
  if (t != t ? y == y : memcmp(&y, &t, 8) != 0) {
    if (bad++ < 5) printf("%a: %a, not %a\n", x, y, t);
  }
}
int main() {
  const uint64_t edges[] = {0x0ull, 0x0010000000000000ull, 0x0020000000000000ull, 0x0030000000000000ull,
                            0x7fdfffffffffffffull, 0x7ff0000000000000ull, 0x7ff8000000000000ull, 0x3ff0000000000000ull};
  for (uint64_t e : edges)
    for (long d = -2000; d <= 2000; ++d) {
      check(e + (uint64_t)d);
      check((e + (uint64_t)d) ^ 0x8000000000000000ull);
    }
  for (long i = 0; i < 1000000; ++i) check(adg::splitmix64((uint64_t)i));
  printf("%ld bad\n", bad);
  return bad != 0;
}
"""


def test_third_is_the_division(tmp_path):
    if not shutil.which("hipcc") and not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("no hipcc")
    src = tmp_path / "third.hip"
    src.write_text(PROGRAM)
    exe = str(tmp_path / "third")
    subprocess.run([build.hipcc(), "--offload-host-only", "-O2", "-ffp-contract=off", f"-I{build.CSRC}", str(src), "-o", exe],
                   check=True, capture_output=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
