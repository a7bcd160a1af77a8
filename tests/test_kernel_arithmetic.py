"""The kernels' time arithmetic on the values that lanes hold whose result nobody looks at, on the CPU."""
import os
import subprocess

from paper_2503_20591_amd import build

NEVER = 2**31 - 1

PROGRAM = r"""
#include "nbos_common.hpp"
#include <stdio.h>
int main() {
  int a, b, c;
  while (scanf("%d %d %d", &a, &b, &c) == 3) {
    printf("%d %d %d %d ", wrap_add(a, b), next_event_time(a, b, c), retry_time(a, b, c), job_finish(a, b));
    printf("%d\n", add_in_range(a & NEVER, b & NEVER));
  }
  return 0;
}
"""


def wrapped(v):
    return (v + 2**31) % 2**32 - 2**31


def test_times_of_unselected_lanes_are_defined(tmp_path):
    # every lane works these sums out; where a lane has no timer its time is NEVER, the rest of the timer what is left
    # of another one, and a signed sum would be undefined there: compiled for the host, any such sum traps
    src, exe = tmp_path / "times.hip", tmp_path / "times"
    src.write_text(PROGRAM)
    check = "signed-integer-overflow"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-host-only", "-std=c++17", "-O1",
                    "-I", os.path.dirname(build.SRC), "-Xarch_host", "-fsanitize=" + check,
                    "-Xarch_host", "-fsanitize-trap=" + check, "-o", str(exe), str(src)], check=True, capture_output=True)
    rows = [(5_000, 2_000, 60_000), (0, 1, 0), (NEVER - 3, 1, 1),            # timers and cells as they are
            (NEVER, 0x0FFFFFFF, NEVER), (NEVER, 1, 0), (NEVER - 1, 0x0FFFFFFF, -1), (NEVER, 16, NEVER), (-1, -1, -1),
            (NEVER - 60_000, 59_999, 0), (NEVER - 60_000, 60_000, 0), (NEVER - 60_000, 60_001, 0),       # a host asked for late
            (86_400_000, NEVER, 0), (NEVER - 1, -2**31, 1)]                  # an earlier job's start, an END event's duration
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, r)) for r in rows), text=True, capture_output=True, check=True)
    got = [tuple(map(int, line.split())) for line in out.stdout.splitlines()]
    assert got == [(wrapped(a + b), wrapped(a + b + c), wrapped(a + b * c), wrapped(a + b),
                    min((a & NEVER) + (b & NEVER), NEVER)) for a, b, c in rows]
