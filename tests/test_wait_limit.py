"""The limit of a device-side wait (csrc/wait.h, host build): a wait that keeps
moving never ends however long the launch lasts, one that stalls ends one limit
after its last movement, and one told of no movement ends one limit after the
launch began."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include "wait.h"
// Polls every `step` ticks from t0 on, moving every `every`-th poll up to tick
// `until`; the tick at which the wait ends (0: not within `end` ticks).
static unsigned long long run(unsigned long long t0, bool whole, unsigned long long limit, unsigned step,
                              unsigned every, unsigned long long until, unsigned long long end) {
  WaitLimit w{t0, !whole};
  unsigned long long now = t0;
  for (unsigned i = 1; now < t0 + end; ++i) {
    now += step;
    if (!whole && i % every == 0 && now <= t0 + until) w.moved = true;
    if (w.expired(now, limit)) return now - t0;
  }
  return 0;
}
int main() {
  const unsigned long long t0s[] = {0, 1ull << 40};
  for (unsigned long long t0 : t0s) {
    if (run(t0, false, 1000, 7, 100, 200000, 200000)) return 1;        // moves every 700 ticks for 200 limits
    const unsigned long long e = run(t0, false, 1000, 7, 100, 50000, 200000);  // then stops at 50,000
    if (e < 50000 + 1000 - 700 || e > 50000 + 1000 + 2 * 7) return 2;
    const unsigned long long s = run(t0, false, 1000, 7, 1, 0, 200000);  // never moves: from the first look on
    if (s <= 1000 || s > 1000 + 3 * 7) return 3;
    const unsigned long long l = run(t0, true, 1000, 7, 1, 200000, 200000);  // limit on the whole launch
    if (l <= 1000 || l > 1000 + 7) return 4;
  }
  std::puts("OK");
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_wait_limit(tmp_path):
    src, exe = tmp_path / "wait.cpp", tmp_path / "wait"
    src.write_text(DRIVER)
    inc = os.path.join(ROOT, "paper_2206_05843_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I" + inc, str(src), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.returncode
