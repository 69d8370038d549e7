"""The sizes up to which a subdomain takes the block-inverse kernels, which
index with 32 bits (am_host.h, compiled with g++; no GPU code)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cstdio>
#include "am_host.h"
int main() {
  using am::tri_indexable;
  const int64_t lim = INT32_MAX;
  int bad = 0;
  auto is = [&](bool want, int64_t np, int64_t kc, int64_t ni) {
    if (tri_indexable(np, kc, ni) != want) {
      std::printf("%lld %lld %lld\n", (long long)np, (long long)kc, (long long)ni);
      ++bad;
    }
  };
  is(true, 64, 0, 0);
  is(true, 512, 1, 6);
  is(true, 4096, 64, 128);
  // couplings: 2 kc np elements
  is(true, 1 << 20, 1023, 1);
  is(false, 1 << 20, 1024, 1);
  // basis functions: ni np values
  is(true, 1 << 24, 1, 127);
  is(false, 1 << 24, 1, 128);
  // 16 columns
  is(true, (lim / 16) / 64 * 64, 1, 1);
  is(false, 1 << 27, 1, 1);
  is(false, (int64_t)1 << 40, 1, 1);
  return bad;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_tri_indexable(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(SRC)
    r = subprocess.run(["g++", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "include"), "-I",
                        os.path.join(ROOT, "paper_2607_22905_amd", "csrc"), str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
