"""Walking a CSR row's entries with int32 offsets (csrc/csr_entries.hpp): every
entry once and nothing else, rows that end at 2^31 - 1 included, and no kernel
walks entries in another way."""

import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_27373_amd", "csrc")

SRC = r"""
#include <cstdio>
#include <initializer_list>
#include "csr_entries.hpp"
int main() {
  const long long last = 2147483647;
  for (int step : {64, 128, 256, 512})
    for (long long end : {0ll, 5ll, 64ll, 1000ll, last - 600, last - 63, last - 1, last})
      for (int size : {0, 1, 2, 63, 64, 65, 127, 128, 129, 511, 512, 513, 1024}) {
        const long long beg = end - size;
        if (beg < 0) continue;
        long long want = beg;
        int steps = 0;
        for (wise::Entries e((int)beg, (int)end); e.more(); e.advance(step)) {
          if (++steps > 1024) return 1;
          for (int i = 0; i < step; ++i)
            if (e.holds(i) && e.at + (long long)i != want++) return 2;
        }
        if (want != end) return 3;
      }
  std::puts("ok");
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no C++ compiler")
def test_entries_up_to_the_last_offset(tmp_path):
    src, exe = tmp_path / "e.cpp", tmp_path / "e"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror",
                    "-I", CSRC, str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout.strip() == "ok", (res.returncode, res.stderr)


def test_kernels_walk_entries_by_it():
    """No loop or lane of a kernel compares a position with a row's end."""
    for path in glob.glob(os.path.join(CSRC, "*.hip")):
        text = open(path).read()
        assert not re.search(r"\w+ \+ (lane|tid) < end|< row_ptr\[\w+ \+ 1\]|< bound\[\w+\]", text), path
