"""Inline assembly names every register that it writes beside its outputs: the
compiler may otherwise keep a value there."""

import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_written_registers_are_clobbered():
    found = 0
    for path in glob.glob(os.path.join(ROOT, "paper_2609_27373_amd", "csrc", "*.h*p")) :
        for body in re.findall(r"asm volatile\((.*?)\);", open(path).read(), re.S):
            code = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', body.split(":")[0])).replace("\\n\\t", "\n")
            clobbers = re.findall(r'"(\w+)"', body.split(":")[-1]) if body.count(":") >= 3 else []
            for ins in code.split("\n"):
                m = re.match(r"\s*[sv]_\w+\s+(m0|vcc|exec|s\[?\d+|v\[?\d+)\b", ins)
                if m:
                    found += 1
                    assert m.group(1) in clobbers, f"{os.path.basename(path)}: {ins.strip()} without a clobber"
    assert found > 0
