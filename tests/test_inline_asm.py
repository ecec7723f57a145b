"""Inline assembly hides no register from the compiler: one that an instruction
writes is an output or a clobber, and m0, where a copy to LDS takes its
address from, is an operand."""

import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def blocks():
    for path in glob.glob(os.path.join(ROOT, "paper_2609_27373_amd", "csrc", "*.h*p")):
        for body in re.findall(r"asm volatile\((.*?)\);", open(path).read(), re.S):
            code = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', body.split(":")[0])).replace("\\n\\t", "\n")
            yield os.path.basename(path), code, body


def test_written_registers_are_declared():
    for path, code, body in blocks():
        clobbers = re.findall(r'"(\w+)"', body.split(":")[-1]) if body.count(":") >= 3 else []
        for ins in code.split("\n"):
            m = re.match(r"\s*[sv]_\w+\s+(m0|vcc|exec|s\[?\d+|v\[?\d+)\b", ins)
            assert not m or m.group(1) in clobbers, f"{path}: {ins.strip()}"


def test_copies_take_m0_from_the_compiler():
    copies = [(path, code, body) for path, code, body in blocks() if re.search(r"buffer_load\w*.* lds", code)]
    assert copies
    for path, code, body in copies:
        assert '"{m0}"' in body and not re.search(r"\bm0,", code), f"{path}: {code}"
