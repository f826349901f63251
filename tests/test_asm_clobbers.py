"""Inline assembly in the kernels names every register that it writes by name: the compiler may keep a value
of its own in a register that is not in the clobber list."""
import glob
import os
import re

import pytest


def statements(text):
    """(template, clobber list) of every asm statement."""
    text = re.sub(r"//[^\n]*", "", text)
    for m in re.finditer(r"\basm\s*(?:volatile\s*)?\(", text):
        depth, at = 1, m.end()
        while depth:
            depth += {"(": 1, ")": -1}.get(text[at], 0)
            at += 1
        parts = re.split(r":(?=(?:[^\"]*\"[^\"]*\")*[^\"]*$)", text[m.end():at - 1])
        yield parts[0], parts[3] if len(parts) > 3 else ""


def test_the_reader_sees_operands_and_clobbers():
    got = list(statements('asm volatile("s_mov_b32 m0, %0\\n\\tx %1, off" :: "s"(f(a)), "v"(p) : "memory", "m0");'))
    assert len(got) == 1 and "m0, %0" in got[0][0] and got[0][1].split(", ")[1].strip() == '"m0"'
    assert list(statements('asm volatile("" ::: "memory");'))[0][1].strip() == '"memory"'


def test_m0_is_declared(repo_root):
    sources = glob.glob(os.path.join(repo_root, "paper_2604_19906_amd", "csrc", "*.h*"))
    found = [(os.path.basename(p), t, c) for p in sources for t, c in statements(open(p).read())
             if re.search(r"\bm0\b", t)]
    assert found
    for name, template, clobbers in found:
        assert '"m0"' in clobbers, (name, template)
