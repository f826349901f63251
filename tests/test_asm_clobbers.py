"""Inline assembly in the kernels leaves registers that it is not given alone: a load straight to LDS takes
its address through an operand tied to m0, and no statement writes m0 itself (the compiler may keep a
value of its own there, and takes no clobber of a reserved register)."""
import glob
import os
import re


def statements(text):
    """(template, operands) of every asm statement."""
    text = re.sub(r"//[^\n]*", "", text)
    for m in re.finditer(r"\basm\s*(?:volatile\s*)?\(", text):
        depth, at = 1, m.end()
        while depth:
            depth += {"(": 1, ")": -1}.get(text[at], 0)
            at += 1
        template, _, operands = text[m.end():at - 1].partition(":")
        yield template, operands


def test_the_reader_splits_statements():
    got = list(statements('asm volatile("x %1, off" :: "{m0}"(f(a)), "v"(p) : "memory"); asm("" : "+s"(A));'))
    assert got == [('"x %1, off" ', ': "{m0}"(f(a)), "v"(p) : "memory"'), ('"" ', ' "+s"(A)')]


def test_m0_is_an_operand(repo_root):
    loads = 0
    for path in glob.glob(os.path.join(repo_root, "paper_2604_19906_amd", "csrc", "*.h*")):
        for template, operands in statements(open(path, encoding="utf-8").read()):
            assert not re.search(r"\bm0\b", template), (path, template)
            if re.search(r"_load\w*_lds_", template):
                assert '"{m0}"' in operands, (path, template)
                loads += 1
    assert loads == 2
