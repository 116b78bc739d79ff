"""What the compiler does not check in hand-written assembly: m0 is the
compiler's own register (a claim of it in an asm statement is not kept), so a
statement that sets m0 saves it first and gives it back, and a load to LDS,
which reads its address from m0, sets m0 in the same statement."""
import glob
import os
import re

import pytest

import paper_2606_19849_amd as vico

SOURCES = sorted(glob.glob(os.path.join(os.path.dirname(vico.__file__), "csrc", "*.h*")))


def _statements(text):
    """The instruction lists of the asm statements of a source."""
    for m in re.finditer(r"\basm\s+volatile\s*\(((?:\s*\"(?:[^\"\\]|\\.)*\")+)", text):
        code = "".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", m.group(1)))
        yield [i.strip() for i in code.replace("\\t", " ").split("\\n") if i.strip()]


@pytest.mark.parametrize("path", SOURCES, ids=[os.path.basename(p) for p in SOURCES])
def test_m0_is_given_back(path):
    for code in _statements(open(path).read()):
        sets = [i for i, x in enumerate(code) if re.match(r"s_mov_b32 m0,", x)]
        loads = [i for i, x in enumerate(code) if x.endswith(" lds")]
        assert not any("m0" in x and not re.match(r"s_mov_b32 (m0, %\d+|%\d+, m0)$", x) for x in code), code
        if loads:
            assert sets and sets[0] < loads[0], code
        if sets:
            saved = [re.match(r"s_mov_b32 (%\d+), m0$", x) for x in code[:sets[0]]]
            saved = [m.group(1) for m in saved if m]
            assert len(saved) == 1 and code[sets[-1]] == f"s_mov_b32 m0, {saved[0]}", code


def test_the_chunk_kernel_is_seen():
    path = [p for p in SOURCES if p.endswith("attn_fwd.hip")][0]
    assert sum(any(x.endswith(" lds") for x in c) for c in _statements(open(path).read())) == 2
