"""What inline assembly has to tell the compiler."""

import glob
import os
import re

import pytest

from paper_2402_00518_amd.build import CSRC

SOURCES = sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip")))
ASM = [(os.path.basename(p), m.group(0)) for p in SOURCES
       for m in re.finditer(r"\basm volatile\((?:[^;\"]|\"[^\"]*\")*\);", open(p).read())]


def _sections(stmt):
    """(template, outputs, inputs, clobbers) of an asm statement."""
    texts = []
    bare = re.sub(r'"[^"]*"', lambda m: texts.append(m.group(0)) or f"@{len(texts) - 1}@", stmt)
    parts = [re.sub(r"@(\d+)@", lambda m: texts[int(m.group(1))], s) for s in bare.split("(", 1)[1].split(":")]
    return parts + [""] * (4 - len(parts))


def test_statements_are_found():
    assert any("global_load_lds" in s for _, s in ASM) and len(ASM) >= 4


@pytest.mark.parametrize("name,stmt", ASM, ids=[f"{n}-{i}" for i, (n, _) in enumerate(ASM)])
def test_clobbers(name, stmt):
    template, outputs, _, clobbers = _sections(stmt)
    if re.search(r"\bs_mov_b32 m0\b", template):
        assert '"m0"' in clobbers
    if "load" in template:  # in flight past the statement: no register may receive it
        assert not outputs.strip() and '"memory"' in clobbers
