"""Inline assembly of the kernels: what a statement writes beside its operands stands in its clobber list.  Nothing else tells the
compiler that a value of its own is gone."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2409_17870_amd", "csrc")
SOURCES = sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip")))
STRINGS = r'"(?:[^"\\]|\\.)*"'


def statements(text):
    for m in re.finditer(r"\basm(?:\s+volatile)?\s*\(", text):
        depth, at = 1, m.end()
        while depth:
            depth += {"(": 1, ")": -1}.get(text[at], 0)
            at += 1
        yield text[m.end():at - 1]


@pytest.mark.parametrize("path", SOURCES, ids=os.path.basename)
def test_named_registers_are_clobbered(path):
    for body in statements(open(path).read()):
        template = re.match(r"(?:\s*%s)+" % STRINGS, body)
        if template is None:
            continue
        code = "".join(re.findall(STRINGS, template.group(0))).replace('"', " ").replace("\\n\\t", "\n").replace("\\n", "\n")
        written = {m.group(1) for m in re.finditer(r"^\s*[sv]_\w+\s+(m0|vcc|exec|s\d+|v\d+)\b", code, re.M)}
        clobbers = re.findall(STRINGS, body[template.end():])
        assert all('"%s"' % r in clobbers for r in written), body
