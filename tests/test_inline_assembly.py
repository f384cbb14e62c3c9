"""Inline assembly of the kernels (read as text, no GPU): a special register that a statement writes is among its clobbers,
as the compiler may keep a value of its own there."""
import glob
import os
import re

import pytest

import paper_2503_17922_amd as W

CSRC = os.path.join(os.path.dirname(os.path.abspath(W.__file__)), "csrc")
SOURCES = sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h")))


def statements(text):
    """(template, clobbers) of every asm statement."""
    for m in re.finditer(r"\basm\s*(?:volatile)?\s*\(", text):
        depth, i, quoted = 1, m.end(), False
        while depth:                                     # to the closing parenthesis, strings skipped
            c = text[i]
            if c == "\\" and quoted:
                i += 1
            elif c == '"':
                quoted = not quoted
            elif not quoted:
                depth += (c == "(") - (c == ")")
            i += 1
        body = text[m.end():i - 1]
        parts, at, quoted = [], 0, False
        for j, c in enumerate(body):                     # template : outputs : inputs : clobbers
            if c == '"' and body[j - 1] != "\\":
                quoted = not quoted
            elif c == ":" and not quoted:
                parts.append(body[at:j])
                at = j + 1
        parts.append(body[at:])
        yield parts[0], parts[3] if len(parts) > 3 else ""


@pytest.mark.parametrize("path", SOURCES, ids=os.path.basename)
def test_special_registers_written_are_clobbers(path):
    for template, clobbers in statements(open(path).read()):
        for line in re.findall(r'"([^"]*)"', template):
            for instruction in re.split(r"\\n(?:\\t)?|;", line):
                written = re.match(r"\s*[sv]_\w+\s+(m0|vcc|exec|scc)\b", instruction)
                assert not written or f'"{written[1]}"' in clobbers, f"{instruction!r} without its clobber"


def test_the_statements_are_found():
    text = open(os.path.join(CSRC, "wkv_score.hip")).read()
    found = list(statements(text))
    assert len(found) == len(re.findall(r"\basm volatile\(", text)) and sum("m0" in t for t, _ in found) >= 1
