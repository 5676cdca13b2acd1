"""Inline assembly names every register it depends on: what the compiler is not told, it may change between two statements."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_25149_amd", "csrc")


def asm_statements(text):
    """The text of every asm volatile (...) in a source file, strings and operands."""
    for m in re.finditer(r"\basm\s+volatile\s*\(", text):
        depth, i, in_string = 1, m.end(), False
        while depth:
            c = text[i]
            if c == '"' and text[i - 1] != "\\":
                in_string = not in_string
            elif not in_string:
                depth += (c == "(") - (c == ")")
            i += 1
        yield text[m.end():i - 1]


@pytest.mark.parametrize("name", ["gemm_f16.hip", "gemm_mx.hip"])
def test_lds_loads_name_their_lds_address(name):
    # a global -> LDS load takes its LDS address from M0: the statement sets it itself or has it as an operand
    with open(os.path.join(CSRC, name)) as fh:
        loads = [s for s in asm_statements(fh.read()) if "global_load_lds" in s]
    assert loads
    for s in loads:
        assert "s_mov_b32 m0" in s.split("global_load_lds")[0] or '"{m0}"' in s, s


def test_no_other_file_has_such_loads():
    for path in glob.glob(os.path.join(CSRC, "*")):
        if os.path.basename(path) not in ("gemm_f16.hip", "gemm_mx.hip"):
            with open(path) as fh:
                assert not [s for s in asm_statements(fh.read()) if "global_load_lds" in s], path
