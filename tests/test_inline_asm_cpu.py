"""No inline asm of the kernels writes a register.  The compiler puts no wait states between a matrix instruction and an asm
statement, and an asm output may get the register of an accumulator that a matrix instruction still reads or writes; an empty
asm that only hides a value from the optimiser holds no instruction."""
import glob
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCES = sorted(glob.glob(os.path.join(ROOT, "paper_2311_10090_amd", "csrc", "*.h*")))


def asm_statements(text):
    """(template, output operands) of every asm statement."""
    text = re.sub(r"//[^\n]*", "", text)
    for m in re.finditer(r"\basm\s*(?:volatile\s*)?\(", text):
        depth, end = 1, m.end()
        while depth:
            depth += {"(": 1, ")": -1}.get(text[end], 0)
            end += 1
        template, *operands = re.split(r'(?<=["\s]):', text[m.end():end - 1])
        yield "".join(re.findall(r'"([^"]*)"', template)), (operands[0].strip() if operands else "")


def test_statements_are_found():
    text = 'asm("v_mov_b32 %0, %1" : "=v"(a) : "v"(b)); asm volatile("" : "+v"(c)); asm("s_nop 0" : : "s"(f(d)) : "scc");'
    assert list(asm_statements(text)) == [("v_mov_b32 %0, %1", '"=v"(a)'), ("", '"+v"(c)'), ("s_nop 0", "")]


@pytest.mark.parametrize("path", SOURCES, ids=os.path.basename)
def test_asm_instructions_write_no_register(path):
    for template, outputs in asm_statements(open(path).read()):
        assert template.strip() == "" or outputs == "", (template, outputs)
