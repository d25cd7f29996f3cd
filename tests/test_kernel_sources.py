"""What the compiler has to be told about the hand-written instructions, checked on the kernel sources: it sees neither the
registers an inline instruction overwrites nor that a barrier orders LDS reads after other wavefronts' copies."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_12598_amd", "csrc")
FILES = sorted(f for f in os.listdir(CSRC) if f.endswith((".h", ".hip")))


def _code(name):
    return re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, name)).read())


def _asm_statements(name):
    """The operand text of every asm statement, parentheses balanced."""
    code = _code(name)
    for m in re.finditer(r"\basm\s*(?:volatile\s*)?\(", code):
        depth, i, quoted = 1, m.end(), False
        while depth:
            c = code[i]
            if c == '"':
                quoted = not quoted
            elif not quoted:
                depth += {"(": 1, ")": -1}.get(c, 0)
            i += 1
        yield code[m.end():i - 1]


@pytest.mark.parametrize("name", FILES)
def test_inline_instructions_name_m0_as_overwritten(name):
    for text in _asm_statements(name):
        if re.search(r"\bs_mov_b32\s+m0\b", text):
            assert '"m0"' in text, text


@pytest.mark.parametrize("name", FILES)
def test_reads_of_copied_lds_cannot_pass_the_barrier(name):
    # kernels that copy memory straight into LDS: the barrier is part of a statement that memory accesses do not pass
    if not any(" lds" in text for text in _asm_statements(name)):
        return
    assert "__builtin_amdgcn_s_barrier" not in _code(name)
    barriers = [text for text in _asm_statements(name) if "s_barrier" in text]
    assert barriers and all('"memory"' in text for text in barriers)
