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


def _unnamed(text):
    """Registers that the instructions of an asm statement write without naming them as overwritten: m0 as a scalar instruction's
    destination, the condition bit of scalar arithmetic, comparisons and logic."""
    out = []
    if re.search(r"\bs_\w+\s+m0\b", text) and '"m0"' not in text:
        out.append("m0")
    if re.search(r"\bs_(add|sub|min|max|and|or|xor|not|nand|nor|xnor|lshl|lshr|ashr|bfe|abs|cmp|bitcmp)\w*_[iub](32|64)\b", text) and '"scc"' not in text:
        out.append("scc")
    return out


@pytest.mark.parametrize("name", FILES)
def test_inline_instructions_name_what_they_overwrite(name):
    for text in _asm_statements(name):
        assert not _unnamed(text), text


def test_the_statements_that_copy_into_lds_are_seen():
    writes = [text for text in _asm_statements("gemm_dma.h") if re.search(r"\bs_\w+\s+m0\b", text)]
    assert len(writes) == 2 and all(" lds" in text for text in writes)


@pytest.mark.parametrize("text,missing", [
    ('"s_mov_b32 m0, %0" :: "s"(a) : "memory", "m0"', []), ('"s_mov_b32 m0, %0" :: "s"(a) : "memory"', ["m0"]),
    ('"s_add_u32 m0, %0, %1" :: "s"(a), "n"(b) : "m0", "scc"', []), ('"s_add_u32 m0, %0, %1" :: "s"(a), "n"(b) : "m0"', ["scc"]),
    ('"s_add_u32 m0, %0, %1" :: "s"(a), "n"(b) : "memory"', ["m0", "scc"]), ('"s_lshl_b32 m0, %0, 2" :: "s"(a)', ["m0", "scc"]),
    ('"s_cmp_lt_i32 %0, %1" :: "s"(a), "s"(b)', ["scc"]), ('"s_and_b64 %0, %1, %2" : "=s"(c) : "s"(a), "s"(b)', ["scc"]),
    ('"s_nop 3"', []), ('"s_waitcnt vmcnt(0)\\n\\ts_barrier" ::: "memory"', []),
])
def test_what_the_check_sees(text, missing):
    assert _unnamed(text) == missing


@pytest.mark.parametrize("name", FILES)
def test_reads_of_copied_lds_cannot_pass_the_barrier(name):
    # kernels that copy memory straight into LDS: the barrier is part of a statement that memory accesses do not pass
    if not any(" lds" in text for text in _asm_statements(name)):
        return
    assert "__builtin_amdgcn_s_barrier" not in _code(name)
    barriers = [text for text in _asm_statements(name) if "s_barrier" in text]
    assert barriers and all('"memory"' in text for text in barriers)
