"""Checks on the text of the HIP sources, for rules that no run can show to be kept."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2411_00850_amd", "csrc")


def asm_statements(text):
    """The operand lists of the inline-asm statements in `text`, comments removed."""
    text = re.sub(r"//[^\n]*|/\*.*?\*/", "", text, flags=re.S)
    for m in re.finditer(r"\basm\s*(?:volatile\s*)?\(", text):
        depth, at, quoted = 1, m.end(), False
        while depth:
            c = text[at]
            if c == "\\":
                at += 1
            elif c == '"':
                quoted = not quoted
            elif not quoted:
                depth += (c == "(") - (c == ")")
            at += 1
        yield text[m.end():at - 1]


def loads_in_flight(text):
    """Inline-asm loads into registers that do not wait for them before the statement ends."""
    load = re.compile(r"\b(?:global|flat|buffer|scratch|ds|s)_(?:load|read)_(?!lds)\w+[^\"]*")
    return [a for a in asm_statements(text) if any("_lds_" not in m for m in load.findall(a)) and "s_waitcnt" not in a]


@pytest.mark.parametrize("name", sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".h"))))
def test_asm_loads_wait_in_their_own_statement(name):
    """The compiler takes the output registers of an asm statement as written when it ends: it may copy, spill or reuse
    them while a load inside is still on its way, and nothing would say so."""
    assert loads_in_flight(open(os.path.join(CSRC, name)).read()) == []


def test_the_check_tells_the_forms_apart():
    bad = 'asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(piece[i]) : "v"(off), "s"(base) : "memory");'
    good = ['asm volatile("global_load_ushort %0, %1, off\\n\\ts_waitcnt vmcnt(0)" : "=v"(v) : "v"(p) : "memory");',
            'asm volatile("s_mov_b32 m0, %0\\n\\ts_nop 0\\n\\tglobal_load_lds_dwordx4 %1, %2" ::"s"(d), "v"(o), "s"(b) : "memory");',
            'asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");  // asm("global_load_dword")']
    assert len(loads_in_flight(bad)) == 1 and not any(loads_in_flight(g) for g in good)


@pytest.mark.parametrize("name", sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".h"))))
def test_wave_barriers_order_memory(name):
    """Lanes of a wave that hand data to each other through the LDS need no wait, but the barrier of a wave orders no memory
    accesses for the compiler: it stands between fences of the wave's scope."""
    text = re.sub(r"//[^\n]*|/\*.*?\*/", "", open(os.path.join(CSRC, name)).read(), flags=re.S)
    fenced = (r'__builtin_amdgcn_fence\(__ATOMIC_RELEASE, "wavefront"\);\s*__builtin_amdgcn_wave_barrier\(\);\s*'
              r'__builtin_amdgcn_fence\(__ATOMIC_ACQUIRE, "wavefront"\);')
    assert "__builtin_amdgcn_wave_barrier" not in re.sub(fenced, "", text)
