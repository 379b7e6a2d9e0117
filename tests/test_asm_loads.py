"""Loads written in inline asm.  The compiler takes an asm statement's output registers as written when it ends: a load that
is still on its way may then be copied or spilled before it arrives, or land on a register that is in use for something
else.  Such a statement therefore waits itself; loads that name no output register (global memory to LDS) need not."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_18145_amd", "csrc")
LOAD = re.compile(r"\b(?:global|flat|buffer|scratch|s|s_buffer)_load_\w+|\bds_read\w*|\bds_load\w*")
STRING = re.compile(r'"((?:[^"\\]|\\.)*)"')


def asm_statements(text):
    """(template, operand text) of every asm statement."""
    for m in re.finditer(r"\basm\s*(?:volatile)?\s*\(", text):
        depth, i, quoted = 1, m.end(), False
        while depth:
            c = text[i]
            if c == "\\" and quoted:
                i += 1
            elif c == '"':
                quoted = not quoted
            elif not quoted:
                depth += {"(": 1, ")": -1}.get(c, 0)
            i += 1
        body = text[m.end():i - 1]
        at = 0
        while True:                                # the adjacent strings that make up the template
            s = re.match(r"\s*" + STRING.pattern, body[at:])
            if not s:
                break
            at += s.end()
        template = "".join(STRING.findall(body[:at]))
        yield re.sub(r"\\[nt]", " ", template), body[at:]


def unwaited(text):
    bad = []
    for template, operands in asm_statements(text):
        parts = operands.split(":")
        outputs = parts[1] if len(parts) > 1 else ""
        loads = list(LOAD.finditer(template))
        if loads and '"' in outputs and "s_waitcnt" not in template[loads[-1].end():]:
            bad.append(template)
    return bad


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.h*"))), ids=os.path.basename)
def test_asm_loads_into_registers_wait(path):
    with open(path) as f:
        assert unwaited(f.read()) == []


def test_the_scan_finds_them():
    assert unwaited('asm volatile("global_load_dword %0, %1, %2" : "=v"(v) : "v"(o), "s"(p) : "memory");')
    assert unwaited('asm("s_waitcnt vmcnt(0)\\n\\tds_read_b32 %0, %1" : "=v"(v) : "v"(o));')
    assert not unwaited('asm volatile("global_load_dword %0, %1, off\\n\\t" "s_waitcnt vmcnt(0)" : "=v"(v) : "v"(p));')
    assert not unwaited('asm volatile("s_mov_b32 m0, %0\\n\\tglobal_load_lds_dwordx4 %1, %2" :: "s"(a), "v"(o), "s"(p));')
