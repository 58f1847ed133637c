"""Inline assembly tells the compiler which fixed registers it touches: one that a template names and neither the operands nor the clobbers declare may be
overwritten under a value that the compiler keeps there (M0 holds the LDS base of direct loads and the index of register-indexed moves)."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_07878_amd", "csrc")
FIXED = re.compile(r"\b(m0|vcc|exec|scc|[sv]\d+|[sv]\[\d+:\d+\])\b")


def undeclared(source):
    """(registers named in a template, rest of the statement) of each inline assembly that leaves one undeclared."""
    bad = []
    for m in re.finditer(r"\basm\b\s*(?:volatile)?\s*\((.*?)\)\s*;", source, re.S):
        template, _, rest = m.group(1).partition(":")
        bad += [(r, rest) for r in FIXED.findall(template) if f'"{r}"' not in rest and f"{{{r}}}" not in rest]
    return bad


def test_fixed_registers_of_inline_assembly_are_declared():
    files = glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))
    assert files
    for f in files:
        with open(f) as src:
            assert not undeclared(src.read()), f


def test_the_check_sees_an_undeclared_register():
    assert undeclared('asm volatile("s_mov_b32 m0, %0" ::"s"(x) : "memory");')
    assert not undeclared('asm volatile("s_mov_b32 m0, %0" ::"s"(x) : "memory", "m0");')
    assert not undeclared('asm volatile("s_nop 0\\n\\tglobal_load_lds_dwordx4 %1, %2" ::"{m0}"(l), "v"(o), "s"(b) : "memory");')
