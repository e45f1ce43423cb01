"""Waits that the kernel sources have to write out themselves.

On gfx9 a load into LDS that reads M0 must not directly follow a scalar write
of M0: one wait state (an s_nop, or any other instruction) belongs between.
The compiler inserts it between instructions of its own, never inside an
assembly string, so every string in the kernel sources is checked here.
"""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_04263_amd", "csrc")


def asm_instructions(source):
    """The instruction lists of the asm statements of a C++ source."""
    for m in re.finditer(r"\basm\s*(?:volatile)?\s*\(((?:\s*\"(?:[^\"\\]|\\.)*\")+)", source):
        text = "".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", m.group(1)))
        yield [i.strip() for i in re.split(r"\\n|;", text.replace("\\t", " ")) if i.strip()]


def m0_hazards(instructions):
    """Pairs (M0 write, LDS load) with no instruction between them."""
    writes = re.compile(r"s_\w+\s+m0\b")
    reads = re.compile(r"(?:global|buffer|scratch)_load_lds|\blds\b")
    return [(a, b) for a, b in zip(instructions, instructions[1:]) if writes.match(a) and reads.search(b)]


def test_scan_finds_a_missing_wait():
    src = 'asm volatile("s_mov_b32 m0, %0\\n\\tglobal_load_lds_dwordx4 %1, %2" : : "s"(a));'
    assert [m0_hazards(i) for i in asm_instructions(src)] == [[("s_mov_b32 m0, %0", "global_load_lds_dwordx4 %1, %2")]]


def test_no_lds_load_directly_after_an_m0_write():
    copies = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(path) as f:
            source = f.read()
        for instructions in asm_instructions(source):
            copies += any("load_lds" in i for i in instructions)
            assert not m0_hazards(instructions), f"{os.path.basename(path)}: {instructions}"
    assert copies >= 2  # the copies of the projection and the prefill kernels


def test_bare_barriers_hold_back_earlier_products():
    # __builtin_amdgcn_s_barrier alone lets the compiler sink register-only
    # products, and the wait for the LDS reads that feed them, below the barrier,
    # after which another wave's copy may overwrite what they read
    bare = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(path) as f:
            lines = f.read().splitlines()
        for i, line in enumerate(lines):
            if "__builtin_amdgcn_s_barrier()" in line:
                bare += 1
                assert any("__builtin_amdgcn_sched_barrier(0)" in x for x in lines[max(0, i - 3):i]), f"{path}:{i + 1}"
    assert bare >= 4
