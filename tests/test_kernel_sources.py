"""Rules of the kernel sources that no run can show to be broken: code that breaks them may pass every test."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1410_7455_amd", "csrc")


def sources():
    for name in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, name)) as f:
            yield name, re.sub(r"//[^\n]*", "", f.read())


def test_wavefront_barriers_are_fenced():
    """A wave barrier does not order memory for the compiler: lanes that exchange data through LDS need a release before it
    and an acquire behind it."""
    fenced = (r'__builtin_amdgcn_fence\(__ATOMIC_RELEASE, "wavefront"\);\s*__builtin_amdgcn_wave_barrier\(\);\s*'
              r'__builtin_amdgcn_fence\(__ATOMIC_ACQUIRE, "wavefront"\);')
    seen = 0
    for name, text in sources():
        all_of_them = len(re.findall(r"__builtin_amdgcn_wave_barrier\(\)", text))
        assert all_of_them == len(re.findall(fenced, text)), name
        seen += all_of_them
    assert seen > 0


def test_no_load_in_inline_assembly():
    """The compiler takes the output of an assembly statement as written at once: with the wait in another statement it
    may use or reuse the register while the load is in flight."""
    for name, text in sources():
        assert not re.search(r'asm[^;]*"[^"]*(global|buffer|flat|ds|s)_(load|read)', text), name
