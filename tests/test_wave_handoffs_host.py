"""LDS exchanges between the lanes of one wave in the carry-less kernels (CPU).

A wave needs no barrier for them, but the compiler does need fences: the
scheduling barrier alone leaves it free to move a load above another lane's
store of a different type.  The build shows no fault by itself, so the source
is checked: the scheduling barrier stands between a release and an acquire
fence, in one helper, and each kernel calls that helper wherever lanes read
what other lanes of their wave wrote.
"""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_1809_07592_amd", "csrc", "pa_gf2_kernels.h")

# kernel: handoffs (direct: before a chunk's words are written and before they
# are read; forward: zeros, sums, periodic form; product: halfwords to words;
# inverse: a word and its successor)
HANDOFFS = {"k_gf_direct": 2, "k_gf_fwd": 2, "k_gf_mul": 1, "k_gf_inv": 1}


def code():
    return re.sub(r"//[^\n]*", "", open(SRC).read())


def body(text, at):
    """The brace block that starts at or after `at`."""
    i = text.index("{", at)
    depth = 0
    for j in range(i, len(text)):
        depth += {"{": 1, "}": -1}.get(text[j], 0)
        if depth == 0:
            return text[i:j + 1]
    raise AssertionError("unbalanced braces")


def test_the_scheduling_barrier_stands_between_fences():
    text = code()
    helper = body(text, text.index("void wave_handoff()"))
    assert re.findall(r"__builtin_amdgcn_\w+\([^)]*\)", helper) == [
        '__builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront")',
        "__builtin_amdgcn_wave_barrier()",
        '__builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront")',
    ]
    assert text.count("__builtin_amdgcn_wave_barrier") == 1


def test_every_handoff_has_its_fence():
    text = code()
    for name, count in HANDOFFS.items():
        k = body(text, re.search(r"\b%s\(JobArgs" % name, text).end())
        assert k.count("wave_handoff();") == count, name
