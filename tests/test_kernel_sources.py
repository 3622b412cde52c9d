"""Promises that the kernels' sources make to the compiler, which no run can be relied on to show broken."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2306_06446_amd", "csrc")


def parameters(text, function):
    """The parameter lists under which `function` is declared."""
    return re.findall(r"\bvoid %s\(([^{;]*?)\) \{" % function, text, flags=re.S)


def test_memory_that_a_kernel_reads_back_is_not_declared_restrict():
    """K^T V is written by ktv_block and, in the kernel of both products, read again through AddFused::kv_in."""
    text = open(os.path.join(CSRC, "additive_mfma.hip")).read()
    for function, name in (("ktv_block", "dst"), ("ktv_qkv_kernel", "kv")):
        lists = parameters(text, function)
        assert len(lists) == 1
        assert re.search(r"float \*%s\b" % name, lists[0]), (function, lists[0])


def test_hand_placed_waits_hold_for_the_compiler_too():
    """s_waitcnt is no memory access to the compiler: it stands in helpers only, between two statements that are."""
    found = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        lines = [l.strip() for l in open(path)]
        for i, l in enumerate(lines):
            if "__builtin_amdgcn_s_waitcnt" in l:
                fence = 'asm volatile("" ::: "memory");'
                assert os.path.basename(path) == "common.h" and lines[i - 1] == fence and lines[i + 1] == fence, (path, i + 1)
                found += 1
    assert found == 2
