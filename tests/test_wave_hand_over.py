"""The lanes of a wave pass data through LDS in pconv_small.hip without a barrier of the workgroup; the hardware keeps a wave's
LDS accesses in order, the compiler has to be told.  Read from the source: no run can show what a compiler may reorder."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2001_07710_amd", "csrc")


def test_every_hand_over_of_a_patch_is_ordered():
    src = open(os.path.join(CSRC, "pconv_small.hip")).read()
    src = re.sub(r"//[^\n]*", "", src)
    fence = re.search(r"auto hand_over = \[\] \{(.*?)\};", src, flags=re.S)
    assert fence, "no hand_over()"
    assert '__builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront")' in fence.group(1)
    assert "__builtin_amdgcn_wave_barrier()" in fence.group(1)
    body = re.search(r"auto multiply = \[&\]\(int b, auto more\) \{(.*?)\n    \};", src, flags=re.S).group(1)
    events = re.findall(r"write_patch\(\)|hand_over\(\)|read_b\(", body)
    assert events[:2] == ["write_patch()", "hand_over()"], "pieces are read before they are known to be written"
    assert events[-1] == "hand_over()", "the next block's pieces may overtake this block's reads"
    assert src.count("write_patch();") == body.count("write_patch();") == 1
