"""A tile's products (float for FP32 and BF16) and its partials (double) lie in
the same LDS words.  To the compiler, accesses of different types, or by other
lanes, are independent; only a fence keeps them in order, and a bare
wave_barrier is none.  So every hand-over goes through lds_handover, which has
both."""
import os
import re

from paper_1504_06474_amd import build


def test_every_hand_over_has_its_fence():
    with open(os.path.join(build.HERE, "csrc", "sss_spmv.hip")) as f:
        src = re.sub(r"//.*", "", f.read())
    body = re.search(r"void lds_handover\(\) \{(.*?)\n\}", src, re.S).group(1)
    assert re.search(r'amdgcn_fence\(__ATOMIC_SEQ_CST, "wavefront"\);\s*__builtin_amdgcn_wave_barrier\(\);', body)
    assert src.count("__builtin_amdgcn_wave_barrier") == 1
    assert src.count("lds_handover();") >= 16
