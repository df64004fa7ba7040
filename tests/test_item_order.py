"""Which item a workgroup computes follows from its id: no kernel reads the hardware's XCD number, which
would leave items out wherever a group of workgroups does not cover every XCD (a probe that only
records it excepted)."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2302_14858_amd", "csrc")


def test_no_kernel_takes_work_by_the_die_it_runs_on():
    readers = []
    for f in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(f) as fh:
            text = re.sub(r"//[^\n]*", "", fh.read())
        for m in re.finditer(r"s_getreg|XCC_ID", text):
            start = text.rfind("__global__", 0, m.start())
            readers.append((os.path.basename(f), text[start:m.start()].split("(")[0].split()[-1]))
    assert readers == [("cfd_kernels.hip", "k_xcc_probe")], readers
