"""The names chopper_time_kernel takes are those of the kernels that the
sources launch."""
import glob
import os
import re

from conftest import ROOT


def test_names_are_the_launched_kernels():
    import paper_2512_08242_amd as ch
    text = ""
    for ext in ("hip", "h"):
        for f in glob.glob(os.path.join(ROOT, "paper_2512_08242_amd", "csrc",
                                        "*." + ext)):
            with open(f) as fh:
                text += fh.read()
    launched = set(re.findall(r'\blaunch(?:_shm)?\(\s*"(\w+)"', text))
    names = list(ch.binding.kernel_names())
    assert len(names) == len(set(names))
    assert set(names) == launched
