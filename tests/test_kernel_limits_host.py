"""Kernel attributes are properties of a kernel on a device, shared by all
threads and captured graphs: they are set where the kernels are loaded
(preload_*), to a constant, and nowhere else in the library's sources."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1401_7441_amd", "csrc")


def test_kernel_attributes_are_set_only_when_kernels_are_loaded():
    found = 0
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith((".hip", ".cpp", ".h")):
            continue
        src = open(os.path.join(CSRC, name)).read()
        for m in re.finditer(r"hipFuncSetAttribute\(([^;]*?)\)\)", src):
            found += 1
            # the last function that opens at the start of a line before the call
            head = re.findall(r"^(?:\w[\w:<>*& ]*) (\w+)\([^;{]*\{", src[:m.start()], re.M)[-1]
            assert head.startswith("preload_"), (name, head)
            assert re.search(r"\(int\)k\w+\)?", m.group(1)), (name, m.group(1))
    assert found > 0
