"""k_root_build's block-shared scalars: one thread sets them and every wavefront
branches on what it read, so a barrier has to lie between any read and the next
store, or the wavefronts part ways at the following barrier."""
import os
import re

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2403_07858_amd", "csrc",
                   "bc_kernels.hip")


def kernel_text():
    text = open(SRC).read()
    start = text.index("k_root_build(RootParams prm)\n")
    text = text[start:text.index("\nhipError_t launch_root_build", start)]
    return re.sub(r"//[^\n]*", "", text)


@pytest.mark.parametrize("name", ["s_flag", "s_claimed", "s_item"])
def test_barrier_between_read_and_store(name):
    text = kernel_text()
    pending, stores, reads = None, 0, 0
    # in order of the text: barriers, plain stores, reads (not declarations or addresses taken)
    for m in re.finditer(r"__syncthreads\(\)|__shared__[^;]*;|&?\b%s\b(\s*=(?!=))?" % name, text):
        t = m.group(0)
        if t.startswith("__syncthreads"):
            pending = None
        elif t.startswith("__shared__") or t.startswith("&"):
            continue
        elif m.group(1):
            stores += 1
            assert pending is None, f"{name} is stored with no barrier after: {pending}"
        else:
            reads += 1
            pending = text[text.rfind("\n", 0, m.start()) + 1:text.find("\n", m.start())].strip()
    assert stores and reads
