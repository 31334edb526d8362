"""A counter summary counts only for the sources it was taken on: the hash over
them has to cover all that the Leja kernels are compiled from (CPU)."""
import os
import re

from paper_2310_08344_amd.profsummary import CSRC, SWEEP_SOURCES


def test_the_source_hash_covers_every_header_of_the_leja_kernels():
    todo, seen = ["kernels.hip", "pair.hip", "block.hip", "stream.hip", "rtile.hip"], set()
    while todo:
        name = todo.pop()
        if name in seen:
            continue
        seen.add(name)
        with open(os.path.join(CSRC, name)) as f:
            todo += re.findall(r'#include "([^"]+)"', f.read())
    assert seen <= set(SWEEP_SOURCES), seen - set(SWEEP_SOURCES)
