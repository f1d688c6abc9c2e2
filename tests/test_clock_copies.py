"""A kernel may read a clock through the constant address space (scalar_copy)
only where it does not write the fields it reads: the compiler takes such
memory as unchanged while the kernel runs, and may load a field again after a
store to it. Read from the kernels' source."""
import os
import re

import pytest

from paper_2609_05494_amd import build as hb

SRC = open(os.path.join(hb.CSRC, "wcsph_kernels.hip")).read()


def _kernels():
    """Name and body of every kernel (a body ends at the first line that is a bare brace)."""
    for m in re.finditer(r"__global__[^;{]*?\bvoid\s+(\w+)\(", SRC):
        yield m.group(1), SRC[m.end():SRC.index("\n}\n", m.end())]


COPYING = {k: b for k, b in _kernels() if "scalar_copy(d.clk" in b}


@pytest.mark.parametrize("kernel", sorted(COPYING))
def test_no_field_is_both_copied_and_written(kernel):
    body = COPYING[kernel]
    copies = set(re.findall(r"(\w+) = scalar_copy\(d\.clk", body))
    copies |= {a for a, rhs in re.findall(r"const Clock& (\w+) = ([^;]*);", body)
               if copies & set(re.findall(r"\w+", rhs))}
    read = {f for c in copies for f in re.findall(rf"\b{c}\.(\w+)\b(?!\s*[-+|]?=[^=])", body)}
    refs = set(re.findall(r"(?<!const )Clock& (\w+) = ", body)) - copies
    written = {f for r in refs for f in re.findall(rf"\b{r}\.(\w+)\s*[-+|]?=[^=]", body)}
    written |= set(re.findall(r"atomic\w+\(&\w*\.?clk\[[^\]]*\]\.(\w+)", body))
    assert read and not read & written, (kernel, read & written)


def test_the_passes_that_copy_a_clock_are_looked_at():
    assert {"k_ghost", "k_pair"} <= set(COPYING)
