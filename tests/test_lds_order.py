"""CPU check of the gfx950 code this repository builds: in the pipelined passes
a wavefront reads one row of its predecessor's from LDS between two barriers.
The compiler has moved the first row's reads past the barrier that the
predecessor's next stores wait for (two rows then stand between two barriers),
and a few sites next to the lattice's first rows came out wrong now and then;
this test keeps that order from coming back."""
import os
import re

import pytest

from test_store_form import BUILD, disassemble

# object, kernel, 128-bit LDS reads per row and wavefront
KERNELS = [("pipe.hip", "k_pipe", 7), ("batch.hip", "k_batch_pipe", 7), ("pipe_rev.hip", "k_rev_pipe", 12)]


def reads_between_barriers(asm, kernel):
    """128-bit LDS reads between consecutive barriers of the named kernels."""
    counts, inside, n = [], False, 0
    for line in asm.splitlines():
        head = re.match(r"^[0-9a-f]+ <(\S+)>:", line)
        if head:
            inside, n = bool(re.search(r"\d" + kernel + r"I", head.group(1))), 0
        elif inside and "ds_read_b128" in line:
            n += 1
        elif inside and re.match(r"^\s*s_barrier", line):
            counts.append(n)
            n = 0
    return counts


def test_parser_counts_reads():
    asm = ("0000 <_ZN1x6k_pipeILi0EEEv>:\n\tds_read_b128 v[0:3], v4\n\ts_barrier // 0\n"
           "\tds_read_b128 v[0:3], v4\n\tds_read_b128 v[0:3], v4\n\ts_barrier\n")
    assert reads_between_barriers(asm, "k_pipe") == [1, 2]


@pytest.mark.parametrize("src,kernel,row", KERNELS)
def test_one_row_of_reads_between_barriers(src, kernel, row, tmp_path):
    counts = reads_between_barriers(disassemble(os.path.join(BUILD, src + ".o"), tmp_path), kernel)
    assert counts and max(counts) == row, sorted(set(counts))
    assert set(counts) <= {0, row}, sorted(set(counts))
