"""CPU check of the gfx950 code this repository builds: where a wavefront of the
pipelined passes reaches a barrier, every LDS read that it issued has returned,
so that the wavefront which may then store to those words cannot overtake it."""
import os
import re

import pytest

from test_store_form import BUILD, disassemble

KERNELS = [("pipe.hip", "k_pipe"), ("batch.hip", "k_batch_pipe"), ("pipe_rev.hip", "k_rev_pipe"),
           ("ribbon_tile.hip", "k_ribbon_tile")]


def reads_in_flight(asm, kernel):
    """LDS reads that may be in flight at each barrier of the named kernels."""
    out, inside, flying = [], False, 0
    for line in asm.splitlines():
        head = re.match(r"^[0-9a-f]+ <(\S+)>:", line)
        wait = re.search(r"s_waitcnt.*lgkmcnt\((\d+)\)", line)
        if head:
            inside, flying = bool(re.search(r"\d" + kernel + r"I", head.group(1))), 0
        elif inside and "ds_read" in line:
            flying += 1
        elif inside and wait:
            flying = min(flying, int(wait.group(1)))
        elif inside and re.match(r"^\s*s_barrier", line):
            out.append(flying)
    return out


def test_parser_counts_reads_in_flight():
    asm = ("0000 <_ZN1x6k_pipeILi0EEEv>:\n\tds_read_b128 v[0:3], v4\n\ts_barrier // 0\n"
           "\ts_waitcnt vmcnt(2) lgkmcnt(0)\n\tds_read_b128 v[0:3], v4\n\tds_read_b64 v[0:1], v4\n"
           "\ts_waitcnt lgkmcnt(1)\n\ts_barrier\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier\n")
    assert reads_in_flight(asm, "k_pipe") == [1, 1, 0]


@pytest.mark.parametrize("src,kernel", KERNELS)
def test_no_lds_read_in_flight_at_a_barrier(src, kernel, tmp_path):
    counts = reads_in_flight(disassemble(os.path.join(BUILD, src + ".o"), tmp_path), kernel)
    assert counts and max(counts) == 0, sorted(set(counts))
