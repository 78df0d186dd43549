"""Filters that leave positions of a primer out (specific primers at few
mismatches): run on the CPU as the other generated filters are, they pass every
site, their planned pass rate holds, and it stays below the planner's limit."""
import re

import numpy as np
import pytest

from paper_2509_13300_amd import _lib as L
from test_scan_filter_host import check_pair, planned_rate

LIMIT = 5e-7
CASES = [
    ("ATGTAGCGGAGGAGATTGCAGTTTACG", "GMSAACSTGRATGSACGGT", 0, 0),
    ("TACGACTCCAGGTKCCGCGCTAGCAAAACC", "GAGCTAACACTTKAGCACCCTCAACGTA", 1, 0),
    ("ATCGATGCCGTCATGACTCACGSAAACACG", "TGGCATTCAGGGCACGCGTGATGGGGCCAG", 2, 0),
    ("CCSTCTGTACCTGCACCACRGAMTCTACCCGG", "TGACATTACACGCATYCCGTCGAACTGACC", 1, 5),
    ("NNNNACGTTGCAAGGCTTAACCGGTTAACC", "BDHVACGTTGCAAGGCTTAACCGG", 0, 3),
]


def _tested(body, i):
    fn = body.split(f"u32 ah_pf_{i}(")[1].split("\n}\n")[0].split("{", 1)[1]
    return {int(m) for m in re.findall(r"\bp[acgthlx]\[(\d+)\]", fn)}


@pytest.mark.parametrize("case", CASES)
def test_filters_that_leave_positions_out_pass_every_site(case):
    body = L.ah_scan_program_source([case]).split("---- generated pattern program follows ----")[1]
    left = 0
    for i in range(4):
        primer = case[i // 2]
        assert planned_rate(body, i) <= LIMIT
        left += sum(ch != "N" for ch in primer) - len(_tested(body, i))
    assert left > 0
    check_pair(*case, rs=np.random.RandomState(23), n_words=32)
