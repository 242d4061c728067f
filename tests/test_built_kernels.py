"""Which kernels the library carries: one per form that some call launches."""
import re

import pytest

from paper_1412_4907_amd import bf


def _instances(kernel):
    """Template arguments of every instance of a kernel, from the symbol names
    the library registers."""
    try:
        with open(bf.LIB_PATH, "rb") as f:
            data = f.read()
    except FileNotFoundError:
        pytest.skip("library not built")
    pat = (r"_ZN2bf\d+%s(I(?:L[ib]n?\d+E)+)EEv" % kernel).encode()
    return {tuple(re.findall(rb"L[ib](n?\d+)E", m)) for m in re.findall(pat, data)}


def test_eight_wave_table_kernels_are_those_tables_launch():
    """bf_table_create takes the eight-wave kernel in FP16 and BF16 at I == 1
    (mode 0) and I % 4 == 0 (mode 3)."""
    want = {(p, m, i) for p in (b"1", b"2") for m in (b"0", b"3") for i in (b"0", b"1")}
    assert _instances("beamform_wide_table_kernel") == want
    # every precision and detecting mode has its batching kernels
    every = {(p, m, i) for p in (b"0", b"1", b"2") for m in (b"0", b"1", b"2", b"3")
             for i in (b"0", b"1")}
    assert _instances("beamform_wide_multi_kernel") == every
    assert _instances("beamform_table_kernel") == every
