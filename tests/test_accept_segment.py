"""Which segment of a row the rejection step's second launch rescans, without a GPU."""
import ctypes

import paper_2311_04951_amd as sv


def test_the_segment_lies_inside_the_row_whatever_the_lanes_say():
    """The first whose running sum passes the threshold; where none does (a threshold that is not below the total), the last - an index of
    -1 would read in front of the row."""
    L = sv.lib()
    L.ss_dev_accept_segment.argtypes = [ctypes.c_ulonglong, ctypes.c_int]
    L.ss_dev_accept_segment.restype = ctypes.c_int
    for nseg in range(1, 17):
        assert L.ss_dev_accept_segment(0, nseg) == nseg - 1
        for first in range(nseg):
            for passed in (1 << first, (1 << nseg) - (1 << first)):
                assert L.ss_dev_accept_segment(passed, nseg) == first
