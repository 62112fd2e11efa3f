"""Types of several groups whose shapes nest deeper than the layout program's loops commit (the expansion of such a
shape into groups ends) and list the oracle's segments."""
import numpy as np
import pytest

from oracle import build_type as obuild
from paper_2402_12274_amd import inputs, mdt

DARRAY = ("darray", 8, 3, [93, 104, 104], ["cyclic"] * 3, [5] * 3, [2, 2, 2], "C", inputs.DOUBLE)


@pytest.mark.timeout(60, method="thread")
def test_block_cyclic_share_ragged_in_the_slowest_dimension():
    t, o = mdt.build_type(DARRAY), obuild(DARRAY)
    n, size = t.iov_len(-1)
    on, osize = o.iov_len(-1)
    assert (n, size) == (on, osize)
    (base, ln), (obase, oln) = t.iov(0, n), o.iov(0, n)
    assert np.array_equal(base, obase) and np.array_equal(ln, oln)
