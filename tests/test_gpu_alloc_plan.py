"""The allocation plan over the table counts where it changes: one thread's tables, all of
them kept in registers (4096 tables), rounds of 1024; and its refusals."""
import numpy as np
import pytest
from gpu_util import assert_state_equal, dev_cache_from_oracle, layouts, t

from oracle import oracle as orc
from paper_2412_03131_amd import diffkv as dk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tables", [1, 1023, 1025, 4096, 4097, 8192, 8193, 20000])
def test_alloc_plan(tables):
    rng = np.random.default_rng(tables)
    Lo, Ld = layouts(max_seq_len=240)  # 16 slots per table
    pages = tables * 9 + 5
    oc = orc.Cache(Lo, pages, tables, 1, ring=rng.permutation(pages))
    dc = dev_cache_from_oracle(Ld, oc, with_pool=False)

    def both(demand):
        orc.alloc_pages(oc, demand)
        dk.alloc_pages(dc, t(demand))

    print("case: allocation plan, %d tables" % tables, flush=True)
    both(rng.integers(0, 4, (tables, 2)).astype(np.int32))
    both(np.zeros((tables, 2), np.int32))
    assert oc.status[0] == 0
    assert_state_equal(dc, oc, with_pool=False, what="allocated")
    one = np.zeros((tables, 2), np.int32)
    for bad in ((17, 0), (-1, 2), (5, 4)):  # too many slots, a negative count, too many pages in all
        demand = one.copy()
        demand[tables // 2] = bad
        if bad == (5, 4):
            demand[:] = bad
        if bad[0] < 0:  # (the oracle takes no negative counts)
            dk.alloc_pages(dc, t(demand))
            oc.status[0] |= dk.ST_BAD_INPUT
        else:
            both(demand)
        assert oc.status[0] != 0
        assert_state_equal(dc, oc, with_pool=False, what="refused %s" % (bad,))
