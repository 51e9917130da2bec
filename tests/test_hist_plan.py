"""Which path reduce_by_index takes, asked of the library on the host: the
lines between the LDS bin cache, the ranges of bins and the buckets."""
import ctypes

import pytest

from paper_2202_10297_amd import capi


def path(op, dtype, n, m, counts=False):
    info = (ctypes.c_int64 * 4)()
    capi.call("pvjp_hist_plan_info", op, dtype, n, m, int(counts), ctypes.cast(info, ctypes.c_void_p))
    return info[0]


# Uniform indices where the cache took up to three times the partition's time
# (n = 1,048,000 with counts into 100,000 bins: 127 us, 33)
@pytest.mark.parametrize("op", [capi.ADD, capi.MIN, capi.MAX])
@pytest.mark.parametrize("n,m,counts", [(500000, 30000, False), (800000, 60000, False), (800000, 100000, False),
                                        (1048000, 300000, False), (1000000, 1000000, False), (500000, 60000, True),
                                        (800000, 30000, True), (1048000, 100000, True), (1048000, 1000000, True)])
def test_short_inputs_leave_the_cache(op, n, m, counts):
    assert path(op, capi.F32, n, m, counts) == capi.HIST_PATH_PARTITION


def test_shortest_inputs_keep_it():
    for m in (20000, 100000, 1000000):
        for counts in (False, True):
            assert path(capi.ADD, capi.F32, 100000, m, counts) == capi.HIST_PATH_CACHE
