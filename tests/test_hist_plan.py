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


# Lengths and bin counts around every line between the forms, and around those
# where a form changes its own parameters
LENGTHS = sorted({x + d for x in [1 << k for k in range(10, 28)] + [3 << 16, 3 << 17, 5 << 17, 7 << 16, 15 << 16, 3 << 19,
                                                                   400000, 5000000, 20000001, 48 << 20]
                  for d in (-1, 0, 1)})
BINS = [8193, 9000, 13632, 13633, 20480, 20481, 32768, 61440, 65537, 81921, 102400, 102401, 122881, 300000, 1 << 19,
        (1 << 19) + 1, 1 << 20, 1 << 22]


@pytest.mark.parametrize("dtype", [capi.F32, capi.F64])
@pytest.mark.parametrize("op", [capi.ADD, capi.MUL, capi.MIN, capi.MAX, "lae", "gather"])
def test_workspace_of_the_longest_input_serves_shorter_ones(op, dtype):
    L = capi.lib()

    def need(n, m):
        if op == "lae":
            return L.pvjp_hist_lae_ws_bytes(dtype, n, m)
        if op == "gather":
            return L.pvjp_gather_map_ws_bytes(dtype, max(m, 16385), n)
        return L.pvjp_hist_ws_bytes(op, dtype, n, m)

    for m in BINS:
        sizes = [need(n, m) for n in LENGTHS]
        assert all(a <= b for a, b in zip(sizes, sizes[1:])), m
    for n in LENGTHS:
        sizes = [need(n, m) for m in BINS]
        assert all(a <= b for a, b in zip(sizes, sizes[1:])), n
