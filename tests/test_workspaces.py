"""The workspace queries: the bytes for the longest input serve the shorter ones,
so that a program may size one workspace once.  Asked of the library on the host."""
import pytest

from paper_2202_10297_amd import capi

# Lengths and bin counts around every line between the forms, and around those
# where a form changes its own parameters
LENGTHS = sorted({x + d for x in [1 << k for k in range(10, 28)] + [3 << 16, 3 << 17, 5 << 17, 7 << 16, 15 << 16, 3 << 19,
                                                                   400000, 5000000, 20000001, 48 << 20]
                  for d in (-1, 0, 1)})
BINS = [8193, 9000, 13632, 13633, 20480, 20481, 32768, 61440, 65537, 81921, 102400, 102401, 122881, 300000, 1 << 19,
        (1 << 19) + 1, 1 << 20, 1 << 22]


@pytest.mark.parametrize("op", [capi.ADD, capi.MUL, capi.MIN, capi.MAX, "lae", "gather"])
def test_workspace_of_the_longest_input_serves_shorter_ones(op):
    L, dtype = capi.lib(), capi.F32  # FP64 calls take the form that their workspace has room for

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


@pytest.mark.parametrize("op", [capi.ADD, capi.MUL, capi.MIN, capi.MAX])
def test_long_f64_inputs_ask_for_words_per_bin(op):
    for m in BINS:
        if m > 102400 or op in (capi.MIN, capi.MAX):  # fewer bins: partials in ranges
            assert capi.lib().pvjp_hist_ws_bytes(op, capi.F64, (1 << 25) + 1, m) <= 12 * m + 512


def _sizes(need):
    return [need(n) for n in LENGTHS]


@pytest.mark.parametrize("dtype", [capi.F32, capi.F64])
def test_other_workspaces_serve_shorter_inputs(dtype):
    L = capi.lib()
    for op in (capi.GOP_LOGADDEXP, capi.GOP_LINREC, capi.GOP_MAT2):
        for m in (1, 300, 513, 1 << 18, 1 << 24):
            s = _sizes(lambda n: L.pvjp_hist_generic_ws_bytes(op, dtype, n, m))
            assert all(a <= b for a, b in zip(s, s[1:])), (op, m)
    for m in (1, 131, 5000, 1000000):  # arrays of more elements, the same updates
        s = _sizes(lambda n: L.pvjp_scatter_plan_bytes(dtype, n, m))
        assert all(a <= b for a, b in zip(s, s[1:])), m


@pytest.mark.parametrize("D", [2, 35, 64, 256])
@pytest.mark.parametrize("K", [5, 19, 64, 77, 256, 1024])
def test_kmeans_workspace_serves_fewer_points(D, K):
    s = _sizes(lambda n: capi.lib().pvjp_kmeans_ws_bytes(n, D, K))
    assert all(a <= b for a, b in zip(s, s[1:]))


@pytest.mark.parametrize("D", [32, 64])
@pytest.mark.parametrize("K", [1, 4, 5, 8, 25, 50, 200, 5000])
def test_gmm_workspace_serves_fewer_points(D, K):
    s = _sizes(lambda n: capi.lib().pvjp_gmm_ws_bytes(n, D, K))
    assert all(a <= b for a, b in zip(s, s[1:]))
