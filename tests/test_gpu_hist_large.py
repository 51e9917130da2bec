"""Element-wise parity of reduce_by_index (Sec. 5.1.2) at n = 2^24 FP32
against the oracle, on the paths that the full-size calls take: bins
m in {2^10, 2^16, 2^20}, indices uniform and Zipf(1.1), operators + and max,
primal and VJP.  Winners, counts and the max/+ adjoints are compared bit for
bit (a winner is an index, the adjoints are copies of hs_bar), the + bin sums
within the FP32 bar (relative L2 2e-5).  Where the plan is the partitioned one,
the test checks on the host that at least one bucket holds more records than
one work item takes, so the merge of a bucket's items is exercised.
"""
import ctypes

import numpy as np
import pytest

from _util import TOL_F32, rel_l2
from paper_2202_10297_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N = 1 << 24


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.fixture(scope="module")
def ops():
    from paper_2202_10297_amd import capi, ops as o

    capi.lib()
    return o


def plan(op, n, m, counts):
    from paper_2202_10297_amd import capi

    info = (ctypes.c_int64 * 4)()
    capi.call("pvjp_hist_plan_info", {"add": capi.ADD, "max": capi.MAX}[op], capi.F32, n, m, int(counts),
              ctypes.cast(info, ctypes.c_void_p))
    return list(info)


def split_buckets(inds, m, info):
    """Number of buckets whose records span more than one work item."""
    bins_per_bucket, per_item = info[1], info[2]
    per_bucket = np.bincount(inds[(inds >= 0) & (inds < m)] // bins_per_bucket)
    return int((per_bucket > per_item).sum())


@pytest.mark.parametrize("dist", ["uniform", "zipf"])
@pytest.mark.parametrize("m", [1 << 10, 1 << 16, 1 << 20])
def test_hist_add_large(ops, orc, m, dist):
    from paper_2202_10297_amd import capi

    inds, vs, hb = workloads.hist(N, m, dist, "f32", seed=m + (dist == "zipf"))
    info = plan("add", N, m, True)
    if info[0] == capi.HIST_PATH_PARTITION and not (m == 1 << 20 and dist == "uniform"):
        assert split_buckets(inds, m, info) >= 1
    di = dev(inds)
    hs, aux = ops.hist("add", di, dev(vs), m, counts=True)
    ref = orc.hist("add", inds, vs, m)
    assert np.array_equal(host(aux["count"]), ref["count"])
    assert rel_l2(host(hs), ref["hs"]) <= TOL_F32
    hs2, _ = ops.hist("add", di, dev(vs), m)  # the plan without counts
    assert rel_l2(host(hs2), ref["hs"]) <= TOL_F32
    vb = host(ops.hist_vjp("add", di, None, m, aux, dev(hb)))
    assert np.array_equal(vb, orc.hist_vjp("add", inds, vs, hb).astype(np.float32))


@pytest.mark.parametrize("dist", ["uniform", "zipf"])
@pytest.mark.parametrize("m", [1 << 10, 1 << 16, 1 << 20])
def test_hist_max_large(ops, orc, m, dist):
    from paper_2202_10297_amd import capi

    inds, vs, hb = workloads.hist(N, m, dist, "f32", seed=m + 2 + (dist == "zipf"))
    # coarse values: ties inside a bin are common, so the lowest-index rule
    # decides many winners
    vs = (np.round(vs * 8) / 8).astype(np.float32)
    vs[::13] = -0.0
    info = plan("max", N, m, False)
    if info[0] == capi.HIST_PATH_PARTITION and not (m == 1 << 20 and dist == "uniform"):
        assert split_buckets(inds, m, info) >= 1
    di = dev(inds)
    hs, aux = ops.hist("max", di, dev(vs), m)
    ref = orc.hist("max", inds, vs, m)
    assert np.array_equal(host(aux["winner"]), ref["winner"])
    got = host(hs)
    assert np.array_equal(got, ref["hs"]) and np.array_equal(np.signbit(got), np.signbit(ref["hs"]))
    vb = host(ops.hist_vjp("max", di, None, m, aux, dev(hb)))
    assert np.array_equal(vb, orc.hist_vjp("max", inds, vs, hb).astype(np.float32))


def test_plan_info_names_the_paths(ops):
    from paper_2202_10297_amd import capi

    assert plan("add", N, 1 << 10, False)[0] == capi.HIST_PATH_LDS
    for m in (1 << 16, 1 << 20):
        for op in ("add", "max"):
            info = plan(op, N, m, False)
            assert info[0] in (capi.HIST_PATH_CACHE, capi.HIST_PATH_PARTITION)


# On either side of the lengths where the partition takes over, bins around one
# block's LDS and whole buckets: every operator and type, indices out of range,
# ties and zeros.
EDGES = [(op, n, m, dist) for op in ("add", "max", "min")
         for n, m, dist in (((3 << 19) - 1, 8193, "zipf"), (3 << 19, 8193, "zipf"), ((3 << 19) + 4097, 20480, "uniform"),
                            ((1 << 20) - 1, 131073, "zipf"), (1 << 20, 131073, "uniform"), (1 << 21, 20481, "zipf"))]
EDGES += [("mul", n, m, "uniform") for n, m in (((1 << 17) - 1, 8193), (1 << 17, 8193), ((1 << 17) + 8193, 20480))]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("op,n,m,dist", EDGES)
def test_partition_edges(ops, orc, op, n, m, dist, dtype):
    inds, vs, hb = workloads.hist(n, m, dist, dtype, seed=n + m)
    inds[::101] = -1
    inds[7::103] = m
    if op == "mul":
        # factors near one, so that a hot bin's product stays in range; some zeros
        vs = np.exp(1e-3 * vs).astype(vs.dtype)
        vs[::5003] = 0.0
        vs[2501::5003] = -0.0
    elif op != "add":
        vs = (np.round(vs * 8) / 8).astype(vs.dtype)
        vs[::13] = -0.0
    di, dv = dev(inds), dev(vs)
    ref = orc.hist(op, inds, vs, m)
    bar = TOL_F32 if dtype == "f32" else 1e-12
    for counts in (False, True):
        hs, aux = ops.hist(op, di, dv, m, counts=counts)
        if counts:
            assert np.array_equal(host(aux["count"]), ref["count"])
        if op in ("min", "max"):
            assert np.array_equal(host(aux["winner"]), ref["winner"])
            got = host(hs)
            assert np.array_equal(got, ref["hs"]) and np.array_equal(np.signbit(got), np.signbit(ref["hs"]))
        else:
            assert rel_l2(host(hs), ref["hs"]) <= bar
        if op == "mul":
            assert np.array_equal(host(aux["z"]), ref["z"])
            assert rel_l2(host(aux["p"]), ref["p"]) <= bar


# The form in ranges of bins: either side of its lines, one to six ranges, a
# last range of one bin, ragged chunks, an unaligned view, empty bins.
RANGES = [("add", (3 << 17) - 1, 8193), ("add", 3 << 17, 8193), ("add", (15 << 16) + 4097, 20481),
          ("add", 1 << 21, 4096), ("add", (1 << 21) + 5, 102400), ("add", 1 << 20, 102401), ("max", 15 << 16, 40961),
          ("min", (1 << 20) + 1, 122880), ("max", 1 << 21, 8192), ("min", 3 << 17, 20480), ("mul", 1 << 17, 13633),
          ("mul", (1 << 18) + 3, 54528), ("mul", 1 << 18, 54529), ("mul", 1 << 17, 5462)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("op,n,m", RANGES)
def test_range_edges(ops, orc, op, n, m, shift, dtype):
    inds, vs, _ = workloads.hist(n + shift, m, "uniform", dtype, seed=n + m)
    inds[::101] = -1
    inds[7::103] = m
    inds[inds % 17 == 3] = m - 1  # empty bins, and a hot last one
    if op == "mul":
        vs = np.exp(1e-3 * vs).astype(vs.dtype)
        vs[::5003] = 0.0
    elif op != "add":
        vs = (np.round(vs * 8) / 8).astype(vs.dtype)
        vs[::13] = -0.0
        vs[5::999] = np.inf if op == "max" else -np.inf
        vs[6::999] = -np.inf if op == "max" else np.inf
    hs, aux = ops.hist(op, dev(inds)[shift:], dev(vs)[shift:], m)
    ref = orc.hist(op, inds[shift:], vs[shift:], m)
    bar = TOL_F32 if dtype == "f32" else 1e-12
    if op in ("min", "max"):
        assert np.array_equal(host(aux["winner"]), ref["winner"])
        got = host(hs)
        assert np.array_equal(got, ref["hs"]) and np.array_equal(np.signbit(got), np.signbit(ref["hs"]))
    else:
        assert rel_l2(host(hs), ref["hs"]) <= bar
    if op == "mul":
        assert np.array_equal(host(aux["z"]), ref["z"])
        assert rel_l2(host(aux["p"]), ref["p"]) <= bar


def clustered(kind, n, m, g):
    """Indices whose equal ones lie together, or of which one bin has most."""
    if kind == "sorted":
        return np.sort(g.integers(0, m, n)).astype(np.int32)
    if kind == "falling":
        return np.sort(g.integers(0, m, n))[::-1].astype(np.int32)
    if kind == "const":
        return np.full(n, m // 3, np.int32)
    if kind == "runs":  # runs of 5,000 elements and some of a few
        lens = np.where(g.random(n // 1000 + 2) < 0.5, 5000, g.integers(1, 70, n // 1000 + 2))
        return np.resize(np.repeat(g.integers(0, m, lens.size), lens), n).astype(np.int32)
    hot = g.random(n) < 0.8  # one bin with four fifths of the elements
    return np.where(hot, m - 5, g.integers(0, m, n)).astype(np.int32)


# One range of bins, several, buckets with few and with many records an item.
@pytest.mark.parametrize("kind", ["sorted", "falling", "const", "runs", "hot"])
@pytest.mark.parametrize("n,m", [(700001, 9001), (1 << 20, 60000), (1050001, 100003), (1 << 21, 131073)])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("op", ["add", "mul", "max", "min"])
def test_clustered_indices(ops, orc, op, dtype, n, m, kind):
    g = workloads.rng(n + m)
    inds = clustered(kind, n, m, g)
    inds[::1009] = -1
    inds[500::1013] = m
    vs = g.standard_normal(n).astype(np.float32 if dtype == "f32" else np.float64)
    if op == "mul":
        vs = np.exp(1e-3 * vs).astype(vs.dtype)
        vs[::5003] = 0.0
        vs[2501::5003] = -0.0
    elif op != "add":
        vs = (np.round(vs * 8) / 8).astype(vs.dtype)
        vs[::13] = -0.0
    ref = orc.hist(op, inds, vs, m)
    bar = TOL_F32 if dtype == "f32" else 1e-12
    pad = np.zeros(1, np.int32), np.zeros(1, vs.dtype)
    odd = dev(np.r_[pad[0], inds])[1:], dev(np.r_[pad[1], vs])[1:]  # no 16-byte alignment
    for di, dv, counts in ((dev(inds), dev(vs), False), (dev(inds), dev(vs), True), (*odd, False)):
        hs, aux = ops.hist(op, di, dv, m, counts=counts)
        if counts:
            assert np.array_equal(host(aux["count"]), ref["count"])
        if op in ("min", "max"):
            assert np.array_equal(host(aux["winner"]), ref["winner"])
            got = host(hs)
            assert np.array_equal(got, ref["hs"]) and np.array_equal(np.signbit(got), np.signbit(ref["hs"]))
        else:
            assert rel_l2(host(hs), ref["hs"]) <= bar
        if op == "mul":
            assert np.array_equal(host(aux["z"]), ref["z"])
            assert rel_l2(host(aux["p"]), ref["p"]) <= bar


@pytest.mark.parametrize("op", ["add", "mul", "max"])
@pytest.mark.parametrize("n,m", [(5000, 100), (100001, 30000), (1 << 20, 50000), (1 << 20, 300000)])
def test_indices_far_outside_are_skipped(ops, orc, op, n, m):
    # every form's test of the range: no difference to a range's first bin wraps
    g = workloads.rng(n + m)
    inds = g.integers(0, m, n).astype(np.int32)
    inds[::7] = np.iinfo(np.int32).min + np.arange(inds[::7].size, dtype=np.int32) % 70000
    inds[3::7] = np.iinfo(np.int32).max
    vs = np.exp(1e-3 * g.standard_normal(n)).astype(np.float32)
    ref = orc.hist(op, inds, vs, m)
    hs, aux = ops.hist(op, dev(inds), dev(vs), m)
    if op == "max":
        assert np.array_equal(host(aux["winner"]), ref["winner"]) and np.array_equal(host(hs), ref["hs"])
    else:
        assert rel_l2(host(hs), ref["hs"]) <= TOL_F32


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n", [1 << 17, 8192 * 236, 8192 * 236 + 1])
@pytest.mark.parametrize("kind", ["uniform", "sorted", "const"])
def test_product_items_of_one_tile(ops, orc, dtype, n, kind):
    # products take items of a tile's records up to 256 of them: 236 tiles and 20
    # buckets, one tile more, and the shortest input that is sorted by bucket
    m = 81920
    g = workloads.rng(n)
    inds = g.integers(0, m, n).astype(np.int32) if kind == "uniform" else clustered(kind, n, m, g)
    vs = np.exp(1e-3 * g.standard_normal(n)).astype(np.float32 if dtype == "f32" else np.float64)
    vs[::5003] = 0.0
    ref = orc.hist("mul", inds, vs, m)
    hs, aux = ops.hist("mul", dev(inds), dev(vs), m)
    bar = TOL_F32 if dtype == "f32" else 1e-12
    assert np.array_equal(host(aux["z"]), ref["z"])
    assert rel_l2(host(hs), ref["hs"]) <= bar and rel_l2(host(aux["p"]), ref["p"]) <= bar


@pytest.mark.parametrize("op,dtype,n,m", [("add", "f32", 1 << 24, 65536), ("mul", "f32", 1 << 21, 40000),
                                          ("mul", "f32", 1 << 21, 300000), ("max", "f64", 1 << 22, 100000),
                                          ("add", "f64", 1 << 22, 300000)])
def test_clustered_indices_take_no_multiple(ops, op, dtype, n, m):
    # sorted indices, or all in one bin, within four times the uniform ones' time
    # (they were 6 to 560 times it where equal neighbours queued at one word or
    # one block of a chunk, or few waves of an item, had all the work)
    g = workloads.rng(n + m)
    vs = dev(np.exp(1e-3 * g.standard_normal(n)).astype(np.float32 if dtype == "f32" else np.float64))

    def best(inds):
        di, ts = dev(inds), []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            ops.hist(op, di, vs, m)
            b.record()
            b.synchronize()
            ts.append(a.elapsed_time(b))
        return min(ts)

    uniform = best(g.integers(0, m, n).astype(np.int32))
    for kind in ("sorted", "const"):
        assert best(clustered(kind, n, m, g)) <= 4 * uniform, kind


# On either side of the lengths where FP32 inputs leave the bin cache.
@pytest.mark.parametrize("op", ["add", "max"])
@pytest.mark.parametrize("n,m,counts", [(3 << 17, 40000, False), (3 << 17, 61440, False), (1 << 19, 61441, False),
                                        (1 << 19, 102400, False), (5 << 17, 122881, False), (15 << 16, 600000, False),
                                        (5 << 17, 9000, True), (3 << 16, 20480, True), (7 << 16, 600000, True)])
@pytest.mark.parametrize("below", [1, 0])
def test_short_input_lines(ops, orc, op, n, m, counts, below):
    n -= below
    inds, vs, _ = workloads.hist(n, m, "zipf", "f32", seed=n + m)
    inds[::101] = -1
    inds[7::103] = m
    if op == "max":
        vs = (np.round(vs * 8) / 8).astype(vs.dtype)
        vs[::13] = -0.0
    ref = orc.hist(op, inds, vs, m)
    hs, aux = ops.hist(op, dev(inds), dev(vs), m, counts=counts)
    if counts:
        assert np.array_equal(host(aux["count"]), ref["count"])
    if op == "max":
        assert np.array_equal(host(aux["winner"]), ref["winner"]) and np.array_equal(host(hs), ref["hs"])
    else:
        assert rel_l2(host(hs), ref["hs"]) <= TOL_F32


@pytest.mark.parametrize("op", ["add", "max", "mul"])
def test_long_f64(ops, orc, op):
    # more than 2^25 FP64 records of 12 bytes
    n, m = (1 << 25) + 4097, 131073
    inds, vs, _ = workloads.hist(n, m, "uniform", "f64", seed=7)
    if op == "mul":
        vs = np.exp(1e-3 * vs)
        vs[::50003] = 0.0
    ref = orc.hist(op, inds, vs, m)
    hs, aux = ops.hist(op, dev(inds), dev(vs), m)
    if op == "max":
        assert np.array_equal(host(aux["winner"]), ref["winner"]) and np.array_equal(host(hs), ref["hs"])
    else:
        assert rel_l2(host(hs), ref["hs"]) <= 1e-12


@pytest.mark.parametrize("m", [9000, 131073])
@pytest.mark.parametrize("n", [1 << 25, 1200001, 3000])
@pytest.mark.parametrize("op", ["add", "max", "mul"])
def test_f64_in_the_workspace_of_a_longer_input(ops, orc, op, n, m):
    # the bytes for more than 2^25 elements are a few words a bin: shorter calls
    # that would sort their records take the bin cache instead
    from paper_2202_10297_amd import capi

    inds, vs, _ = workloads.hist(n, m, "uniform", "f64", seed=8)
    if op == "mul":
        vs = np.exp(1e-3 * vs)
        vs[::50003] = 0.0
    o = {"add": capi.ADD, "max": capi.MAX, "mul": capi.MUL}[op]
    ws = torch.zeros(capi.lib().pvjp_hist_ws_bytes(o, capi.F64, (1 << 25) + 4097, m), dtype=torch.uint8, device="cuda")
    i, v = dev(inds), dev(vs)
    hs, p = (torch.empty(m, dtype=torch.float64, device="cuda") for _ in range(2))
    w, z = (torch.empty(m, dtype=torch.int32, device="cuda") for _ in range(2))
    capi.call("pvjp_hist", o, capi.F64, i.data_ptr(), v.data_ptr(), n, m, hs.data_ptr(),
              w.data_ptr() if op == "max" else None, p.data_ptr() if op == "mul" else None,
              z.data_ptr() if op == "mul" else None, None, ws.data_ptr(), ws.numel(), None)
    ref = orc.hist(op, inds, vs, m)
    if op == "max":
        assert np.array_equal(host(w), ref["winner"]) and np.array_equal(host(hs), ref["hs"])
    else:
        assert rel_l2(host(hs), ref["hs"]) <= 1e-12
    if op == "mul":
        assert np.array_equal(host(z), ref["z"])


def test_f64_log_add_exp_and_gather_in_the_workspace_of_a_longer_input(ops, orc):
    from paper_2202_10297_amd import capi

    n, m, more = 1 << 21, 131073, (1 << 25) + 4097
    inds, vs, yb = workloads.hist(n, m, "uniform", "f64", seed=9)
    i, v = dev(inds), dev(vs)
    out = torch.empty(m, dtype=torch.float64, device="cuda")
    ws = torch.zeros(capi.lib().pvjp_hist_lae_ws_bytes(capi.F64, more, m) - 8 * (more - n), dtype=torch.uint8,
                     device="cuda")  # but for the terms, of which there are n
    capi.call("pvjp_hist_lae", capi.F64, i.data_ptr(), v.data_ptr(), n, m, out.data_ptr(), ws.data_ptr(),
              ws.numel(), None)
    ref = host(ops.hist_lae(i, v, m))
    both = np.isfinite(ref)
    assert np.array_equal(both, np.isfinite(host(out))) and rel_l2(host(out)[both], ref[both]) <= 1e-12
    ws = torch.zeros(capi.lib().pvjp_gather_map_ws_bytes(capi.F64, m, more) - 8 * (more - n), dtype=torch.uint8,
                     device="cuda")
    capi.call("pvjp_gather_map_vjp", capi.GMAP["gather"], capi.F64, out.data_ptr(), m, i.data_ptr(), None, n,
              v.data_ptr(), out.data_ptr(), None, 0, ws.data_ptr(), ws.numel(), None)
    assert rel_l2(host(out), orc.hist("add", inds, vs, m)["hs"]) <= 1e-12
