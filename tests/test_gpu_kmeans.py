"""GPU parity of dense k-means (Sec. 7.4) through the C ABI against the
oracle: the objective, the nearest-centre assignments (bit-exact: both sides
decide on the same FP64 distance chain), the gradient and the jvp of the
VJP (Hessian-vector product), at the paper's two workload shapes (k, n, d) =
(5, 494019, 35) and (1024, 10000, 256) and at small and ragged sizes.
"""
import numpy as np
import pytest

from _util import TOL_F32, rel_l2
from paper_2202_10297_amd import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


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


# small and ragged sizes; K = 16 / 17 on either side of the register-accumulator
# gradient; D > 256 (the listed-point gradient at small K) and D = 1024 (the
# largest, 8 centres per slice); the paper's two shapes
CASES = [(1, 1, 1), (5, 3, 2), (100, 35, 5), (1000, 17, 33), (777, 64, 70), (3000, 256, 40),
         (3001, 40, 16), (3001, 40, 17), (2000, 300, 3), (600, 1024, 20),
         (494019, 35, 5), (10000, 256, 1024)]


@pytest.mark.parametrize("N,D,K", CASES)
def test_kmeans_objective_gradient_hvp(ops, orc, N, D, K):
    X, C = workloads.kmeans(N, D, K, "f32", seed=N + D + K)
    Xd, Cd = dev(X), dev(C)
    f, a = ops.kmeans_objective(Xd, Cd)
    rf, ra = orc.kmeans_objective(X, C)
    assert np.array_equal(host(a), ra)
    assert abs(host(f)[0] - rf) <= 1e-12 * max(1.0, rf)
    Cdot = workloads.rng(5).standard_normal(C.shape).astype(np.float32)
    cb, hv = ops.kmeans_vjp(Xd, Cd, a, f_bar=0.5, C_dot=dev(Cdot))
    assert rel_l2(host(cb), orc.kmeans_vjp(X, C, 0.5)) <= TOL_F32
    assert rel_l2(host(hv), orc.kmeans_hvp(X, C, Cdot, 0.5)) <= TOL_F32


def test_kmeans_accumulate_and_newton_step(ops, orc):
    N, D, K = 20000, 35, 5
    X, C = workloads.kmeans(N, D, K, "f32", seed=1)
    Xd, Cd = dev(X), dev(C)
    _, a = ops.kmeans_objective(Xd, Cd)
    base = [workloads.rng(i).standard_normal(C.shape).astype(np.float32) for i in (2, 3)]
    out = (dev(base[0]), dev(base[1]))
    ops.kmeans_vjp(Xd, Cd, a, f_bar=1.0, C_dot=torch.ones_like(Cd), out=out, accumulate=True)
    g = orc.kmeans_vjp(X, C, 1.0)
    h = orc.kmeans_hvp(X, C, np.ones_like(C), 1.0)
    assert rel_l2(host(out[0]) - base[0], g) <= 2 * TOL_F32
    assert rel_l2(host(out[1]) - base[1], h) <= 2 * TOL_F32
    # the Newton step with the Hessian diagonal is the mean of each cluster
    cb, hv = ops.kmeans_vjp(Xd, Cd, a, f_bar=1.0, C_dot=torch.ones_like(Cd))
    cbn, hvn = host(cb).astype(np.float64), host(hv).astype(np.float64)
    an = host(a)
    n = np.bincount(an, minlength=K)
    S = np.zeros((K, D))
    np.add.at(S, an, X.astype(np.float64))
    nz = n > 0
    newton = C - cbn / np.where(hvn == 0, 1, hvn)
    assert rel_l2(newton[nz], (S / np.maximum(n, 1)[:, None])[nz]) <= 1e-5


def test_kmeans_empty_input_and_ties(ops, orc):
    X = np.array([[0.0, 0.0], [1.0, 0.0]], dtype=np.float32)
    C = np.array([[1.0, 1.0], [1.0, -1.0], [-1.0, 1.0]], dtype=np.float32)
    f, a = ops.kmeans_objective(dev(X), dev(C))
    assert list(host(a)) == [0, 0] and host(f)[0] == 3.0
    f, a = ops.kmeans_objective(dev(np.zeros((0, 2), dtype=np.float32)), dev(C))
    assert host(f)[0] == 0.0
    cb, _ = ops.kmeans_vjp(dev(np.zeros((0, 2), dtype=np.float32)), dev(C), a)
    assert np.all(host(cb) == 0)


def test_autograd(orc):
    from paper_2202_10297_amd import autograd

    X, C = workloads.kmeans(5000, 35, 5, "f32", seed=14)
    c = dev(C).requires_grad_()
    f = autograd.kmeans_objective(dev(X), c)
    (0.5 * f).backward()
    ref = orc.kmeans_vjp(X.astype(np.float64), C.astype(np.float64), 0.5)
    assert rel_l2(host(c.grad), ref) <= TOL_F32
    fv = float(f.detach())
    assert abs(fv - orc.kmeans_objective(X, C)[0]) <= 1e-12 * fv


# searches large enough for the bounded form (D from 16 to 256, K >= 64): widths
# around its fragments, rows that are no whole 16 bytes, a ragged last tile of
# centres and block of points
@pytest.mark.parametrize("N,D,K,off", [(262145, 16, 64, 0.0), (60003, 35, 515, 0.0), (70001, 64, 65, 1000.0),
                                       (20011, 100, 257, -30.0), (8099, 255, 530, 0.0), (17000, 256, 64, 3.0e4)])
def test_bounded_search(ops, orc, N, D, K, off):
    X, C = workloads.kmeans(N, D, K, "f32", seed=N + D + K)
    X, C = X + np.float32(off), C + np.float32(off)
    # ties: equal centres, in pairs and in a row of five, the lowest wins
    C[K - 1] = C[0]
    C[20:25] = C[20]
    f, a = ops.kmeans_objective(dev(X), dev(C))
    rf, ra = orc.kmeans_objective(X, C)
    assert np.array_equal(host(a), ra)
    assert abs(host(f)[0] - rf) <= 1e-12 * rf


def test_bounded_search_close_centres(ops, orc):
    # every centre within rounding of the others' distance: the FP64 chains decide
    N, D, K = 9000, 128, 256
    g = workloads.rng(77)
    X = g.standard_normal((N, D)).astype(np.float32)
    C = (1e-5 * g.standard_normal((K, D))).astype(np.float32)
    f, a = ops.kmeans_objective(dev(X), dev(C))
    rf, ra = orc.kmeans_objective(X, C)
    assert np.array_equal(host(a), ra) and abs(host(f)[0] - rf) <= 1e-12 * rf


def test_bounded_search_extreme_values(ops, orc):
    # points beyond the FP32 norms, tiny ones, zero centres
    N, D, K = 40000, 64, 128
    X, C = workloads.kmeans(N, D, K, "f32", seed=9)
    X[5], X[6, 3], X[7] = 1e19, 3e30, 1e-30
    C[3] = 0.0
    f, a = ops.kmeans_objective(dev(X), dev(C))
    _, ra = orc.kmeans_objective(X, C)
    assert np.array_equal(host(a), ra)
    # a point that is no number: all its distances are, centre 0 keeps it
    X[5], X[6, 3] = 0.0, 0.0
    X[11, 5] = np.nan
    _, a = ops.kmeans_objective(dev(X), dev(C))
    _, ra = orc.kmeans_objective(np.delete(X, 11, 0), C)
    assert np.array_equal(np.delete(host(a), 11), ra) and host(a)[11] == 0
    # a centre that is no number wins nothing; one out of FP32's reach neither
    X[11, 5] = 0.0
    for v in (np.nan, 1e25):
        D_ = C.copy()
        D_[5, 2] = v
        _, a = ops.kmeans_objective(dev(X), dev(D_))
        far = C.copy()
        far[5] = 1e15
        _, ra = orc.kmeans_objective(X, far)
        assert np.array_equal(host(a), ra)


# Few points: slices of fewer centres than the kernel's width, a last slice of
# one, and chunk partials of eight and a remainder.
@pytest.mark.parametrize("N,D,K", [(255, 16, 33), (3117, 64, 19), (2049, 128, 41), (16385, 24, 17), (65537, 8, 9)])
def test_small_slices(ops, orc, N, D, K):
    X, C = workloads.kmeans(N, D, K, "f32", seed=N)
    C[K - 1] = C[1]  # equal centres in different slices: the lower one wins
    f, a = ops.kmeans_objective(dev(X), dev(C))
    rf, ra = orc.kmeans_objective(X, C)
    assert np.array_equal(host(a), ra)
    assert abs(host(f)[0] - rf) <= 1e-12 * max(1.0, rf)
    cb, _ = ops.kmeans_vjp(dev(X), dev(C), a, f_bar=0.5)
    assert rel_l2(host(cb), orc.kmeans_vjp(X, C, 0.5)) <= TOL_F32


@pytest.mark.parametrize("N,D,K", [(270000, 16, 64), (140000, 32, 64), (70000, 64, 64)])
def test_bounded_search_worst_products(ops, orc, N, D, K):
    # relative to the first centre (zero) every coordinate is near 1 + 2^-8 times
    # a power of two, where a bf16 product leaves out the most, all of one sign;
    # the centres differ by a few units in the last place
    g = workloads.rng(D)

    def rows(n):
        s = 1.0 + 2.0 ** -8 + g.integers(-64, 65, (n, D)) * 2.0 ** -23
        return (s * 2.0 ** g.integers(-1, 2, (1, D))).astype(np.float32)

    X, C = rows(N), rows(K)
    C[0] = 0.0
    f, a = ops.kmeans_objective(dev(X), dev(C))
    rf, ra = orc.kmeans_objective(X, C)
    assert np.array_equal(host(a), ra)
    assert abs(host(f)[0] - rf) <= 1e-12 * rf


@pytest.mark.parametrize("N,D,K", [(9001, 256, 257), (70003, 35, 1000), (66001, 64, 65), (270001, 16, 64)])
@pytest.mark.parametrize("kind", ["equal", "groups", "some"])
def test_bounded_search_left_open(ops, orc, N, D, K, kind):
    # too many centres within reach of the bound: blocks of points go to the FP64
    # search, all of them or (some) a few beside blocks that are decided
    g = workloads.rng(N + K)
    X, C = workloads.kmeans(N, D, K, "f32", seed=N)
    if kind == "equal":
        C[:] = C[K // 2]
    else:
        far = (1000.0 * g.standard_normal((8, D))).astype(np.float32)
        at = np.arange(N) if kind == "groups" else np.r_[300:340, 5000:5400, N - 30:N]
        X[at] = far[g.integers(0, 8, at.size)] + g.standard_normal((at.size, D)).astype(np.float32)
        k0 = 0 if kind == "groups" else K // 2
        C[k0:] = far[g.integers(0, 8, K - k0)] + g.standard_normal((K - k0, D)).astype(np.float32)
    C[K - 1] = C[1]
    sub = np.unique(np.r_[0:600, 4900:5500, N - 300:N])  # the oracle's share
    f, a = ops.kmeans_objective(dev(X), dev(C))
    _, ra = orc.kmeans_objective(X[sub], C)
    assert np.array_equal(host(a)[sub], ra)
    # a second call on the same workspace, whose flags the first one set
    X2, C2 = workloads.kmeans(N, D, K, "f32", seed=N + 1)
    f2, a2 = ops.kmeans_objective(dev(X2), dev(C2))
    _, ra2 = orc.kmeans_objective(X2[sub], C2)
    assert np.array_equal(host(a2)[sub], ra2)
    # f is the sum of the points' distances to their centres
    d = torch.sum((dev(X2).double() - dev(C2).double()[a2.long()]) ** 2)
    assert abs(host(f2)[0] - host(d)) <= 1e-12 * host(d)
