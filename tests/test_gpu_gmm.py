"""GPU parity of the Gaussian-mixture objective and gradient against the taped
FP64 oracle (FP32 inputs, relative L2 per parameter group <= 2e-5)."""
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


CASES = [(1, 32, 1), (7, 32, 3), (130, 32, 5), (300, 64, 4), (1000, 64, 20), (2049, 32, 50), (200, 64, 200)]


@pytest.mark.parametrize("N,D,K", CASES)
def test_gmm_objective_and_gradient(ops, orc, N, D, K):
    X, alpha, mu, q, l = workloads.gmm(N, D, K, seed=N + D + K)
    ll, lse = ops.gmm_objective(dev(X), dev(alpha), dev(mu), dev(q), dev(l))
    rll, rlse = orc.gmm_objective(X, alpha, mu, q, l)
    assert abs(host(ll)[0] - rll) <= TOL_F32 * abs(rll)
    assert rel_l2(host(lse), rlse) <= TOL_F32
    got = ops.gmm_vjp(dev(X), dev(alpha), dev(mu), dev(q), dev(l), lse=lse, ell_bar=1.0)
    ref = orc.gmm_vjp(X, alpha, mu, q, l, 1.0)
    for name, g, r in zip(["alpha", "mu", "q", "l"], got, ref):
        err = rel_l2(host(g), r)
        assert err <= TOL_F32, (name, err)
    assert rel_l2([host(g) for g in got], list(ref)) <= TOL_F32


@pytest.mark.parametrize("N,D,K", CASES)
def test_gmm_gradient_from_s_checkpoint(ops, orc, N, D, K):
    # the forward also keeps every s_ik; the reverse sweep then contracts
    # S_k = sum w y y^T and forms G_k = Q_k S_k instead of recomputing z
    X, alpha, mu, q, l = workloads.gmm(N, D, K, seed=N + D + K)
    ll, lse, sck = ops.gmm_objective_ckpt(dev(X), dev(alpha), dev(mu), dev(q), dev(l))
    rll, rlse = orc.gmm_objective(X, alpha, mu, q, l)
    assert rel_l2(host(lse), rlse) <= TOL_F32
    # the kept s_ik are the forward's: LSE over k of each point's s is lse
    sv = host(sck)
    mx = sv.max(axis=0)
    assert np.allclose(mx + np.log(np.exp(sv - mx).sum(axis=0)), host(lse), rtol=1e-13, atol=1e-12)
    got = ops.gmm_vjp(dev(X), dev(alpha), dev(mu), dev(q), dev(l), lse=lse, s=sck, ell_bar=1.0)
    ref = orc.gmm_vjp(X, alpha, mu, q, l, 1.0)
    for name, g, r in zip(["alpha", "mu", "q", "l"], got, ref):
        err = rel_l2(host(g), r)
        assert err <= TOL_F32, (name, err)
    # accumulate on top of a base
    base = [workloads.rng(i + 9).standard_normal(a.shape).astype(np.float32) for i, a in enumerate((alpha, mu, q, l))]
    out = tuple(dev(b) for b in base)
    ops.gmm_vjp(dev(X), dev(alpha), dev(mu), dev(q), dev(l), lse=lse, s=sck, ell_bar=1.0, out=out, accumulate=True)
    for g, b, r in zip(out, base, ref):
        assert rel_l2(host(g) - b, r) <= 2 * TOL_F32


def test_gmm_several_point_chunks(ops, orc):
    # 40000 points span three point chunks of the objective and the gradient,
    # so the FP64 merge across chunks is checked element by element
    N, D, K = 40000, 32, 5
    X, alpha, mu, q, l = workloads.gmm(N, D, K, seed=11)
    ll, lse = ops.gmm_objective(dev(X), dev(alpha), dev(mu), dev(q), dev(l))
    rll, rlse = orc.gmm_objective(X, alpha, mu, q, l)
    assert abs(host(ll)[0] - rll) <= TOL_F32 * abs(rll)
    assert rel_l2(host(lse), rlse) <= TOL_F32
    ref = orc.gmm_vjp(X, alpha, mu, q, l, 1.0)
    for s in (None, "ckpt"):
        if s is None:
            got = ops.gmm_vjp(dev(X), dev(alpha), dev(mu), dev(q), dev(l), lse=lse, ell_bar=1.0)
        else:
            _, lse2, sck = ops.gmm_objective_ckpt(dev(X), dev(alpha), dev(mu), dev(q), dev(l))
            got = ops.gmm_vjp(dev(X), dev(alpha), dev(mu), dev(q), dev(l), lse=lse2, s=sck, ell_bar=1.0)
        for name, g, r in zip(["alpha", "mu", "q", "l"], got, ref):
            err = rel_l2(host(g), r)
            assert err <= TOL_F32, (s, name, err)


@pytest.mark.parametrize("N,D,K", [(127, 32, 4), (128, 64, 2), (129, 32, 9), (4095, 64, 3), (130944, 32, 7),
                                   (130945, 32, 7)])
def test_gmm_lse_over_component_ranges(ops, orc, N, D, K):
    # up to 1,023 blocks of 128 points the objective splits the components
    # over block rows and merges each point's (max, sum); one point more and
    # a block takes all components.  K around whole batches of components.
    X, alpha, mu, q, l = workloads.gmm(N, D, K, seed=7 * N + K)
    ll, lse = ops.gmm_objective(dev(X), dev(alpha), dev(mu), dev(q), dev(l))
    idx = np.unique(np.r_[0:min(N, 20), max(0, N - 20):N])
    _, rlse = orc.gmm_objective(X[idx], alpha, mu, q, l)
    assert rel_l2(host(lse)[idx], rlse) <= TOL_F32
    from scipy.special import logsumexp

    expect = host(lse).sum() - N * logsumexp(alpha.astype(np.float64)) - 0.5 * N * D * np.log(2 * np.pi)
    assert abs(host(ll)[0] - expect) <= 1e-12 * abs(expect)
    # weights over the components sum to one: so do the objective's alpha adjoints with the softmax term
    ab = host(ops.gmm_vjp(dev(X), dev(alpha), dev(mu), dev(q), dev(l), lse=lse)[0])
    assert abs(ab.sum()) <= TOL_F32 * N


@pytest.mark.parametrize("N,D,K", [(131072, 64, 5), (131073, 32, 8), (131135, 64, 9), (200001, 32, 17),
                                   (262143, 64, 33)])
def test_gmm_large_n_form(ops, orc, N, D, K):
    # from 2^17 points the contractions run as bf16 triples: around a tile, a
    # block of eight components and a component range.  LSE_i against the oracle
    # on sampled points; the gradient against the sum over two parts, which are
    # short enough for the FP32 form (each side within TOL_F32, so twice that).
    X, alpha, mu, q, l = workloads.gmm(N, D, K, seed=N + K)
    Xd, P = dev(X), [dev(a) for a in (alpha, mu, q, l)]
    ll, lse, sck = ops.gmm_objective_ckpt(Xd, *P)
    idx = np.unique(np.r_[0:10, N // 2:N // 2 + 10, N - 40:N])
    _, rlse = orc.gmm_objective(X[idx], alpha, mu, q, l)
    assert rel_l2(host(lse)[idx], rlse) <= TOL_F32
    cut = [0, 100001, min(N, 220001), N] if N > 231071 else [0, 100001, N]
    parts = [[host(g) for g in ops.gmm_vjp(dev(X[a:b]), *P, ell_bar=-0.75)] for a, b in zip(cut, cut[1:]) if b > a]
    ref = [sum(p[i].astype(np.float64) for p in parts) for i in range(4)]
    base = [workloads.rng(i).standard_normal(a.shape).astype(np.float32) for i, a in enumerate((alpha, mu, q, l))]
    for s in (None, sck):
        out = tuple(dev(b) for b in base)
        ops.gmm_vjp(Xd, *P, lse=lse, s=s, ell_bar=-0.75, out=out, accumulate=True)
        got = ops.gmm_vjp(Xd, *P, lse=lse, s=s, ell_bar=-0.75)
        for g, o, b, r in zip(got, out, base, ref):
            assert rel_l2(host(g), r) <= 2 * TOL_F32
            assert rel_l2(host(o), b + r) <= 2 * TOL_F32


def test_gmm_vjp_without_checkpoint_and_accumulate(ops, orc):
    N, D, K = 500, 64, 6
    X, alpha, mu, q, l = workloads.gmm(N, D, K, seed=3)
    ref = orc.gmm_vjp(X, alpha, mu, q, l, 0.5)
    got = ops.gmm_vjp(dev(X), dev(alpha), dev(mu), dev(q), dev(l), lse=None, ell_bar=0.5)
    assert rel_l2([host(g) for g in got], list(ref)) <= TOL_F32
    base = [workloads.rng(i).standard_normal(a.shape).astype(np.float32) for i, a in enumerate((alpha, mu, q, l))]
    out = tuple(dev(b) for b in base)
    ops.gmm_vjp(dev(X), dev(alpha), dev(mu), dev(q), dev(l), ell_bar=0.5, out=out, accumulate=True)
    for g, b, r in zip(out, base, ref):
        assert rel_l2(host(g), b + r) <= TOL_F32


def test_gmm_empty_and_unsupported(ops):
    from paper_2202_10297_amd import capi

    X, alpha, mu, q, l = workloads.gmm(0, 32, 3, seed=1)
    X = np.zeros((0, 32), dtype=np.float32)
    ll, _ = ops.gmm_objective(dev(X).reshape(0, 32), dev(alpha), dev(mu), dev(q), dev(l))
    assert host(ll)[0] == 0.0
    ab, mb, qb, lb = ops.gmm_vjp(dev(X).reshape(0, 32), dev(alpha), dev(mu), dev(q), dev(l))
    assert np.all(host(ab) == 0) and np.all(host(mb) == 0) and np.all(host(lb) == 0)
    assert np.all(host(qb) == 0)
    # D outside the built shapes is refused before any launch
    L = capi.lib()
    assert L.pvjp_gmm_objective(8, 10, 48, 3, 8, 8, 8, 8, 8, None, None, 256, 1 << 20, None) == capi.PVJP_EUNSUPPORTED


def test_gmm_full_size_sampled(ops, orc):
    # N = 10^6, D = 64, K = 200: per-point LSE on sampled points against the
    # oracle (each LSE_i depends on point i only), and properties of the full
    # gradient: sum(alpha_bar) = 0, and additivity over two halves of the data.
    N, D, K = 1_000_000, 64, 200
    X, alpha, mu, q, l = workloads.gmm(N, D, K, seed=0)
    Xd = dev(X)
    P = [dev(a) for a in (alpha, mu, q, l)]
    ll, lse = ops.gmm_objective(Xd, *P)
    idx = np.random.default_rng(5).choice(N, 24, replace=False)
    _, rl = orc.gmm_objective(X[idx], alpha, mu, q, l)
    assert rel_l2(host(lse)[idx], rl) <= TOL_F32
    from scipy.special import logsumexp

    expect = host(lse).sum() - N * logsumexp(alpha.astype(np.float64)) - 0.5 * N * D * np.log(2 * np.pi)
    assert abs(host(ll)[0] - expect) <= 1e-12 * abs(expect)
    g = [host(t) for t in ops.gmm_vjp(Xd, *P, lse=lse)]
    assert abs(g[0].sum()) <= 1e-5 * np.abs(g[0]).sum()
    h = N // 2
    g1 = [host(t) for t in ops.gmm_vjp(dev(X[:h]), *P)]
    g2 = [host(t) for t in ops.gmm_vjp(dev(X[h:]), *P)]
    # alpha_bar's -N softmax(alpha) term splits with N as well
    for a, b, c in zip(g, g1, g2):
        assert rel_l2(b + c, a) <= TOL_F32
    # the s_ik checkpoint form at full size: same gradient as the recomputing
    # form within the FP32 bar (both are checked against the oracle at small N)
    _, lse2, sck = ops.gmm_objective_ckpt(Xd, *P)
    assert np.array_equal(host(lse2), host(lse))
    gs = [host(t) for t in ops.gmm_vjp(Xd, *P, lse=lse2, s=sck)]
    for name, a, b in zip(["alpha", "mu", "q", "l"], g, gs):
        assert rel_l2(b, a) <= TOL_F32, name


def _q_of(q, l, D):
    Q = torch.diag_embed(torch.exp(q))
    r, c = np.tril_indices(D, -1)  # row-major below the diagonal: the packing of l
    Q[:, r, c] = l
    return Q


def _exact(X, alpha, mu, q, l, comps, ell_bar=1.0):
    """(loglik, LSE_i, the adjoints of the components `comps`) in FP64 torch."""
    X, alpha, mu, q, l = [dev(a).double() for a in (X, alpha, mu, q, l)]
    N, D = X.shape
    Q = _q_of(q, l, D)

    def z(k):
        return (X - mu[k]) @ Q[k].T.contiguous()

    s = torch.stack([alpha[k] + q[k].sum() - 0.5 * (z(k) ** 2).sum(1) for k in range(alpha.numel())])
    lse = torch.logsumexp(s, 0)
    lse_a = torch.logsumexp(alpha, 0)
    ll = lse.sum() - N * lse_a - 0.5 * N * D * np.log(2 * np.pi)
    r, c = np.tril_indices(D, -1)
    out = [[], [], [], []]
    for k in comps:
        w = ell_bar * torch.exp(s[k] - lse)
        zk, y = z(k), X - mu[k]
        G = (w[:, None] * zk).T.contiguous() @ y
        out[0].append(w.sum() - N * ell_bar * torch.exp(alpha[k] - lse_a))
        out[1].append(Q[k].T @ (w[:, None] * zk).sum(0))
        out[2].append(w.sum() - torch.exp(q[k]) * torch.diagonal(G))
        out[3].append(-G[r, c])
    return host(ll), host(lse), [host(torch.stack(o)) for o in out]


@pytest.mark.parametrize("N,D,K", [(127, 32, 50), (10007, 32, 50), (3001, 64, 21), (131073, 32, 50),
                                   (140001, 64, 41)])
@pytest.mark.parametrize("where", ["first", "starts", "inside", "range", "all_but_one"])
def test_gmm_components_of_weight_zero(ops, N, D, K, where):
    # alpha = -inf at k = 0, at the starts of the ranges that the objective
    # splits the components into (multiples of four, two in D = 64, and of the
    # long form's 16 or more), inside one and over whole ones: such components
    # add nothing, and the others' results are finite.
    X, alpha, mu, q, l = workloads.gmm(N, D, K, seed=N + K)
    off = {"first": [0], "starts": list(range(4, K, 4)), "inside": [1, 6, K - 1], "range": list(range(4, 12)) +
           list(range(K // 2, K)), "all_but_one": [k for k in range(K) if k != K // 3]}[where]
    alpha[off] = -np.inf
    comps = sorted({0, 1, 4, 5, K // 3, K // 2, K - 1})
    rll, rlse, ref = _exact(X, alpha, mu, q, l, comps, -0.75)
    Xd, P = dev(X), [dev(a) for a in (alpha, mu, q, l)]
    ll, lse, sck = ops.gmm_objective_ckpt(Xd, *P)
    assert abs(host(ll)[0] - rll) <= TOL_F32 * abs(rll)
    assert rel_l2(host(lse), rlse) <= TOL_F32
    for s in (None, sck):
        got = [host(g) for g in ops.gmm_vjp(Xd, *P, lse=lse, s=s, ell_bar=-0.75)]
        assert all(np.isfinite(g).all() for g in got)
        for g, r in zip(got, ref):
            assert rel_l2(g[comps], r) <= TOL_F32


@pytest.mark.parametrize("D", [32, 64])
def test_gmm_long_chunks_exact(ops, D):
    # K = 64 at 10^6 points: chunks of 31,296, near the 32,768 that the bf16 form
    # sums in FP32 at most; its gradient against 64 bits, with and without s.
    N, K = 1_000_000, 64
    X, alpha, mu, q, l = workloads.gmm(N, D, K, seed=D)
    comps = [0, 7, 8, 63]
    rll, rlse, ref = _exact(X, alpha, mu, q, l, comps)
    Xd, P = dev(X), [dev(a) for a in (alpha, mu, q, l)]
    ll, lse, sck = ops.gmm_objective_ckpt(Xd, *P)
    assert abs(host(ll)[0] - rll) <= TOL_F32 * abs(rll)
    assert rel_l2(host(lse), rlse) <= TOL_F32
    for s in (None, sck):
        got = ops.gmm_vjp(Xd, *P, lse=lse, s=s)
        for g, r in zip(got, ref):
            assert rel_l2(host(g)[comps], r) <= TOL_F32
