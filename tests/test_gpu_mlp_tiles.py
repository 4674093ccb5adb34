"""Cost-model kernels at the edges of their tiles (32 samples), of the
single-workgroup batches (below 64) and of several tiles per workgroup (above
16384), against the fp64 reference.

Tolerance of the small batches: an element is a sum of products of sums; with u
= 2^-24 its error is at most (roundings on a path) u times the same expression
with every term replaced by its absolute value.  A path has at most 16 + 64 +
64 + 10 roundings to an output, 64 + 10 more to a delta and 32 + 8 + 64 more to
a gradient: 400 u covers all.  A hidden unit within that error of zero may be
cut on one side only, so inputs (seeds) are taken where the reference has none.
"""
import numpy as np
import pytest

from oracle import mlp_ref as R

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

U = 400 * 2.0 ** -24


@pytest.fixture(scope="module")
def mods():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_00806_amd import _lib as L, costmodel as CM
    return CM, L


def layers(p):
    return (p[:1024].reshape(64, 16), p[1024:1088], p[1088:5184].reshape(64, 64), p[5184:5248],
            p[5248:5376].reshape(2, 64), p[5376:])


def absolute(p, norm, X, T):
    """Bounds: outputs, gradients and loss with every term made positive."""
    W1, b1, W2, b2, W3, b3 = (np.abs(a) for a in layers(p))
    xn = (np.abs(X) + np.abs(norm[:16])) / norm[16:32]
    a1 = xn @ W1.T + b1
    a2 = a1 @ W2.T + b2
    y = a2 @ W3.T + b3
    e = y + (np.abs(T) + np.abs(norm[32:34])) / norm[34:36]
    dy = 2.0 * e / e.size
    d2 = dy @ W3
    d1 = d2 @ W2
    g = np.concatenate([(d1.T @ xn).reshape(-1), d1.sum(0), (d2.T @ a1).reshape(-1), d2.sum(0),
                        (dy.T @ a2).reshape(-1), dy.sum(0)])
    return y * norm[34:36] + np.abs(norm[32:34]), g, np.mean(e * e), a1, a2


def inputs(CM, B):
    for seed in range(200):
        rng = np.random.default_rng(1000 * B + seed)
        X = rng.normal(1.0, 2.0, (B, 16)).astype(np.float32)
        T = rng.normal(0.0, 1.5, (B, 2)).astype(np.float32)
        p, norm = CM.init_params(seed), np.concatenate([rng.normal(size=16), rng.uniform(0.5, 2, 16),
                                                        rng.normal(size=2), rng.uniform(0.5, 2, 2)]).astype(np.float32)
        p64, n64, X64, T64 = (a.astype(np.float64) for a in (p, norm, X, T))
        W1, b1, W2, b2, _, _ = layers(p64)
        z1 = ((X64 - n64[:16]) / n64[16:32]) @ W1.T + b1
        z2 = np.maximum(z1, 0) @ W2.T + b2
        _, _, _, A1, A2 = absolute(p64, n64, X64, T64)
        if (np.abs(z1) > U * A1).all() and (np.abs(z2) > U * A2).all():
            return X, T, p, norm, (p64, n64, X64, T64)
    raise AssertionError("no inputs away from the cuts")


def gradient(CM, L, m, X, T):
    Xd, Td = torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda()
    n = int(L.lib().wpm_mlp_work_floats(len(X)))
    work = torch.full((n + 64,), 7.0, dtype=torch.float32, device="cuda")
    g = torch.full((L.MLP_PARAMS,), 7.0, dtype=torch.float32, device="cuda")
    loss = torch.full((1,), 7.0, dtype=torch.float32, device="cuda")
    m.grad(Xd, Td, work, g, loss)
    assert bool((work[n:] == 7.0).all()), "work buffer overrun"
    return g.cpu().numpy().astype(np.float64), float(loss.item())


@pytest.mark.parametrize("B", [1, 2, 31, 32, 33, 39, 63, 64, 65, 97])
def test_edges_of_tiles(mods, B):
    CM, L = mods
    X, T, p, norm, ref = inputs(CM, B)
    print(f"[gpu] cost model, batch {B}", flush=True)
    m = CM.CostModel(p, norm)
    ya, ga, la, _, _ = absolute(*ref)
    want, _ = R.forward(ref[0], ref[1], ref[2])
    assert (np.abs(m.predict(X) - want) <= U * ya).all()
    lref, gref = R.loss_and_grad(*ref)
    g, loss = gradient(CM, L, m, X, T)
    assert (np.abs(g - gref) <= U * ga).all(), np.max(np.abs(g - gref) / ga)
    assert abs(loss - lref) <= U * la
    assert np.array_equal(gradient(CM, L, m, X, T)[0], g)


def test_several_tiles_per_workgroup(mods):
    """A batch of more tiles than workgroups against its pieces: each sample's
    share is the same in both, the sums differ by their roundings."""
    CM, L = mods
    B, step = 512 * 32 * 2 + 77, 4096
    rng = np.random.default_rng(5)
    X = rng.normal(1.0, 2.0, (B, 16)).astype(np.float32)
    T = rng.normal(0.0, 1.5, (B, 2)).astype(np.float32)
    p, norm = CM.init_params(9), CM.make_norm(X, T)
    m = CM.CostModel(p, norm)
    g, loss = gradient(CM, L, m, X, T)
    _, ga, la, _, _ = absolute(*(a.astype(np.float64) for a in (p, norm, X, T)))
    gs, ls = np.zeros(L.MLP_PARAMS), 0.0
    for s in range(0, B, step):
        gi, li = gradient(CM, L, m, X[s:s + step], T[s:s + step])
        n = min(step, B - s)
        gs, ls = gs + gi * n / B, ls + li * n / B
    assert (np.abs(g - gs) <= U * ga).all()
    assert abs(loss - ls) <= U * la
