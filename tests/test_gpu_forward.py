"""The full forward pass at the edges of its kernels' tiles (rows of 64 and
128, 128 columns, chunks of 32 k, logit layers in blocks of 128 k, reduction
widths that are no multiple of four), against 64-bit numpy.

Tolerance: the first-order bound of fp32 sums.  With u = 2^-24, a layer's field
is off by at most (n + 16) u sum |w| |a| for its n terms and the operands'
rounding, plus the error of its inputs through |w|; tanh and relu do not
enlarge an error and add 8 u.  A sample's loss moves by at most twice the
largest logit error, plus 32 u of its own size.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [((17, 17, 2), 1), ((33, 129, 10), 129), ((100, 64, 16), 63), ((31, 65, 130, 3), 200),
          ((16, 100, 10), 127), ((257, 300, 33, 7), 1001), ((784, 512, 10), 2050), ((32, 8, 9), 128),
          ((21, 4100, 11), 2051), ((64, 4096, 10), 2048)]


@pytest.mark.parametrize("act", ["tanh", "relu"])
@pytest.mark.parametrize("widths,N", SHAPES, ids=["-".join(map(str, w)) + f"x{n}" for w, n in SHAPES])
def test_forward_edges(widths, N, act):
    from paper_2607_08406_amd import mca

    rng = np.random.default_rng(sum(widths) + N)
    X = (rng.random((N, widths[0])) * (rng.random((N, widths[0])) < 0.5)).astype(np.float32)
    y = rng.integers(0, widths[-1], N).astype(np.int32)
    W = [((rng.random((m, n)) * 2 - 1) * np.sqrt(3.0 / n)).astype(np.float32)
         for n, m in zip(widths[:-1], widths[1:])]
    ctx = mca.Context(mca.mlp_desc(list(widths), act, delta=0.1, seed=1, stream_tag=1), W, X, y, k_max=1)
    u = 2.0 ** -24
    a, err = X.astype(np.float64), 0.0
    for l, w in enumerate(W):
        w = w.astype(np.float64)
        z = a @ w.T
        size = np.abs(a) @ np.abs(w).T
        err = (w.shape[1] + 16) * u * size + (0.0 if l == 0 else err @ np.abs(w).T)
        a = np.tanh(z) if act == "tanh" else np.maximum(z, 0.0)
        if l < len(W) - 1:
            err = err + 8 * u
    top = z.max(1)
    loss = np.log(np.exp(z - top[:, None]).sum(1)) + top - z[np.arange(N), y]
    tol = 2 * err.max(1) + 32 * u * (1 + np.abs(loss) + np.abs(z).max(1))
    for again in range(2):
        got = ctx.sample_losses()
        ratio = np.abs(got - loss) / tol
        assert got.shape == (N,) and ratio.max() <= 1, (again, ratio.max(), int(ratio.argmax()))
        ctx.refresh()
    ctx.close()


@pytest.mark.parametrize("widths,lit", [((784, 64, 2), 0.2), ((101, 257, 2), 1.0), ((64, 256, 256, 2), 0.5)])
def test_forward_rounds_to_neither_side(widths, lit):
    """The fields' errors have mean zero: a sample's loss is the sum of its last
    hidden units (ReLU; near 30, where the other class's share is below an ulp),
    so its error adds up theirs.  Over 20000 samples the mean of rounding errors
    stays within a few of its standard errors (their deviation over
    sqrt(20000)); 10 is allowed, and sums rounded towards one side were off by
    60 and more."""
    from paper_2607_08406_amd import mca

    N, H = 20000, widths[-2]
    rng = np.random.default_rng(sum(widths))
    X = (rng.random((N, widths[0])) * (rng.random((N, widths[0])) < lit)).astype(np.float32)
    W = [((rng.random((m, n)) * 2 - 1) * np.sqrt(3.0 / n)).astype(np.float32)
         for n, m in zip(widths[:-2], widths[1:-1])]
    a = X.astype(np.float64)
    for w in W:
        a = np.maximum(a @ w.astype(np.float64).T, 0.0)
    top = np.zeros((2, H), np.float32)
    top[0] = np.float32(2.0 ** np.ceil(np.log2(30.0 / a.sum(1).min())))
    loss = a.sum(1) * float(top[0, 0])
    assert loss.min() >= 30.0
    ctx = mca.Context(mca.mlp_desc(list(widths), "relu", delta=0.1, seed=1, stream_tag=1), W + [top], X,
                      np.ones(N, np.int32), k_max=1)
    err = (ctx.sample_losses() - loss) / loss
    off = err.mean() / (err.std() / np.sqrt(N))
    print(f"[gpu] {widths} mean {err.mean():.2e} deviation {err.std():.2e}: {off:+.1f} standard errors", flush=True)
    assert abs(off) <= 10
    ctx.close()


@pytest.mark.parametrize("N,H", [(300, 64), (70, 200)])
def test_forward_of_tiny_activations(N, H):
    """Gaussian units far out (exp(-z^2) near 2^-123) under weights of 2^118: the
    next layer's fields are of ordinary size.  Relative error of an activation:
    its exponent, about 85, in fp32 (z, z^2 and its product with log2 e each
    rounded, 4 x 2^-24 of it), 2e-5; split as they are, such values have 10 bits."""
    from paper_2607_08406_amd import mca

    rng = np.random.default_rng(N)
    X = np.full((N, 4), 1.0, np.float32)
    X[:, 1:] = rng.random((N, 3))
    W0 = np.zeros((H, 4), np.float32)
    W0[:, 0] = 9.16
    W0[:, 1:] = rng.random((H, 3)) * 0.05
    W1 = ((rng.random((20, H)) * 2 - 1) * 2.0 ** 118).astype(np.float32)
    W2 = (rng.random((3, 20)) * 2 - 1).astype(np.float32)
    y = rng.integers(0, 3, N).astype(np.int32)
    ctx = mca.Context(mca.mlp_desc([4, H, 20, 3], "gauss", delta=0.1, seed=1, stream_tag=1), [W0, W1, W2], X, y, k_max=1)
    a = X.astype(np.float64)
    z0 = a @ W0.astype(np.float64).T
    h = np.exp(-z0 * z0)
    err = h * 4 * 2.0 ** -24 * z0 * z0 @ np.abs(W1.astype(np.float64)).T
    z1 = h @ W1.astype(np.float64).T
    a1 = np.exp(-z1 * z1)
    z2 = a1 @ W2.astype(np.float64).T
    loss = np.log(np.exp(z2).sum(1)) - z2[np.arange(N), y]
    # |d exp(-z^2)| <= 0.86 |dz|, the logits' error through |W2|, twice it on the loss
    tol = 2 * ((0.86 * err + 2.0 ** -20) @ np.abs(W2.astype(np.float64)).T).max(1)
    got = ctx.sample_losses()
    assert 0.05 < np.abs(z1).mean() < 20 and (h < 2.0 ** -121).mean() > 0.9 and h.min() > 2.0 ** -126
    ratio = np.abs(got - loss) / tol
    print(f"[gpu] worst error over its bound {ratio.max():.3f}", flush=True)
    assert ratio.max() <= 1
    ctx.close()
