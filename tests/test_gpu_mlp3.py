"""GPU parity of three-layer MLPs against the fp64 oracle (through the C ABI).

A first-layer mutation moves one unit of the first hidden layer, every unit
of the second hidden layer for each affected sample (rank-1), and then the
logits; second- and third-layer mutations are the column cases of the
two-layer path.  Workloads: reduced ternary Gaussian and tanh nets whose
sample counts span several 16-sample tiles (12 for class counts other than ten)
and a ragged tail, and the full
ternary 784-1024-1024-10 net on 8,192 samples at K = 64.
"""
import numpy as np
import pytest
import torch

from oracle import mca as omca
from oracle.mlp import FullMLP, MLPState, per_sample_ce
from parity_util import (REL_TOL, ParityStats, assert_cands_equal, assert_state_equal,
                         check_batch, check_step, explicit_steps, kappa_of, make_pair,
                         replay_trace)
from workloads import CONFIGS, mlp_workload

pytestmark = pytest.mark.gpu


def banner(msg):
    print(f"[gpu] {msg}", flush=True)


@pytest.fixture(scope="module")
def mca():
    from paper_2607_08406_amd import mca as m
    m.load_library()
    assert torch.cuda.is_available()
    return m


def assert_caches_match(ctx, ref, rel=1e-5):
    """The device's cached per-sample losses against the oracle's (recomputed
    from its own fp64 caches)."""
    got = ctx.sample_losses()
    exp = per_sample_ce(ref.Z[-1], ref.y)
    np.testing.assert_allclose(got, exp, rtol=rel, atol=1e-6)


def layer_counts(ref, cfg, t0, n, K):
    counts = np.zeros(cfg.n_layers, dtype=int)
    for t in range(t0, t0 + n):
        _, rc, _, _ = omca.evaluate(ref, t, K, cfg.seed_stream, cfg.stream_tag, cfg.delta,
                                    cfg.layer_pick, cfg.accept_ties)
        for c in rc:
            counts[c.layer] += 1
    return counts


def test_ternary_three_layer_small(mca):
    """784-96-80-10 Gaussian ternary net on 333 samples (20 full tiles of 16
    and a tail of 13): explicit steps, then a device run replayed."""
    cfg = CONFIGS["ternary"].scaled(name="t3_small", widths=(784, 96, 80, 10), n_samples=333,
                                    K=16)
    banner(f"{cfg.name} {cfg.widths} N={cfg.n_samples}")
    w = mlp_workload(cfg)
    ctx, ref = make_pair(cfg, w, k_max=16)
    L, _ = ctx.loss()
    assert abs(L - ref.loss()) <= REL_TOL * ref.loss()
    ps = ParityStats("ternary 784-96-80-10")
    _, acc = explicit_steps(ctx, ref, cfg, 0, 40, 16, ps)
    assert acc > 5
    assert_state_equal(ctx, ref)
    assert_caches_match(ctx, ref)
    ctx.set_step(40)
    st, ch, dl = ctx.run_steps(60, 16, trace=True, trace_dloss=True)
    assert st.steps == 60
    replay_trace(ref, cfg, 40, ch, dl, 16, ps)
    assert_state_equal(ctx, ref)
    assert_caches_match(ctx, ref)
    # first-layer candidates were drawn and some were committed
    first = [int(c) for n, c in enumerate(ch) if c >= 0]
    assert len(first) > 5
    ctx.close()


def test_three_layer_other_class_count(mca):
    """784-64-48-13 Gaussian ternary net on 250 template images: thirteen
    classes run the general variant of the layer-(L-3) kernel (12-sample
    tiles) and of the column kernels."""
    cfg = CONFIGS["ternary"].scaled(name="t3_c13", widths=(784, 64, 48, 13), n_samples=250, K=16)
    banner(f"{cfg.name} {cfg.widths} N={cfg.n_samples}")
    w = mlp_workload(cfg)
    ctx, ref = make_pair(cfg, w, k_max=16)
    L, _ = ctx.loss()
    assert abs(L - ref.loss()) <= REL_TOL * ref.loss()
    counts = layer_counts(ref, cfg, 0, 30, 16)
    assert counts[0] > 20  # the first layer is exercised
    ps = ParityStats("ternary 784-64-48-13")
    explicit_steps(ctx, ref, cfg, 0, 30, 16, ps)
    assert_state_equal(ctx, ref)
    assert_caches_match(ctx, ref)
    ctx.set_step(30)
    st, ch, dl = ctx.run_steps(30, 16, trace=True, trace_dloss=True)
    replay_trace(ref, cfg, 30, ch, dl, 16, ps)
    assert_state_equal(ctx, ref)
    assert_caches_match(ctx, ref)
    ctx.close()


def test_tanh_three_layer_continuous(mca):
    """64-48-40-10 tanh net with continuous weights on 500 samples, K = 8."""
    cfg = CONFIGS["tiny"].scaled(name="tanh3", widths=(64, 48, 40, 10), n_samples=500, K=8)
    banner(f"{cfg.name} {cfg.widths} N={cfg.n_samples}")
    w = mlp_workload(cfg)
    ctx, ref = make_pair(cfg, w, k_max=8)
    counts = layer_counts(ref, cfg, 0, 50, 8)
    assert counts[0] > 20  # the first layer is exercised
    ps = ParityStats("tanh 64-48-40-10")
    explicit_steps(ctx, ref, cfg, 0, 50, 8, ps)
    assert_state_equal(ctx, ref)
    assert_caches_match(ctx, ref)
    ctx.set_step(50)
    st, ch, dl = ctx.run_steps(150, 8, trace=True, trace_dloss=True)
    replay_trace(ref, cfg, 50, ch, dl, 8, ps)
    assert_state_equal(ctx, ref)
    assert_caches_match(ctx, ref)
    ctx.close()


@pytest.mark.parametrize("N", [1, 15, 16, 17, 23, 24, 25, 49])
def test_three_layer_tile_edges(mca, N):
    cfg = CONFIGS["ternary"].scaled(name=f"t3_n{N}", widths=(784, 40, 36, 10), n_samples=N, K=8)
    w = mlp_workload(cfg)
    ctx, ref = make_pair(cfg, w, k_max=8)
    explicit_steps(ctx, ref, cfg, 0, 25, 8, ParityStats(f"ternary 784-40-36-10 N={N}"))
    assert_state_equal(ctx, ref)
    assert_caches_match(ctx, ref)
    ctx.close()


@pytest.mark.parametrize("n2,ternary", [(192, False), (193, False), (384, True), (385, True)])
def test_three_layer_lanes_per_pair(mca, n2, ternary):
    """Columns at the line between half a wave and a whole one for a pair of samples
    (192 entries, half of a ternary net's units)."""
    base = CONFIGS["ternary"] if ternary else CONFIGS["tiny"]
    cfg = base.scaled(name=f"t3_lanes{n2}", widths=(64, 48, n2, 10), data="sparse_uniform", n_samples=150, K=12)
    banner(f"{cfg.name} {cfg.widths}")
    w = mlp_workload(cfg)
    ctx, ref = make_pair(cfg, w, k_max=12)
    ps = ParityStats(f"three layers, {n2} units, ternary {int(ternary)}")
    explicit_steps(ctx, ref, cfg, 0, 20, 12, ps)
    ctx.set_step(20)
    _, ch, dl = ctx.run_steps(20, 12, trace=True, trace_dloss=True)
    replay_trace(ref, cfg, 20, ch, dl, 12, ps)
    assert_state_equal(ctx, ref)
    assert_caches_match(ctx, ref)
    ctx.close()


def test_rollback_three_layer_is_byte_identical(mca):
    cfg = CONFIGS["ternary"].scaled(name="t3_rb", widths=(784, 64, 48, 10), n_samples=200, K=16)
    w = mlp_workload(cfg)
    ctx, ref = make_pair(cfg, w, k_max=16)
    before_p, before_c = ctx.params()
    before_l = ctx.sample_losses()
    cands = ctx.propose(0, 16)
    ctx.eval_losses(cands)
    ctx.rollback()
    after_p, after_c = ctx.params()
    for a, b in zip(before_p, after_p):
        assert a.tobytes() == b.tobytes()
    for a, b in zip(before_c, after_c):
        assert a.tobytes() == b.tobytes()
    assert before_l.tobytes() == ctx.sample_losses().tobytes()
    ctx.close()


def test_full_ternary_workload(mca):
    """784-1024-1024-10 Gaussian ternary net on 8,192 samples, K = 64: init
    loss, one explicit step with every candidate against the incremental
    oracle and two first-layer candidates against full recomputation, then a
    short device run replayed."""
    cfg = CONFIGS["ternary"]
    banner("ternary 784-1024-1024-10 N=8192 K=64")
    w = mlp_workload(cfg)
    ctx, ref = make_pair(cfg, w, k_max=64)
    L, _ = ctx.loss()
    assert abs(L - ref.loss()) <= REL_TOL * ref.loss()
    ps = ParityStats("ternary 784-1024-1024-10 full")
    cands = ctx.propose(0, 64)
    losses, dl = ctx.eval_losses(cands)
    L_t, rc, dls, chosen = check_batch(ps, dl, ref, cfg, 0, 64)
    assert_cands_equal(cands, rc)
    full = FullMLP(MLPState(w["weights"], w["codes"], w["scales"]), w["X"], w["y"], cfg.act,
                   cfg.gamma)
    firsts = [k for k, c in enumerate(rc) if c.layer == 0][:2]
    assert firsts
    for k in firsts:
        assert abs(losses[k] - full.eval(rc[k])) <= REL_TOL * losses[k]
        d, _ = full.delta(rc[k])
        assert abs(dl[k] - d) <= 1e-5 * abs(d) + 1e-13, (k, dl[k], d)
    ctx.rollback()
    st, ch, dl = ctx.run_steps(50, 64, trace=True, trace_dloss=True)
    assert st.steps == 50
    replay_trace(ref, cfg, 0, ch, dl, 64, ps)
    assert_state_equal(ctx, ref)
    assert_caches_match(ctx, ref)
    ctx.close()


@pytest.mark.parametrize("kind", ["ternary", "deep"])
@pytest.mark.parametrize("empty", [1, 2])
def test_batch_with_empty_groups(mca, kind, empty):
    """A batch of 150 candidates whose first `empty` groups of 64 hold none of
    layer L-3: the tile kernel lists its candidates group by group and goes past
    a group that has none."""
    K = 150
    if kind == "ternary":
        cfg = CONFIGS["ternary"].scaled(name="t3_groups", widths=(784, 96, 80, 10), n_samples=333, K=K)
    else:
        cfg = CONFIGS["deep"].scaled(name="deep_groups", widths=(64, 256, 256, 256, 256, 10),
                                     data="sparse_uniform", n_samples=200, K=K, delta=0.1)
    banner(f"{cfg.name} {cfg.widths} N={cfg.n_samples} K={K} first {empty} groups empty")
    w = mlp_workload(cfg)
    ctx, ref = make_pair(cfg, w, k_max=K)
    tile_layer = cfg.n_layers - 3
    tile, other = [], []
    for t in range(16):
        rc = [ref.candidate(cfg.seed_stream, cfg.stream_tag, t, k, cfg.delta, cfg.layer_pick) for k in range(K)]
        for g, c in zip(ctx.propose(t, K), rc):
            (tile if c.layer == tile_layer else other).append((g, c))
    n = 64 * empty
    batch = other[:n] + tile[:K - n - 4] + other[n:n + 4 + max(0, K - n - 4 - len(tile))]
    assert len(batch) == K and sum(c.layer == tile_layer for _, c in batch) >= 15
    _, dl = ctx.eval_losses(np.array([g for g, _ in batch], dtype=batch[0][0].dtype))
    ctx.rollback()
    ps = ParityStats(f"{kind} batch of 150, {empty} empty groups")
    exp, mags = zip(*[omca._delta(ref, c) for _, c in batch])
    check_step(ps, dl, exp, mags, [kappa_of(cfg, c) for _, c in batch], [0.0] * K, cfg.accept_ties, -1, -1)
    ctx.close()
