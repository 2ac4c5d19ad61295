"""The dense products on bf16 parts, at the edges of their tiles, against the
fp64 oracle: sample counts around the 48-sample tile of the deep nets' chain,
with candidates in every layer kind (the longest chains first in the grid), and a
resume that rebuilds the split copy of the weights; commits of every layer of
every net kind, each of which must leave that copy equal to the weights (bit for
bit against a context made from them); changes near the end of fp32; batches
larger than the lists of moved samples."""
import numpy as np
import pytest
import torch

from parity_util import (ParityStats, _oracle_step, assert_state_equal, make_pair,
                         replay_trace)
from workloads import CONFIGS, mlp_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act,N", [("tanh", 47), ("relu", 48), ("gauss", 49), ("tanh", 97)])
def test_chain_tiles(act, N):
    assert torch.cuda.is_available()
    cfg = CONFIGS["deep"].scaled(name=f"split_{act}_{N}", widths=(64, 256, 256, 256, 256, 10),
                                 act=act, gamma=0.4 if act == "gauss" else 1.0,
                                 data="sparse_uniform", n_samples=N, K=13, delta=0.1,
                                 seed_stream=5000 + N)
    print(f"[gpu] {cfg.name} {cfg.widths}", flush=True)
    w = mlp_workload(cfg)
    ctx, ref = make_pair(cfg, w, k_max=13)
    ps = ParityStats(cfg.name)
    st, ch, dl = ctx.run_steps(30, 13, trace=True, trace_dloss=True)
    _, acc = replay_trace(ref, cfg, 0, ch, dl, 13, ps)
    assert st.accepted == acc >= 5
    assert_state_equal(ctx, ref)
    # after a resume, which makes the split copy anew, the same candidates score
    # the same
    cands = ctx.propose(99, 13)
    _, before = ctx.eval_losses(cands)
    ctx.rollback()
    ctx.set_state(ctx.params()[0], None, 30)
    _, after = ctx.eval_losses(cands)
    ctx.rollback()
    # (the caches are recomputed: fields differ in their last bits)
    np.testing.assert_allclose(before, after, rtol=1e-3, atol=1e-9)
    ctx.close()


@pytest.mark.parametrize("base,net", [
    ("deep", dict(widths=(64, 256, 256, 256, 256, 10))),
    ("deep", dict(widths=(64, 512, 512, 512, 512, 10))),
    ("deepln", dict(widths=(64, 256, 256, 256, 10), layer_pick="layer")),
    ("deepln", dict(widths=(64, 1024, 1024, 1024, 10), layer_pick="layer", layer_norm=False)),
    ("channel", dict(widths=(64, 256, 256, 256, 10))),
], ids=["chain", "wide", "normalized", "bias", "channel"])
def test_split_copy_after_each_commit(base, net):
    """After a commit in each layer (a channel: in all of them) and a forward pass,
    candidates score to the same bits as on a context made from the parameters: a
    split weight that a commit left behind would move every change that passes
    through it."""
    K = 40
    cfg = CONFIGS[base].scaled(name=f"copy_{base}", act="tanh", data="sparse_uniform", n_samples=70, K=K,
                               delta=0.3, seed_stream=5100, **net)
    print(f"[gpu] {cfg.name} {cfg.widths}", flush=True)
    w = mlp_workload(cfg)
    ctx, _ = make_pair(cfg, w, k_max=K)
    channel = cfg.mutation != "single"
    propose = lambda c, t: c.propose_channels(t, K) if channel else c.propose(t, K)
    score = lambda c, r: (c.eval_channels(r) if channel else c.eval_losses(r))[1]
    for n, layer in enumerate([None] * 3 if channel else range(cfg.n_layers)):
        cands = propose(ctx, n)
        pick = range(K) if channel else np.flatnonzero(cands["layer"] == layer)
        score(ctx, cands)
        before = ctx.params()[0]
        ctx.commit(int(pick[0]))
        after = ctx.params()[0]
        moved = [l for l in range(cfg.n_layers) if (before[l] != after[l]).any()]
        assert moved == (list(range(cfg.n_layers)) if channel else [layer])
        ctx.refresh()
        fresh, _ = make_pair(cfg, dict(w, weights=after), k_max=K)
        cands = propose(ctx, 100 + n)
        assert score(ctx, cands).tobytes() == score(fresh, cands).tobytes(), layer
        ctx.rollback()
        fresh.close()
    ctx.close()


@pytest.mark.parametrize("base,net", [
    ("deep", dict(widths=(64, 256, 256, 256, 256, 10))),
    ("deep", dict(widths=(64, 512, 512, 512, 512, 10))),
    ("deep", dict(widths=(64, 1024, 1024, 1024, 10))),
    ("deepln", dict(widths=(64, 256, 256, 256, 10), layer_norm=False, layer_pick="layer")),
], ids=["chain", "wide512", "wide1024", "bias"])
def test_changes_near_the_end_of_fp32(base, net):
    """First-layer mutations through a second layer with weights of 2^-115: the
    activation changes that the dense layers take on are of about 2^-122 and keep
    their relative accuracy.  The errors' rms stays below 2^-24 of the rms size of
    the changes' first-order terms (each is an average over the samples' roundings:
    4e-9 to 5e-9 is seen, and 2e-6 to 1e-5 from values split as they are)."""
    cfg = CONFIGS[base].scaled(name=f"tiny_{base}_{net['widths'][1]}", act="tanh", data="sparse_uniform",
                               n_samples=150, K=24, delta=0.1, seed_stream=5200, **net)
    print(f"[gpu] {cfg.name} {cfg.widths}", flush=True)
    w = mlp_workload(cfg)
    w["weights"][1] = w["weights"][1] * np.float32(2.0 ** -111)
    ctx, ref = make_pair(cfg, w, k_max=24)
    err, size = [], []
    for t in range(6):
        _, rc, dls, mags, _, _, _ = _oracle_step(ref, cfg, t, 24, 0.0, 0.0, 0)
        _, dl = ctx.eval_losses(ctx.propose(t, 24))
        ctx.rollback()
        first = [k for k in range(24) if rc[k].layer == 0]
        err += [dl[k] - dls[k] for k in first]
        size += [mags[k] for k in first]
    assert len(err) >= 15 and max(size) < 1e-35
    ratio = np.sqrt(np.sum(np.square(np.array(err) * 1e38)) / np.sum(np.square(np.array(size) * 1e38)))
    print(f"[gpu] rms error over rms size {ratio:.2e}", flush=True)
    assert ratio <= 2.0 ** -24
    ctx.close()


@pytest.mark.parametrize("base,net", [
    ("deepln", dict(widths=(64, 256, 256, 10), layer_pick="layer")),
    ("deep", dict(widths=(64, 512, 512, 512, 10))),
    ("channel", dict(widths=(64, 256, 256, 256, 10))),
], ids=["normalized", "wide", "channel"])
@pytest.mark.parametrize("N", [130, 65537])
def test_batch_past_the_lists(base, net, N):
    """150 candidates at once are scored to the same bits as 50 at a time (lists
    are held for 64 on 65537 samples), one past the first 64 commits as it does
    alone, and reading
    the parameters between evaluation and commit changes nothing (a biased net's
    pass through the lists' memory)."""
    K = 150
    cfg = CONFIGS[base].scaled(name=f"lists_{base}", data="sparse_uniform", n_samples=N, K=K,
                               delta=0.1, seed_stream=5300, **net)
    print(f"[gpu] {cfg.name} {cfg.widths}", flush=True)
    w = mlp_workload(cfg)
    ctx, _ = make_pair(cfg, w, k_max=K)
    alone, _ = make_pair(cfg, w, k_max=50)
    channel = cfg.mutation != "single"
    cands = ctx.propose_channels(0, K) if channel else ctx.propose(0, K)
    score = lambda c, r: (c.eval_channels(r) if channel else c.eval_losses(r))[1]
    parts = []
    for g in range(0, K, 50):
        parts.append(score(alone, cands[g:g + 50]))
        alone.rollback()
    dl = score(ctx, cands)
    assert dl.tobytes() == np.concatenate(parts).tobytes()
    k = 64 + int(np.argmax(np.abs(dl[64:])))
    assert dl[k] != 0.0
    before = ctx.params()[0]
    ctx.commit(k)
    score(alone, cands[k:k + 1])
    alone.commit(0)
    assert ctx.loss()[0] == alone.loss()[0]
    assert ctx.sample_losses().tobytes() == alone.sample_losses().tobytes()
    after = ctx.params()[0]
    assert [a.tobytes() for a in after] == [a.tobytes() for a in alone.params()[0]]
    assert sum(int((a != b).sum()) for a, b in zip(before, after)) >= 1
    ctx.close()
    alone.close()
