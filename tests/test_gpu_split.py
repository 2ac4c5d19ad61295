"""The dense products on bf16 parts, at the edges of their tiles, against the
fp64 oracle: sample counts around the 48-sample tile of the deep nets' chain,
with candidates in every layer kind (the longest chains first in the grid),
commits of every layer (each must leave the split copy of the weights equal to
the weights: later steps read it), and a resume that rebuilds it."""
import numpy as np
import pytest
import torch

from parity_util import ParityStats, assert_state_equal, make_pair, replay_trace
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
    # the split copy kept through the commits equals one made from the weights
    cands = ctx.propose(99, 13)
    _, before = ctx.eval_losses(cands)
    ctx.rollback()
    ctx.set_state(ctx.params()[0], None, 30)
    _, after = ctx.eval_losses(cands)
    ctx.rollback()
    # (the caches are recomputed: fields differ in their last bits)
    np.testing.assert_allclose(before, after, rtol=1e-3, atol=1e-9)
    ctx.close()
