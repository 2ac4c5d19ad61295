"""Class counts other than ten on the GPU against the fp64 oracle: the slab,
chain, channel and dense-layer kernels have variants for exactly ten classes,
and nets with fewer (or more) take the general ones.  A ten-class variant
given a net of fewer classes would read and write rows past its logits."""
import numpy as np
import pytest
import torch

from parity_util import ParityStats, assert_state_equal, make_pair, replay_trace
from workloads import CONFIGS, mlp_workload

pytestmark = pytest.mark.gpu

NETS = [
    ("ternary", dict(widths=(784, 96, 80)), 12),
    ("deep", dict(widths=(784, 256, 256, 256)), 8),
    ("channel", dict(widths=(784, 256, 256, 256)), 4),
    ("deepln", dict(widths=(784, 256, 256), layer_pick="layer", delta=0.05), 8),
]


@pytest.mark.parametrize("C", [3, 9, 13])
@pytest.mark.parametrize("base,net,K", NETS)
def test_class_count(base, net, K, C):
    assert torch.cuda.is_available()
    net = dict(net, widths=net["widths"] + (C,))
    cfg = CONFIGS[base].scaled(name=f"{base}_c{C}", n_samples=333, K=K, seed_stream=4900 + C, **net)
    print(f"[gpu] {cfg.name} {cfg.widths}", flush=True)
    w = mlp_workload(cfg)
    ctx, ref = make_pair(cfg, w, k_max=K)
    ps = ParityStats(f"{cfg.name} {'-'.join(map(str, cfg.widths))}")
    st, ch, dl = ctx.run_steps(12, K, trace=True, trace_dloss=True)
    _, acc = replay_trace(ref, cfg, 0, ch, dl, K, ps)
    assert st.accepted == acc >= 1
    assert_state_equal(ctx, ref)
    before = ctx.sample_losses()
    ctx.refresh()
    np.testing.assert_allclose(before, ctx.sample_losses(), rtol=3e-5, atol=3e-6)
    ctx.close()
