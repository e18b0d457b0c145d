"""The whole-network fp32 MLP kernel at the edges of its tiles: widths around 64 / 128 / 256, ragged observations and
batches, one to three hidden layers, one to four head tiles, both state-tile counts (32 states per workgroup above 4096 states of
256 units or 8192 of 128, else 16) and a width that stays on the layer-by-layer path.  The bound is the forward error bound of the
sums themselves: a dot product of K terms in any order is within (K + 2) eps of sum |w||x| + |b|, and |W| carries the error of the
layer before."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from helpers import check_sampler_self_consistency

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,hidden,A,relu,B", [
    (4, [64, 64], 2, True, 1), (4, [64, 64], 2, True, 33), (24, [256, 256], 4, True, 4096), (24, [256, 256], 4, True, 4113),
    (1, [1], 1, True, 17), (65, [63, 127, 128], 18, True, 50), (200, [255], 63, False, 31), (256, [256, 3, 129], 15, False, 16),
    (17, [33, 65], 16, True, 5000), (8, [257], 3, True, 40),
    (17, [33, 65], 16, True, 8209), (9, [64, 30], 5, True, 8209),
])
def test_whole_network_kernel(D, hidden, A, relu, B):
    import paper_2211_15023_amd as Amd
    rng = np.random.default_rng(D * 1000 + B)
    dims = [D] + hidden
    layers = [dict(kind="dense", cin=i, cout=o, relu=relu) for i, o in zip(dims, hidden)]
    net = SimpleNamespace(name="mlp", obs_dtype="f32", obs_shape=(D,), n_actions=A, layers=layers)
    tensors = [dict(w=(rng.uniform(-1, 1, (o, i)) * (3.0 / i) ** 0.5).astype(np.float32), b=rng.uniform(-0.5, 0.5, o).astype(np.float32))
               for i, o in zip(dims, hidden + [A + 1])]
    x = rng.standard_normal((B, D)).astype(np.float32)
    u = rng.random(B).astype(np.float32) * np.float32(0.999)
    pol = Amd.Policy(net, "fp32", tensors)
    plan = Amd.accerl_plan_describe(pol.arch, Amd.pack_weights(tensors))
    assert ("whole_network=1" in plan) == (max(dims) <= 256)
    print(f"fp32 mlp D={D} hidden={hidden} A={A} B={B}", flush=True)
    logits, value, action = (t.cpu().numpy() for t in pol.forward(torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda()))
    ref, err, eps = x.astype(np.float64), np.zeros((B, D)), 2.0 ** -24
    for t, last in zip(tensors, [False] * len(hidden) + [True]):
        w, b = t["w"].astype(np.float64), t["b"].astype(np.float64)
        err = err @ np.abs(w).T + (w.shape[1] + 2) * eps * ((np.abs(ref) + err) @ np.abs(w).T + np.abs(b))
        ref = ref @ w.T + b
        if relu and not last:
            ref = np.maximum(ref, 0)
    got = np.concatenate([logits, value[:, None]], axis=1)
    assert np.all(np.abs(got - ref) <= err)
    check_sampler_self_consistency(action, logits, u)


def test_infinite_observations_stay_in_their_units():
    """Padded units and padded inputs must not turn an infinity into NaN (0 * inf): a ReLU network with positive weights
    carries +inf to every logit, as its layers do one by one."""
    import paper_2211_15023_amd as Amd
    net = SimpleNamespace(name="mlp", obs_dtype="f32", obs_shape=(3,), n_actions=2,
                          layers=[dict(kind="dense", cin=3, cout=5, relu=True), dict(kind="dense", cin=5, cout=7, relu=True)])
    tensors = [dict(w=np.ones((o, i), np.float32), b=np.zeros(o, np.float32)) for i, o in ((3, 5), (5, 7), (7, 3))]
    x = np.ones((20, 3), np.float32)
    x[4, 1] = np.inf
    logits, value, _ = Amd.Policy(net, "fp32", tensors).forward(torch.from_numpy(x).cuda(), torch.zeros(20, device="cuda"))
    logits = logits.cpu().numpy()
    assert np.all(np.isposinf(logits[4])) and np.all(np.delete(logits, 4, 0) == 105.0) and np.isposinf(value[4].item())


def test_more_states_than_one_launch_takes():
    """2^29 + 69 states: workgroups of 256 lanes over 16 or 32 states each exceed the work-items of one launch, so the batch goes
    out in pieces.  The states repeat with a period that divides neither piece: every period must give the bits of the first."""
    import paper_2211_15023_amd as Amd
    rng = np.random.default_rng(5)
    net = SimpleNamespace(name="mlp", obs_dtype="f32", obs_shape=(1,), n_actions=1, layers=[dict(kind="dense", cin=1, cout=8, relu=True)])
    tensors = [dict(w=rng.uniform(-1, 1, s).astype(np.float32), b=rng.uniform(-1, 1, s[0]).astype(np.float32)) for s in ((8, 1), (2, 8))]
    pol = Amd.Policy(net, "fp32", tensors)
    period, B = 5003, (1 << 29) + 69
    n = B // period
    base = torch.from_numpy(rng.standard_normal((period, 1)).astype(np.float32)).cuda()
    x = base.repeat(n + 1, 1)[:B]
    u = torch.zeros(B, device="cuda")
    print(f"fp32 mlp B={B}", flush=True)
    out = pol.forward(x, u)
    want = pol.forward(base, u[:period])
    for got, first in zip(out, want):
        got, first = got.view(-1), first.view(-1)
        assert bool((got[:n * period].view(n, period) == first).all()) and torch.equal(got[n * period:], first[:B - n * period])
