"""The int8 MLP kernel that takes 64 states per wavefront (many states, at most 32 features, at most four actions) against
the one that takes 16 (the same states in smaller calls): whole numbers, so every bit, with a last group of any length, one to
four layers, and the oracle on a few rows."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,hidden,A,extra", [(24, (64, 64), 4, 0), (24, (64, 64), 3, 1), (4, (64, 64), 2, 17), (32, (48,), 4, 63),
                                              (8, (64, 20, 64), 1, 65), (12, (64, 64, 64, 64), 4, 62)])
def test_sixty_four_states_per_wavefront_give_the_same_numbers(D, hidden, A, extra):
    import paper_2211_15023_amd as P
    widths = (D,) + hidden
    net = SimpleNamespace(name="mlp", obs_dtype="f32", obs_shape=(D,), n_actions=A,
                          layers=[dict(kind="dense", cin=a, cout=b, relu=True) for a, b in zip(widths, widths[1:])])
    params = wl.init_params(net, wl.STREAM["weights_student"])
    qp = oracle.quantize_policy(net, params, wl.make_obs_f32(64, D, stream=wl.STREAM["calibration"]))
    pol = P.Policy(net, "int8", qp.tensors, qp.act_scales)
    B, part = (1 << 17) + extra, 60000
    gen = torch.Generator(device="cuda").manual_seed(D)
    x, u = torch.randn((B, D), device="cuda", generator=gen), torch.rand(B, device="cuda", generator=gen)
    x[5], x[B - 1] = 1e30, -1e30                                  # saturated observations
    print(f"int8 MLP {widths} A={A} B={B}", flush=True)
    got = pol.forward(x, u)
    for i in range(0, B, part):
        for a, b in zip(got, pol.forward(x[i:i + part].contiguous(), u[i:i + part].contiguous())):
            assert torch.equal(a[i:i + part], b)
    rows = [0, 5, 63, 64, B - 2, B - 1]
    ref = oracle.forward_int8(net, qp, x[rows].cpu().numpy(), u[rows].cpu().numpy())
    assert np.array_equal(got[0][rows].cpu().numpy(), ref["logits"])
