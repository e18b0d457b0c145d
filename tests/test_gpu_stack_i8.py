"""The int8 student's whole-stack kernels against the layer-by-layer kernels and the oracle: whole numbers, so every bit, at
the batch sizes where the work split changes (one image; the third stack's batches of five one short, full and one over; a
second round of the resident workgroups), with states that drive the sums to both ends of int8."""
import copy

import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from helpers import policies, student_tensors

pytestmark = pytest.mark.gpu


def states(B):
    x = wl.make_frames_u8(B, first=23)
    x[0], x[B // 2, :, 40:, :40], x[-1, 1] = 255, 0, 255         # saturated planes, and an edge between the extremes
    return x


@pytest.mark.parametrize("B", [1, 4, 5, 6, 11, 1029])
def test_int8_stacks_give_the_layerwise_bytes(monkeypatch, B):
    import paper_2211_15023_amd as A
    nt, pt, ns, ps, qp = policies(3)
    x, u = states(B), wl.make_uniforms(B)
    dx, du = torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda()
    out = []
    for fused in (True, False):
        if not fused:
            monkeypatch.setenv("ACCERL_NO_STACK_FUSE", "1")       # read when the policy is created
        pol = A.Policy(ns, "int8", student_tensors(qp), qp.act_scales)
        print(f"int8 student B={B} {'stacks' if fused else 'layer by layer'}", flush=True)
        out.append([t.cpu().numpy() for t in pol.forward(dx, du)])
        pol.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    rows = np.unique(np.r_[0:min(B, 3), B // 2, B - 1])
    ref = oracle.forward_int8(ns, qp, x[rows], u[rows])
    assert np.array_equal(out[0][0][rows], ref["logits"])


@pytest.mark.parametrize("bias", [1 << 22, -(1 << 22)])
@pytest.mark.parametrize("tensor", [0, 2, 9])
def test_int8_stacks_convert_sums_that_may_leave_22_bits(tensor, bias):
    """A bias that takes a stack convolution's or a block's second convolution's sums out of +-2^22 (the sums of the same
    layer's other channels stay far below): the kernel may no longer read them as floats, and converts them."""
    import paper_2211_15023_amd as A
    from oracle.ptq import derived_constants
    nt, pt, ns, ps, qp = copy.deepcopy(policies(3))               # policies() is cached
    i = next(i for i, k in derived_constants(ns, qp)["layers"].items() if any(v is qp.tensors[tensor]["wq"] for v in k.values()))
    name = "biasq" if tensor in (0, 5, 10) else "biasqB"
    t = qp.tensors[tensor]
    t["b"] = np.array(t["b"], np.float32)
    t["b"][3] = 1.0
    t["b"][3] = bias * 1.01 / derived_constants(ns, qp)["layers"][i][name][3]
    assert abs(derived_constants(ns, qp)["layers"][i][name][3]) >= 1 << 22
    x, u = states(6), wl.make_uniforms(6)
    pol = A.Policy(ns, "int8", student_tensors(qp), qp.act_scales)
    print(f"int8 student, tensor {tensor} bias {bias}", flush=True)
    got = [o.cpu().numpy() for o in pol.forward(torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda())]
    pol.close()
    assert np.array_equal(got[0], oracle.forward_int8(ns, qp, x, u)["logits"])
