"""The bf16 teacher's whole-stack kernels against the layer-by-layer kernels: the same bits, at the batch sizes where the
work split changes (one image, an odd image left over in the two-image batches of the third stack, a second and third
round of the resident workgroups), and within the bf16 bound of the oracle."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from helpers import policies, rel_err_rows, teacher_tensors, check_actions

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 2, 7, 515])
def test_bf16_stacks_give_the_layerwise_bits(monkeypatch, B):
    import paper_2211_15023_amd as A
    nt, pt, ns, ps, qp = policies(3)
    x, u = wl.make_frames_u8(B, first=11), wl.make_uniforms(B)
    dx, du = torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda()
    out = []
    for fused in (True, False):
        if not fused:
            monkeypatch.setenv("ACCERL_NO_STACK_FUSE", "1")       # read when the policy is created
        pol = A.Policy(nt, "bf16", teacher_tensors(pt))
        plan = A.accerl_plan_describe(pol.arch, A.pack_weights(teacher_tensors(pt)))
        assert plan.count("stack_bf16=1") == (3 if fused else 0)
        print(f"bf16 teacher B={B} {'stacks' if fused else 'layer by layer'}", flush=True)
        out.append([t.cpu().numpy() for t in pol.forward(dx, du)])
        pol.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    rows = np.unique(np.r_[0:min(B, 4), B - 1])
    ref = oracle.forward_float(nt, pt, x[rows], u[rows], "bf16")
    assert rel_err_rows(out[0][0][rows], ref["logits"]).max() <= 2e-2     # the bf16 bound of the parity tests
    check_actions(out[0][2][rows], ref["action"], ref["logits"], u[rows], 2e-2)
