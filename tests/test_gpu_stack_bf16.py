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


@pytest.mark.parametrize("bad_bits", [np.uint32(0x7fc00000), np.uint32(0xffc00000)])
@pytest.mark.parametrize("stack,block", [(0, 0), (1, 1), (2, 0)])
def test_relu_inside_a_block_turns_nan_sums_into_zero(stack, block, bad_bits):
    """As in the oracle, max(NaN, 0) = 0: a filter of a block's first convolution with a NaN weight computes the bits of a
    filter of zeros."""
    import paper_2211_15023_amd as A
    nt, pt, ns, ps, qp = policies(3)
    x, u = torch.from_numpy(wl.make_frames_u8(5, first=11)).cuda(), torch.from_numpy(wl.make_uniforms(5)).cuda()
    at = 5 * stack + 1 + 2 * block                                 # stack convolution, then two blocks of two
    out = []
    for bad in (bad_bits.view(np.float32), np.float32(0)):
        params = [(n, w.copy(), b.copy()) for n, w, b in pt]
        assert params[at][0].endswith("convA")
        params[at][1][7] = 0
        params[at][1][7, 0, 0, 0] = bad
        params[at][2][7] = 0
        out.append([t.cpu().numpy() for t in A.Policy(nt, "bf16", teacher_tensors(params)).forward(x, u)])
    assert np.isfinite(out[0][0]).all()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
