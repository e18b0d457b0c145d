"""The int8 front kernel takes one observation per workgroup while the chip has a workgroup for each, pairs beyond: the same
whole numbers on both sides of the line, for the smallest batches and for odd ones.  Small calls of the paper's network have the third
convolution in that launch too; the two layers alone are those of a network whose third layer is another one."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from workloads import Net, conv, dense, flatten
from helpers import kernel_names, make_states, policies, student_tensors, teacher_tensors

pytestmark = pytest.mark.gpu


def test_single_observations_and_pairs_agree():
    import paper_2211_15023_amd as A
    nt, pt, ns, ps, qp = policies(2)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    x, u = wl.make_frames_u8(2 * cus + 3, first=5), wl.make_uniforms(2 * cus + 3)
    x[1], x[2, :, 40:] = 255, 0
    pol = A.Policy(ns, "int8", student_tensors(qp), qp.act_scales)
    dx, du = torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda()
    pairs = pol.forward(dx, du)                                   # two rounds of pairs
    for B in (1, 2, 3, cus - 1, cus, cus + 1):
        print(f"front kernel B={B}", flush=True)
        for got, ref in zip(pol.forward(dx[:B], du[:B]), pairs):
            assert torch.equal(got, ref[:B])
    rows = [0, 1, 2, cus - 1, cus, 2 * cus + 2]
    ref = oracle.forward_int8(ns, qp, x[rows], u[rows])
    assert np.array_equal(pairs[0].cpu().numpy()[rows], ref["logits"])


OTHER_THIRD = Net("other_third", "u8", (4, 84, 84), 18, [conv(4, 32, 8, 4, 0, True), conv(32, 64, 4, 2, 0, True), conv(64, 32, 3, 1, 0, True),
                                                         flatten(), dense(32 * 49, 64, True)])


@pytest.mark.parametrize("rows", [False, True])
def test_two_layers_alone(rows):
    """Without and with a row list, on both sides of the line between single observations and pairs; the kernel's name says which
    instance ran (<three-instruction requantization, row list, third layer>)."""
    import paper_2211_15023_amd as A
    params = wl.init_params(OTHER_THIRD, 4)
    qp = oracle.quantize_policy(OTHER_THIRD, params, make_states(OTHER_THIRD, 16, wl.STREAM["calibration"]))
    pol = A.Policy(OTHER_THIRD, "int8", student_tensors(qp), qp.act_scales)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    most = 2 * cus + 3
    x, u = wl.make_frames_u8(most, first=5), wl.make_uniforms(most)
    dx, du = torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda()
    pairs = pol.forward(dx, du)
    some = [0, 1, cus, most - 1]
    assert np.array_equal(pairs[0].cpu().numpy()[some], oracle.forward_int8(OTHER_THIRD, qp, x[some], u[some])["logits"])
    other = A.Policy(OTHER_THIRD, "bf16", teacher_tensors(params)) if rows else None
    for B in (1, 2, 3, cus - 1, cus, cus + 1):
        print(f"two layers alone, row list {rows}, B={B}", flush=True)
        if not rows:
            got, names = kernel_names(lambda: pol.forward(dx[:B], du[:B]))
            at = torch.arange(B, device="cuda")
        else:                                                     # B rows for the int8 policy among all
            use = np.zeros(most, np.uint8)
            use[np.random.default_rng(B).permutation(most)[:B]] = 1
            got = pol.alloc_outputs(most)
            _, names = kernel_names(lambda: A.accerl_actor_forward_mixture(pol.handle, other.handle, dx, du, use, *got))
            at = torch.from_numpy(use.astype(bool)).cuda().nonzero()[:, 0]
        assert any(f"conv_front_kernel<true, {str(rows).lower()}, false>" in n for n in names), names
        for a, ref in zip(got, pairs):
            assert torch.equal(a[at] if rows else a, ref[at])
    pol.close()
