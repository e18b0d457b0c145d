"""The int8 front kernel takes one observation per workgroup while the chip has a workgroup for each, pairs beyond: the same
whole numbers on both sides of the line, for the smallest batches and for odd ones."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from helpers import policies, student_tensors

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
