"""The streaming int8 dense kernel on row-major states behind a ReLU, with rows that end inside an MFMA step, and both: every
bit against the oracle, on the first, the middle and the last (cut) tiles of 128 states.  The smallest batch has exactly one
workgroup per compute unit of 256, below which another kernel is used."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from workloads import Net, conv, dense, relu, flatten
from helpers import make_states

pytestmark = pytest.mark.gpu


def _behind_conv(cout, act, width, side):
    return Net("rows", "u8", (4, side + 1, side + 1), 5,
               [conv(4, cout, 2, 1, 0, False)] + ([relu()] if act else []) + [flatten(), dense(cout * side * side, width, True)])


NETS = {
    "relu, 30.25 steps": (_behind_conv(16, True, 256, 11), [8065, 8192, 8321]),
    "56.25 steps, 500 of 512 features": (_behind_conv(16, False, 500, 15), [4001, 4100]),
    "relu, 8 whole steps": (Net("rows", "u8", (4, 8, 8), 5, [conv(4, 16, 2, 1, 0, False), flatten(), dense(784, 512, False), relu(), dense(512, 512, True)]), [4001, 4100]),
    "12.25 steps": (_behind_conv(16, False, 512, 7), [4001]),
}


@pytest.mark.parametrize("name", list(NETS))
def test_rows_through_the_streaming_kernel(name):
    import paper_2211_15023_amd as A
    net, batches = NETS[name]
    qp = oracle.quantize_policy(net, wl.init_params(net, 2), make_states(net, 16, wl.STREAM["calibration"]))
    pol = A.Policy(net, "int8", qp.tensors, qp.act_scales)
    x, u = make_states(net, max(batches), wl.STREAM["states"]), wl.make_uniforms(max(batches))
    dx, du = torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda()
    for B in batches:
        print(f"{name} B={B}", flush=True)
        logits, value, _ = pol.forward(dx[:B], du[:B])
        rows = np.unique(np.r_[0:40, B // 2:B // 2 + 140, B - 140:B])
        ref = oracle.forward_int8(net, qp, x[rows], u[rows])
        assert np.array_equal(logits.cpu().numpy()[rows], ref["logits"])
        assert np.array_equal(value.cpu().numpy()[rows], ref["value"])
    pol.close()
