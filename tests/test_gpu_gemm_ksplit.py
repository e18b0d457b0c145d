"""The dense kernels whose wavefronts split K, at every tile they can take: the batch picks the tile (layers of about 512
features: 1, 100 states 16x16; 160 16x32; 500 32x32; 900 32x64; 2000 64x64; bf16 at 2400 128x64 or, with fewer than 64 steps, the
kernel that walks K in one wavefront; int8 layers of at most 256 features: 16x64 from 513 or, of 128, from 1025 states on), the
layer's rows end inside a 16-byte chunk or inside an MFMA step, with and without a ReLU on the input, with a
partly filled last feature tile.  int8: the oracle's bits.  bf16: the oracle's tolerance, and a state's result does not depend on the tile or the kernel (the split of K and the order of its sums are fixed)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from workloads import Net, conv, dense, relu, flatten
from helpers import make_states, rel_err_rows, teacher_tensors

pytestmark = pytest.mark.gpu

BATCHES = [1, 100, 160, 500, 900, 2000, 2400]


def _net(cout, act, width, side=15):
    # 15 x 15 pixels of cout channels: int8 900 bytes (14.06 steps, the last chunk holds 4 bytes), 16 channels: whole chunks;
    # bf16 3600 bytes (8 channels, 56.25 steps, the last chunk whole), 1800 bytes (4 channels, 28.1 steps, the last chunk holds
    # 8 bytes), 7200 bytes (16 channels, 112.5 steps).  11 x 11
    # pixels of 16 channels are the 1936 inputs behind the IMPALA student's stacks
    return Net("ksplit", "u8", (4, side + 1, side + 1), 5,
               [conv(4, cout, 2, 1, 0, False)] + ([relu()] if act else []) + [flatten(), dense(cout * side * side, width, True)])


@pytest.mark.parametrize("cout,act,width,side", [(4, True, 512, 15), (16, False, 500, 15), (16, True, 256, 11), (4, False, 120, 15)])
def test_int8_all_tiles(cout, act, width, side):
    import paper_2211_15023_amd as A
    net = _net(cout, act, width, side)
    qp = oracle.quantize_policy(net, wl.init_params(net, 2), make_states(net, 16, wl.STREAM["calibration"]))
    pol = A.Policy(net, "int8", qp.tensors, qp.act_scales)
    x, u = make_states(net, max(BATCHES), wl.STREAM["states"]), wl.make_uniforms(max(BATCHES))
    ref = oracle.forward_int8(net, qp, x, u)
    dx, du = torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda()
    for B in BATCHES:
        print(f"int8 {cout} channels, B={B}", flush=True)
        logits, value, _ = pol.forward(dx[:B], du[:B])
        assert np.array_equal(logits.cpu().numpy(), ref["logits"][:B])
        assert np.array_equal(value.cpu().numpy(), ref["value"][:B])


@pytest.mark.parametrize("cout,act,width", [(4, True, 512), (8, False, 500), (16, True, 500)])
def test_bf16_all_tiles(cout, act, width):
    import paper_2211_15023_amd as A
    net = _net(cout, act, width)
    params = wl.init_params(net, 2)
    pol = A.Policy(net, "bf16", teacher_tensors(params))
    x, u = make_states(net, max(BATCHES), wl.STREAM["states"]), wl.make_uniforms(max(BATCHES))
    dx, du = torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda()
    whole = pol.forward(dx, du)[0].cpu().numpy()
    rows = np.r_[0:40, len(x) - 40:len(x)]
    assert rel_err_rows(whole[rows], oracle.forward_float(net, params, x[rows], u[rows], "bf16")["logits"]).max() <= 2e-2
    for B in BATCHES:
        print(f"bf16 {cout} channels, B={B}", flush=True)
        assert np.array_equal(pol.forward(dx[:B], du[:B])[0].cpu().numpy(), whole[:B])
