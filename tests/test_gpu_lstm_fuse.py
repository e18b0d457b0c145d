"""The dense layer in front of an LSTM writes the operand of the LSTM's product itself (its own outputs and the state h, cleared
where an episode ended) where its wavefronts split K; every other plan packs it in a kernel of its own.  Both give the same bits
of everything, at each tile the dense kernel takes (the batch picks it), with more and fewer units than inputs, shares of h that
do not divide evenly among a row's workgroups or are empty, a cut last tile of states, and a ReLU between the two layers.  The
student's rows are padded to 16 features: it packs only where the inputs are a multiple of that, and the other sizes compare its
plan with itself."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from helpers import make_states, teacher_tensors

pytestmark = pytest.mark.gpu

BATCHES = [1, 37, 100, 160, 500, 613, 900, 2000, 2400]


@pytest.mark.parametrize("role", ["student", "teacher"])
@pytest.mark.parametrize("In,Hd,act", [(256, 256, True), (24, 104, False), (200, 56, True), (504, 8, False), (512, 128, False),
                                        (48, 80, False), (208, 48, True), (240, 16, False)])
def test_fused_operand_gives_the_same_bits(monkeypatch, role, In, Hd, act):
    import paper_2211_15023_amd as A
    layers = [wl.nets.conv(4, 16, 2, 1, 0, False), wl.nets.flatten(), wl.nets.dense(16 * 11 * 11, In, not act)] \
        + ([wl.nets.relu()] if act else []) + [wl.nets.lstm(In, Hd)]
    net = wl.Net("lstm_fuse", "u8", (4, 12, 12), 5, layers)
    params = wl.init_params(net, 3)
    qp = oracle.quantize_policy(net, params, make_states(net, 16, wl.STREAM["calibration"])) if role == "student" else None
    make = lambda: A.Policy(net, "int8", qp.tensors, qp.act_scales) if qp else A.Policy(net, "bf16", teacher_tensors(params))
    fused = make()
    monkeypatch.setenv("ACCERL_NO_LSTM_FUSE", "1")               # read when the policy is created
    plain = make()

    def packs():
        tensors = qp.tensors if qp else teacher_tensors(params)
        scales = A.pack_scales(qp.act_scales, qp.tensors) if qp else None
        plan = A.accerl_plan_describe(A.make_arch(net, "int8" if qp else "bf16"), A.pack_weights(tensors), scales)
        return ["packs_next=1" in line for line in plan.splitlines() if " gemm " in line][0]
    assert not packs()
    monkeypatch.delenv("ACCERL_NO_LSTM_FUSE")
    assert packs() == (role == "teacher" or In % 16 == 0)
    top = max(BATCHES)
    x, u = make_states(net, top, wl.STREAM["states"]), wl.make_uniforms(top)
    h0, c0 = wl.make_hc(top, Hd)
    done = (np.arange(top) % 3 == 1).astype(np.uint8)
    dev = lambda a: torch.from_numpy(a).cuda()
    dx, du, dd = dev(x), dev(u), dev(done)
    for B in BATCHES:
        print(f"lstm {In} + {Hd} {role} B={B}", flush=True)
        out = []
        for pol in (fused, plain):
            h, c = dev(h0[:B].copy()), dev(c0[:B].copy())
            res = [pol.forward(dx[:B], du[:B], done=dd[:B] if B != 500 else None, h=h, c=c) for _ in range(2)]   # two steps in a row
            out.append([t.cpu().numpy() for r in res for t in r] + [h.cpu().numpy(), c.cpu().numpy()])
        for a, b in zip(*out):
            assert np.array_equal(a, b)
    fused.close()
    plain.close()
