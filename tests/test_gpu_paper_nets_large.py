"""The paper's two-convolution networks beyond one round of their convolutions' workgroups: batches with the planned number of images, the
next one staged while one is multiplied, a last one that is short, first layers that read through a row list in several rounds.  The plan
says that the instances with weights in registers are meant; every row equals, bit for bit, what calls of 100 states give, and some are
checked against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from helpers import make_states, rel_err_rows, student_tensors, teacher_tensors

pytestmark = pytest.mark.gpu

# (element, steps held in registers, staging registers, images per batch) of the convolutions, first and second
PLANS = {("net1", "int8"): [(4, 8, 1), None], ("net2", "int8"): [(6, 8, 1), (2, 8, 3)], ("net3", "int8"): [(10, 8, 1), (1, 8, 9)],
         ("net1", "bf16"): [(8, 4, 1), None], ("net2", "bf16"): [(12, 4, 1), (4, 10, 6)], ("net3", "bf16"): [None, None]}


def _policy(A, name, precision):
    net = wl.configs.PAPER_STUDENTS[name]
    params = wl.init_params(net, wl.STREAM["weights_student"])
    qp = oracle.quantize_policy(net, params, make_states(net, 16, wl.STREAM["calibration"])) if precision == "int8" else None
    tensors = student_tensors(qp) if qp else teacher_tensors(params)
    scales = qp.act_scales if qp else None
    pol = A.Policy(net, precision, tensors, scales)
    plan = A.accerl_plan_describe(pol.arch, A.pack_weights(tensors), A.pack_scales(scales, tensors) if qp else None).splitlines()
    for line, want in zip([l for l in plan if " conv " in l], PLANS[name, precision]):
        have = tuple(int(line.split(f" {k}=")[1].split()[0]) for k in ("KS", "PF", "G"))
        assert want is None or have == want, line
    return net, params, qp, pol


@pytest.mark.parametrize("precision", ["int8", "bf16"])
@pytest.mark.parametrize("name", ["net1", "net2", "net3"])
def test_rows_equal_small_calls(name, precision):
    import paper_2211_15023_amd as A
    net, params, qp, pol = _policy(A, name, precision)
    base = 300
    x, u = make_states(net, base, wl.STREAM["states"]), wl.make_uniforms(base)
    dx, du = torch.from_numpy(x).cuda(), torch.from_numpy(u).cuda()
    parts = [pol.forward(dx[i:i + 100].contiguous(), du[i:i + 100].contiguous()) for i in range(0, base, 100)]
    ref = [torch.cat(t) for t in zip(*parts)]
    rows = np.r_[0:6, base - 6:base]
    got = ref[0].cpu().numpy()[rows]
    if precision == "int8":
        assert np.array_equal(got, oracle.forward_int8(net, qp, x[rows], u[rows])["logits"])
    else:
        assert rel_err_rows(got, oracle.forward_float(net, params, x[rows], u[rows], "bf16")["logits"]).max() <= 2e-2
    times = 28
    dx, du, ref = torch.cat([dx] * times), torch.cat([du] * times), [torch.cat([t] * times) for t in ref]
    # beyond a round of batches of one image, of three and of six, with last batches of one, two and five images
    for B in (1281, 2570, 4609, 4613, 5001, 8191):
        print(f"{name} {precision} B={B}", flush=True)
        for out, want in zip(pol.forward(dx[:B], du[:B]), ref):
            assert torch.equal(out, want[:B])
    pol.close()


@pytest.mark.parametrize("small,other", [(("net2", "int8"), ("net2", "bf16")), (("net3", "int8"), ("net1", "bf16")), (("net1", "int8"), ("net3", "bf16"))])
def test_row_list_of_several_rounds(small, other):
    import paper_2211_15023_amd as A
    ps, po = _policy(A, *small)[3], _policy(A, *other)[3]
    B = 7003
    gen = torch.Generator(device="cuda").manual_seed(B)
    x = torch.randint(0, 256, (B, 4, 84, 84), dtype=torch.uint8, device="cuda", generator=gen)
    u = torch.rand(B, device="cuda", generator=gen)
    use = (np.random.default_rng(B).random(B) < 0.5).astype(np.uint8)
    out = ps.alloc_outputs(B)
    print(f"mixture of {small} and {other}, B={B}, smaller rows={int(use.sum())}", flush=True)
    A.accerl_actor_forward_mixture(ps.handle, po.handle, x, u, use, *out)
    m = torch.from_numpy(use.astype(bool)).cuda()
    for got, a, b in zip(out, ps.forward(x, u), po.forward(x, u)):
        assert torch.equal(got, torch.where(m.view(-1, *[1] * (got.dim() - 1)), a, b))
    ps.close(); po.close()
