"""The two ways arguments reach the library (compiled for plain tensors, in Python for the rest): the same results, and what was refused
is refused with the same errors."""
import pytest
import torch

import workloads as wl
from helpers import make_states, teacher_tensors

pytestmark = pytest.mark.gpu


class Sub(torch.Tensor):
    pass


def _policy():
    import paper_2211_15023_amd as A
    net = wl.CONFIGS[0]["teacher"]
    pol = A.Policy(net, "fp32", teacher_tensors(wl.init_params(net, 6)))
    return A, net, pol, torch.from_numpy(make_states(net, 40, wl.STREAM["states"])).cuda(), torch.from_numpy(wl.make_uniforms(40)).cuda()


def test_forward_either_way():
    A, net, pol, x, u = _policy()
    ref = pol.forward(x, u)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    ways = {"subclass": (x.as_subclass(Sub), u, None), "parameter": (torch.nn.Parameter(x), u, None), "stream": (x, u, side),
            "raw stream": (x, u, side.cuda_stream), "slice": (x[4:], u[4:], None)}
    for name, (a, b, stream) in ways.items():
        got = pol.forward(a, b, stream=stream)
        torch.cuda.synchronize()
        for g, w in zip(got, ref):
            assert torch.equal(g, w[-len(a):]), name
    with torch.cuda.stream(side):
        got = pol.forward(x, u)
    with torch.overrides.BaseTorchFunctionMode():
        mode = pol.forward(x, u)
    torch.cuda.synchronize()
    for g, m, w in zip(got, mode, ref):
        assert torch.equal(g, w) and torch.equal(m, w)


def test_forward_refusals():
    A, net, pol, x, u = _policy()
    out = pol.alloc_outputs(40)
    call = lambda **k: A.accerl_actor_forward_teacher(*({**dict(handle=pol.handle, states=x, uniforms=u, l=out[0], v=out[1], a=out[2]), **k}.values()))
    for bad in (dict(states=x.cpu()), dict(states=x.t()), dict(uniforms=u.double()), dict(a=out[2].long()), dict(l=out[0].half())):
        with pytest.raises(ValueError):
            call(**bad)
    for bad in (dict(uniforms=None), dict(v=None), dict(states=x.view(-1)[1:5].view(1, 4))):
        with pytest.raises(A.AccerlError) as e:
            call(**bad)
        assert e.value.code < 0 and A.accerl_last_error()
    with pytest.raises(A.AccerlError):
        A.accerl_actor_forward(pol.handle, x, u, *out)                # an fp32 policy
    with pytest.raises(IndexError):
        call(states=torch.tensor(1.0, device="cuda"))
    with pytest.raises(RuntimeError, match="storage"):
        torch.func.vmap(lambda s: (call(states=s), s)[1])(x.view(2, 20, 4))


def test_corrector_either_way():
    import paper_2211_15023_amd as A
    T, B, acts = 7, 33, 5
    g = torch.Generator(device="cuda").manual_seed(3)
    o, s = (torch.randn(T, B, acts, device="cuda", generator=g) for _ in range(2))
    act = torch.randint(0, acts, (T, B), dtype=torch.int32, device="cuda", generator=g)
    r, d, v = (torch.rand(T, B, device="cuda", generator=g) for _ in range(3))
    boot = torch.rand(B, device="cuda", generator=g)

    def run(wrap, one):
        outs = [torch.empty(T, B, device="cuda") for _ in range(3)]
        A.accerl_vtrace(wrap(o), s, act, r, d, v, boot, one, one, *outs)
        kl, ent, st = torch.empty(T * B, device="cuda"), torch.empty(T * B, device="cuda"), torch.empty(4, dtype=torch.float64, device="cuda")
        A.accerl_monitor_kl(wrap(o.view(T * B, acts)), s.view(T * B, acts), kl, ent, st)
        return outs + [kl, ent, st]

    for a, b in zip(run(lambda t: t, 1.0), run(lambda t: t.as_subclass(Sub), 1)):
        assert torch.equal(a, b)
    outs = [torch.empty(T, B, device="cuda") for _ in range(3)]
    for bad in (dict(act=act[:-1]), dict(s=s[..., :-1]), dict(r=r.t()), dict(act=act.float())):
        k = {**dict(o=o, s=s, act=act, r=r, d=d, v=v, boot=boot), **bad}
        with pytest.raises(ValueError):
            A.accerl_vtrace(*k.values(), 1.0, 1.0, *outs)
    A.accerl_vtrace(o, s, act, r, d, v, boot, 1.0, 1.0, outs[0], None, outs[2])    # advantages are optional
