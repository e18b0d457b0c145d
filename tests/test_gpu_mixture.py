"""alpha-mixture of the smaller and the original policy (Section 3.2): every row must hold exactly what
the network chosen for it produces on that row alone — int8 rows bit-exact against the oracle, bf16
rows within the bf16 tolerance, and equal to the same policy's own forward on the GPU."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from helpers import policies, make_states, rel_err_rows, student_tensors, teacher_tensors, check_actions, check_sampler_self_consistency

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    import paper_2211_15023_amd as A
    A.load_library()
    return A


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("B,alpha", [(64, 0.5), (37, 0.3), (160, 0.9), (33, 0.0), (33, 1.0), (5, 0.5)])
def test_mixture_rows_match_their_network(A, B, alpha):
    # smaller = the paper's Net3 quantized to int8; original = the paper's conv 32/64/64 network in bf16
    small = wl.configs.PAPER_STUDENTS["net3"]
    ps = wl.init_params(small, wl.STREAM["weights_student"])
    qp = oracle.quantize_policy(small, ps, make_states(small, 64, wl.STREAM["calibration"]))
    orig = wl.nature_cnn()
    po = wl.init_params(orig, wl.STREAM["weights_teacher"])
    p_small = A.Policy(small, "int8", qp.tensors, qp.act_scales)
    p_orig = A.Policy(orig, "bf16", teacher_tensors(po))
    x = make_states(small, B, wl.STREAM["states"])
    u = wl.make_uniforms(B)
    use = (wl.uniform01(wl.BASE_SEED, 41, 0, B) < np.float32(alpha)).astype(np.uint8)   # Bernoulli(alpha) per row
    print(f"mixture B={B} alpha={alpha} smaller rows={int(use.sum())}", flush=True)
    ref = oracle.forward_mixture(small, qp, orig, po, "bf16", x, u, use)
    nA = small.n_actions
    logits = torch.full((B, nA), float("nan"), dtype=torch.float32, device="cuda")
    value = torch.full((B,), float("nan"), dtype=torch.float32, device="cuda")
    action = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    dx, du = _dev(x), _dev(u)
    A.accerl_actor_forward_mixture(p_small.handle, p_orig.handle, dx, du, use, logits, value, action)
    torch.cuda.synchronize()
    gl, gv, ga = logits.cpu().numpy(), value.cpu().numpy(), action.cpu().numpy()
    m = use.astype(bool)
    assert np.array_equal(gl[m], ref["logits"][m]) and np.array_equal(gv[m], ref["value"][m])
    if m.any():
        check_actions(ga[m], ref["action"][m], ref["logits"][m], u[m], 1e-5)
    if (~m).any():
        assert rel_err_rows(gl[~m], ref["logits"][~m]).max() <= 2e-2
        assert rel_err_rows(gv[~m], ref["value"][~m]).max() <= 2e-2
        check_actions(ga[~m], ref["action"][~m], ref["logits"][~m], u[~m], 2e-2)
    check_sampler_self_consistency(ga, gl, u)      # every row, whichever network produced it
    # and bit-identical to what each policy computes for those rows in a plain forward
    ls, vs, as_ = p_small.forward(dx, du)
    lo, vo, ao = p_orig.forward(dx, du)
    torch.cuda.synchronize()
    tm = torch.from_numpy(m).cuda()
    assert torch.equal(logits[tm], ls[tm]) and torch.equal(action[tm], as_[tm]) and torch.equal(value[tm], vs[tm])
    assert torch.equal(logits[~tm], lo[~tm]) and torch.equal(action[~tm], ao[~tm]) and torch.equal(value[~tm], vo[~tm])
    # a second call with another draw reuses the buffers
    use2 = 1 - use
    A.accerl_actor_forward_mixture(p_small.handle, p_orig.handle, dx, du, use2, logits, value, action)
    torch.cuda.synchronize()
    tm2 = ~tm
    assert torch.equal(logits[tm2], ls[tm2]) and torch.equal(logits[~tm2], lo[~tm2])
    p_small.close(); p_orig.close()


def test_mixture_alpha_schedule(A):
    from oracle import layers as L
    for k in (0.0, 0.1, 0.2, 0.3, 0.45, 0.5, 2.0):
        assert A.accerl_mixture_alpha(k, 0.1, 0.5) == L.mixture_alpha(k, 0.1, 0.5)


def test_mixture_rejects_mismatched_policies(A):
    nt, pt, ns, ps, qp = policies(0)
    mlp = A.Policy(ns, "int8", student_tensors(qp), qp.act_scales)
    small = wl.configs.PAPER_STUDENTS["net3"]
    p3 = A.Policy(small, "bf16", teacher_tensors(wl.init_params(small, wl.STREAM["weights_student"])))
    x = _dev(make_states(small, 4, wl.STREAM["states"]))
    u = _dev(wl.make_uniforms(4))
    lg = torch.empty(4, 18, device="cuda"); v = torch.empty(4, device="cuda"); a = torch.empty(4, dtype=torch.int32, device="cuda")
    with pytest.raises(A.AccerlError):
        A.accerl_actor_forward_mixture(mlp.handle, p3.handle, x, u, np.ones(4, np.uint8), lg, v, a)
    mlp.close(); p3.close()


def test_mixture_of_more_rows_than_one_launch_takes(A):
    """2^24 + 1000 rows of 16 bytes: a workgroup of 256 lanes per copied row exceeds the work-items of one launch, so rows are
    gathered and scattered in pieces.  Two fp32 MLPs of 4 features; every row against the plain forward of its network."""
    B, nA = (1 << 24) + 1000, 2
    net = SimpleNamespace(name="mlp", obs_dtype="f32", obs_shape=(4,), n_actions=nA, layers=[dict(kind="dense", cin=4, cout=8, relu=True)])
    rng = np.random.default_rng(3)
    small, orig = (A.Policy(net, "fp32", [dict(w=rng.uniform(-1, 1, s).astype(np.float32), b=rng.uniform(-1, 1, s[0]).astype(np.float32))
                                          for s in ((8, 4), (nA + 1, 8))]) for _ in range(2))
    use = (rng.random(B, np.float32) < 0.6).astype(np.uint8)
    gen = torch.Generator(device="cuda").manual_seed(1)
    x, u = torch.randn((B, 4), device="cuda", generator=gen), torch.rand(B, device="cuda", generator=gen)
    out = small.alloc_outputs(B)
    print(f"mixture of two MLPs, B={B}", flush=True)
    A.accerl_actor_forward_mixture(small.handle, orig.handle, x, u, use, *out)
    m = _dev(use).bool()
    for got, a, b in zip(out, small.forward(x, u), orig.forward(x, u)):
        assert torch.equal(got, torch.where(m.view(-1, *[1] * (got.dim() - 1)), a, b))


def _wide_head_net(cout):
    return SimpleNamespace(name="wide", obs_dtype="u8", obs_shape=(4, 84, 84), n_actions=40,
                           layers=[dict(kind="conv", cin=4, cout=cout, k=8, stride=4, pad=0, relu=True),
                                   dict(kind="conv", cin=cout, cout=8, k=4, stride=2, pad=0, relu=True),
                                   dict(kind="flatten"), dict(kind="dense", cin=8 * 81, cout=64, relu=True)])


@pytest.mark.parametrize("passes", [False, True])
@pytest.mark.parametrize("pair", ["nature", "impala", "net1", "net2", "wide heads", "odd size", "two convolutions"])
def test_mixture_rows_are_read_and_written_in_place(A, monkeypatch, pair, passes):
    """Every kernel that can be the first of an image policy reads through the row list, and both forms of the heads kernel
    write through it: bit for bit what the policies compute on those rows alone, also when a policy runs in several passes.  (Calls
    of one round: the next test has several.)"""
    if passes:
        monkeypatch.setenv("ACCERL_CHUNK", "64")                  # read when the policy is created
    rng = np.random.default_rng(5)

    def float_policy(net, prec="bf16"):
        return A.Policy(net, prec, teacher_tensors(wl.init_params(net, wl.STREAM["weights_teacher"])))

    def int8_policy(net):
        params = wl.init_params(net, wl.STREAM["weights_student"])
        qp = oracle.quantize_policy(net, params, make_states(net, 16, wl.STREAM["calibration"]))
        return A.Policy(net, "int8", qp.tensors, qp.act_scales)

    if pair in ("nature", "impala"):
        nt, pt, ns, ps, qp = policies(2 if pair == "nature" else 3)
        net, small, orig = ns, A.Policy(ns, "int8", student_tensors(qp), qp.act_scales), A.Policy(nt, "bf16", teacher_tensors(pt))
    elif pair == "wide heads":
        net = _wide_head_net(8)
        small, orig = int8_policy(net), float_policy(_wide_head_net(20))
    elif pair == "odd size":                                      # the generic first kernel, one image at a time in calls of this size
        net = SimpleNamespace(name="odd", obs_dtype="u8", obs_shape=(3, 12, 16), n_actions=3,
                              layers=[dict(kind="conv", cin=3, cout=12, k=3, stride=1, pad=1, relu=True),
                                      dict(kind="flatten"), dict(kind="dense", cin=12 * 192, cout=24, relu=True)])
        small, orig = int8_policy(net), float_policy(net)
    elif pair == "two convolutions":                              # the generic kernel of the first two layers
        net = SimpleNamespace(name="two", obs_dtype="u8", obs_shape=(4, 60, 60), n_actions=6,
                              layers=[dict(kind="conv", cin=4, cout=16, k=8, stride=4, pad=0, relu=True),
                                      dict(kind="conv", cin=16, cout=64, k=4, stride=2, pad=0, relu=True),
                                      dict(kind="flatten"), dict(kind="dense", cin=64 * 36, cout=24, relu=False)])
        small, orig = int8_policy(net), float_policy(net)
    else:
        net = wl.configs.PAPER_STUDENTS[pair]
        small, orig = int8_policy(net), float_policy(net)
    B = 150
    x = make_states(net, B, wl.STREAM["states"])
    dx, du = _dev(x), _dev(wl.make_uniforms(B))
    use = (rng.random(B) < 0.55).astype(np.uint8)
    out = small.alloc_outputs(B)
    print(f"mixture in place: {pair}, B={B}, {'passes of 64' if passes else 'one pass'}", flush=True)
    A.accerl_actor_forward_mixture(small.handle, orig.handle, dx, du, use, *out)
    m = _dev(use).bool()
    for got, a, b in zip(out, small.forward(dx, du), orig.forward(dx, du)):
        assert torch.equal(got, torch.where(m.view(-1, *[1] * (got.dim() - 1)), a, b))


@pytest.mark.parametrize("pair", ["nature", "impala"])
def test_mixture_rows_beyond_one_round(A, pair):
    """An odd number of rows for each policy, more than its first kernel takes in a round: the second observation of a workgroup, the
    one requested ahead and the last, single one are looked up in the list too."""
    ci = 2 if pair == "nature" else 3
    nt, pt, ns, ps, qp = policies(ci)
    small, orig = A.Policy(ns, "int8", student_tensors(qp), qp.act_scales), A.Policy(nt, "bf16", teacher_tensors(pt))
    n = 4 * torch.cuda.get_device_properties(0).multi_processor_count + 3
    B = 2 * n
    gen = torch.Generator(device="cuda").manual_seed(B)
    x = torch.randint(0, 256, (B, 4, 84, 84), dtype=torch.uint8, device="cuda", generator=gen)
    u = torch.rand(B, device="cuda", generator=gen)
    use = np.zeros(B, np.uint8)
    use[np.random.default_rng(7).permutation(B)[:n]] = 1
    out = small.alloc_outputs(B)
    print(f"mixture beyond one round: {pair}, {n} rows each", flush=True)
    A.accerl_actor_forward_mixture(small.handle, orig.handle, x, u, use, *out)
    m = _dev(use).bool()
    for got, a, b in zip(out, small.forward(x, u), orig.forward(x, u)):
        assert torch.equal(got, torch.where(m.view(-1, *[1] * (got.dim() - 1)), a, b))


@pytest.mark.parametrize("B", [6001, 30011])
@pytest.mark.parametrize("shape,convs", [((3, 12, 16), [(12, 3, 1, 1)]), ((4, 20, 20), [(16, 4, 2, 0)]), ((4, 40, 40), [(16, 8, 4, 0), (32, 4, 2, 0)])])
def test_mixture_of_small_images_in_batches(A, shape, convs, B):
    """Small images are staged several at a time, neighbours or not: batches with fewer images than planned and with all of them
    (the larger call), a last batch that is not full, a second pass of the larger policy."""
    layers, c, hw = [], shape[0], shape[1:]
    for cout, k, stride, pad in convs:
        layers.append(dict(kind="conv", cin=c, cout=cout, k=k, stride=stride, pad=pad, relu=True))
        c, hw = cout, [(v + 2 * pad - k) // stride + 1 for v in hw]
    layers += [dict(kind="flatten"), dict(kind="dense", cin=c * hw[0] * hw[1], cout=24, relu=True)]
    net = SimpleNamespace(name="small", obs_dtype="u8", obs_shape=shape, n_actions=3, layers=layers)
    params = wl.init_params(net, wl.STREAM["weights_student"])
    qp = oracle.quantize_policy(net, params, make_states(net, 16, wl.STREAM["calibration"]))
    small, orig = A.Policy(net, "int8", qp.tensors, qp.act_scales), A.Policy(net, "bf16", teacher_tensors(params))
    for prec, tensors, scales in (("int8", qp.tensors, A.pack_scales(qp.act_scales, qp.tensors)), ("bf16", teacher_tensors(params), None)):
        plan = A.accerl_plan_describe(A.make_arch(net, prec), A.pack_weights(tensors), scales).splitlines()[1]
        assert int(plan.split(" G=")[1].split()[0]) > 1 and "fuse_next=0" in plan
    gen = torch.Generator(device="cuda").manual_seed(B)
    x = torch.randint(0, 256, (B, *shape), dtype=torch.uint8, device="cuda", generator=gen)
    u = torch.rand(B, device="cuda", generator=gen)
    use = (np.random.default_rng(B).random(B) < 0.55).astype(np.uint8)
    out = small.alloc_outputs(B)
    print(f"mixture of {shape}, B={B}, smaller rows={int(use.sum())}", flush=True)
    A.accerl_actor_forward_mixture(small.handle, orig.handle, x, u, use, *out)
    m = _dev(use).bool()
    for got, a, b in zip(out, small.forward(x, u), orig.forward(x, u)):
        assert torch.equal(got, torch.where(m.view(-1, *[1] * (got.dim() - 1)), a, b))
