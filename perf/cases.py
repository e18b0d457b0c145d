"""The work that is timed: calls of the library's public entry points over the sizes its users run them at.

A case is a plain dict.  `kind` names the program around the calls:

  forward    one policy forward per pass (int8 student, bf16 or fp32 teacher) on a batch of states
  unroll     `steps` forwards of a recurrent policy with the state carried from one to the next
  mixture    one pass of the alpha-mixture of a small int8 policy and the original bf16 policy
  corrector  V-trace and the Monitor's KL / entropy indicators on one unroll of both policies' logits

The networks are the benchmark configurations of this repository (classic-control and Box2D MLPs, the Nature-DQN CNN,
the IMPALA ResNet with and without an LSTM core; teachers in their full width, IMPALA students at half the channels)
and the two-convolution network `net2` of the paper's table.  Weights are seeded uniform draws; the int8 policies are
quantized per output channel with activation scales from a float pass over a few calibration states.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch
import torch.nn.functional as F

import paper_2211_15023_amd as A

FRAME = (4, 84, 84)


def _conv(cin, cout, k, stride, pad, relu):
    return dict(kind="conv", cin=cin, cout=cout, k=k, stride=stride, pad=pad, relu=relu)


def _dense(cin, cout):
    return dict(kind="dense", cin=cin, cout=cout, relu=True)


def _mlp(d, hidden):
    return [_dense(d, hidden), _dense(hidden, hidden)]


def _impala(ch, lstm):
    layers, c = [], 4
    for n in ch:
        layers += [_conv(c, n, 3, 1, 1, False), dict(kind="maxpool", k=3, stride=2, pad=1),
                   dict(kind="resblock", ch=n), dict(kind="resblock", ch=n)]
        c = n
    layers += [dict(kind="relu"), dict(kind="flatten"), _dense(c * 121, 256)]
    if lstm:
        layers.append(dict(kind="lstm", cin=256, hidden=256))
    return layers


def _network(net, precision, actions):
    """The layer list of a named network; students of the IMPALA networks have half the channels of the teachers and
    the Box2D student is the narrow distilled one."""
    student = precision == "int8"
    if net == "classic_mlp":
        shape, layers = (4,), _mlp(4, 64)
    elif net == "box2d_mlp":
        shape, layers = (24,), _mlp(24, 64 if student else 256)
    elif net == "nature_cnn":
        shape, layers = FRAME, [_conv(4, 32, 8, 4, 0, True), _conv(32, 64, 4, 2, 0, True), _conv(64, 64, 3, 1, 0, True),
                                dict(kind="flatten"), _dense(64 * 49, 512)]
    elif net == "net2":
        shape, layers = FRAME, [_conv(4, 8, 8, 4, 0, True), _conv(8, 16, 4, 2, 0, True), dict(kind="flatten"),
                                _dense(16 * 81, 128)]
    else:
        shape, layers = FRAME, _impala((8, 16, 16) if student else (16, 32, 32), net == "impala_lstm")
    return SimpleNamespace(name=net, obs_dtype="f32" if len(shape) == 1 else "u8", obs_shape=shape, n_actions=actions,
                           layers=layers)


def _walk(net):
    """(layer index or None for the heads, weight shape, outputs per weight row) of every weight matrix in blob order."""
    shape, out = tuple(net.obs_shape), []
    for i, l in enumerate(net.layers):
        if l["kind"] == "conv":
            hw = [(v + 2 * l["pad"] - l["k"]) // l["stride"] + 1 for v in shape[1:]]
            shape = (l["cout"], *hw)
            out.append((i, (l["cout"], l["cin"], l["k"], l["k"]), hw[0] * hw[1]))
        elif l["kind"] == "maxpool":
            shape = (shape[0], *[(v - 1) // 2 + 1 for v in shape[1:]])
        elif l["kind"] == "resblock":
            out += [(i, (l["ch"], l["ch"], 3, 3), shape[1] * shape[2])] * 2
        elif l["kind"] == "flatten":
            shape = (int(np.prod(shape)),)
        elif l["kind"] == "dense":
            shape = (l["cout"],)
            out.append((i, (l["cout"], l["cin"]), 1))
        elif l["kind"] == "lstm":
            shape = (l["hidden"],)
            out += [(i, (4 * l["hidden"], l["cin"]), 1), (i, (4 * l["hidden"], l["hidden"]), 1)]
    out.append((None, (net.n_actions + 1, shape[0]), 1))
    return out


def _weights(net, rng):
    """Uniform weights with the variance that keeps activations level, in blob order: (layer, W, b or None).  The second
    convolution of a residual block is halved, as deep residual networks are initialised, so that the stream does not
    double from block to block and drive the LSTM's gates into saturation."""
    out, last = [], None
    for i, shape, _ in _walk(net):
        lstm = i is not None and net.layers[i]["kind"] == "lstm"
        fan = shape[0] // 4 if lstm else int(np.prod(shape[1:]))
        bound = math.sqrt((1.0 if lstm else 6.0) / fan)
        w = rng.uniform(-bound, bound, shape).astype(np.float32)
        second_of_lstm = lstm and last == i
        if last == i and not lstm:
            w *= 0.5
        b = None if second_of_lstm else rng.uniform(-fan ** -0.5, fan ** -0.5, shape[0]).astype(np.float32)
        out.append((i, w, b))
        last = i
    return out


def _act_scales(net, params, states):
    """max|a| / 127 of every quantized activation in a float pass over `states` (a CPU tensor)."""
    u8 = net.obs_dtype == "u8"
    x = states.float() / 255.0 if u8 else states
    scales = [1.0 / 255.0 if u8 else float(x.abs().max()) / 127.0]
    it = iter(params)

    def tensors():
        _, w, b = next(it)
        return torch.from_numpy(w), torch.from_numpy(b)

    def keep(v):
        scales.append(float(v.abs().max()) / 127.0)
        return v

    for l in net.layers:
        if l["kind"] == "conv":
            w, b = tensors()
            x = F.conv2d(x, w, b, stride=l["stride"], padding=l["pad"])
            x = keep(F.relu(x) if l["relu"] else x)
        elif l["kind"] == "dense":
            w, b = tensors()
            x = keep(F.relu(F.linear(x, w, b)))
        elif l["kind"] == "maxpool":
            x = F.max_pool2d(x, 3, 2, 1)
        elif l["kind"] == "resblock":
            w, b = tensors()
            mid = keep(F.relu(F.conv2d(F.relu(x), w, b, padding=1)))
            w, b = tensors()
            x = keep(x + F.conv2d(mid, w, b, padding=1))
        elif l["kind"] == "relu":
            x = F.relu(x)
        elif l["kind"] == "flatten":
            x = x.flatten(1)
    return np.asarray(scales, np.float32)


def _policy(net, precision, rng):
    params = _weights(net, rng)
    if precision != "int8":
        return A.Policy(net, precision, [dict(w=w, b=b) for _, w, b in params])
    n = 16
    if net.obs_dtype == "u8":
        calib = _frames(n, torch.Generator(device="cuda").manual_seed(int(rng.integers(1 << 30)))).cpu()
    else:
        calib = torch.from_numpy(rng.standard_normal((256, *net.obs_shape), np.float32))
    scales = _act_scales(net, params, calib)
    lstm = any(l["kind"] == "lstm" for l in net.layers)
    tensors = []
    for i, w, b in params:
        if lstm and (i is None or net.layers[i]["kind"] == "lstm"):
            tensors.append(dict(w=w, b=b))               # the recurrent core and the heads behind it stay in float
            continue
        flat = w.reshape(w.shape[0], -1)
        s = (np.abs(flat).max(axis=1) / 127.0).astype(np.float32)
        q = np.clip(np.rint(flat / s[:, None]), -127, 127).astype(np.int8)
        tensors.append(dict(wq=q.reshape(w.shape), s_w=s, b=b))
    return A.Policy(net, "int8", tensors, scales)


def _frames(n, gen):
    """uint8 frames [n, 4, 84, 84]: noise with six flat rectangles per plane (Atari's flat regions)."""
    x = torch.randint(0, 256, (n, *FRAME), dtype=torch.uint8, device="cuda", generator=gen)
    at = torch.arange(84, device="cuda")
    for i in range(0, n, 2048):
        part = x[i:i + 2048]
        m = part.shape[0]
        for _ in range(6):
            r = torch.randint(0, 1 << 20, (5, m, 4, 1), device="cuda", generator=gen)
            w, h, value = r[0] % 37 + 4, r[1] % 37 + 4, (r[4] % 256).to(torch.uint8)
            x0, y0 = r[2] % (85 - w), r[3] % (85 - h)
            inside = ((at >= y0) & (at < y0 + h)).unsqueeze(3) & ((at >= x0) & (at < x0 + w)).unsqueeze(2)
            part.copy_(torch.where(inside, value.unsqueeze(3), part))
    return x


def _states(net, n, gen):
    return _frames(n, gen) if net.obs_dtype == "u8" else torch.randn((n, *net.obs_shape), device="cuda", generator=gen)


def _forward(name, net, precision, batch, actions):
    return dict(name=name, kind="forward", net=net, precision=precision, batch=batch, actions=actions)


def listed():
    return [
        # an actor stepping 32 classic-control environments: the smallest call, pure latency
        _forward("classic_mlp_int8_32", "classic_mlp", "int8", 32, 2),
        # very many vectorised Box2D-style environments through the distilled student; a ragged batch
        _forward("box2d_mlp_int8_1000003", "box2d_mlp", "int8", 1000003, 4),
        # the wide fp32 teacher on the configured batch (distillation targets, Monitor)
        _forward("box2d_mlp_fp32_8192", "box2d_mlp", "fp32", 8192, 4),
        # the paper's Atari network as the actors run it: ten agents x 16 states, and the large batch
        _forward("nature_cnn_int8_160", "nature_cnn", "int8", 160, 18),
        _forward("nature_cnn_int8_4096", "nature_cnn", "int8", 4096, 18),
        # the original network on the same states (Corrector and Monitor need both distributions)
        _forward("nature_cnn_bf16_4096", "nature_cnn", "bf16", 4096, 18),
        # the pruned IMPALA student at its largest configured batch, and its teacher at an ordinary one
        _forward("impala_int8_16384", "impala", "int8", 16384, 18),
        _forward("impala_bf16_1024", "impala", "bf16", 1024, 18),
        # the configured recurrent unroll of the student; a short unroll of its teacher at a ragged batch
        dict(name="impala_lstm_int8_16x4096", kind="unroll", net="impala_lstm", precision="int8", batch=4096, steps=16, actions=18),
        dict(name="impala_lstm_bf16_4x999", kind="unroll", net="impala_lstm", precision="bf16", batch=999, steps=4, actions=18),
        # half the states of 1000 environments through net2, the others through the original network
        dict(name="mixture_1000", kind="mixture", batch=1000, alpha=0.5, actions=18),
        # one long unroll corrected and monitored at once
        dict(name="corrector_256x4096", kind="corrector", steps=256, batch=4096, actions=18),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """A case of the same families: batch sizes over the logarithm of their range, any number of actions up to Atari's 18."""
    actions = rng.randint(2, 18)
    pick = rng.randrange(10)
    if pick == 0:
        return dict(kind="forward", net=rng.choice(("classic_mlp", "box2d_mlp")), precision="int8", batch=_log(rng, 1, 1000003), actions=actions)
    if pick == 1:
        return dict(kind="forward", net=rng.choice(("classic_mlp", "box2d_mlp")), precision="fp32", batch=_log(rng, 1, 65536), actions=actions)
    if pick == 2:
        return dict(kind="forward", net=rng.choice(("nature_cnn", "net2")), precision="int8", batch=_log(rng, 1, 8192), actions=actions)
    if pick == 3:
        return dict(kind="forward", net=rng.choice(("nature_cnn", "net2")), precision="bf16", batch=_log(rng, 1, 8192), actions=actions)
    if pick == 4:
        return dict(kind="forward", net="impala", precision="int8", batch=_log(rng, 1, 16384), actions=actions)
    if pick == 5:
        return dict(kind="forward", net="impala", precision="bf16", batch=_log(rng, 1, 4096), actions=actions)
    if pick == 6:
        steps = rng.randint(1, 16)
        return dict(kind="unroll", net="impala_lstm", precision="int8", batch=_log(rng, 1, 4096), steps=steps, actions=actions)
    if pick == 7:
        steps = rng.randint(1, 4)
        return dict(kind="unroll", net="impala_lstm", precision="bf16", batch=_log(rng, 1, 1024), steps=steps, actions=actions)
    if pick == 8:
        return dict(kind="mixture", batch=_log(rng, 2, 4096), alpha=rng.choice((0.1, 0.25, 0.5, 0.75, 0.9)), actions=actions)
    return dict(kind="corrector", steps=_log(rng, 1, 256), batch=_log(rng, 1, 4096), actions=actions)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    rng = np.random.default_rng(int(seed))
    B, acts = case["batch"], case["actions"]
    s = SimpleNamespace(case=case)
    if case["kind"] == "corrector":
        T = case["steps"]
        normal = lambda *shape: torch.randn(shape, device="cuda", generator=gen)
        chance = lambda p: torch.rand((T, B), device="cuda", generator=gen) < p
        s.original = 2.0 * normal(T, B, acts)
        s.smaller = s.original + 0.3 * normal(T, B, acts)     # a compressed policy tracks its original
        s.actions = torch.randint(0, acts, (T, B), dtype=torch.int32, device="cuda", generator=gen)
        s.rewards = normal(T, B) * chance(0.1)                # sparse, as in Atari
        s.discounts = 0.99 * (~chance(0.01)).float()
        s.values, s.bootstrap = normal(T, B), normal(B)
        s.vs, s.advantage, s.rho, s.kl, s.entropy = (torch.empty((T, B), device="cuda") for _ in range(5))
        s.stats = torch.empty(4, dtype=torch.float64, device="cuda")
        return s
    if case["kind"] == "mixture":
        net = _network("nature_cnn", "bf16", acts)
        s.policy = _policy(_network("net2", "int8", acts), "int8", rng)
        s.original = _policy(net, "bf16", rng)
        s.use_smaller = (rng.random(B) < case["alpha"]).astype(np.uint8)
    else:
        net = _network(case["net"], case["precision"], acts)
        s.policy = _policy(net, case["precision"], rng)
    uniforms = lambda: torch.rand(B, device="cuda", generator=gen)
    if case["kind"] == "unroll":
        T = case["steps"]
        s.states = [_states(net, B, gen) for _ in range(T)]
        s.uniforms = [uniforms() for _ in range(T)]
        s.done = [(uniforms() < 0.01).to(torch.uint8) for _ in range(T)]
        s.h0, s.c0 = (0.1 * torch.randn((B, 256), device="cuda", generator=gen) for _ in range(2))
        s.h, s.c = torch.empty_like(s.h0), torch.empty_like(s.c0)
        s.outputs = [s.policy.alloc_outputs(B) for _ in range(T)]
    else:
        s.states, s.uniforms = _states(net, B, gen), uniforms()
        s.outputs = s.policy.alloc_outputs(B)
    return s


def run(s):
    kind = s.case["kind"]
    if kind == "forward":
        return s.policy.forward(s.states, s.uniforms, outputs=s.outputs)
    if kind == "mixture":
        A.accerl_actor_forward_mixture(s.policy.handle, s.original.handle, s.states, s.uniforms, s.use_smaller, *s.outputs)
        return s.outputs
    if kind == "unroll":
        s.h.copy_(s.h0)
        s.c.copy_(s.c0)
        for x, u, done, out in zip(s.states, s.uniforms, s.done, s.outputs):
            s.policy.forward(x, u, done, s.h, s.c, outputs=out)
        return s.outputs, s.h, s.c
    A.accerl_vtrace(s.original, s.smaller, s.actions, s.rewards, s.discounts, s.values, s.bootstrap, 1.0, 1.0,
                    s.vs, s.advantage, s.rho)
    n = s.case["steps"] * s.case["batch"]
    A.accerl_monitor_kl(s.original.view(n, -1), s.smaller.view(n, -1), s.kl.view(n), s.entropy.view(n), s.stats)
    return s.vs, s.advantage, s.rho, s.kl, s.entropy, s.stats


def _cost(net, precision, batch):
    """Bytes and operations of one forward: observations, uniforms, outputs and weights once; two per multiply-add."""
    size = {"int8": 1, "bf16": 2, "fp32": 4}[precision]
    macs = sum(int(np.prod(shape)) * n for _, shape, n in _walk(net))
    weights = sum(int(np.prod(shape)) * size for _, shape, _ in _walk(net))
    obs = int(np.prod(net.obs_shape)) * (1 if net.obs_dtype == "u8" else 4)
    return batch * (obs + 4 + 4 * net.n_actions + 8) + weights, 2 * macs * batch


def work(case):
    B, acts = case["batch"], case["actions"]
    if case["kind"] == "corrector":
        n = case["steps"] * B
        # both logit tables; actions, rewards, discounts, values; the five outputs.  Per action two exponentials and a few
        # operations around them for either network
        return dict(bytes=n * (2 * 4 * acts + 4 * 4 + 5 * 4) + 4 * B + 32, flops=n * (16 * acts + 20))
    if case["kind"] == "mixture":
        small = round(B * case["alpha"])
        b0, f0 = _cost(_network("net2", "int8", acts), "int8", small)
        b1, f1 = _cost(_network("nature_cnn", "bf16", acts), "bf16", B - small)
        return dict(bytes=b0 + b1 + B, flops=f0 + f1)
    steps = case.get("steps", 1)
    net = _network(case["net"], case["precision"], acts)
    bytes_, flops = _cost(net, case["precision"], B * steps)
    if case["kind"] == "unroll":
        bytes_ += B * steps + 4 * 4 * 256 * B        # the done flags; h and c read and written
    return dict(bytes=bytes_, flops=flops)


def tolerance(case):
    """About four times what each path differs by from a float64 evaluation that rounds where the path stores a value.
    `differ` concerns the sampled actions: a uniform next to a boundary of the CDF."""
    if case["kind"] == "corrector":
        return {"rel": 1.2e-5, "max": 8e-5}                       # measured 3.1e-6 / 1.8e-5 (KL; 6e-7 elsewhere)
    precision = case.get("precision", "bf16")
    recurrent = case["kind"] == "unroll"
    if precision == "fp32":
        return {"rel": 1.5e-6, "max": 5e-6, "differ": 1e-4}       # 3.7e-7 / 1.2e-6
    if precision == "int8" and not recurrent:
        return {"rel": 1e-7, "max": 1e-6, "differ": 2e-5}         # one multiply of an exact integer; actions 0 of 1000003
    if precision == "int8":
        return {"rel": 8e-4, "max": 1.2e-2, "differ": 1e-3}       # exact torso, bf16 LSTM: 1.8e-4 / 2.9e-3
    if case.get("net") in ("impala", "impala_lstm"):
        return {"rel": 3e-2, "max": 0.25, "differ": 1e-2}         # fifteen rounded layers: up to 1.6e-2 / 6.3e-2, actions 8e-3
    return {"rel": 4e-3, "max": 3e-2, "differ": 5e-3}             # 9.5e-4 / 7.3e-3
