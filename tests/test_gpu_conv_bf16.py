"""The bf16 kernels of the paper's original network's convolutions (first two in one launch; third with fixed sizes, storing
the FC's fragment order) against the generic kernels, which run in a child process: the same bits, at the batch sizes where
the work split changes: one observation, an odd image beside an empty slot, a partly filled tile of 16 states; a second and an
uneven third round of the front kernel's resident workgroups (257, 700), a third and a fifth of the third convolution's with an
odd last image (2101, 4133); the FC's 64x64 and 128x64 tiles on fragment-order input (2101, 3001) and, at 4133, the kernel that
walks K in one wavefront."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import workloads as wl
from helpers import policies, teacher_tensors

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BATCHES = [1, 3, 17, 257, 700, 2101, 3001, 4133]


def _forwards(path=None):
    import paper_2211_15023_amd as A
    nt, pt, ns, ps, qp = policies(2)
    pol = A.Policy(nt, "bf16", teacher_tensors(pt))
    plan = A.accerl_plan_describe(pol.arch, A.pack_weights(teacher_tensors(pt)))
    x, u = torch.from_numpy(wl.make_frames_u8(max(BATCHES), first=5)).cuda(), torch.from_numpy(wl.make_uniforms(max(BATCHES))).cuda()
    out = {}
    for B in BATCHES:
        print(f"bf16 teacher B={B}", flush=True)
        out[str(B)] = pol.forward(x[:B], u[:B])[0].cpu().numpy()
    if path:
        np.savez(path, fused=int("fuse_next=1" in plan or "out_frag=1" in plan), **out)
    return plan, out


def test_bf16_convolutions_give_the_generic_bits(tmp_path):
    path = str(tmp_path / "generic.npz")
    code = f"import sys; sys.path[:0] = [{ROOT!r}, {os.path.join(ROOT, 'tests')!r}]; import test_gpu_conv_bf16 as t; t._forwards({path!r})"
    r = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, ACCERL_NO_CONV_FRONT="1", ACCERL_NO_CONV_TAIL="1"),
                       capture_output=True, text=True, timeout=110)
    assert r.returncode == 0, r.stderr[-2000:]
    generic = np.load(path)
    assert not generic["fused"]
    plan, got = _forwards()
    assert plan.count("fuse_next=1 front=1") == 1 and plan.count("tail=1 out_frag=1") == 1
    for B in BATCHES:
        assert np.array_equal(got[str(B)], generic[str(B)]), B


@pytest.mark.parametrize("B,alpha", [(5, 0.5), (600, 0.4)])
def test_mixture_reads_rows_in_place(B, alpha):
    """Both policies of the mixture are bf16 networks of that shape, so neither's rows are gathered: every row holds what its
    policy's plain forward computes, bit for bit."""
    import paper_2211_15023_amd as A
    nt, pt, ns, ps, qp = policies(2)
    first = A.Policy(nt, "bf16", teacher_tensors(pt))
    other = A.Policy(nt, "bf16", teacher_tensors(wl.init_params(nt, wl.STREAM["weights_student"])))
    x, u = torch.from_numpy(wl.make_frames_u8(B, first=9)).cuda(), torch.from_numpy(wl.make_uniforms(B)).cuda()
    use = (wl.uniform01(wl.BASE_SEED, 43, 0, B) < np.float32(alpha)).astype(np.uint8)
    out = first.alloc_outputs(B)
    print(f"mixture of two bf16 networks, B={B}", flush=True)
    A.accerl_actor_forward_mixture(first.handle, other.handle, x, u, use, *out)
    m = torch.from_numpy(use.astype(bool)).cuda()
    for got, a, b in zip(out, first.forward(x, u), other.forward(x, u)):
        assert torch.equal(got[m], a[m]) and torch.equal(got[~m], b[~m])


NAN = [np.uint32(0x7fc00000), np.uint32(0xffc00000)]          # of either sign


@pytest.mark.parametrize("bad_bits", NAN)
@pytest.mark.parametrize("layer", [0, 1, 2])
def test_relu_turns_nan_sums_into_zero(layer, bad_bits):
    """A filter with a NaN weight sums to NaN everywhere; the ReLU behind it gives zeros (max(NaN, 0) = 0, as in the oracle), so the
    network computes the bits it computes with that filter set to zero."""
    import paper_2211_15023_amd as A
    nt, pt, ns, ps, qp = policies(2)
    x, u = torch.from_numpy(wl.make_frames_u8(19, first=5)).cuda(), torch.from_numpy(wl.make_uniforms(19)).cuda()
    out = []
    for bad in (bad_bits.view(np.float32), np.float32(0)):
        params = [(n, w.copy(), b.copy()) for n, w, b in pt]
        params[layer][1][5] = 0
        params[layer][1][5, 0, 0, 0] = bad
        params[layer][2][5] = 0
        out.append([t.cpu().numpy() for t in A.Policy(nt, "bf16", teacher_tensors(params)).forward(x, u)])
    assert np.isfinite(out[0][0]).all()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
