"""bf16 dense layers of states in fragment order around the lines of their dispatch: one and several rounds of 128 x 64 tiles, a cut last
tile, weights of more than 8 MB whose rounds are full enough or not.  Every row equals, bit for bit, what calls of 100 states give."""
import pytest
import torch

import workloads as wl
from helpers import make_states, teacher_tensors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [512, 2048])
def test_rows_equal_small_calls(width):
    import paper_2211_15023_amd as A
    net = wl.nature_cnn("dense%d" % width, fc=width)
    pol = A.Policy(net, "bf16", teacher_tensors(wl.init_params(net, 6)))
    dx = torch.from_numpy(make_states(net, 300, wl.STREAM["states"])).cuda()
    du = torch.from_numpy(wl.make_uniforms(300)).cuda()
    parts = [pol.forward(dx[i:i + 100].contiguous(), du[i:i + 100].contiguous()) for i in range(0, 300, 100)]
    ref = [torch.cat(t * 20) for t in zip(*parts)]
    dx, du = torch.cat([dx] * 20), torch.cat([du] * 20)
    for B in (513, 640, 1025, 1050, 2305, 2561, 2600, 3072, 3073, 4096, 4225, 6000):
        print(f"{width} B={B}", flush=True)
        for got, want in zip(pol.forward(dx[:B], du[:B]), ref):
            assert torch.equal(got, want[:B])
    pol.close()
