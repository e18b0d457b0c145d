"""Dense layers whose wavefronts split K, at numbers of tiles that the eight XCDs do and do not share evenly (the order of the tiles
depends on it, and on the size of the weights beyond one round), at the two sides of the
lines between 64 x 64 and 128 x 64 tiles, and with a cut last tile: a state's result does not depend on the batch it is in, so
every row equals, bit for bit, what calls of 100 states (other tiles, another order of them) give."""
import pytest
import torch

import oracle
import workloads as wl
from workloads import Net, conv, dense, flatten
from helpers import make_states, policies, student_tensors, teacher_tensors

pytestmark = pytest.mark.gpu

# 4096 states are two 64 x 64 tiles per compute unit of 256; row-major states behind the small convolution, fragment order in the
# Nature network
WIDE = Net("wide", "u8", (4, 16, 16), 5, [conv(4, 16, 2, 1, 0, True), flatten(), dense(16 * 15 * 15, 2048, True)])
SMALL = Net("order", "u8", (4, 16, 16), 5, [conv(4, 16, 2, 1, 0, True), flatten(), dense(16 * 15 * 15, 500, True)])


@pytest.mark.parametrize("net", ["rows", "nature", "wide"])
@pytest.mark.parametrize("precision", ["int8", "bf16"])
def test_results_do_not_depend_on_the_batch(precision, net):
    import paper_2211_15023_amd as A
    if net == "nature":
        nt, pt, ns, ps, qp = policies(2)
    else:
        nt = ns = SMALL if net == "rows" else WIDE
        pt = wl.init_params(ns, 4)
        qp = oracle.quantize_policy(ns, pt, make_states(ns, 16, wl.STREAM["calibration"]))
    pol = A.Policy(ns, "int8", student_tensors(qp), qp.act_scales) if precision == "int8" else A.Policy(nt, "bf16", teacher_tensors(pt))
    base, times = 300, 14                                         # 300 is no multiple of a tile's states
    dx = torch.from_numpy(make_states(nt, base, wl.STREAM["states"])).cuda()
    du = torch.from_numpy(wl.make_uniforms(base)).cuda()
    parts = [pol.forward(dx[i:i + 100].contiguous(), du[i:i + 100].contiguous()) for i in range(0, base, 100)]
    ref = [torch.cat(t * times) for t in zip(*parts)]
    dx, du = torch.cat([dx] * times), torch.cat([du] * times)
    for B in (1, 17, 128, 130, 300, 512, 575, 1100, 1900, 2048, 2049, 2305, 2311, 3009, 3600, 4096, 4097, 4200):
        print(f"{net} {precision} B={B}", flush=True)
        for got, want in zip(pol.forward(dx[:B], du[:B]), ref):
            assert torch.equal(got, want[:B])
    pol.close()
