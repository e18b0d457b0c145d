"""Which kernel a dense layer takes on either side of the lines of its dispatch (names from a kernel trace), and that a row's result does not
depend on it: every row equals, bit for bit, what a call of 100 states gives."""
import pytest
import torch

import oracle
import workloads as wl
from workloads import Net, conv, dense, relu, flatten
from helpers import kernel_names, make_states, student_tensors, teacher_tensors

pytestmark = pytest.mark.gpu

CUS = torch.cuda.get_device_properties(0).multi_processor_count if torch.cuda.is_available() else 256


def _row_major(cout, side, width):
    return Net("routes", "u8", (4, side + 1, side + 1), 5,
               [conv(4, cout, 2, 1, 0, False), relu(), flatten(), dense(cout * side * side, width, True)])


# states at which `per` workgroups a tile of `rows` states fill the compute units once
def _full(rows, per):
    return rows * (CUS // per)


ROUTES = [
    # int8 of at most 256 features: 16 x 32 tiles up to one workgroup per compute unit, then four wavefronts on 16 x 64
    ("int8", lambda: _row_major(16, 11, 256), [(_full(16, 8), "ksplit_kernel<0, 0, 1, 2,"), (_full(16, 8) + 1, "ksplit_small_i8_kernel"),
                                               (_full(16, 8) + 64, "ksplit_small_i8_kernel")]),
    ("int8", lambda: wl.configs.PAPER_STUDENTS["net2"], [(_full(16, 4), "ksplit_kernel<0, 0, 1, 2,"), (_full(16, 4) + 1, "ksplit_small_i8_kernel")]),
    # int8 with more than 4 MB of weights: 64 x 64 tiles beyond one 32 x 64 tile per compute unit, the streaming kernel beyond an eighth more
    ("int8", lambda: wl.nature_cnn("wide", fc=2048), [(_full(32, 32), "ksplit_kernel<0, 0, 2, 4,"), (_full(32, 32) + 1, "ksplit_kernel<0, 0, 4, 4,"),
                                                      (_full(36, 32), "ksplit_kernel<0, 0, 4, 4,"), (_full(36, 32) + 1, "gemm_stream_i8_kernel")]),
    # bf16 beyond one 64 x 64 tile per compute unit: 41 steps of K go to the kernel that walks K in one wavefront, 61 stay (128 x 64 tiles) up
    # to an eighth more
    ("bf16", lambda: wl.configs.PAPER_STUDENTS["net2"], [(_full(64, 2), "ksplit_kernel<1, 2, 4, 4,"), (_full(64, 2) + 1, "gemm_kernel<1, 2, 8>")]),
    ("bf16", lambda: _row_major(16, 11, 256), [(_full(64, 4), "ksplit_kernel<1, 2, 4, 4,"), (_full(64, 4) + 1, "ksplit_kernel<1, 2, 8, 4,"),
                                               (_full(72, 4), "ksplit_kernel<1, 2, 8, 4,"), (_full(72, 4) + 1, "gemm_kernel<1, 2, 8>")]),
]


@pytest.mark.parametrize("case", range(len(ROUTES)))
def test_route(case):
    import paper_2211_15023_amd as A
    precision, make, lines = ROUTES[case]
    net = make()
    params = wl.init_params(net, 6)
    if precision == "int8":
        qp = oracle.quantize_policy(net, params, make_states(net, 16, wl.STREAM["calibration"]))
        pol = A.Policy(net, "int8", student_tensors(qp), qp.act_scales)
    else:
        pol = A.Policy(net, precision, teacher_tensors(params))
    dx = torch.from_numpy(make_states(net, 100, wl.STREAM["states"])).cuda()
    du = torch.from_numpy(wl.make_uniforms(100)).cuda()
    ref = pol.forward(dx, du)
    times = -(-max(B for B, _ in lines) // 100)
    dx, du, ref = torch.cat([dx] * times), torch.cat([du] * times), [torch.cat([t] * times) for t in ref]
    for B, kernel in lines:
        print(f"{net.name} {precision} B={B}: {kernel}", flush=True)
        out, names = kernel_names(lambda: pol.forward(dx[:B], du[:B]))
        assert any(kernel in n for n in names), names
        for got, want in zip(out, ref):
            assert torch.equal(got, want[:B])
    pol.close()
