"""Small calls of the paper's network compute all three convolutions in one launch: the same whole numbers as the launches it replaces,
with the plain layout behind it and with the four-instruction requantization, for the smallest call, a ragged and the largest one."""
import pytest

import test_gpu_generic_paths as generic

pytestmark = pytest.mark.gpu

ENVS = dict(two_launches=dict(ACCERL_NO_CONV_TAIL="1"), plain_layout=dict(ACCERL_NO_FRAG_HANDOFF="1"),
            plain_requant_and_layout=dict(ACCERL_NO_P23="1", ACCERL_NO_FRAG_HANDOFF="1"))


@pytest.mark.parametrize("env,B", [("two_launches", 2), ("plain_layout", 77), ("plain_requant_and_layout", 256)])
def test_three_convolutions_in_one_launch(tmp_path, env, B):
    generic.test_kernel_choices_agree(tmp_path, env, ENVS[env], 2, B, "student")
