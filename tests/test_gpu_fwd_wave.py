"""GPU parity of the forward kernel for up to 16 token rows against the CPU oracle at the edges of its dispatch: every
number of weight rows a workgroup takes (chosen so that the launch is one round of 256 workgroups), wave counts that do not
divide the chunks of a row, one request's worth of token rows and more, ranks formed in the kernel, handed in and absent."""
import pytest

from parity import check_layer, small_inputs

pytestmark = pytest.mark.gpu

# N: 16-row blocks that take 1, 2, 3, 4, 2 x 3 and 2 x 4 blocks per workgroup, and more than one round
CASES = [(M, K, N, bits, r, dtype)
         for i, (N, K) in enumerate([(8, 128), (4104, 1152), (8200, 384), (12296, 256), (16392, 640), (24584, 128), (32776, 128)])
         for bits, M, r, dtype in [(2, (1, 16)[i % 2], (8, 16)[i % 2], "f16"), (4, (16, 4)[i % 2], (16, 8)[i % 2], "f16"),
                                   (8, (5, 1)[i % 2], (0, 8)[i % 2], "f16"), (3, (4, 13)[i % 2], 8, "f16"),
                                   (2, (16, 3)[i % 2], 40, "bf16"), (4, (2, 9)[i % 2], 8, "bf16")]]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "M{}_K{}_N{}_b{}_r{}_{}".format(*c))
def test_forward_blocks_per_workgroup(case):
    M, K, N, bits, r, dtype = case
    check_layer(small_inputs(M + 3 * K + N + bits, M, K, N, bits, 128, r, dtype))
