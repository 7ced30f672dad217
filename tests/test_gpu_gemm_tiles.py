"""GPU parity of the tiled GEMM against the CPU oracle where its dispatch changes from 128- to 256-row tiles: one round of
256 tiles of 128 x 128 (and one tile row or column more) in each direction, with and without the masked epilogue."""
import pytest

from parity import check_layer, small_inputs

pytestmark = pytest.mark.gpu

CASES = [(M, K, N, bits, dtype)
         for M, K, N in [(130, 128, 16384), (130, 128, 16392), (250, 128, 16448), (130, 16384, 64), (129, 16416, 64),
                         (257, 10944, 72), (300, 192, 10928)]
         for bits, dtype in [(4, "f16"), (2, "bf16"), (3, "f16"), (8, "bf16")]]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "M{}_K{}_N{}_b{}_{}".format(*c))
def test_tile_height_boundary(case):
    M, K, N, bits, dtype = case
    check_layer(small_inputs(M + 3 * K + N + bits, M, K, N, bits, 32, 8, dtype))
