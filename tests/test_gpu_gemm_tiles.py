"""GPU parity of the tiled GEMM against the CPU oracle where its dispatch changes from 128- to 256-row tiles: one round of
256 tiles of 128 x 128 (and one tile row or column more) in each direction, with and without the masked epilogue; and where
it splits its contraction and forms t or u beside the GEMM."""
import numpy as np
import pytest

from parity import announce, check_layer, rel_fro, small_inputs, unit_roundoff

pytestmark = pytest.mark.gpu

CASES = [(M, K, N, bits, dtype)
         for M, K, N in [(130, 128, 16384), (130, 128, 16392), (250, 128, 16448), (130, 16384, 64), (129, 16416, 64),
                         (257, 10944, 72), (300, 192, 10928)]
         for bits, dtype in [(4, "f16"), (2, "bf16"), (3, "f16"), (8, "bf16")]]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "M{}_K{}_N{}_b{}_{}".format(*c))
def test_tile_height_boundary(case):
    M, K, N, bits, dtype = case
    check_layer(small_inputs(M + 3 * K + N + bits, M, K, N, bits, 32, 8, dtype))


# launches of several rounds: two of 128-row tiles (430) instead of two of 256-row tiles (258), one of 256 x 256 tiles (129) instead
# of the same two, four of 128-row tiles (946) instead of three (516); forward into many columns, then backward
ROUNDS = [(577, 128, 11008, 4, "f16"), (577, 11008, 128, 2, "bf16"), (700, 128, 11008, 3, "f16"), (700, 11008, 128, 4, "f16"),
          (1290, 128, 11008, 8, "f16"), (1290, 11008, 128, 3, "f16")]


@pytest.mark.parametrize("case", ROUNDS, ids=lambda c: "M{}_K{}_N{}_b{}_{}".format(*c))
def test_tile_shape_by_rounds(case):
    M, K, N, bits, dtype = case
    check_layer(small_inputs(M + K + N + bits, M, K, N, bits, 32, 8, dtype))


# split contractions at ranks 8 and 16: fewer tile columns than stages of a split (33), a contraction that ends inside a stage
# (2080, 1032), a last split shorter than the tile columns (4160), 8-bit codes at 28 tokens (tiled backward pass only)
SIDE = [(33, 4096, 512, 4, 8, "f16"), (130, 2080, 1032, 3, 8, "bf16"), (40, 1024, 4160, 2, 16, "f16"),
        (200, 1056, 2056, 2, 16, "bf16"), (28, 1024, 1024, 8, 8, "f16"), (129, 2048, 136, 8, 8, "f16")]


@pytest.mark.parametrize("case", SIDE, ids=lambda c: "M{}_K{}_N{}_b{}_r{}_{}".format(*c))
def test_adapter_products_beside_a_split_gemm(case):
    import torch
    from paper_2306_08162_amd.device import DeviceLayer
    M, K, N, bits, r, dtype = case
    inp = small_inputs(M + K + N + bits, M, K, N, bits, 32, r, dtype)
    check_layer(inp)
    # a workspace without the room for the partial sums of t and u: they come from launches of their own.  Both forms round
    # the same fp32 sums, taken in another order, to 16 bits: half a unit in the last place each
    announce(f"smaller workspace: {inp.cfg.name}")
    full, less = DeviceLayer(inp), DeviceLayer(inp)
    less.workspace = less.workspace[:-256]
    for layer in (full, less):
        layer.forward()
        layer.backward()
    torch.cuda.synchronize()
    import oracle
    for name in ("host_y", "host_dx"):
        a, b = (np.asarray(oracle.widen(getattr(l, name)(), dtype), np.float64) for l in (full, less))
        assert rel_fro(a, b) <= unit_roundoff(dtype), name


# an infinity among the last elements of a contraction that ends inside a stage: it reaches t (u) as an infinity of the other
# factor's sign, and dB (dA) through it; the elements staged past the end must not make a NaN of it
@pytest.mark.parametrize("case", [(40, 1056, 2056, 2, 8, "f16"), (130, 2080, 1032, 3, 8, "bf16"), (45, 1056, 1032, 4, 16, "f16")],
                         ids=lambda c: "M{}_K{}_N{}_b{}_r{}_{}".format(*c))
def test_infinity_at_the_end_of_a_split_contraction(case):
    import torch
    import oracle
    from paper_2306_08162_amd.device import DeviceLayer
    M, K, N, bits, r, dtype = case
    inp = small_inputs(M + K + N + bits, M, K, N, bits, 32, r, dtype)
    announce(f"infinity at the end: {inp.cfg.name}")
    inf, mx, kx, my, ny = 0x7c00 if dtype == "f16" else 0x7f80, 5, K - 3, 7, N - 2
    inp.x[mx, kx], inp.dy[my, ny] = inf, inf
    x, dy, A, B = (oracle.widen(v, dtype) for v in (inp.x, inp.dy, inp.A, inp.B))
    layer = DeviceLayer(inp)
    layer.forward()
    layer.backward()
    torch.cuda.synchronize()
    t = oracle.widen(layer.host_t(), dtype)
    finite = np.arange(M) != mx
    assert np.isfinite(t[finite]).all()
    assert np.array_equal(t[mx], np.sign(A[:, kx]) * np.inf)
    k, n = np.arange(K) != kx, np.arange(N) != ny
    assert np.array_equal(layer.host_dA()[:, k], np.outer(np.sign(B[ny]), np.sign(x[my, k])) * np.inf)
    assert np.array_equal(layer.host_dB()[n], np.outer(np.sign(dy[mx, n]), np.sign(A[:, kx])) * np.inf)
