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


# 624 of 768 places of 256 x 256 tiles: taken with one stage, or with a rank above 32; 256 x 128 tiles at two stages and rank 8
NEARLY_FULL = [(1290, 64, 26376, 4, 64, "bf16"), (1290, 26400, 64, 2, 8, "f16"), (1290, 128, 26376, 3, 48, "f16"),
               (1290, 128, 26376, 8, 8, "bf16")]


@pytest.mark.parametrize("case", NEARLY_FULL, ids=lambda c: "M{}_K{}_N{}_b{}_r{}_{}".format(*c))
def test_nearly_full_rounds_of_large_tiles(case):
    M, K, N, bits, r, dtype = case
    check_layer(small_inputs(M + K + N + bits, M, K, N, bits, 32, r, dtype))


# split contractions at ranks 8 and 16: fewer tile columns than stages of a split (33), a contraction that ends inside a stage
# (2080, 1032), a last split shorter than the tile columns (4160), 8-bit codes at 28 tokens (tiled backward pass only), u
# with one tile column, with two and more token rows, t in four partial sums
SIDE = [(33, 4096, 512, 4, 8, "f16"), (130, 2080, 1032, 3, 8, "bf16"), (40, 1024, 4160, 2, 16, "f16"),
        (200, 1056, 2056, 2, 16, "bf16"), (28, 1024, 1024, 8, 8, "f16"), (129, 2048, 136, 8, 8, "f16"),
        (100, 96, 6664, 4, 16, "f16"), (600, 224, 2056, 3, 8, "bf16"), (1290, 2080, 72, 2, 8, "f16")]


PATTERN = 0x5a


def _in_room(inp, room, alloc, packed_zeros=False):
    """Outputs of both passes with the first `room` bytes of `alloc`, which holds PATTERN, as their workspace."""
    import torch
    import oracle
    from paper_2306_08162_amd.device import DeviceLayer
    layer = DeviceLayer(inp)
    if packed_zeros:
        layer.use_packed_zeros(oracle.pack_zeros(inp.zeros, inp.cfg.bits))
    alloc.fill_(PATTERN)
    layer.workspace = alloc[:room]
    layer.forward()
    layer.backward()
    torch.cuda.synchronize()
    assert bool((alloc[room:] == PATTERN).all()), f"bytes behind the {room} of the workspace were written"
    return {"y": layer.host_y().copy(), "t": layer.host_t().copy(), "dx": layer.host_dx().copy(), "dA": layer.host_dA().copy(),
            "dB": layer.host_dB().copy()}


@pytest.mark.parametrize("case", SIDE, ids=lambda c: "M{}_K{}_N{}_b{}_r{}_{}".format(*c))
def test_adapter_products_beside_a_split_gemm(case):
    import torch
    import oracle
    from paper_2306_08162_amd import binding as ql
    M, K, N, bits, r, dtype = case
    inp = small_inputs(M + K + N + bits, M, K, N, bits, 32, r, dtype)
    check_layer(inp)
    # the room without the partial sums of t and u: what the layer needs without an adapter, and t and u
    announce(f"smaller workspace: {inp.cfg.name}")
    total = ql.qlora_workspace_bytes(M, N, K, bits, 32, r)
    base = ql.qlora_workspace_bytes(M, N, K, bits, 32, 0) + 2 * ((M * r * 2 + 255) // 256 * 256)
    zeros = (N * (K // 32) + 255) // 256 * 256
    assert base < total and ql.qlora_workspace_bytes_zp(M, N, K, bits, 32, r) == total + zeros
    alloc = torch.empty(total + zeros + 4096, dtype=torch.uint8, device="cuda:0")
    full = _in_room(inp, total, alloc)
    assert bool((alloc[base:total] != PATTERN).any()), "t and u were formed by launches of their own"
    less = _in_room(inp, base, alloc)
    with pytest.raises(ql.QLoraError):
        _in_room(inp, base - 256, alloc)
    # t and, through it, dB: the same bits.  y, dx: the same fp32 sums in another order, half a unit in the last place each.  dA:
    # of u rounded so, at most a unit in the last place (two roundoffs) apart
    for name, got in full.items():
        if name in ("t", "dB"):
            assert np.array_equal(got, less[name]), name
        elif name == "dA":
            assert rel_fro(less[name], got) <= 2 * unit_roundoff(dtype), name
        else:
            wide = [np.asarray(oracle.widen(v, dtype), np.float64) for v in (less[name], got)]
            assert rel_fro(*wide) <= unit_roundoff(dtype), name
    # bit-packed zero-points, unpacked behind whichever of the two the buffer has room for: the bits of the calls above
    announce(f"smaller workspace, packed zero-points: {inp.cfg.name}")
    for room, want in ((total + zeros, full), (total + zeros - 256, less), (base + zeros, less)):
        got = _in_room(inp, room, alloc, packed_zeros=True)
        if room == total + zeros - 256:
            assert bool((alloc[base + zeros:] == PATTERN).all())
        for name in want:
            assert np.array_equal(got[name], want[name]), (name, room)


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
