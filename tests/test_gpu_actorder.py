"""GPU parity for checkpoints quantized in activation order (App. A): the host sort, the permuted pack and the
column gather are exact integer / byte work; the layer called in sorted coordinates is compared with the oracle's
plain per-column-group definition in the checkpoint's own column order."""
import numpy as np
import pytest

import oracle
from paper_2306_08162_amd import binding as ql
from paper_2306_08162_amd import workloads as wl
from parity import Report, announce, layer_bounds, small_inputs

pytestmark = pytest.mark.gpu

CASES = [
    # (M, K, N, bits, G, r, dtype): weight-streaming, forward-only streaming, tiled paths; ragged everywhere
    (5, 256, 72, 4, 32, 8, "f16"),
    (16, 1376, 520, 2, 32, 16, "bf16"),
    (40, 384, 264, 3, 128, 16, "f16"),
    (300, 640, 392, 4, 128, 8, "f16"),
    (131, 1024, 136, 8, 64, 64, "bf16"),
    (77, 2080, 200, 3, 32, 0, "f16"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "M{}_K{}_N{}_b{}_G{}_r{}_{}".format(*c))
def test_actorder_layer(case):
    import torch
    from paper_2306_08162_amd.device import ActOrderLayer
    M, K, N, bits, G, r, dtype = case
    inp = small_inputs(11 * M + K + bits, M, K, N, bits, G, r, dtype)
    c = inp.cfg
    g_idx = wl.actorder_g_idx(c.seed, K, G)
    announce(f"act-order {c.name}")
    layer = ActOrderLayer(inp, g_idx)
    layer.forward()
    layer.backward()
    torch.cuda.synchronize()

    # integer and byte work: bit-exact
    perm_ref, inv_ref = oracle.actorder_perm(g_idx)
    assert np.array_equal(layer.perm.cpu().numpy(), perm_ref)
    assert np.array_equal(layer.inv_perm.cpu().numpy(), inv_ref)
    assert np.array_equal(layer.host_packed(), oracle.pack(inp.codes[:, perm_ref], bits))
    assert np.array_equal(layer.x.cpu().numpy().view(np.uint16), inp.x[:, perm_ref])

    # the layer, against the per-column-group definition in checkpoint order (A is held in sorted order)
    s = oracle.widen(inp.scales, "f16")
    Wd = oracle.dequant_actorder(inp.codes, s, inp.zeros, g_idx)
    x, dy = oracle.widen(inp.x, dtype), oracle.widen(inp.dy, dtype)
    A_sorted, B = oracle.widen(inp.A, dtype), oracle.widen(inp.B, dtype)
    A_ckpt = A_sorted[:, inv_ref] if r else A_sorted
    y_ref, _ = oracle.forward(x, Wd, A_ckpt, B, c.alpha)
    dx_ref = oracle.backward_dx(dy, Wd, A_ckpt, B, c.alpha)
    sc = c.alpha / r if r else 0.0
    t_ref = oracle.lora_down(x, A_ckpt) if r else None
    u_ref = oracle.lora_u(dy, B) if r else None
    b = layer_bounds(Wd, A_ckpt, B, sc, x=x, dy=dy, t=t_ref, u=u_ref, x_adapter=x)
    rep = Report(f"act-order {c.name}", dtype)
    rep.add("y", oracle.widen(layer.host_y(), dtype), y_ref, lines="rows", bound=b["y"])
    rep.add("dx", oracle.widen(layer.host_dx(), dtype), dx_ref, lines="rows", bound=b["dx"])
    if r:
        dA_ref, dB_ref = oracle.backward_adapters(dy, x, A_ckpt, B, c.alpha)
        rep.add("dA", layer.host_dA(), dA_ref[:, perm_ref], lines="rows", bound=b["dA"][:, perm_ref])
        rep.add("dB", layer.host_dB(), dB_ref, lines="cols", bound=b["dB"])
    rep.finish()


def test_gather_columns_out_of_range_index_gives_zero():
    import torch
    M, K = 9, 64
    src = torch.arange(1, M * K + 1, dtype=torch.int16, device="cuda:0").reshape(M, K)
    index = np.arange(K, dtype=np.int32)[::-1].copy()
    index[3], index[40] = -1, K
    idx = torch.from_numpy(index).to("cuda:0")
    dst = torch.full((M, K), 77, dtype=torch.int16, device="cuda:0")
    ql.qlora_gather_columns(src, idx, dst, M, K)
    torch.cuda.synchronize()
    ref = src.cpu().numpy()[:, np.clip(index, 0, K - 1)]
    ref[:, [3, 40]] = 0
    assert np.array_equal(dst.cpu().numpy(), ref)


def test_gather_full_size_is_exact():
    """The headline shape (2048 x 4096), sorted and back: the round trip returns the input bit for bit."""
    import torch
    M, K, G = 2048, 4096, 128
    g_idx = wl.actorder_g_idx(4242, K, G)
    perm = np.empty(K, dtype=np.int32)
    inv = np.empty(K, dtype=np.int32)
    ql.qlora_actorder_perm(g_idx, perm, inv, K, G)
    p_ref, i_ref = oracle.actorder_perm(g_idx)
    assert np.array_equal(perm, p_ref) and np.array_equal(inv, i_ref)
    x = wl.to_f16_bits(wl.normal(4243, M * K)).reshape(M, K)
    xd = torch.from_numpy(x.view(np.int16)).to("cuda:0")
    xs, xb = torch.empty_like(xd), torch.empty_like(xd)
    ql.qlora_gather_columns(xd, torch.from_numpy(perm).to("cuda:0"), xs, M, K)
    ql.qlora_gather_columns(xs, torch.from_numpy(inv).to("cuda:0"), xb, M, K)
    torch.cuda.synchronize()
    assert np.array_equal(xs.cpu().numpy().view(np.uint16), x[:, p_ref])
    assert np.array_equal(xb.cpu().numpy().view(np.uint16), x)


@pytest.mark.parametrize("bits", [2, 3, 4, 8])
@pytest.mark.parametrize("groups", [1, 11, 32, 86, 344])
def test_packed_zero_points_bit_exact(bits, groups):
    """Zero-points in their checkpoint storage form: pack and unpack against the oracle, bit for bit."""
    import torch
    N = 136
    z = wl.uniform_ints(77 + bits + groups, N * groups, 1 << bits).reshape(N, groups)
    zd = torch.from_numpy(z).to("cuda:0")
    words = ql.qlora_packed_zero_words(N, groups, bits)
    assert words == N * oracle.zero_words(groups, bits)
    pd = torch.full((N, words // N), -1, dtype=torch.int32, device="cuda:0")
    ql.qlora_pack_zeros(zd, pd, N, groups, bits)
    back = torch.full((N, groups), 255, dtype=torch.uint8, device="cuda:0")
    ql.qlora_unpack_zeros(pd, back, N, groups, bits)
    torch.cuda.synchronize()
    ref = oracle.pack_zeros(z, bits)
    assert np.array_equal(pd.cpu().numpy().view(np.uint32), ref)
    assert np.array_equal(back.cpu().numpy(), z)
    # and from the oracle's words, as a loader would hand them over
    pd2 = torch.from_numpy(ref.view(np.int32)).to("cuda:0")
    ql.qlora_unpack_zeros(pd2, back.fill_(255), N, groups, bits)
    torch.cuda.synchronize()
    assert np.array_equal(back.cpu().numpy(), oracle.unpack_zeros(ref, groups, bits))


def test_gather_rows_wider_than_the_lds_staging():
    """Rows of more than 32768 columns do not fit the kernel that stages a row in LDS: the direct kernel takes them.
    Seeded permutation with two indices out of range; every element compared."""
    import torch
    M, K = 5, 40000
    x = wl.to_f16_bits(wl.normal(77, M * K)).reshape(M, K)
    order = np.argsort(wl.uniform01(78, 0, K), kind="stable").astype(np.int32)
    order[11], order[39999] = -5, K + 3
    xd = torch.from_numpy(x.view(np.int16)).to("cuda:0")
    out = torch.full((M, K), 77, dtype=torch.int16, device="cuda:0")
    ql.qlora_gather_columns(xd, torch.from_numpy(order).to("cuda:0"), out, M, K)
    torch.cuda.synchronize()
    ref = x[:, np.clip(order, 0, K - 1)].copy()
    ref[:, [11, 39999]] = 0
    assert np.array_equal(out.cpu().numpy().view(np.uint16), ref)


# both sides of the workgroup sizes (2048 and 8192 columns, one or more workgroups), rows that end inside a batch of pieces, the
# longest row that is staged; a few indexes out of range
@pytest.mark.parametrize("M,K", [(1, 2048), (3, 2048), (3, 2080), (1, 4096), (5, 8192), (3, 8224), (2, 32768), (3, 32),
                                 (1, 2080), (1, 4128), (513, 8224), (770, 4128), (1536, 9216), (1537, 4128)])
def test_gathered_columns_at_the_workgroup_sizes(M, K):
    import torch
    from paper_2306_08162_amd import binding as ql
    g = torch.Generator().manual_seed(M + K)
    src = torch.randint(-2 ** 15, 2 ** 15, (M, K), generator=g, dtype=torch.int16)
    index = torch.randperm(K, generator=g).to(torch.int32)
    index[0], index[K // 2], index[K - 1] = -1, K, 2 ** 31 - 1
    inside = (index >= 0) & (index < K)
    want = torch.where(inside, src[:, index.clamp(0, K - 1).long()], 0)
    dst = torch.full((M, K), 7, dtype=torch.int16, device="cuda")
    announce(f"gather {M} x {K}")
    ql.qlora_gather_columns(src.cuda(), index.cuda(), dst, M, K)
    assert torch.equal(dst.cpu(), want)
