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


def _exact(M, K, Ns, bits, r, dtype, G=128):
    """y (and t where it is formed in the kernel) of projections that share x, on whole-number inputs and power-of-two scales:
    every sum is exact in fp32 whatever its order, so the result is the exact one, rounded once.  The reference is a float64
    product on the GPU."""
    import torch
    from paper_2306_08162_amd import binding as ql

    gen = torch.Generator(device="cuda").manual_seed(M + 3 * K + sum(Ns) + bits + r)
    dt, flag = (torch.bfloat16, ql.QLORA_BF16) if dtype == "bf16" else (torch.float16, ql.QLORA_F16)

    def ints(lo, hi, *shape, keep=1.0):
        v = torch.randint(lo, hi + 1, shape, generator=gen, device="cuda")
        return v if keep == 1.0 else v * (torch.rand(shape, generator=gen, device="cuda") < keep)

    x = ints(-1, 1, M, K).to(dt)
    parts = []
    for N in Ns:
        q, z = ints(0, 2 ** bits - 1, N, K).to(torch.uint8), ints(0, 2 ** bits - 1, N, K // G).to(torch.uint8)
        s = torch.pow(2.0, -bits - ints(3, 4, N, K // G)).to(torch.float16)
        A, B = ints(-1, 1, max(r, 1), K, keep=0.03).to(dt), ints(-1, 1, N, max(r, 1)).to(dt)
        packed = torch.empty(ql.qlora_packed_words(N, K, bits), dtype=torch.int32, device="cuda")
        ql.qlora_pack(q, packed, N, K, bits)
        y, t = torch.zeros((M, N), dtype=dt, device="cuda"), torch.zeros((M, max(r, 1)), dtype=dt, device="cuda")
        parts.append((q, z, s, A, B, packed, y, t))
    ws = torch.empty(ql.qlora_siblings_workspace_bytes(list(Ns), M, K, bits, G, r), dtype=torch.uint8, device="cuda")
    col = lambda i: [p[i] for p in parts]
    ql.qlora_linear_fwd_siblings(x, col(5), col(2), col(1), col(3) if r else None, col(4) if r else None, col(6),
                                 col(7) if r else None, list(Ns), M, K, bits, G, r, float(r), flag, ws)
    for q, z, s, A, B, _, y, t in parts:
        wd = ((q.double().view(q.shape[0], -1, G) - z.double().unsqueeze(2)) * s.double().unsqueeze(2)).view(q.shape[0], K)
        want = x.double() @ wd.t().contiguous()
        if r:
            t_want = x.double() @ A.double().t().contiguous()
            assert t_want.abs().max() <= 256                        # exact in 16 bits
            assert torch.equal(t.double(), t_want)
            want = want + t_want @ B.double().t().contiguous()
        assert want.abs().max() * 2 ** (bits + 4) < 2 ** 24         # exact in fp32
        assert torch.equal(y, want.to(torch.float32).to(dt))


# Two groups of rows per workgroup, and more chunks of a row per wave than its ring holds: every wave waits for a chunk with the
# whole ring in flight, refills it within the first group and on into the second one.  4352 columns are 34 chunks, which eight
# waves share unevenly.
RING_CASES = [(M, 4352, Ns, bits, r, dtype)
              for Ns in [(16392,), (12296, 12280)] for bits in (2, 3, 4, 8)
              for M, r, dtype in [(1, 8, "f16"), (4, 16, "bf16"), (5, 8, "bf16"), (16, 8, "f16"), (16, 16, "f16"), (9, 40, "bf16"),
                                  (16, 0, "f16")]]


@pytest.mark.parametrize("case", RING_CASES, ids=lambda c: "M{}_K{}_N{}_b{}_r{}_{}".format(c[0], c[1], "x".join(map(str, c[2])), *c[3:]))
def test_ring_steady_state(case):
    _exact(*case)


# Launches of more than one round of 256 workgroups: the shape that the plan names once the larger ones do not fit in LDS
@pytest.mark.parametrize("case", [(16, 5120, (13824, 13832), 3, 8, "f16"), (2, 5120, (13824, 13832), 8, 8, "bf16"),
                                  (16, 4096, (32008,), 3, 16, "f16"), (16, 5120, (13832, 13824), 4, 8, "f16"),
                                  (16, 13824, (5128,), 3, 16, "bf16")],
                         ids=lambda c: "M{}_K{}_N{}_b{}_r{}_{}".format(c[0], c[1], "x".join(map(str, c[2])), *c[3:]))
def test_several_rounds(case):
    _exact(*case)


# 8-bit codes in 64-column chunks of one group: weight rows arrive for two chunks at once.  1 to 34 chunk pairs of a row, so that
# waves have none, one, two and more of them; one block of rows beside 16 adapter rows and two beside 8; token rows of one
# request and of two.  (Without an adapter two blocks fit with 128-column chunks.)
PAIR_CASES = [(M, K, (N,), 8, r, dtype)
              for K in (128, 256, 1024, 1152, 2176, 3200, 4352) for N, r in [(4112, 8), (8192, 8), (8192, 0), (264, 16)]
              for M, dtype in [(16, "f16"), (5, "bf16"), (2, "f16")] if N * (K // 128) % 16 == 0]


@pytest.mark.parametrize("case", PAIR_CASES, ids=lambda c: "M{}_K{}_N{}_b{}_r{}_{}".format(c[0], c[1], c[2][0], *c[3:]))
def test_paired_weight_requests(case):
    _exact(*case)
