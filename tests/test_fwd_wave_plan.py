"""The launch plan of the forward kernel for up to 16 token rows, compiled by itself for the host (whole numbers only): the
shape it names always fits in LDS and is the cheapest that does, and the calls that an earlier fixed order of the shapes
sent to a dearer one keep the cheaper one."""
import itertools
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2306_08162_amd", "csrc")
MAIN = r'''
#include <cstdio>
#include "gemv_fwd_wave_plan.hpp"
using namespace qlora;
int main()
{
    int bits, ar, xr, ng, zrow, count, N[4];
    while (std::scanf("%d %d %d %d %d %d", &bits, &ar, &xr, &ng, &zrow, &count) == 6) {
        for (int i = 0; i < count; ++i)
            if (std::scanf("%d", &N[i]) != 1) return 1;
        std::printf("%d", fw_plan(bits, ar, xr, ng, zrow, count, N));
        for (const FwShape sh : FW_SHAPES)
            std::printf(" %d %d %d", sh.nb, sh.gr, fw_lds(bits, sh, ar, xr, ng, zrow));
        std::printf("\n");
    }
    std::printf("static %d %d %d\n", fw_static(0), fw_static(8), fw_static(16));
    return 0;
}
'''


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "plan")], check=True)

    def ask(calls):
        """calls: (bits, ar, xr, ng, zrow, [N, ...]) -> per call (index or -1, [(nb, gr, lds), ...])"""
        text = "\n".join(" ".join(map(str, [*c[:5], len(c[5]), *c[5]])) for c in calls)
        lines = subprocess.run([str(d / "plan")], input=text, capture_output=True, text=True, check=True).stdout.split("\n")
        out = []
        for line in lines[:len(calls)]:
            v = [int(x) for x in line.split()]
            out.append((v[0], [tuple(v[1 + 3 * i:4 + 3 * i]) for i in range((len(v) - 1) // 3)]))
        statics = [int(x) for x in lines[len(calls)].split()[1:]]
        return out, dict(zip((0, 8, 16), statics))
    return ask


def _rounds(Ns, blocks):
    return -(-sum(-(-(-(-n // 16)) // blocks) for n in Ns) // 256)


def test_cheapest_shape_that_fits(plan):
    calls = [(bits, ar, xr, K // 128, -(-K // 128 * bits // 32) * 4 if packed else K // 128, Ns)
             for bits, ar, xr, K, packed, Ns in itertools.product(
                 (2, 3, 4, 8), (0, 8, 16), (4, 16), (128, 4096, 5120, 11008, 28672, 131072), (False, True),
                 ([8], [4096], [5120], [11008, 11008], [13824, 13824], [4096] * 3, [8192, 1024, 1024], [28672], [40000]))]
    answers, statics = plan(calls)
    chosen = 0
    for (bits, ar, xr, ng, zrow, Ns), (pick, shapes) in zip(calls, answers):
        cost = {}
        for i, (nb, gr, lds) in enumerate(shapes):
            assert lds == 0 or lds + statics[ar] <= 160 * 1024
            rounds = _rounds(Ns, nb * gr)
            if lds and not (nb * gr == 1 and rounds > 1 and ar == 16 and xr == 16):
                cost[i] = rounds * (3 + nb * gr)
        if pick < 0:
            assert not cost
        else:
            assert cost[pick] == min(cost.values())
            chosen += 1
    assert chosen > len(calls) // 2


@pytest.mark.parametrize("bits, ar, xr, K, Ns, rows", [
    (3, 8, 16, 5120, [13824, 13824], 64),       # was 96 rows: 288 workgroups, a second round for 32 of them
    (3, 8, 4, 5120, [13824, 13824], 64),
    (4, 8, 16, 5120, [13824, 13824], 64),
    (8, 8, 4, 5120, [13824, 13824], 64),
    (3, 8, 16, 8192, [28672], 64),              # was 96 rows
    (3, 16, 16, 4096, [32000], 64),             # was 32 rows: four rounds
    (4, 8, 4, 4096, [11008, 11008], 96),        # one round
    (2, 8, 16, 4096, [4096, 4096, 4096], 64),
    (2, 16, 16, 13824, [5120], 32),
    (8, 8, 16, 13824, [5120], 32),
])
def test_rows_of_a_workgroup(plan, bits, ar, xr, K, Ns, rows):
    (pick, shapes), = plan([(bits, ar, xr, K // 128, K // 128, Ns)])[0]
    assert pick >= 0 and 16 * shapes[pick][0] * shapes[pick][1] == rows


def test_one_block_of_many_rounds_is_left_to_the_older_kernel(plan):
    (pick, _), = plan([(3, 16, 16, 13824 // 128, 13824 // 128, [5120])])[0]
    assert pick == -1


def test_8_bit_rows_come_in_whole_lines(plan):
    """Without an adapter the 64-row shape with 128-column chunks (2 x 2 blocks) stands in for that of four blocks."""
    (pick, shapes), = plan([(8, 0, 16, 5120 // 128, 5120 // 128, [13824])])[0]
    assert shapes[pick][:2] == (2, 2)
