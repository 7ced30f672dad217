// Host side of gemv_fwd_wave.hpp: what a workgroup keeps in LDS, and how many weight rows it takes.  Whole numbers only, so
// that a test can compile it by itself.
#pragma once

namespace qlora {

namespace {

constexpr int FW_NW = 8;                   // waves of a workgroup; wave w takes the chunks w, w + 8, ... of its columns
constexpr int FW_LDS = 160 * 1024;
// Shapes of a workgroup: GR groups of NB 16-row blocks of weight rows
struct FwShape {
    int nb, gr;
};
constexpr FwShape FW_SHAPES[] = {{1, 1}, {2, 1}, {3, 1}, {4, 1}, {2, 2}, {3, 2}, {4, 2}};
constexpr int FW_SHAPE_COUNT = 7;

// columns of a chunk; half as many, so that two chunks fit, for 8-bit codes of several blocks (two blocks fit where no adapter
// rows come with them) and for 16 token rows beside 16 adapter rows (not for 3-bit codes: 64 columns of a row are no
// whole 16-byte pieces)
constexpr int fw_ks(int bits, int nb, int ar, int xr)
{
    return bits != 3 && ((bits == 8 && (nb > 2 || (nb == 2 && ar > 0))) || (ar == 16 && xr == 16)) ? 64 : 128;
}
constexpr int fw_xr(int ks, int xr) { return xr * ks < 512 ? 512 / ks : xr; }       // whole requests
constexpr int fw_chunk(int bits, int nb, int ar, int xr)
{
    const int ks = fw_ks(bits, nb, ar, xr);
    return (fw_xr(ks, xr) + ar) * 2 * ks + nb * 16 * ks * bits / 8;
}
constexpr int fw_tc(int ar) { return ar > 0 ? 16 : 64; }                                        // columns of t kept
constexpr int fw_static(int ar) { return 16 * (fw_tc(ar) + 1) * 4; }
// row pitch of the waves' partial sums: the four rows a wave writes together lie 16 banks apart
constexpr int FW_RS = 20;
constexpr int fw_red(int nb) { return FW_NW * (nb + 1) * 16 * FW_RS * 4; }

// 64 columns of 8-bit codes are half a cache line of a row, and a request of half lines is as many lines to work through for
// the compute unit as one of whole lines (HBM sees every line once: L2 has the other half).  So one wave takes both halves,
// and its weight rows are requested for two chunks at once ("pair"), in two slots of their own; token and adapter rows come
// by the chunk.  16 tokens, rank 8, INT8: 28672 -> 8192 65.8 -> 58.1 us, 13824 -> 5120 29.3 -> 26.4; the two chunks dealt to
// one wave but requested apart took as long as before.  (2- and 4-bit codes, rank 16: 12 to 16 % less at K = 28672, but
// 6 to 9 % more up to K = 384, where half of the waves get no columns: not done.)  Three blocks leave room for too few
// pairs (one token, 4096 -> 11008: 14.1 us apart, 15.1 in pairs), two groups would need a third slot.
constexpr int fw_wbytes(int bits, int nb, int ar, int xr) { return nb * 16 * fw_ks(bits, nb, ar, xr) * bits / 8; }
constexpr int fw_pair_depth(int bits, int nb, int ar, int xr)       // chunks of token and adapter rows beside two pairs
{
    const int w = fw_wbytes(bits, nb, ar, xr), x = fw_chunk(bits, nb, ar, xr) - w;
    const int d = ((FW_LDS - fw_static(ar) - 12 * 1024) / FW_NW - 4 * w) / x;
    return d > 4 ? 4 : d;
}
constexpr bool fw_pair(int bits, FwShape sh, int ar, int xr)
{
    return bits == 8 && sh.gr == 1 && sh.nb <= 2 && fw_ks(bits, sh.nb, ar, xr) == 64 && fw_pair_depth(bits, sh.nb, ar, xr) >= 3;
}

// chunks of a wave in flight: as many as fit beside tables of up to 12 KB (6 KB if that leaves only one), four at most
constexpr int fw_depth(int bits, FwShape sh, int ar, int xr)
{
    if (fw_pair(bits, sh, ar, xr)) return fw_pair_depth(bits, sh.nb, ar, xr);
    const int nb = sh.nb;
    const int chunks = FW_NW * fw_chunk(bits, nb, ar, xr), room = FW_LDS - fw_static(ar);
    const int d = (room - 12 * 1024) / chunks;
    return d > 4 ? 4 : (d >= 2 ? d : (room - 6 * 1024) / chunks);
}
constexpr int fw_ring(int bits, FwShape sh, int ar, int xr)         // bytes of a wave's ring
{
    const int d = fw_depth(bits, sh, ar, xr), c = fw_chunk(bits, sh.nb, ar, xr), w = fw_wbytes(bits, sh.nb, ar, xr);
    return fw_pair(bits, sh, ar, xr) ? d * (c - w) + 4 * w : d * c;
}

// group constants of a workgroup's rows in LDS: scales, zero-points (zrow bytes a row), each filled in whole KB
constexpr int fw_table(int rows, int ng, int zrow) { return ((rows * ng * 2 + 1023) & ~1023) + ((rows * zrow + 1023) & ~1023) + 16; }

// LDS of a workgroup; 0: the ring (two chunks at least) and the tables do not fit
constexpr int fw_lds(int bits, FwShape sh, int ar, int xr, int ng, int zrow)
{
    const int d = fw_depth(bits, sh, ar, xr);
    const int pipe = FW_NW * fw_ring(bits, sh, ar, xr) + fw_table(sh.nb * sh.gr * 16, ng, zrow);
    const int red = fw_red(sh.nb * sh.gr), lds = pipe > red ? pipe : red;
    return d >= 2 && lds <= FW_LDS - fw_static(ar) ? lds : 0;
}

// Index of the shape that serves `count` siblings of N[i] rows soonest, -1 if none fits.  One workgroup fills a compute unit's
// LDS, so a launch is as many rounds of 256 workgroups as it takes, and a round costs about as much as three blocks beside its
// own blocks: the order of rounds * (3 + blocks) is the measured order of the seven shapes at one and sixteen tokens over
// 2- to 8-bit codes and K = 2048 to 28672.  Two launches of 4-block workgroups instead of one round too many of 6-block ones:
// INT3, rank 8, 5120 -> 2 x 13824, 16 tokens 47.4 -> 35.2 us (INT4, rank 16: 48.2 -> 35.2), 8192 -> 28672 60.4 -> 44.6.
// Projections go together: with one shape for all, their rounds together are no more than their rounds apart.  One block
// per workgroup brings in x and A once per 16 rows: with 16 rows of both, more than one round of that is left to the
// kernel that stages x and A only (16 tokens, rank 16, 13824 -> 5120, INT3: 35.4 against 31.9 us; rank 8, INT2: 21.7
// against 26.3, so with fewer rows it stays).  Of two shapes at the same cost the one with whole cache lines is taken (INT8 without
// an adapter, 5120 -> 13824, 16 tokens: 2 x 2 blocks 19.6 us, four blocks 20.7).
inline int fw_plan(int bits, int ar, int xr, int ng, int zrow, int count, const int *N)
{
    int pick = -1, best = 0;
    for (int i = 0; i < FW_SHAPE_COUNT; ++i) {
        const int blocks = FW_SHAPES[i].nb * FW_SHAPES[i].gr;
        if (fw_lds(bits, FW_SHAPES[i], ar, xr, ng, zrow) == 0) continue;
        int wgs = 0;
        for (int p = 0; p < count; ++p) wgs += ((N[p] + 15) / 16 + blocks - 1) / blocks;
        const int rounds = (wgs + 255) / 256, cost = rounds * (3 + blocks);
        if (blocks == 1 && rounds > 1 && ar == 16 && xr == 16) continue;
        const int ks = fw_ks(bits, FW_SHAPES[i].nb, ar, xr);
        if (pick < 0 || cost < best || (cost == best && ks > fw_ks(bits, FW_SHAPES[pick].nb, ar, xr))) {
            pick = i;
            best = cost;
        }
    }
    return pick;
}

}  // namespace

}  // namespace qlora
