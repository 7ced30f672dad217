// Forward pass for up to 16 token rows, one private pipeline per wave (included by gemv_fwd_impl.hpp).
//
// What bounds the pass is latency and the work inside a compute unit, not HBM: at 4096 x 4096, 16 workgroups take as long
// as 256.  A stage shared by the workgroup costs two barriers, and every wave then waits for the slowest request of all
// (the kernel this replaces).  Here the contraction is cut into chunks of 128 columns dealt to eight waves, and a wave
// brings in everything its chunk needs -- packed words of all rows, token rows, adapter rows -- with direct-to-LDS loads
// into a ring of its own, two to four chunks in flight, waiting on its own requests only.  No barrier in the loop; the
// waves meet once, to add their partial sums.  Rows of a workgroup are taken in up to two groups (GR) of NB 16-row blocks,
// one after the other through the same ring, so that q/k/v and gate/up are one launch and one round of the compute units.
// Measured (cold weights, from a graph; before: one launch per stage-wide kernel): INT4, one token, q/k/v 22.7 -> 11.8 us,
// gate/up 24.5 -> 17.4, o 7.2 -> 6.5, down 14.0 -> 11.6; INT2, 16 tokens, 13.4 -> 11.9, 24.3 -> 16.6, 7.7 -> 6.8,
// 16.4 -> 13.8.  Sixteen waves instead of eight, group constants laid out without bank conflicts and a converted table of
// them were no faster.
#pragma once
#include "gemv_fwd_wave_plan.hpp"

namespace qlora {

namespace {

// slot of the 16-byte piece `piece` of weight row n inside the row's PPR pieces of a chunk (its own inverse)
template <int BITS, int PPR>
__device__ __forceinline__ int fw_slot(int n, int piece)
{
    if constexpr (PPR == 8) return piece ^ ((n >> 1) & 7);
    else if constexpr (PPR == 4) return piece ^ ((n >> 2) & 3);
    else if constexpr (PPR == 2) return piece ^ ((n >> 3) & 1);
    else return piece;
}

// Eight codes of a word as an MFMA operand of exact integers q - z with the fewest instructions: codes that lie 16 bits
// apart are masked out together and land in the mantissas of (1024.0, 1024.0), one and-or per pair; a packed fma takes
// 1024 and z off.  The operand's order is then (0,4)(1,5)(2,6)(3,7) for 4-bit codes and (0,8)(1,9)(2,10)(3,11) |
// (4,12)(5,13)(6,14)(7,15) for the sixteen codes of a 2-bit word: fw_order() brings the activations into the same order.
// 3- and 8-bit codes keep their order (dequant8).
template <int BITS, bool BF16>
struct FwConst {
    static constexpr int NP = BITS == 2 ? 4 : 2;
    half2_t off[NP];      // -(1024 * 2^-p + z), p = BITS i
    float offf[NP];
    __device__ __forceinline__ void set(half_t nz)       // -z
    {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const float c = 1024.f / (float)(1 << (BITS * i));
            if constexpr (BF16) offf[i] = (float)nz - c;
            else off[i] = half2_t{nz, nz} + half2_t{(half_t)(-c), (half_t)(-c)};
        }
    }
};

template <int BITS, bool BF16>
__device__ __forceinline__ u16x8_t fw_dequant8(const uint32_t (&w)[BITS], int part, const FwConst<BITS, BF16> &c)
{
    static_assert(BITS == 2 || BITS == 4, "code widths whose codes meet 16 bits apart");
    typedef float float2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    const uint32_t word = BITS == 4 ? w[part] : w[part >> 1];
    u32x4_t out;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // pair i of the operand: bits p .. p + BITS of both halves of the (shifted) word
        const int p = BITS == 4 ? 4 * (i & 1) : 2 * i;
        const uint32_t x = (BITS == 4 ? i >= 2 : (part & 1)) ? word >> 8 : word;
        const uint32_t m = ((1u << BITS) - 1u) << p;
        const half2_t h = __builtin_bit_cast(half2_t, and_or(x, m | (m << 16), 0x64006400u));
        const float inv = 1.f / (float)(1 << p);
        if constexpr (BF16) {
            const float2_t f = {__builtin_fmaf((float)h[0], inv, c.offf[p / BITS]), __builtin_fmaf((float)h[1], inv, c.offf[p / BITS])};
            out[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
        } else {
            const half2_t hi = {(half_t)inv, (half_t)inv};
            out[i] = __builtin_bit_cast(uint32_t, p == 0 ? h + c.off[0] : h * hi + c.off[p / BITS]);
        }
    }
    return __builtin_bit_cast(u16x8_t, out);
}

// activations x[32 q' ..] in natural order (SS fragments of eight) -> the order of fw_dequant8
template <int BITS, int SS>
__device__ __forceinline__ void fw_order(const u16x8_t (&x)[SS], u16x8_t (&o)[SS])
{
    auto lo = [](uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); };
    auto hi = [](uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); };
#pragma unroll
    for (int s = 0; s < SS; ++s) {
        u32x4_t r;
        if constexpr (BITS == 4) {
            const u32x4_t d = __builtin_bit_cast(u32x4_t, x[s]);
            r = u32x4_t{lo(d[0], d[2]), hi(d[0], d[2]), lo(d[1], d[3]), hi(d[1], d[3])};
        } else {
            const u32x4_t a = __builtin_bit_cast(u32x4_t, x[s & ~1]), b = __builtin_bit_cast(u32x4_t, x[s | 1]);
            const int h = 2 * (s & 1);
            r = u32x4_t{lo(a[h], b[h]), hi(a[h], b[h]), lo(a[h + 1], b[h + 1]), hi(a[h + 1], b[h + 1])};
        }
        o[s] = __builtin_bit_cast(u16x8_t, r);
    }
}

template <int N>
__device__ __forceinline__ void fw_wait_pending(int chunks)       // at most `chunks` younger chunks of N requests in flight
{
    if (chunks >= 3) wait_vm<3 * N>();
    else if (chunks == 2) wait_vm<2 * N>();
    else if (chunks == 1) wait_vm<N>();
    else wait_vm<0>();
}

template <int BITS, bool BF16, int NB, int GR, int AR, int XMIN>
__device__ __forceinline__ void gemv_fwd_wave_body(const FwdArgs &a, const int wg)
{
    constexpr int NW = FW_NW, NT = NW * 64, R = 16 * NB, RT = R * GR;
    constexpr int KS = fw_ks(BITS, NB, AR, XMIN), SS = KS / 32, UB = KS * BITS / 32;      // MFMA steps; bytes of a lane's codes
    constexpr FwShape SHAPE = {NB, GR};
    constexpr bool PAIR = fw_pair(BITS, SHAPE, AR, XMIN);
    constexpr int PPC = KS * BITS / 128, PPR = PAIR ? 2 * PPC : PPC;        // pieces of a weight row per chunk, per request
    constexpr int PR = KS / 8, RPI = 64 / PR;                               // pieces of an activation row; rows per request
    constexpr int XR = fw_xr(KS, XMIN);
    constexpr int D = fw_depth(BITS, SHAPE, AR, XMIN), RING = fw_ring(BITS, SHAPE, AR, XMIN);
    constexpr int WB = R * PPR * 16, XB = (XR + AR) * 2 * KS;               // bytes of a slot: weight rows; token and adapter rows
    constexpr int CHUNK = PAIR ? XB : WB + XB;                              // PAIR: two weight slots ahead of the others
    constexpr int WI = (R * PPR + 63) / 64, XI = XR / RPI, AI = AR / RPI;   // requests of a chunk
    constexpr int RQ = WI + XI + AI, RQ1 = WI + XI;                         // of the first group, of a later one
    constexpr int NBT = NB * GR;
    constexpr int XOFF = PAIR ? 2 * WB : WB, AOFF = XOFF + XR * 2 * KS;
    constexpr int TC = fw_tc(AR);
    static_assert(D >= 2 && (D - 1) * RQ <= 63 && (!PAIR || D >= 3), "two chunks in flight, countable");
    static_assert(RING == (PAIR ? 2 * WB + D * XB : D * CHUNK), "the launch sizes LDS for this");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    __shared__ float tfull[16][TC + 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 15, q = lane >> 4;
    const int n0 = wg * RT, K = a.K, Kw = K * BITS / 32, r = a.r, ng = a.ng;
    const int rows_here = min(RT, a.N - n0);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)lds;
    constexpr int TABLES = NW * RING;
    const uint16_t *sct = (const uint16_t *)(lds + TABLES);
    const uint8_t *zt = lds + TABLES + ((RT * ng * 2 + 1023) & ~1023);
    const int zrow = a.zpacked ? a.zw * 4 : ng;

    // ---- group constants of the workgroup's rows: copied as they lie (the rows are neighbours), 1 KB per request; a piece
    //      past the end of the array repeats the array's first one (it belongs to rows past N)
    const uint32_t s_row = (uint32_t)ng * 2u, z_row = (uint32_t)zrow;
    auto copy_table = [&](const void *src, uint32_t row_bytes, uint32_t dst) {
        const uint32_t bytes = (uint32_t)RT * row_bytes, all = (uint32_t)a.N * row_bytes, first = (uint32_t)n0 * row_bytes;
        for (uint32_t o = (uint32_t)wave * 1024u; o < bytes; o += NW * 1024u) {
            const uint32_t at = first + o + lane * 16u;
            dma16(src, at + 16u <= all ? at : 0u, dst + o);
        }
    };
    {
        const uint32_t tb = lds0 + TABLES;
        copy_table(a.scales, s_row, tb);
        copy_table(a.zpacked ? (const void *)a.zpacked : (const void *)a.zeros, z_row, tb + ((RT * s_row + 1023u) & ~1023u));
    }

    // ---- this lane's part of the requests of a chunk
    const uint32_t *wbase = a.packed + (long)n0 * Kw;
    uint32_t w_src[GR][WI], x_src[XI], a_src[AI > 0 ? AI : 1];
#pragma unroll
    for (int g = 0; g < GR; ++g)
#pragma unroll
        for (int i = 0; i < WI; ++i) {
            const int e = min(64 * i + lane, R * PPR - 1), n = e / PPR, slot = e % PPR;
            w_src[g][i] = (uint32_t)min(g * R + n, rows_here - 1) * ((uint32_t)Kw * 4u) + (uint32_t)fw_slot<BITS, PPR>(n, slot) * 16u;
        }
    auto xkey = [](int row) { return PR == 16 ? row & 15 : (row >> 1) & 7; };
#pragma unroll
    for (int j = 0; j < XI; ++j) {
        const int row = RPI * j + lane / PR, piece = (lane % PR) ^ xkey(row);
        x_src[j] = (uint32_t)(((long)min(row, a.M - 1) * K + 8 * piece) * 2);
    }
#pragma unroll
    for (int j = 0; j < AI; ++j) {
        const int row = RPI * j + lane / PR, piece = (lane % PR) ^ xkey(row);
        a_src[j] = (uint32_t)(((long)min(row, r - 1) * K + 8 * piece) * 2);
    }
    // units are dealt to the waves in turn: a chunk, or a pair of them (K % 128 == 0: pairs are whole)
    const int units = K / (PAIR ? 2 * KS : KS), n_units = wave < units ? (units - wave + NW - 1) / NW : 0;
    const int n_it = PAIR ? 2 * n_units : n_units;
    auto chunk_at = [&](int i) { return PAIR ? 2 * (wave + NW * (i >> 1)) + (i & 1) : wave + NW * i; };
    const uint32_t mine = lds0 + (uint32_t)wave * RING;
    auto issue_w = [&](int g, int unit, uint32_t base) {
        const uint32_t c = (uint32_t)(wave + NW * unit);
#pragma unroll
        for (int j = 0; j < WI; ++j) {
            if ((j + 1) * 64 <= R * PPR || lane < R * PPR - 64 * j)      // a last request of fewer lanes
                dma16(wbase, w_src[g][j] + c * (uint32_t)(PPR * 16), base + j * 1024u);
        }
    };
    auto issue = [&](int g, int i, int slot) {
        const uint32_t c = (uint32_t)chunk_at(i), base = mine + (uint32_t)slot * CHUNK;
        if constexpr (!PAIR) issue_w(g, i, base);
#pragma unroll
        for (int j = 0; j < XI; ++j) dma16(a.x, x_src[j] + c * (uint32_t)(KS * 2), base + XOFF + j * 1024u);
        if (g == 0) {
#pragma unroll
            for (int j = 0; j < AI; ++j) dma16(a.A, a_src[j] + c * (uint32_t)(KS * 2), base + AOFF + j * 1024u);
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d) {
        if (PAIR && (d == 0 || d == 2) && d < n_it) issue_w(0, d / 2, mine + (d / 2) * WB);
        if (d < n_it) issue(0, d, d);
        else if (GR > 1 && n_it > 0 && d < 2 * n_it) issue(1, d - n_it, d);
    }

    // the rows of B the outputs need at the very end
    constexpr int EPT = (NBT * 256 + NT - 1) / NT, BV = AR > 0 ? AR / 8 : 1;
    u16x8_t bpre[EPT][BV];
    if constexpr (AR > 0) {
#pragma unroll
        for (int x = 0; x < EPT; ++x) {
            const int e = threadIdx.x + x * NT, nn = n0 + (e >> 8) * 16 + (e & 15);
            const bool live = e < NBT * 256 && nn < a.N;
#pragma unroll
            for (int h = 0; h < BV; ++h)
                bpre[x][h] = (live && 8 * h < r) ? *(const u16x8_t *)(a.B + (long)nn * r + 8 * h) : ZERO8;
        }
    }

    float4_t acc[NBT], tacc = float4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int nb = 0; nb < NBT; ++nb) acc[nb] = float4_t{0.f, 0.f, 0.f, 0.f};
    // where this lane's fragments lie in a chunk
    uint32_t x_at[SS], a_at[SS];
#pragma unroll
    for (int s = 0; s < SS; ++s) {
        const int piece = SS * q + s, xr = li & (XR - 1), ar = AR > 0 ? li & (AR - 1) : 0;
        x_at[s] = (uint32_t)(XOFF + (xr * PR + (piece ^ xkey(xr))) * 16);
        a_at[s] = (uint32_t)(AOFF + (ar * PR + (piece ^ xkey(ar))) * 16);   // adapter columns past r repeat: never used
    }
    const uint8_t *const ring = lds + (size_t)wave * RING;

    // the tables are this wave's oldest requests: they have landed with its first chunk; the barrier publishes them
    fw_wait_pending<PAIR ? XI + AI : (GR == 1 ? RQ : RQ1)>(min(D, n_it * GR) - 1);
    asm volatile("s_barrier" ::: "memory");
    const bool zpk = a.zpacked != nullptr;
    const uint32_t zbits = zpk ? BITS : 8;
    int slot = 0;
#pragma unroll
    for (int g = 0; g < GR; ++g) {
#pragma unroll 1
        for (int i = 0; i < n_it; ++i) {
            // chunk (g, i) has landed when at most the requests of the chunks behind it are in flight (chunks of later groups
            // bring no adapter rows: where one of them may be among those, all are counted as that short)
            constexpr int FULL = (D - 1) * (GR == 1 ? RQ : RQ1);
            // PAIR: behind the younger of this chunk's requests and its pair's stand those of the D - 1 chunks that follow and, if
            // another pair follows, those of exactly one pair: pair p is requested before chunk 2 p (the first two pairs) or
            // when pair p - 2 has been read, before chunk 2 p - 3 + D
            if constexpr (PAIR) {
                if (i + D <= n_it) wait_vm<(D - 1) * (XI + AI) + WI>();
                else fw_wait_pending<XI + AI>(n_it - 1 - i);
            } else if (GR == 2 && g == 0 && i + D <= n_it) wait_vm<(D - 1) * RQ>();
            else if (i + D <= n_it * (GR - g)) wait_vm<FULL>();
            else fw_wait_pending<GR == 1 ? RQ : RQ1>(n_it * (GR - g) - 1 - i);
            const uint8_t *buf = ring + slot * CHUNK, *wbuf = PAIR ? ring + ((i >> 1) & 1) * WB : buf;
            const int first = PAIR ? (i & 1) * PPC : 0;      // the chunk's first piece in a weight row
            const int grp = group_of(chunk_at(i) * KS, a.magic);
            const uint32_t zoff = zpk ? (uint32_t)(grp * BITS) >> 3 : (uint32_t)grp, zshift = zpk ? (grp * BITS) & 7 : 0;
            const uint32_t s_at = (uint32_t)li * s_row + (uint32_t)grp * 2u, z_at = (uint32_t)li * z_row + zoff;
            u16x8_t xf[SS], af[SS], xo[SS];
            uint32_t w[NB][BITS];
            half_t sc[NB];
            uint32_t zp[NB];
#pragma unroll
            for (int s = 0; s < SS; ++s) {
                xf[s] = *(const u16x8_t *)(buf + x_at[s]);
                if (AR > 0 && g == 0) af[s] = *(const u16x8_t *)(buf + a_at[s]);
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int n = nb * 16 + li;
                const uint8_t *rowp = wbuf + n * (PPR * 16);
                if constexpr (BITS == 3) {
                    const uint32_t *p = (const uint32_t *)(rowp + 12 * q);
#pragma unroll
                    for (int h = 0; h < 3; ++h) w[nb][h] = p[h];
                } else if constexpr (UB == 32) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const u32x4_t v = *(const u32x4_t *)(rowp + fw_slot<BITS, PPR>(n, first + 2 * q + h) * 16);
#pragma unroll
                        for (int e = 0; e < 4; ++e) w[nb][(4 * h + e) % BITS] = v[e];
                    }
                } else if constexpr (UB == 16) {
                    const u32x4_t v = *(const u32x4_t *)(rowp + fw_slot<BITS, PPR>(n, first + q) * 16);
#pragma unroll
                    for (int h = 0; h < 4; ++h) w[nb][h] = v[h];
#pragma unroll
                    for (int h = 4; h < BITS; ++h) w[nb][h] = 0u;
                } else if constexpr (UB == 8) {
                    const u32x2_t v = *(const u32x2_t *)(rowp + fw_slot<BITS, PPR>(n, q >> 1) * 16 + (q & 1) * 8);
                    w[nb][0] = v[0];
                    w[nb][1] = v[1];
#pragma unroll
                    for (int h = 2; h < BITS; ++h) w[nb][h] = 0u;
                } else {
                    w[nb][0] = *(const uint32_t *)(rowp + q * 4);
                    w[nb][1] = 0u;
                }
                sc[nb] = *(const half_t *)((const uint8_t *)sct + (s_at + (uint32_t)(g * NB + nb) * 16u * s_row));
                // one byte read for both storage forms of the zero-points, no branch: a branch per block would wait for its
                // own read (3-bit fields may reach into the next byte)
                const uint8_t *zq = zt + (z_at + (uint32_t)(g * NB + nb) * 16u * z_row);
                uint32_t z = zq[0];
                if constexpr (BITS == 3) z |= (uint32_t)zq[1] << 8;
                zp[nb] = __builtin_amdgcn_ubfe(z, (uint32_t)zshift, zbits);
            }
            wait_lds();                                      // the chunk is in registers: its slot may be refilled
            if (PAIR && (i & 1) && i + 3 < n_it) issue_w(0, (i >> 1) + 2, mine + ((i >> 1) & 1) * WB);
            if (i + D < n_it) issue(g, i + D, slot);
            else if (g + 1 < GR && i + D - n_it < n_it) issue(g + 1, i + D - n_it, slot);
            slot = slot + 1 == D ? 0 : slot + 1;
            if constexpr (BITS == 2 || BITS == 4) {
                fw_order<BITS, SS>(xf, xo);
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                // the chunk lies in one group: the MFMAs sum x (q - z), exact integers times x, and the scale is applied
                // to the four sums of the lane's weight row
                float4_t part = {0.f, 0.f, 0.f, 0.f};
                if constexpr (BITS == 2 || BITS == 4) {
                    FwConst<BITS, BF16> dq;
                    dq.set(-(half_t)(uint16_t)zp[nb]);
#pragma unroll
                    for (int s = 0; s < SS; ++s) part = mfma16<BF16>(xo[s], fw_dequant8<BITS, BF16>(w[nb], s, dq), part);
                } else {
                    DequantConst<BITS, BF16> dq;
                    dq.set(1.f, (float)zp[nb]);
#pragma unroll
                    for (int s = 0; s < SS; ++s)
                        part = mfma16<BF16>(xf[s], dequant8<BITS, BF16, false>(w[nb], s, dq), part);   // D[m = 4q+v][n = li]
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[g * NB + nb][v] = fmaf((float)sc[nb], part[v], acc[g * NB + nb][v]);
            }
            if (AR > 0 && g == 0) {
#pragma unroll
                for (int s = 0; s < SS; ++s) tacc = mfma16<BF16>(xf[s], af[s], tacc);   // D[m][j = li]
            }
        }
    }

    // ---- the waves' partial sums meet in LDS
    __syncthreads();
    float *red = (float *)lds;                               // [NW][NBT + 1][16][FW_RS]
    auto red_at = [&](int w, int blk, int row, int col) -> float & { return red[((w * (NBT + 1) + blk) * 16 + row) * FW_RS + col]; };
#pragma unroll
    for (int v = 0; v < 4; ++v) {
#pragma unroll
        for (int nb = 0; nb < NBT; ++nb) red_at(wave, nb, 4 * q + v, li) = acc[nb][v];
        if constexpr (AR > 0) red_at(wave, NBT, 4 * q + v, li) = tacc[v];
    }
    __syncthreads();
    if constexpr (AR > 0) {
        if (threadIdx.x < 256) {
            const int m = threadIdx.x >> 4, j = threadIdx.x & 15;
            float tv = 0.f;
            if (j < r && m < a.M) {
#pragma unroll
                for (int w = 0; w < NW; ++w) tv += red_at(w, NBT, m, j);
                tv = cvt16<BF16>(to16<BF16>(tv));            // the value every consumer of t sees
                if (wg == 0 && a.t_out) a.t_out[(long)m * r + j] = to16<BF16>(tv);
            }
            tfull[m][j] = tv;
        }
    } else {
        for (int e = threadIdx.x; e < a.M * r; e += NT) tfull[e / r][e % r] = cvt16<BF16>(a.t_in[e]);
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < EPT; ++x) {
        const int e = threadIdx.x + x * NT;
        const int nb = e >> 8, m = (e >> 4) & 15, nl = e & 15, nn = n0 + nb * 16 + nl;
        if (e >= NBT * 256 || m >= a.M || nn >= a.N) continue;
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += red_at(w, nb, m, nl);
        float lo = 0.f;
        if constexpr (AR > 0) {
#pragma unroll
            for (int h = 0; h < BV; ++h)
#pragma unroll
                for (int c = 0; c < 8; ++c) lo += tfull[m][8 * h + c] * cvt16<BF16>(bpre[x][h][c]);   // zero past r
        } else {
            for (int j0 = 0; j0 < r; j0 += 8) {
                const u16x8_t bv = *(const u16x8_t *)(a.B + (long)nn * r + j0);
#pragma unroll
                for (int h = 0; h < 8; ++h) lo += tfull[m][j0 + h] * cvt16<BF16>(bv[h]);
            }
        }
        a.y[(long)m * a.N + nn] = to16<BF16>(v + a.sc * lo);
    }
}

// A workgroup's stages fill a compute unit's LDS, which the compiler cannot know: two waves per SIMD is all there ever are.
// Left to spare registers for more, it requested the rows of B one by one where t is handed in (rank 64, one token,
// 1024 -> 4096, INT2: 9.3 against 8.3 us).
template <int BITS, bool BF16, int NB, int GR, int AR, int XR>
__global__ __launch_bounds__(FW_NW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemv_fwd_wave_kernel(const FwdMulti ma)
{
    int pi = 0;
    while (pi + 1 < ma.count && (int)blockIdx.x >= ma.wg_end[pi]) ++pi;          // wave-uniform
    const FwdArgs a = ma.p[pi];
    gemv_fwd_wave_body<BITS, BF16, NB, GR, AR, XR>(a, (int)blockIdx.x - (pi ? ma.wg_end[pi - 1] : 0));
}

template <int BITS, bool BF16, int AR, int XR, int SHAPE>
void launch_fwd_wave_one(FwdMulti m, hipStream_t s)
{
    constexpr int NB = FW_SHAPES[SHAPE].nb, GR = FW_SHAPES[SHAPE].gr;
    if constexpr (fw_depth(BITS, FW_SHAPES[SHAPE], AR, XR) >= 2) {            // (else the plan never names it)
        const FwdArgs &a = m.p[0];
        int wgs = 0;
        for (int i = 0; i < m.count; ++i) {
            wgs += (blocks16(m.p[i].N) + NB * GR - 1) / (NB * GR);
            m.wg_end[i] = wgs;
        }
        auto kern = gemv_fwd_wave_kernel<BITS, BF16, NB, GR, AR, XR>;
        ensure_dynamic_lds((const void *)kern, FW_LDS - fw_static(AR));
        QLORA_LAUNCH(kern, dim3(wgs), dim3(FW_NW * 64),
                     fw_lds(BITS, FW_SHAPES[SHAPE], AR, XR, a.ng, a.zpacked ? a.zw * 4 : a.ng), s, m);
    }
}

template <int BITS, bool BF16, int AR, int XR>
bool launch_fwd_wave_nb(const FwdMulti &m, hipStream_t s)
{
    const FwdArgs &a = m.p[0];
    int N[MAX_SIBLINGS];
    for (int i = 0; i < m.count; ++i) N[i] = m.p[i].N;
    switch (fw_plan(BITS, AR, XR, a.ng, a.zpacked ? a.zw * 4 : a.ng, m.count, N)) {
    case 0: launch_fwd_wave_one<BITS, BF16, AR, XR, 0>(m, s); return true;
    case 1: launch_fwd_wave_one<BITS, BF16, AR, XR, 1>(m, s); return true;
    case 2: launch_fwd_wave_one<BITS, BF16, AR, XR, 2>(m, s); return true;
    case 3: launch_fwd_wave_one<BITS, BF16, AR, XR, 3>(m, s); return true;
    case 4: launch_fwd_wave_one<BITS, BF16, AR, XR, 4>(m, s); return true;
    case 5: launch_fwd_wave_one<BITS, BF16, AR, XR, 5>(m, s); return true;
    case 6: launch_fwd_wave_one<BITS, BF16, AR, XR, 6>(m, s); return true;
    default: return false;
    }
}

// Serves the call if its shape allows: up to 16 token rows, K and the group size multiples of 128 (a chunk then shares its
// group constants), t formed here from at most 16 adapter rows or handed in, arrays that can be read in 16-byte pieces.
template <int BITS, bool BF16>
bool launch_fwd_wave(const FwdMulti &m, int rg, hipStream_t s)
{
    const FwdArgs &a = m.p[0];
    if (a.M > 16 || a.K % 128 != 0 || (a.K / a.ng) % 128 != 0 || rg > 1 || (rg == 0 && a.r > 64)) return false;
    for (int i = 0; i < m.count; ++i) {
        const FwdArgs &b = m.p[i];
        const uintptr_t bits_or = (uintptr_t)b.x | (uintptr_t)b.packed | (uintptr_t)b.scales | (uintptr_t)b.zeros |
                                  (uintptr_t)b.zpacked | (rg ? (uintptr_t)b.A : 0);
        const long zrow = b.zpacked ? b.zw * 4 : b.ng;
        if ((bits_or & 15) != 0 || ((long)b.N * b.ng) % 16 != 0 || ((long)b.N * zrow) % 16 != 0) return false;
    }
    // token rows in LDS: one request's worth (four rows of 128 columns) or sixteen
    const bool few = a.M <= 4;
    if (rg == 0) return few ? launch_fwd_wave_nb<BITS, BF16, 0, 4>(m, s) : launch_fwd_wave_nb<BITS, BF16, 0, 16>(m, s);
    if (a.r <= 8) return few ? launch_fwd_wave_nb<BITS, BF16, 8, 4>(m, s) : launch_fwd_wave_nb<BITS, BF16, 8, 16>(m, s);
    return few ? launch_fwd_wave_nb<BITS, BF16, 16, 4>(m, s) : launch_fwd_wave_nb<BITS, BF16, 16, 16>(m, s);
}

}  // namespace

}  // namespace qlora
