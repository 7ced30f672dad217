// Tiled MFMA GEMM over the packed weight with dequantisation fused into the operand staging.
//
//   forward   (TRANS = false):  y [M,N]  = x [M,K]  * Wd[N,K]^T  + sc * t[M,r] * B[N,r]^T      (Fig. 1, forward path)
//   backward  (TRANS = true):   dX[M,K]  = dY[M,N]  * Wd[N,K]    + sc * u[M,r] * A[r,K]        (Sec. 3.1: the packed
//             weight is consumed transposed; transpose + unpack + matmul happen inside this one kernel)
//
// Both are C[M,NO] = Act[M,KC] * W^T with W viewed as [NO,KC]; only the way a packed tile is fetched and laid
// into LDS differs.  A workgroup owns a BM x BN output tile and walks the contraction in steps of 64.  Its eight
// waves are specialised: four staging waves move packed words global -> registers -> (unpack, s*(q-z), round to
// 16 bit) -> LDS (two stages); four MFMA waves pull the activation tile global -> LDS directly (three stages, no
// registers) and read 16-byte fragments of both operands into v_mfma_f32_16x16x32.  One barrier per stage.
// The dequantised weight never reaches HBM.  The rank-r LoRA term is folded in as extra contraction steps.
//
// What bounds the large launches is power: the matrix pipe's clock falls with the operand bits that change.  A
// register-resident loop on random fp16 operands sustains 1620 to 1660 TFLOP/s with 32x32x16 MFMAs and 1890 with 16x16x32
// in the order used here (qlora_mfma_probe; half the accumulator traffic per flop).  The 16x16x32 form, weights as the
// first operand and the MFMAs of a step in serpentine order take the fp16 step at 2048 x 4096 x 4096, INT4, from 153 to
// 144 us, 4096 x 11008 -> 4096, INT3, from 725 to 679 us and the bf16 forward pass at 8192 x 4096 -> 11008 from 725 to
// 693 us.  Launches of 128-row tiles are not held back by power: against 32x32x16 MFMAs, activations first, they take 0 to
// 9 % less in bf16 and in the forward pass, and between 2 % less and 2 % more in the fp16 backward pass.
// Launches that give every compute unit at least one 256 x 256 tile use a second arrangement of the same parts
// (SYM below): eight waves that each stage, load and multiply an eighth.
#include "common.hpp"
#include "dequant.hpp"
#include "kernels.hpp"

namespace qlora {

namespace {

constexpr int BK = 64;               // contraction elements per LDS stage
constexpr int GEMM_NXS = 3;     // activation stages in LDS
constexpr int LDS_STRIDE = BK + 8;   // 144-byte rows: the 16-byte reads of 8 consecutive rows fall in distinct bank groups
constexpr int STAGERS = 256;        // staging threads (4 waves); the MFMA waves come on top

struct GemmArgs {
    const uint16_t *act;      // x (forward) or dY (backward): [M, KC]
    const uint32_t *packed;   // [N, K*BITS/32]
    const uint16_t *scales;   // fp16 [N, K/G]
    const uint8_t *zeros;     // [N, K/G]
    const uint16_t *ext_act;  // t (forward) or u (backward): [M, r]; unused when r == 0
    const uint16_t *ext_w;    // B [N,r] (forward) or A [r,K] (backward)
    uint16_t *out;            // y [M,N] or dX [M,K]
    int M, N, K, G, r;
    float sc;
    int tiles_m, tiles_n;
    uint32_t g32_magic;       // see group_magic(): (k/32) / (G/32) == umulhi(k/32, magic), 0 meaning G == 32
    float *part;              // splits > 1: fp32 partial products [splits][M][NO], summed by splitk_sum_kernel
    int splits, kt_split;     // workgroups per tile along the contraction, 64-deep stages per workgroup
    const uint8_t *keep;      // LoRA dropout (backward only): keep bit of x[m, k] is bit k % 8 of keep[m * K/8 + k/8]
    float keep_sc;            // sc * keep_scale
    // split contraction: t (or u) formed beside the GEMM, see "side product"; side_r == 0: it is not
    const uint16_t *side_w;   // A [r,K] (forward) or B [N,r] (backward)
    float *side;              // partial sums [M][splits * side_p][side_r]
    int side_r, side_p;       // side_p: workgroups of a tile row and split that hold some
};

template <bool BF16>
__device__ __forceinline__ float4_t mfma16(u16x8_t a, u16x8_t b, float4_t c)
{
    if constexpr (BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b),
                                                       c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a), __builtin_bit_cast(half8_t, b), c,
                                                      0, 0, 0);
}

// 32 consecutive codes of one row are exactly BITS words.
template <int BITS>
__device__ __forceinline__ void load_unit(const uint32_t *__restrict__ p, uint32_t (&w)[BITS])
{
    if constexpr (BITS == 2) {
        const u32x2_t v = *(const u32x2_t *)p;
        w[0] = v[0];
        w[1] = v[1];
    } else if constexpr (BITS == 4) {
        const u32x4_t v = *(const u32x4_t *)p;
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = v[i];
    } else if constexpr (BITS == 8) {
        const u32x4_t v0 = *(const u32x4_t *)p, v1 = *(const u32x4_t *)(p + 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            w[i] = v0[i];
            w[4 + i] = v1[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < BITS; ++i) w[i] = p[i];
    }
}

// What one staging thread fetches for one 64-deep stage of the weight: WU packed units with their group's scale
// and zero-point, kept exactly as loaded.
template <int BITS, int WU>
struct StageRegs {
    uint32_t w[WU][BITS];
    uint16_t s[WU];     // raw fp16 bits: nothing may touch loaded values before they are staged, or the
    uint8_t z[WU];      // in-order memory counter would make that instruction wait for every load issued so far
    bool ok[WU];        // (not SYM) false: the unit lies outside the weight, stage zeros
};

// wait until at most N vector-memory operations of this wave are outstanding, then meet the workgroup
template <int N>
__device__ __forceinline__ void wait_vm_and_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// Swizzle key of a row of the backward weight stage.  Its upper two bits run through 0..3 over any 4 consecutive
// rows starting at a multiple of 4 (the transposing reads), its lower three bits through 0..7 over any 8 consecutive
// rows starting at a multiple of 8 (the 16-byte writes, one row per lane: eight lanes per clock into a bank space of
// 128 bytes.  Counters: with a key whose lower three bits took four values, a write took 16 LDS cycles instead of 8).
__device__ __forceinline__ constexpr int wswz(int row) { return ((row & 3) << 2) | ((row & 2) ^ ((row >> 2) & 2)) | ((row >> 2) & 1); }
// Slot key of a row of the forward weight stage of the symmetric arrangement (128-byte rows): eight different values
// over the even and over the odd rows of any 16 consecutive rows (16-byte reads: sixteen lanes per clock, two rows
// fill the 256-byte bank space), four different values mod 4 over any 4 consecutive rows (16-byte writes: two
// lanes per row, pieces p and p + 4, eight lanes per clock into 128 bytes).
__device__ __forceinline__ constexpr int fswz(int row) { return ((row & 3) ^ ((row >> 2) & 1)) | (((row >> 3) & 1) << 2); }

// MASKED (backward under LoRA dropout, ranks up to 32, no split): the adapter's share of dX is masked per element,
// dX = dY Wd + keep_sc * keep (.) (u A), so it cannot ride in the accumulators.  The LoRA steps are left out; the
// staging waves lay the tile's rows of u and columns of A (both fetched at kernel start) beside the epilogue area, and
// the copy-out adds the masked product to every 8-element piece before it is stored.
//
// SYM (256 x 256 tiles, for launches of at least one such tile per compute unit): eight waves, two per SIMD, each with
// a 128 x 64 block of accumulators and each doing an eighth of everything: activation loads, weight staging and the
// MFMAs.  The accumulators are half of a wave's 256 registers; a spilled register would be reloaded through the
// vector-memory counter that the stages wait on (a build with a dozen spills took 1.4 times as long), so addresses are
// formed when they are needed, two sets of packed words are in flight and two block rows of fragments are held.
//
// SIDE (launches of 128-row tiles whose contraction is split): t (forward) or u (backward) is formed as well, see "side
// product".  A template argument: a branch that is never taken cost the unsplit launches 1 to 4 %.
template <int BITS, bool BF16, bool TRANS, int BM, int BN, int WM, int WN, bool MASKED = false, bool SYM = false, bool SIDE = false>
__global__ __launch_bounds__(WM * WN * 64 + (SYM ? 0 : STAGERS)) void qgemm_kernel(const GemmArgs a)
{
    static_assert(!MASKED || TRANS, "the dropout mask acts on dX only");
    constexpr int MW = WM * WN;                     // MFMA waves
    constexpr int THREADS = MW * 64 + (SYM ? 0 : STAGERS);
    static_assert(MW == 4 || MW == 8, "one or two MFMA waves per SIMD");
    static_assert(!SYM || !MASKED, "symmetric waves: no masked epilogue");
    constexpr int NSTG = SYM ? MW * 64 : STAGERS;   // staging threads: all of them, or the four staging waves
    static_assert(BN % 128 == 0 && BM % 128 == 0, "tile shape");
    constexpr int TM = BM / WM, TN = BN / WN;       // per-wave output tile
    constexpr int MI = TM / 16, NI = TN / 16;       // 16x16 MFMA blocks per wave
    // block rows multiplied from one set of fragments (SYM: the staging registers leave room for two), sets per k-step
    constexpr int MH = SYM ? 2 : 4, AH = MI / MH;
    static_assert(MI % MH == 0, "a stage is made of whole steps of MH x NI MFMAs");
    constexpr int STEPS = AH * BK / 32;             // such steps per stage
    // The symmetric bf16 backward kernel holds its addresses and group constants for one use only and dequantises behind a
    // step's MFMAs: 5 to 23 registers spilled otherwise (4096 x 4096 x 4096, INT2: 167 us against 140)
    constexpr bool TIGHT = SYM && BF16 && TRANS;
    constexpr int XDMA = BM / 8 / MW;               // direct-to-LDS loads per MFMA wave per stage (8 rows each)
    static_assert(XDMA >= 4 && XDMA % 4 == 0, "loads are spread over the steps of a stage");
    constexpr int WU = 2 * BN / NSTG;               // 32-code weight units per staging thread per stage
    constexpr int XS = BM * BK;                     // halfs per activation stage (128-byte rows, swizzled)
    constexpr int NXS = GEMM_NXS;                   // (2 would let two workgroups share a CU's LDS: measured slower)
    static_assert(NXS == 2 || NXS == 3, "activation stages");
    // Weight stage.  Forward: [BN rows n][64 k + 8] (144-byte rows), fragments are 16-byte reads.  Backward: the
    // staging threads own rows n of the contraction, so the stage is kept as they produce it, [64 rows n][BN k],
    // and the fragments are gathered with the transposing LDS read (ds_read_b64_tr_b16), two per fragment.  The
    // 16-byte pieces of a row are XOR-swizzled with wswz(row): eight consecutive rows put the same piece into
    // eight different bank quads of the 128 bytes a write cycle covers (the stagers' 16-byte writes, one row per
    // lane), and four consecutive rows put four consecutive pieces into disjoint runs of 16 banks (the transposing
    // reads: 4 rows x 64 bytes per half wave).  Unpadded 320-byte rows served the reads equally well but made the
    // writes collide four ways.
    // SYM, forward: 128-byte rows with a slot swizzle (fswz) instead of the padding (LDS is full).
    constexpr int WPITCH = TRANS ? BN : (SYM ? BK : LDS_STRIDE);
    constexpr int WS = TRANS ? BK * WPITCH : BN * WPITCH;       // halfs per weight stage
    using Regs = StageRegs<BITS, WU>;

    static_assert(!SIDE || (BM == 128 && !SYM && !MASKED), "launches whose contraction is split");
    constexpr int SIDE_I = MI / WN;                 // side product: block rows per wave

    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    uint16_t *const xs = smem;                      // [NXS][BM][64]
    uint16_t *const wsm = smem + NXS * XS;          // [2] weight stages

    // The first MW waves feed the matrix cores: LDS fragment reads, MFMAs, and the direct-to-LDS loads of the
    // activation tile (no registers, no ALU work).  The last four waves stage the weight: packed words global ->
    // registers -> dequantise -> LDS.  Every SIMD hosts waves of both kinds (and, with MW = 8, two MFMA waves), so
    // one wave's fragment reads, loads and dequantisation issue in the shadow of another wave's MFMAs: a single
    // wave cannot hide its own instruction issue behind its MFMAs.
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave-uniform, kept in a scalar register
    const bool stager = SYM || wave >= MW, feeder = SYM || wave < MW;
    const int stid = SYM ? tid : tid - MW * 64;     // index among the staging threads
    const int cw = wave, wm = cw / WN, wn = cw % WN;
    const int NO = TRANS ? a.K : a.N;    // output columns
    const int KC = TRANS ? a.N : a.K;    // contraction length
    const int ng = a.K / a.G, Kw = a.K * BITS / 32;
    // a workgroup owns the stages kt_first .. kt_first + KT of its tile's contraction (all of them unless the
    // contraction is split over several workgroups)
    const int nt = a.tiles_m * a.tiles_n;
    const int split = __builtin_amdgcn_readfirstlane(a.splits > 1 ? (int)blockIdx.x / nt : 0);
    const int kt_first = split * a.kt_split;
    const int KT = min((KC + BK - 1) / BK - kt_first, a.kt_split);

    // --- which tile: consecutive workgroups land on different XCDs, so hand each XCD a contiguous run of tile
    //     ids, and order ids so that a run covers a compact block of tiles (shared rows and columns hit in L2)
    int pm, pn;
    {
        const int bid = a.splits > 1 ? (int)blockIdx.x % nt : (int)blockIdx.x;
        const int xcd = bid & 7, loc = bid >> 3, per = nt >> 3, rem = nt & 7;
        const int t = xcd * per + min(xcd, rem) + loc;
        // Tile ids run down GM tile rows before they move to the next tile column.  An activation tile row is 32 / bits
        // times the bytes of a packed weight tile column, so a run should be wide rather than tall: with 32 tiles per
        // XCD (the headline launch) GM = 2 makes it 2 x 16 and the launch fetches 69 MB where GM = 4 (4 x 8) fetched
        // 85 MB; the time is the same (the fetches are not what the kernel waits for).
        constexpr int GM = 2;
        const int in_group = GM * a.tiles_n, group = t / in_group, first_m = group * GM;
        const int gsz = min(a.tiles_m - first_m, GM), o = t % in_group;
        pm = first_m + o % gsz;
        pn = o / gsz;
    }
    const int row0 = pm * BM, col0 = pn * BN;

    float4_t acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};

    // Activation tile in LDS: row r is 128 bytes = eight 16-byte slots; slot s holds the row's chunk
    // s ^ ((r >> 1) & 7).  A 16-byte LDS read serves 16 lanes per clock out of a 256-byte-wide bank space, i.e. two
    // rows; with this key the 16 consecutive rows read by 16 lanes fall into 16 different slots of that space.
    // A direct-to-LDS load lays the 64 lanes' 16 bytes down contiguously (8 rows), so the swizzle is applied by
    // choosing which global chunk each lane fetches.
    // A step multiplies MH block rows of the activation tile with all NI block columns of the weight tile over 32
    // contraction elements; a k-step of 32 is AH steps that share the weight fragments.
    struct AFrags {
        u16x8_t a[MH];
    };
    struct BFrags {
        u16x8_t b[NI];
    };
    const int fr = lane & 15, fq = lane >> 4;
    int aoff[BK / 32];                              // per k-step: this lane's offset into an activation stage
#pragma unroll
    for (int ks = 0; ks < BK / 32; ++ks) aoff[ks] = (wm * TM + fr) * BK + ((4 * ks + fq) ^ ((fr >> 1) & 7)) * 8;
    // and into a weight stage (a k-step adds 32 contraction elements).  Transposing read: in every block of 16
    // lanes, lane 4e+g supplies the address of four consecutive 16-bit columns of one row, and lane i receives, as
    // element e, column i%4 of the row supplied by lane 4e + i/4.  Lane (e, g) of block b therefore points at row
    // 8 b + e, columns 4g .. +4 of the 32 x 16 slab of a block column, and lane l ends up with contraction elements
    // 8 (l/16) .. +4 of column l % 16: half an MFMA operand; the second read starts four rows further down.
    // The row's swizzle key differs between the two reads, so each of the 2 NI reads has its own offset.
    const int boff = TRANS ? 0 : (wn * TN + fr) * WPITCH + (SYM ? 0 : fq * 8);
    uint32_t toff[2] = {0, 0};                      // byte offsets for block column 0; block column j: ^ 32 j
    if constexpr (TRANS) {
        const int row = 8 * (lane >> 4) + ((lane & 15) >> 2);
        const int piece = (lane & 3) >> 1;                               // 16-byte piece within the 32-byte run
#pragma unroll
        for (int hi = 0; hi < 2; ++hi)
            toff[hi] = (uint32_t)((row + 4 * hi) * WPITCH * 2 + ((wn * TN / 8 + piece) ^ wswz(row + 4 * hi)) * 16 + 8 * (lane & 1));
        static_assert(!TRANS || TN == 64, "the pieces of a wave's block columns differ in slot bits 1 and 2 only");
    }
    auto load_a = [&](int xstage, int ks, int half, AFrags &f) {
        int at = aoff[ks];
        if constexpr (TIGHT) asm volatile("" : "+v"(at));
        const uint16_t *As = xs + xstage * XS + at + half * MH * 16 * BK;
#pragma unroll
        for (int i = 0; i < MH; ++i) f.a[i] = *(const u16x8_t *)(As + i * 16 * BK);
    };
    auto load_b = [&](int wstage, int ks, BFrags &f) {
        if constexpr (TRANS) {
            const uint8_t *Bs = (const uint8_t *)(wsm + wstage * WS + ks * 32 * WPITCH);   // 32 rows further: same swizzle keys
            uint32_t t0 = toff[0], t1 = toff[1];
            if constexpr (SYM) asm("" : "+v"(t0), "+v"(t1));            // formed when needed: registers are short
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                typedef short s16x4_t __attribute__((ext_vector_type(4)));
                typedef __attribute__((address_space(3))) s16x4_t *lds4_t;
                const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(Bs + (t0 ^ (32u * j))));
                const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(Bs + (t1 ^ (32u * j))));
                f.b[j] = u16x8_t{(uint16_t)lo[0], (uint16_t)lo[1], (uint16_t)lo[2], (uint16_t)lo[3],
                                 (uint16_t)hi[0], (uint16_t)hi[1], (uint16_t)hi[2], (uint16_t)hi[3]};
            }
        } else {
            // (SYM: the slot key depends on the row's lower four bits: the same 16 rows further down)
            const uint16_t *Bs = wsm + wstage * WS + boff + (SYM ? ((4 * ks + fq) ^ fswz(fr)) * 8 : ks * 32);
#pragma unroll
            for (int j = 0; j < NI; ++j) f.b[j] = *(const u16x8_t *)(Bs + j * 16 * WPITCH);
        }
    };
    // The weight is the MFMA's first operand: a lane then holds four neighbouring output columns of one token row.  The
    // order of a step's MFMAs is a serpentine, so that each shares one operand with the one before: what the matrix
    // pipe draws, and with it the clock, follows how many operand bits change (register-resident loop on random fp16
    // operands, one box: 1835 TFLOP/s in plain order, 1934 as a serpentine).  Launches of 128-row tiles are not held back by power, and
    // in plain order a step's first MFMAs need the fragments that arrive first (backward pass 2 % faster than as a serpentine).
    auto mfma_step = [&](int half, const AFrags &fa, const BFrags &fb) {
#pragma unroll
        for (int i = 0; i < MH; ++i)
#pragma unroll
            for (int jj = 0; jj < NI; ++jj) {
                const int j = BM > 128 && (i & 1) ? NI - 1 - jj : jj;
                acc[half * MH + i][j] = mfma16<BF16>(fb.b[j], fa.a[i], acc[half * MH + i][j]);
            }
    };
    // a step's MFMAs with the LDS reads of later steps slotted between them, one behind each MFMA
    auto spread = [&](int reads) {
#pragma unroll
        for (int i = 0; i < MH * NI; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                        // one MFMA
            if (i < reads) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);         // one LDS read
        }
    };
    constexpr int A_READS = MH, B_READS = TRANS ? 2 * NI : NI;
    AFrags fa[2];
    BFrags fb[2];
    [[maybe_unused]] u16x8_t sf[BK / 32];           // side product: the small operand's fragments of one stage
    [[maybe_unused]] float4_t sacc[SIDE_I];
#pragma unroll
    for (int i = 0; i < SIDE_I; ++i) sacc[i] = float4_t{0.f, 0.f, 0.f, 0.f};
    // The steps of one stage.  `work(s)` runs before step s's MFMAs are issued (loads, staging), `turn()` between the
    // last but one step and the last: the wait and barrier behind which the next stage's fragments may be read; the
    // last step runs from registers, over the LDS latency of those.
    auto stage_steps = [&](int xstage, int wstage, int xnext, auto &&work, auto &&turn) {
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            const int ks = st / AH, half = st % AH;
            const bool last = st + 1 == STEPS;
            if (!TIGHT || last) work(st);
            if (last) turn();
            const bool next_b = half + 1 == AH;                    // the step after starts a new k-step
            if (last) load_a(xnext, 0, 0, fa[(st + 1) & 1]);
            else load_a(xstage, (st + 1) / AH, (st + 1) % AH, fa[(st + 1) & 1]);
            if (next_b) {
                if (last) load_b(wstage ^ 1, 0, fb[(ks + 1) & 1]);
                else load_b(wstage, ks + 1, fb[(ks + 1) & 1]);
            }
            mfma_step(half, fa[st & 1], fb[ks & 1]);
            if (TIGHT && !last) work(st);
            spread(A_READS + (next_b ? B_READS : 0));
            if constexpr (SYM) __builtin_amdgcn_sched_barrier(0);
        }
    };

    // The same in pieces of one block row (256-row tiles, MFMA waves): NI MFMAs with the fragment reads of the same row of
    // the next step, then `slot(q)`, q = 0 .. SLOTS - 1 through the stage.  An activation request holds the compute unit's
    // address path for sixteen clocks and the wave until it is accepted; one behind every second row keeps MFMAs queued meanwhile,
    // where two in a row at the start of a step, by four waves at once, let the matrix pipe run dry.  Forward / backward, us:
    // 2048 x 4096 <- 4096, INT4 73.5 -> 71.9 / 80.6 -> 79.3; 4096 <- 11008, INT3 186.2 -> 186.3 / 196.0 -> 190.5; 5000 x 5120 <- 5120,
    // INT2 307 -> 300 / 323 -> 309 (all operands zero, 2048 x 4096, INT4: 59.5 -> 56.4 / 67.9 -> 64.1).  Requests behind the other
    // rows, or the eight of them behind the first eight, gain half of that; slots that differ from wave to wave lose 5 %, and
    // 128-row tiles, whose waves wait for the weight more than for this, lose 0 to 8 %.
    constexpr int SLOTS = STEPS * MH, SLOT_STEP = SLOTS / XDMA;     // slots of a stage; a request in every SLOT_STEP-th
    auto stage_rows = [&](int xstage, int wstage, int xnext, auto &&slot, auto &&turn) {
        auto read_a = [&](int stage, int ks, int half, int i) {
            return *(const u16x8_t *)(xs + stage * XS + aoff[ks] + (half * MH + i) * 16 * BK);
        };
        auto read_b = [&](int stage, int ks, int j) {
            if constexpr (TRANS) {
                const uint8_t *Bs = (const uint8_t *)(wsm + stage * WS + ks * 32 * WPITCH);
                typedef short s16x4_t __attribute__((ext_vector_type(4)));
                typedef __attribute__((address_space(3))) s16x4_t *lds4_t;
                const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(Bs + (toff[0] ^ (32u * j))));
                const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4_t)(Bs + (toff[1] ^ (32u * j))));
                return u16x8_t{(uint16_t)lo[0], (uint16_t)lo[1], (uint16_t)lo[2], (uint16_t)lo[3],
                               (uint16_t)hi[0], (uint16_t)hi[1], (uint16_t)hi[2], (uint16_t)hi[3]};
            } else return *(const u16x8_t *)(wsm + stage * WS + boff + ks * 32 + j * 16 * WPITCH);
        };
        static_assert(MH == NI || SYM, "a row of either operand per piece");
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            const int ks = st / AH, half = st % AH;
            const bool last = st + 1 == STEPS, next_b = half + 1 == AH;
            if (last) turn();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < MH; ++i) {
                fa[(st + 1) & 1].a[i] = last ? read_a(xnext, 0, 0, i) : read_a(xstage, (st + 1) / AH, (st + 1) % AH, i);
                if (next_b) fb[(ks + 1) & 1].b[i] = last ? read_b(wstage ^ 1, 0, i) : read_b(wstage, ks + 1, i);
#pragma unroll
                for (int jj = 0; jj < NI; ++jj) {                               // serpentine, as in mfma_step
                    const int j = i & 1 ? NI - 1 - jj : jj;
                    acc[half * MH + i][j] = mfma16<BF16>(fb[ks & 1].b[j], fa[st & 1].a[i], acc[half * MH + i][j]);
                }
#pragma unroll
                for (int h = 0; h < NI; ++h) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                        // one MFMA
                    if (h < 1 + (next_b ? (TRANS ? 2 : 1) : 0)) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
                }
                __builtin_amdgcn_sched_barrier(0);
                slot(st * MH + i);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    constexpr int EXT_STEPS = 2;                                        // LoRA steps whose operands are prefetched
    constexpr int EXT_A = BM * 2 / NSTG, EXT_W = BN * 2 / NSTG;   // pieces per staging thread and LoRA step
    u16x8_t ext_a[EXT_STEPS][EXT_A], ext_w[EXT_STEPS][EXT_W];

    // Where the unit of this thread lies in stage kt: weight row n and first column k0.  TRANS: 64 contraction rows n,
    // UPR units across the output columns k; else BN output rows n, 2 units along the contraction k.
    // TRANS: a wave takes all units of 64 / UPR rows, eight rows to eight neighbouring lanes (what the stage's writes need),
    // so that one of its loads touches 16 rows (BN = 256: 8), not 64: the compute unit works through a load row by
    // row, and the activation requests queue behind it.  Against one unit of each of the stage's 64 rows per wave, the whole
    // backward pass, us: 600 x 4096 <- 11008, INT4, fp16 112 -> 103; 777 x 4096 <- 4096, bf16 52.6 -> 48.9; 2048 x 4096 <- 4096,
    // INT8 82.0 -> 77.4; 4096 x 11008 <- 4096, INT8 377 -> 363.
    static_assert(WU == 1, "one unit per staging thread and stage");
    constexpr int UPR = BN / 32;
    const int t_row = (stid >> 6) * (64 / UPR) + (stid & 63) / (8 * UPR) * 8 + (stid & 7), t_unit = (stid >> 3) % UPR;
    auto unit_row = [&](int kt) { return TRANS ? (kt_first + kt) * BK + t_row : col0 + (stid >> 1); };
    auto unit_col = [&](int kt) { return TRANS ? col0 + t_unit * 32 : (kt_first + kt) * BK + (stid & 1) * 32; };
    // global -> registers for stage kt.  Branch-free: every address is clamped into the valid range and
    // whatever lies beyond the contraction length (or beyond the weight's rows / columns) is neutralised by a
    // zero scale, so stages past the end may be fetched and staged harmlessly.  SYM: a uniform base and one register per
    // address (byte offsets fit 32 bits: the entry points accept fewer than 2^32 codes), because registers are short.  The
    // staging waves have registers to spare and form plain pointers: with the 32-bit form a launch of 128-row tiles took 3 to
    // 9 % longer (513 x 4096 <- 11008, INT3, fp16, backward pass 118 -> 126 us).
    const uint32_t row_bytes = (uint32_t)Kw * 4u;
    const uint32_t g32_one = a.g32_magic ? 0u : ~0u;        // G == 32: the group is q itself (no branch in the loop)
    auto load_global = [&](int kt, Regs &rg) {
#pragma unroll
        for (int i = 0; i < WU; ++i) {
            if constexpr (SYM) {
                const uint32_t n = (uint32_t)min(unit_row(kt), a.N - 1), q = (uint32_t)min(unit_col(kt), a.K - 32) >> 5;
                load_unit<BITS>((const uint32_t *)((const uint8_t *)a.packed + (n * row_bytes + q * (BITS * 4u))), rg.w[i]);
                const uint32_t gi = n * (uint32_t)ng + (__umulhi(q, a.g32_magic) + (q & g32_one));
                rg.s[i] = *(const uint16_t *)((const uint8_t *)a.scales + gi * 2u);
                rg.z[i] = *(a.zeros + gi);
            } else {
                int n = unit_row(kt), k0 = unit_col(kt);
                rg.ok[i] = TRANS ? n < a.N && k0 < a.K : k0 < a.K;
                n = min(n, a.N - 1);
                k0 = min(k0, a.K - 32);
                load_unit<BITS>(a.packed + (long)n * Kw + (k0 >> 5) * BITS, rg.w[i]);
                const long gi = (long)n * ng + (a.g32_magic ? (int)__umulhi((uint32_t)(k0 >> 5), a.g32_magic) : (k0 >> 5));
                rg.s[i] = a.scales[gi];
                rg.z[i] = a.zeros[gi];
            }
        }
    };

    // registers -> LDS: the units of stage kt, dequantised 8 codes at a time; parts p0 .. p1 of unit i.  A unit's four
    // pieces go to slots that differ in their lower two bits only: piece p lies at (address of piece 0) ^ 16 p bytes.
    auto stage_parts = [&](int kt, const Regs &rg, int buf, int i, int p0, int p1) {
        const int u = stid + NSTG * i;
        DequantConst<BITS, BF16> dq;
        bool ok;
        if constexpr (SYM) ok = TRANS ? unit_row(kt) < a.N && unit_col(kt) < a.K : unit_col(kt) < a.K;
        else ok = rg.ok[i];
        uint32_t sr = rg.s[i], zr = rg.z[i];
        if constexpr (TIGHT) asm volatile("" : "+v"(sr), "+v"(zr));      // not kept from one part to the next
        dq.set(ok ? f16_bits_to_f32((uint16_t)sr) : 0.f, (float)zr);
        uint32_t at;                                // byte offset of piece 0 in the stage
        if constexpr (TRANS) at = t_row * (WPITCH * 2) + (((t_unit * 4) ^ wswz(t_row)) * 16);
        else if constexpr (SYM) at = (u >> 1) * (WPITCH * 2) + ((((u & 1) * 4) ^ fswz(u >> 1)) * 16);   // row u / 2
        else at = (u >> 1) * (WPITCH * 2) + (u & 1) * 64;
        if constexpr (SYM) asm("" : "+v"(at));      // the four addresses are formed when needed: four registers fewer
        uint8_t *Bs = (uint8_t *)(wsm + buf * WS);
#pragma unroll
        for (int part = p0; part < p1; ++part) {
            const u16x8_t v = dequant8<BITS, BF16>(rg.w[i], part, dq);
            *(u16x8_t *)(Bs + (TRANS || SYM ? at ^ (uint32_t)(part * 16) : at + (uint32_t)(part * 16))) = v;
        }
    };
    auto stage = [&](int kt, const Regs &rg, int buf) {
#pragma unroll
        for (int i = 0; i < WU; ++i) stage_parts(kt, rg, buf, i, 0, 4);
    };

    if constexpr (SYM) {
        // ---- symmetric waves: every wave requests an MW-th of the activation tile, stages an MW-th of the weight
        //      stage and multiplies its own block.  Per 64-deep stage and wave: eight steps of MH NI MFMAs, every other one
        //      with a quarter of the unit that is dequantised into the other weight buffer, the ones between with one of
        //      the XDMA direct-to-LDS requests; and one unit requested from memory NSETS stages ahead.
        static_assert(NXS == 3, "three activation stages");
        const int drow = lane >> 3;
        const int dchunk = ((lane & 7) ^ ((4 * cw + (drow >> 1)) & 7)) * 8;
        const uint32_t xs_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t *)xs;
        uint32_t xoff[XDMA];
#pragma unroll
        for (int i = 0; i < XDMA; ++i)
            xoff[i] = (uint32_t)min(row0 + (MW * i + cw) * 8 + drow, a.M - 1) * (uint32_t)KC * 2u;
        auto issue_x = [&](int kt, int stage, int i) {
            const uint32_t k2 = (uint32_t)min((kt_first + kt) * BK + dchunk, KC - 8) * 2u;
            const uint32_t dst = xs_lds + (uint32_t)(stage * XS + (MW * i + cw) * 512) * 2u;
            dma16(a.act, xoff[i] + k2, (uint32_t)__builtin_amdgcn_readfirstlane((int)dst));
        };
        // Requests complete in the order they were made.  Per stage a wave first requests its weight units (at least
        // WL instructions), then the XDMA activation pieces for the stage after next; "the activation pieces of the
        // next stage have landed" is therefore "at most XDMA + WL requests are outstanding".
        constexpr int WL = WU * (BITS == 3 ? 3 : (BITS == 8 ? 2 : 1));
        constexpr int NSETS = 2;
        Regs rs[NSETS];
#pragma unroll
        for (int i = 0; i < NSETS; ++i) load_global(i, rs[i]);
#pragma unroll
        for (int i = 0; i < XDMA; ++i) issue_x(0, 0, i);
#pragma unroll
        for (int i = 0; i < XDMA; ++i) issue_x(1, 1, i);
        stage(0, rs[0], 0);
        load_global(NSETS, rs[0]);
        wait_vm_and_barrier<XDMA + WL>();       // activation stage 0 and every wave's share of weight stage 0 are in LDS
        load_a(0, 0, 0, fa[0]);
        load_b(0, 0, fb[0]);
        int xstage = 0;
        static_assert(STEPS == 8 && WU == 1 && XDMA == 4, "a part of the staging or a request per step");
        // stage kt: rg holds the units of stage kt + 1, and is refilled with those of stage kt + 1 + NSETS
        auto step = [&](int kt, Regs &rg) {
            const int wstage = kt & 1, wfill = wstage ^ 1;
            const int xnext = xstage + 1 == NXS ? 0 : xstage + 1;
            const int xfill = xnext + 1 == NXS ? 0 : xnext + 1;
            auto work = [&](int st) {
                if (st % 2 == 0) stage_parts(kt + 1, rg, wfill, 0, st / 2, st / 2 + 1);
                else issue_x(kt + 2, xfill, st / 2);
            };
            auto turn = [&]() {
                wait_vm_and_barrier<XDMA + WL>();    // activation stage kt + 1 has landed; weight stage kt + 1 is written
                load_global(kt + 1 + NSETS, rg);
            };
            stage_steps(xstage, wstage, xnext, work, turn);
            xstage = xnext;
        };
        int kt0 = 0;
        for (; kt0 + NSETS <= KT; kt0 += NSETS) {
#pragma unroll
            for (int i = 0; i < NSETS; ++i) step(kt0 + i, rs[(i + 1) % NSETS]);
        }
#pragma unroll
        for (int i = 0; i < NSETS - 1; ++i)
            if (kt0 + i < KT) step(kt0 + i, rs[(i + 1) % NSETS]);
        wait_vm_and_barrier<0>();               // nothing in flight any more: LDS is quiet
    } else
    if (!stager) {
        // ---- MFMA waves ----
        __builtin_amdgcn_s_setprio(1);          // when both kinds of wave are ready, the matrix pipe's feeder goes first
        // direct-to-LDS loads: this wave's load i covers tile rows (MW i + cw) * 8 .. + 8
        const int drow = lane >> 3;              // row within the 8-row block; block b starts at tile row 8 b
        const int dchunk = ((lane & 7) ^ ((4 * cw + (drow >> 1)) & 7)) * 8;   // MW * i * 4 is a multiple of 8
        const uint32_t xs_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t *)xs;
        uint32_t xoff[XDMA];                    // byte offset of this lane's row within the activation matrix
#pragma unroll
        for (int i = 0; i < XDMA; ++i)
            xoff[i] = (uint32_t)min(row0 + (MW * i + cw) * 8 + drow, a.M - 1) * (uint32_t)KC * 2u;
        auto issue_x = [&](int kt, int stage, int i) {
            // stages past the end and chunks past the contraction length re-read valid data; the weight side is zero there
            const uint32_t k2 = (uint32_t)min((kt_first + kt) * BK + dchunk, KC - 8) * 2u;
            const uint32_t dst = xs_lds + (uint32_t)(stage * XS + (MW * i + cw) * 512) * 2u;   // wave-uniform byte address
            dma16(a.act, xoff[i] + k2, (uint32_t)__builtin_amdgcn_readfirstlane((int)dst));
        };
        // Side product: the workgroups of a tile row all hold the same activation stages, so each of them multiplies some by
        // the small operand as well (stages pn, pn + tiles_n, ... of its run), a half of the tile's rows per wave column, and
        // leaves fp32 partial sums of t (or u) that the kernel which sums the planes adds up.  That is a launch less than with t
        // (or u) by a kernel of its own, which took 5 to 6 us beside 20 of the GEMM.  INT2, fp16, rank 8, forward / backward, us:
        // 64 x 4096 <- 4096 20.8 -> 18.6 / 24.9 -> 20.4; 256 30.3 -> 28.3 / 33.2 -> 28.8; 512 x 4096 <- 11008 74.0 -> 67.4 / 67.4 -> 65.2.
        [[maybe_unused]] int side_kt = SIDE && pn < a.side_p ? pn : KT;
        auto side_load = [&](int kt) {
#pragma unroll
            for (int ks = 0; ks < BK / 32; ++ks) {
                const int k = (kt_first + kt) * BK + 32 * ks + 8 * fq;          // eight contraction elements of this lane
                const bool in = k < KC;
                sf[ks] = u16x8_t{0, 0, 0, 0, 0, 0, 0, 0};
                if (!in || fr >= a.side_r) continue;
                if constexpr (TRANS) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) sf[ks][e] = a.side_w[(long)(k + e) * a.side_r + fr];
                } else sf[ks] = *(const u16x8_t *)(a.side_w + (long)fr * a.K + k);
            }
        };
        auto side_step = [&](int xstage, auto &&inside) {
#pragma unroll
            for (int ks = 0; ks < BK / 32; ++ks)
#pragma unroll
                for (int i = 0; i < SIDE_I; ++i) {
                    u16x8_t x = *(const u16x8_t *)(xs + xstage * XS + aoff[ks] + (wn * SIDE_I + i) * 16 * BK);
                    if (!inside(ks)) x = u16x8_t{0, 0, 0, 0, 0, 0, 0, 0};
                    sacc[i] = mfma16<BF16>(sf[ks], x, sacc[i]);             // D[j = 4 fq + v][m = fr]
                }
        };
        // A contraction that ends inside a stage: past its end lie copies of the row's last elements, which have to be zero
        // beside the zeros of sf, or an infinity among them would make a NaN of the sum.  Zeroing them in every stage costs 2 to
        // 5 % where a workgroup takes most of its stages (642 x 64 <- 28672), so that last stage is taken after the loop.
        [[maybe_unused]] const int side_tail = SIDE && KC % BK != 0 && kt_first + KT == (KC + BK - 1) / BK ? KT - 1 : KT;
        [[maybe_unused]] bool at_tail = false;
        auto side_fetch = [&]() {               // for the next stage, side_kt
            if (side_kt >= KT) return;
            side_load(side_kt);
            if (side_kt == side_tail) {
                at_tail = true;
                side_kt = KT;
            }
        };
        if constexpr (SIDE) side_fetch();       // the oldest requests: they have landed with the first stage
#pragma unroll
        for (int i = 0; i < XDMA; ++i) issue_x(0, 0, i);
        if constexpr (NXS == 3) {
#pragma unroll
            for (int i = 0; i < XDMA; ++i) issue_x(1, 1, i);
        }
        constexpr int AHEAD = NXS == 3 ? XDMA : 0;   // loads that may still be in flight when a stage is needed
        wait_vm_and_barrier<AHEAD>();           // stage 0 of the activations has landed; weights staged by waves 4-7
        if constexpr (SIDE) {
#pragma unroll
            for (int ks = 0; ks < BK / 32; ++ks) asm volatile("" : "+v"(sf[ks]));     // the compiler's wait for them goes here
        }
        load_a(0, 0, 0, fa[0]);
        load_b(0, 0, fb[0]);
        int xstage = 0;                         // kt % NXS
        for (int kt = 0; kt < KT; ++kt) {
            const int xnext = xstage + 1 == NXS ? 0 : xstage + 1;
            const int xfill = NXS == 3 ? (xnext + 1 == NXS ? 0 : xnext + 1) : xnext;   // the stage NXS-1 ahead
            // the activation loads for stage kt+2 are spread over the steps, or over the rows of MFMAs
            auto work = [&](int st) {
#pragma unroll
                for (int i = st * XDMA / STEPS; i < (st + 1) * XDMA / STEPS; ++i) issue_x(kt + NXS - 1, xfill, i);
            };
            // stage kt+1 has landed: only loads for a later one may be pending, with ROWS those issued before the last step
            constexpr bool ROWS = BM > 128;
            auto turn = [&]() { wait_vm_and_barrier<ROWS ? AHEAD - XDMA / STEPS : AHEAD>(); };
            auto slot = [&](int q) {
                if (q % SLOT_STEP == 0) issue_x(kt + NXS - 1, xfill, q / SLOT_STEP);
            };
            if (SIDE && kt == side_kt) {
                side_step(xstage, [](int) { return true; });
                side_kt += a.tiles_n;
                side_fetch();
            }
            if constexpr (ROWS) stage_rows(xstage, kt & 1, xnext, slot, turn);
            else stage_steps(xstage, kt & 1, xnext, work, turn);
            xstage = xnext;
        }
        wait_vm_and_barrier<0>();               // the loads issued past the last stage have landed: LDS is quiet
        if constexpr (SIDE) {
            if (at_tail)
                side_step(xstage == 0 ? NXS - 1 : xstage - 1,
                          [&](int ks) { return (kt_first + KT - 1) * BK + 32 * ks + 8 * fq < KC; });
        }
    } else {
        // ---- weight staging waves ----
        // The operands of the LoRA steps that follow the main loop (up to two steps, ranks up to 32) are requested
        // now, so their memory latency is long gone when they are needed: 8-element pieces of t (or u) and of B (or A);
        // piece (row, half h) of step st holds adapter columns 16 st + 8 h .. + 8.
        const int ext_steps = (a.r + 15) / 16;
        if (a.r > 0 && split == 0 && ext_steps <= EXT_STEPS) {
#pragma unroll
            for (int st = 0; st < EXT_STEPS; ++st) {
#pragma unroll
                for (int i = 0; i < EXT_A; ++i) {
                    const int c = stid + NSTG * i, r = c >> 1, j = 16 * st + (c & 1) * 8;
                    ext_a[st][i] = u16x8_t{0, 0, 0, 0, 0, 0, 0, 0};
                    if (j < a.r) ext_a[st][i] = *(const u16x8_t *)(a.ext_act + (long)min(row0 + r, a.M - 1) * a.r + j);
                }
#pragma unroll
                for (int i = 0; i < EXT_W; ++i) {
                    const int c = stid + NSTG * i;
                    ext_w[st][i] = u16x8_t{0, 0, 0, 0, 0, 0, 0, 0};
                    if constexpr (TRANS) {
                        const int j = 16 * st + c / (BN / 8), col = col0 + (c % (BN / 8)) * 8;
                        if (j < a.r && col < NO) ext_w[st][i] = *(const u16x8_t *)(a.ext_w + (long)j * a.K + col);
                    } else {
                        const int r = c >> 1, j = 16 * st + (c & 1) * 8, col = col0 + r;
                        if (j < a.r && col < NO) ext_w[st][i] = *(const u16x8_t *)(a.ext_w + (long)col * a.r + j);
                    }
                }
            }
        }
        // stage kt+1 is written while the MFMA waves work on stage kt; NSETS later stages are in flight from
        // memory (one register set each)
        // (forward with 128-row tiles, whose stages are half as long, gains 1 to 2 % from a fourth set; backward loses 2 to 4 %
        // where the contraction is split)
        constexpr int NSETS = BM == 128 && !TRANS ? 4 : 3;
        Regs rs[NSETS];
#pragma unroll
        for (int i = 0; i < NSETS; ++i) load_global(i, rs[i]);
        stage(0, rs[0], 0);
        load_global(NSETS, rs[0]);
        __syncthreads();
        auto step = [&](int kt, Regs &rg) {
            stage(kt + 1, rg, (kt + 1) & 1);
            load_global(kt + 1 + NSETS, rg);
            __syncthreads();
        };
        // Whole rotations run without any condition inside: the compiler derives how many loads may stay in flight
        // from the static paths through the loop, and a skippable step would make it assume the shortest one.
        int kt0 = 0;
        for (; kt0 + NSETS <= KT; kt0 += NSETS) {
#pragma unroll
            for (int i = 0; i < NSETS; ++i) step(kt0 + i, rs[(i + 1) % NSETS]);
        }
#pragma unroll
        for (int i = 0; i < NSETS - 1; ++i)
            if (kt0 + i < KT) step(kt0 + i, rs[(i + 1) % NSETS]);
        __syncthreads();                        // pairs with the MFMA waves' final wait-and-barrier
    }

    // --- LoRA term as extra contraction steps: Act' = sc * t (or u), W' = B (or A^T), zero-padded to 32.
    //     Every wave is past the last barrier of the main loop, so every LDS stage is free.
    constexpr int ESTR = TN + 8;                            // row pitch of a wave's epilogue area
    constexpr int SIDE_R = 32;                              // adapter columns of the masked epilogue's side tiles
    uint16_t *const side_u = smem + MW * TM * ESTR;         // [BM][SIDE_R] rows of u, behind the epilogue areas
    uint16_t *const side_a = side_u + BM * SIDE_R;          // [SIDE_R][BN] columns of A
    if constexpr (MASKED) {
        if (stager) {                                       // the prefetched pieces, as they are (zero past the rank)
#pragma unroll
            for (int st = 0; st < EXT_STEPS; ++st) {
#pragma unroll
                for (int i = 0; i < EXT_A; ++i) {
                    const int c = stid + NSTG * i;
                    *(u16x8_t *)(side_u + (c >> 1) * SIDE_R + 16 * st + (c & 1) * 8) = ext_a[st][i];
                }
#pragma unroll
                for (int i = 0; i < EXT_W; ++i) {
                    const int c = stid + NSTG * i;
                    *(u16x8_t *)(side_a + (16 * st + c / (BN / 8)) * BN + (c % (BN / 8)) * 8) = ext_w[st][i];
                }
            }
        }
    }
    if (!MASKED && a.r > 0 && split == 0) {                 // the first workgroup of a split contraction adds it
        const int nsteps = (a.r + 31) / 32, width = nsteps * 32;
        if (!SYM && stager && nsteps == 1) {                // operands already in registers (zero past the rank)
#pragma unroll
            for (int st = 0; st < EXT_STEPS; ++st) {
#pragma unroll
                for (int i = 0; i < EXT_A; ++i) {
                    const int c = stid + NSTG * i, r = c >> 1, jc = 2 * st + (c & 1);
                    u16x8_t p;
#pragma unroll
                    for (int h = 0; h < 8; ++h) p[h] = to16<BF16>(a.sc * cvt16<BF16>(ext_a[st][i][h]));
                    *(u16x8_t *)(xs + r * BK + ((jc ^ ((r >> 1) & 7)) * 8)) = p;  // same swizzle as the main loop
                }
#pragma unroll
                for (int i = 0; i < EXT_W; ++i) {
                    const int c = stid + NSTG * i;
                    if constexpr (TRANS)
                        *(u16x8_t *)(wsm + (16 * st + c / (BN / 8)) * WPITCH
                                     + (((c % (BN / 8)) ^ wswz(c / (BN / 8))) * 8)) = ext_w[st][i];
                    else if constexpr (!SYM)
                        *(u16x8_t *)(wsm + (c >> 1) * LDS_STRIDE + 16 * st + (c & 1) * 8) = ext_w[st][i];
                }
            }
        } else if (stager) {
            const int cpr = width / 8;                      // 8-element chunks per row
            for (int c = stid; c < BM * cpr; c += NSTG) {
                const int r = c / cpr, jc = c % cpr, j = jc * 8;
                u16x8_t p = {0, 0, 0, 0, 0, 0, 0, 0};
                if (j < a.r) {
                    const int gm = min(row0 + r, a.M - 1);
                    const u16x8_t v = *(const u16x8_t *)(a.ext_act + (long)gm * a.r + j);
#pragma unroll
                    for (int h = 0; h < 8; ++h) p[h] = to16<BF16>(a.sc * cvt16<BF16>(v[h]));
                }
                *(u16x8_t *)(xs + r * BK + ((jc ^ ((r >> 1) & 7)) * 8)) = p;  // same swizzle as the main loop
            }
            if constexpr (TRANS) {          // rows j of A, the tile's columns contiguous: the stage's own layout
                for (int c = stid; c < width * (BN / 8); c += NSTG) {
                    const int j = c / (BN / 8), col = col0 + (c % (BN / 8)) * 8;
                    u16x8_t p = {0, 0, 0, 0, 0, 0, 0, 0};
                    if (j < a.r && col < NO) p = *(const u16x8_t *)(a.ext_w + (long)j * a.K + col);
                    *(u16x8_t *)(wsm + j * WPITCH + (((c % (BN / 8)) ^ wswz(j)) * 8)) = p;
                }
            } else {
                for (int c = stid; c < BN * cpr; c += NSTG) {
                    const int r = c / cpr, j = (c % cpr) * 8;
                    const int col = col0 + r;
                    u16x8_t p = {0, 0, 0, 0, 0, 0, 0, 0};
                    if (j < a.r && col < NO) p = *(const u16x8_t *)(a.ext_w + (long)col * a.r + j);
                    if constexpr (SYM) *(u16x8_t *)(wsm + r * WPITCH + (((c % cpr) ^ fswz(r)) * 8)) = p;
                    else *(u16x8_t *)(wsm + r * LDS_STRIDE + j) = p;
                }
            }
        }
        __syncthreads();
        if (feeder) {
            for (int ks = 0; ks < nsteps; ++ks) {
                load_b(0, ks, fb[0]);
#pragma unroll
                for (int half = 0; half < AH; ++half) {
                    load_a(0, ks, half, fa[0]);
                    mfma_step(half, fa[0], fb[0]);
                }
            }
        }
        __syncthreads();
    }

    // --- epilogue: fp32 accumulators -> 16 bit.  Each MFMA wave lays its TM x TN block into its own LDS area in
    //     row-major order; then all waves stream the areas out in 16-byte pieces (8 lanes per 128-byte row
    //     segment).  Rows beyond M and columns beyond NO (always whole 8-element pieces) are dropped.
    if (!SYM && a.splits > 1) {
        // split contraction: the fp32 accumulators go to this split's plane as they are (16 bytes per lane,
        // 64 consecutive bytes of a row); a second kernel sums the planes in order and rounds once
        if (feeder) {
            float *P = a.part + (size_t)split * a.M * NO;
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    const int grow = row0 + wm * TM + i * 16 + (lane & 15), gcol = col0 + wn * TN + j * 16 + (lane >> 4) * 4;
                    if (grow < a.M && gcol < NO) *(float4_t *)(P + (size_t)grow * NO + gcol) = acc[i][j];   // NO % 8 == 0
                }
            if (SIDE && pn < a.side_p) {
#pragma unroll
                for (int i = 0; i < SIDE_I; ++i) {
                    const int m = row0 + wm * TM + (wn * SIDE_I + i) * 16 + fr, j = 4 * fq;
                    if (m < a.M && j < a.side_r)
                        *(float4_t *)(a.side + ((size_t)m * (a.splits * a.side_p) + split * a.side_p + pn) * a.side_r + j) = sacc[i];
                }
            }
        }
        return;
    }
    if (feeder) {
        uint16_t *E = smem + cw * (TM * ESTR);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const u16x4_t h = {to16<BF16>(acc[i][j][0]), to16<BF16>(acc[i][j][1]), to16<BF16>(acc[i][j][2]),
                                   to16<BF16>(acc[i][j][3])};
                *(u16x4_t *)(E + (i * 16 + (lane & 15)) * ESTR + j * 16 + (lane >> 4) * 4) = h;
            }
    }
    __syncthreads();
    {
        constexpr int CPR = TN / 8;                       // 16-byte pieces per row of one wave's area
        constexpr int PER_AREA = TM * CPR;
        for (int c = tid; c < MW * PER_AREA; c += THREADS) {
            const int w = c / PER_AREA, cc = c % PER_AREA;
            const int r = cc / CPR, ch = (cc % CPR) * 8;
            const int grow = row0 + (w / WN) * TM + r, gcol = col0 + (w % WN) * TN + ch;
            u32x4_t v = *(const u32x4_t *)(smem + w * (TM * ESTR) + r * ESTR + ch);
            if constexpr (MASKED) {
                if (grow < a.M && gcol < NO) {
                    const uint32_t bits = a.keep[(size_t)grow * (NO / 8) + gcol / 8];
                    const uint16_t *ur = side_u + ((w / WN) * TM + r) * SIDE_R, *ap = side_a + (w % WN) * TN + ch;
                    float l[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                    const int rp = (a.r + 7) / 8;               // 8-column pieces of the adapter
                    for (int jp = 0; jp < rp; ++jp) {
                        const u16x8_t u8 = *(const u16x8_t *)(ur + 8 * jp);
                        u16x8_t a8[8];
#pragma unroll
                        for (int jj = 0; jj < 8; ++jj) a8[jj] = *(const u16x8_t *)(ap + (8 * jp + jj) * BN);
                        // 128-row tiles, bf16: all eight rows requested before the first is used, for the compiler waits for one
                        // after the other there (rank 32, 91 x 768 <- 64: 16.2 against 18.9 us; fp16 loses 1 %, 256-row tiles 3 %)
                        if constexpr (BF16 && BM == 128) {
#pragma unroll
                            for (int jj = 0; jj < 8; ++jj) asm volatile("" : "+v"(a8[jj]));
                        }
#pragma unroll
                        for (int jj = 0; jj < 8; ++jj) {
                            const float uj = cvt16<BF16>(u8[jj]);
#pragma unroll
                            for (int e = 0; e < 8; ++e) l[e] = fmaf(uj, cvt16<BF16>(a8[jj][e]), l[e]);
                        }
                    }
                    const u16x8_t b8 = __builtin_bit_cast(u16x8_t, v);
                    u16x8_t o8;
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        o8[e] = ((bits >> e) & 1u) ? to16<BF16>(cvt16<BF16>(b8[e]) + a.keep_sc * l[e]) : b8[e];
                    v = __builtin_bit_cast(u32x4_t, o8);
                }
            }
            // written once and not read by this kernel: the non-temporal hint keeps the output from displacing the
            // activation rows and weight columns that other tiles still want from L2 (-1 us per GEMM)
            if (grow < a.M && gcol < NO) __builtin_nontemporal_store(v, (u32x4_t *)(a.out + ((long)grow * NO + gcol)));
        }
    }
}

template <int BITS, bool BF16, bool TRANS, int BM, int BN, int WM, int WN, bool MASKED = false, bool SYM = false, bool SIDE = false>
void launch_variant(const GemmArgs &a, hipStream_t s)
{
    constexpr size_t wstage = TRANS ? (size_t)BK * BN : (size_t)BN * (SYM ? BK : LDS_STRIDE);
    constexpr size_t lds_pipe = (GEMM_NXS * (size_t)BM * BK + 2 * wstage) * sizeof(uint16_t);
    constexpr size_t lds_side = MASKED ? (size_t)32 * (BM + BN) * sizeof(uint16_t) : 0;    // side tiles of the masked epilogue
    constexpr size_t lds_epi = (size_t)WM * WN * (BM / WM) * (BN / WN + 8) * sizeof(uint16_t) + lds_side;
    constexpr size_t lds = lds_pipe > lds_epi ? lds_pipe : lds_epi;
    static_assert(lds <= 160 * 1024, "LDS of a compute unit");
    auto kern = qgemm_kernel<BITS, BF16, TRANS, BM, BN, WM, WN, MASKED, SYM, SIDE>;
    ensure_dynamic_lds((const void *)kern, (int)(lds));
    QLORA_LAUNCH(kern, dim3(a.tiles_m * a.tiles_n * a.splits), dim3(WM * WN * 64 + (SYM ? 0 : STAGERS)), lds, s, a);
}

// out = round16(sum over the S split planes, in order): 4 elements per thread.  The number of planes is a template argument
// so that a thread requests all of its pieces before it adds the first: a loop over them was one memory round trip per
// plane (64 x 4096, 8 planes: the pass took 1.0 us longer).
template <bool BF16, int S>
__global__ __launch_bounds__(256) void splitk_sum_kernel(const float *__restrict__ part, uint16_t *__restrict__ out,
                                                         size_t plane)
{
    const size_t e = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (e >= plane) return;                             // plane is a multiple of 8
    float4_t p[S];
#pragma unroll
    for (int sp = 0; sp < S; ++sp) p[sp] = *(const float4_t *)(part + sp * plane + e);
    float4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int sp = 0; sp < S; ++sp) acc += p[sp];
    *(u16x4_t *)(out + e) = u16x4_t{to16<BF16>(acc[0]), to16<BF16>(acc[1]), to16<BF16>(acc[2]), to16<BF16>(acc[3])};
}

// The same sum where t (or u) was formed beside the GEMM: SIDE_ROWS token rows and 1024 columns per workgroup.  Their partial
// sums of t are added first, rounded as t is, written once (by the first column block) and multiplied with B [N, R]
// (forward) or A [R, K] (backward); sc * t is rounded to 16 bits, as in the extra contraction steps of an unsplit GEMM.
// Bound by the latency of its chain (partial sums, barrier, t, barrier) and the planes' bytes; the planes are requested ahead of
// the partial sums.  B is read once for the SIDE_ROWS rows, the partial sums, a few KB per row, by every column block.  One row
// per workgroup instead of two: 256 x 4096 <- 4096, rank 8 28.3 -> 27.5 us, but 64 rows 18.6 -> 19.9; four: 29.6 and 21.2.
constexpr int SIDE_ROWS = 2;
struct SideSum {
    const float *part, *side;
    const uint16_t *w;        // B (forward) or A (backward)
    uint16_t *out, *t;        // t may be NULL
    int M, NO, P;             // P: partial sums of t per token row
    float sc;
};
template <bool BF16, bool TRANS, int S, int R>
__global__ __launch_bounds__(256) void splitk_sum_side_kernel(const SideSum a)
{
    __shared__ float red[SIDE_ROWS][4][R], st[SIDE_ROWS][R];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m0 = blockIdx.y * SIDE_ROWS, col = (blockIdx.x * 256 + tid) * 4;
    const bool live = col < a.NO;
    const size_t plane = (size_t)a.M * a.NO;
    float4_t p[SIDE_ROWS][S];
#pragma unroll
    for (int i = 0; i < SIDE_ROWS; ++i)
#pragma unroll
        for (int sp = 0; sp < S; ++sp)
            if (live) p[i][sp] = *(const float4_t *)(a.part + sp * plane + (size_t)min(m0 + i, a.M - 1) * a.NO + col);
    u16x8_t wf[TRANS ? 1 : 4 * R / 8];
    u16x4_t wb[TRANS ? R : 1];
    if (live) {
        if constexpr (TRANS) {
#pragma unroll
            for (int j = 0; j < R; ++j) wb[j] = *(const u16x4_t *)(a.w + (size_t)j * a.NO + col);
        } else {
#pragma unroll
            for (int h = 0; h < 4 * R / 8; ++h) wf[h] = *(const u16x8_t *)(a.w + (size_t)col * R + 8 * h);
        }
    }
    const int n = a.P * R;
#pragma unroll
    for (int i = 0; i < SIDE_ROWS; ++i) {
        const float *src = a.side + (size_t)min(m0 + i, a.M - 1) * n;
        float v = 0.f;
        for (int f = tid; f < n; f += 256) v += src[f];         // column f % R = tid % R
#pragma unroll
        for (int d = R; d < 64; d <<= 1) v += __shfl_xor(v, d, 64);
        if (lane < R) red[i][wave][lane] = v;
    }
    __syncthreads();
    if (tid < SIDE_ROWS * R) {
        const int i = tid / R, j = tid % R;
        const uint16_t t = to16<BF16>(red[i][0][j] + red[i][1][j] + red[i][2][j] + red[i][3][j]);
        if (a.t && blockIdx.x == 0 && m0 + i < a.M) a.t[(size_t)(m0 + i) * R + j] = t;
        st[i][j] = cvt16<BF16>(to16<BF16>(a.sc * cvt16<BF16>(t)));
    }
    __syncthreads();
    if (!live) return;
#pragma unroll
    for (int i = 0; i < SIDE_ROWS; ++i) {
        if (m0 + i >= a.M) return;
        float4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int sp = 0; sp < S; ++sp) acc += p[i][sp];
#pragma unroll
        for (int j = 0; j < R; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                acc[c] = fmaf(st[i][j], cvt16<BF16>(TRANS ? wb[TRANS ? j : 0][c] : wf[TRANS ? 0 : (c * R + j) / 8][j & 7]), acc[c]);
        *(u16x4_t *)(a.out + (size_t)(m0 + i) * a.NO + col) =
            u16x4_t{to16<BF16>(acc[0]), to16<BF16>(acc[1]), to16<BF16>(acc[2]), to16<BF16>(acc[3])};
    }
}

template <bool BF16, bool TRANS, int S>
void launch_splitk_sum_side(const SideSum &a, int r, hipStream_t s)      // gemm_side_floats(): r is 8, backward 16 too
{
    const dim3 grid((unsigned)((a.NO / 4 + 255) / 256), (unsigned)((a.M + SIDE_ROWS - 1) / SIDE_ROWS)), block(256);
    if constexpr (TRANS) {
        if (r == 16) {
            QLORA_LAUNCH((splitk_sum_side_kernel<BF16, TRANS, S, 16>), grid, block, 0, s, a);
            return;
        }
    }
    QLORA_LAUNCH((splitk_sum_side_kernel<BF16, TRANS, S, 8>), grid, block, 0, s, a);
}

template <bool BF16>
void launch_splitk_sum(const float *part, uint16_t *out, size_t plane, int splits, hipStream_t s)
{
    const dim3 grid((unsigned)((plane / 4 + 255) / 256)), block(256);
    switch (splits) {                                   // gemm_splits(): 2 to 8
    case 2: QLORA_LAUNCH((splitk_sum_kernel<BF16, 2>), grid, block, 0, s, part, out, plane); break;
    case 3: QLORA_LAUNCH((splitk_sum_kernel<BF16, 3>), grid, block, 0, s, part, out, plane); break;
    case 4: QLORA_LAUNCH((splitk_sum_kernel<BF16, 4>), grid, block, 0, s, part, out, plane); break;
    case 5: QLORA_LAUNCH((splitk_sum_kernel<BF16, 5>), grid, block, 0, s, part, out, plane); break;
    case 6: QLORA_LAUNCH((splitk_sum_kernel<BF16, 6>), grid, block, 0, s, part, out, plane); break;
    case 7: QLORA_LAUNCH((splitk_sum_kernel<BF16, 7>), grid, block, 0, s, part, out, plane); break;
    default: QLORA_LAUNCH((splitk_sum_kernel<BF16, 8>), grid, block, 0, s, part, out, plane); break;
    }
}

template <int BITS, bool BF16, bool TRANS>
void launch_tiles(GemmArgs &a, uint16_t *side_out, hipStream_t s)
{
    constexpr int BM = 256, BN = 128, WM = 2, WN = 2;       // tile shape and grid of MFMA waves
    static_assert(BN == GEMM_SPLIT_BN, "gemm_splits() counts tiles of this width");
    const int NO = TRANS ? a.K : a.N, KC = TRANS ? a.N : a.K;
    a.tiles_n = (NO + BN - 1) / BN;
    a.splits = 1;
    a.kt_split = (KC + BK - 1) / BK;
    // 128-row tiles while they are one round of the 256 CUs (a CU holds one workgroup), and if they are far fewer also the
    // contraction split over several workgroups per tile.  A round of 128-row tiles takes 0.6 to 0.73 times as long as one of
    // 256-row tiles (4096 x 4096, INT4, fp16: 39 and 64 us forward, 42 and 66 backward), so two rounds of them lose to one
    // (M = 1397, 4096 x 4096, bf16 INT4, 352 tiles of 128 rows or 192 of 256: 79 and 52 us forward, 76 and 56 backward) and
    // win against two, as in fp16 four do against three: 595 tokens to 11008 columns are 430 or 258 tiles, forward from 4096
    // 99.8 -> 72.8 us, backward from 5120 121.8 -> 87.0; 1350 tokens 946 or 516, forward 162.7 -> 147.4 (bf16, whose 128-row tiles
    // are slower, 0.94 to 1.03 times as long).  With more rounds the last one is too small a part of the launch (six against four,
    // five and more: 1.04 to 1.4 times as long).  Not forward with more packed words than the 256 MB of the Infinity Cache, which the
    // third tile row reads from HBM again: four rounds 1.09 to 1.12 times as long as three (306 tokens, 34816 <- 11328, INT8: 552
    // and 493 us), up to there 0.89 to 1.01.
    if constexpr (BM == 256) {
        const int tall = (a.M + 255) / 256 * a.tiles_n, flat = (a.M + 127) / 128 * a.tiles_n;
        const bool cached = (long long)NO * KC * BITS <= (2ll << 30);
        if (flat <= 256 || (flat <= 512 && tall > 256) || (!BF16 && flat <= 1024 && tall > 512 && (TRANS || cached))) {
            a.tiles_m = (a.M + 127) / 128;
            if constexpr (TRANS) {
                if (a.keep) {           // the masked epilogue needs the whole contraction in one workgroup
                    launch_variant<BITS, BF16, TRANS, 128, BN, WM, WN, true>(a, s);
                    return;
                }
            }
            const int splits = a.part ? gemm_splits(a.M, NO, KC) : 1;
            if (splits > 1) {
                a.splits = splits;
                a.kt_split = (a.kt_split + splits - 1) / splits;
            }
            if (splits > 1 && a.side_r > 0) {
                a.side_p = min(a.tiles_n, a.kt_split);
                launch_variant<BITS, BF16, TRANS, 128, BN, WM, WN, false, false, true>(a, s);
                const SideSum q{a.part, a.side, a.ext_w, a.out, side_out, a.M, NO, splits * a.side_p, a.sc};
                switch (splits) {
                case 2: launch_splitk_sum_side<BF16, TRANS, 2>(q, a.side_r, s); break;
                case 3: launch_splitk_sum_side<BF16, TRANS, 3>(q, a.side_r, s); break;
                case 4: launch_splitk_sum_side<BF16, TRANS, 4>(q, a.side_r, s); break;
                case 5: launch_splitk_sum_side<BF16, TRANS, 5>(q, a.side_r, s); break;
                case 6: launch_splitk_sum_side<BF16, TRANS, 6>(q, a.side_r, s); break;
                case 7: launch_splitk_sum_side<BF16, TRANS, 7>(q, a.side_r, s); break;
                default: launch_splitk_sum_side<BF16, TRANS, 8>(q, a.side_r, s); break;
                }
                return;
            }
            launch_variant<BITS, BF16, TRANS, 128, BN, WM, WN>(a, s);
            if (splits > 1) launch_splitk_sum<BF16>(a.part, a.out, (size_t)a.M * NO, splits, s);
            return;
        }
    }
    a.tiles_m = (a.M + BM - 1) / BM;
    if constexpr (TRANS) {
        if (a.keep) {
            launch_variant<BITS, BF16, TRANS, BM, BN, WM, WN, true>(a, s);
            return;
        }
    }
    // 256 x 256 tiles, by the symmetric-wave kernel, where they take at most half the rounds of the 256 x 128 tiles or fill
    // theirs nearly (5-11 % less time at M = 4096 and 8192); a launch of 344 tiles, two rounds of which the second is a third
    // full, is 10 % slower than the 688 smaller tiles in three, and 1026 tiles, five rounds, 6 % slower than 2052 in nine.
    // One round of them, up to 4/5 full, beside two of the smaller tiles: fp16 forward 0.83 to 0.99 times as long (1110 tokens,
    // 8192 <- 2048, INT3 55 -> 51 us), fp16 backward with 2 and 4 bits 0.93 to 0.98 (738 tokens, 13824 <- 11008: 260 -> 230 us);
    // 0.95 to 1.04 where it is fuller, where the backward pass unpacks 3 or 8 bits, and in bf16.  Contractions of 128 to 768: 105
    // of 108 calls 0.75 to 0.99 times as long, three 1.01 to 1.04 (1740 tokens, 7216 <- 384, INT4, the most); 1040 calls of other
    // lengths 0.65 to 1.03, seven with 8 bits forward up to 1.08 (129 tokens, 34048 <- 12096).
    // "Nearly full" is 4/5 of a round where a tile's fixed part counts most: a contraction of one stage (the smaller tiles 0.99 to 1.10
    // times as long), and ranks above 32, whose rows the smaller tiles fetch after their last stage only, up to 32 stages (1.06 to
    // 1.44 times as long up to 8: 804 tokens, 52800 <- 64, rank 64 48 and 65 us; 0.99 to 1.10 up to 32).  Elsewhere it is 17/20: between
    // the two the smaller tiles take 0.77 to 1.06 times as long, 0.93 in the mean of 377 calls (one 1.15: 6149 tokens, 6208 <- 384).
    {
        const int tn = (NO + 255) / 256, tiles = a.tiles_m * tn, rounds = (tiles + 255) / 256;
        const int small_rounds = (a.tiles_m * a.tiles_n + 255) / 256;
        const bool half = 2 * rounds <= small_rounds, full = tiles * 10 >= rounds * 256 * 8;
        const bool fixed = KC <= BK || (a.r > 32 && KC <= 32 * BK);
        bool take;
        if (tiles >= 256) take = half ? !BF16 || full : (fixed ? full : tiles * 20 >= rounds * 256 * 17);
        else take = half && !full && !BF16 && (!TRANS || BITS == 2 || BITS == 4);
        if (take) {
            a.tiles_n = tn;
            launch_variant<BITS, BF16, TRANS, 256, 256, 2, 4, false, true>(a, s);
            return;
        }
    }
    launch_variant<BITS, BF16, TRANS, BM, BN, WM, WN>(a, s);
}

// Multiplier m with umulhi(q, m) == q / (G/32) for every q < 2^16 (q = k/32, K < 2^21): m = floor(2^32 / d) + 1
// for d = G/32 >= 2.  d = 1 would need m = 2^32; it is encoded as 0 and the kernel then uses q itself.
inline uint32_t group_magic(int G)
{
    const uint32_t d = (uint32_t)(G / 32);
    return d == 1 ? 0u : (uint32_t)(0x100000000ull / d) + 1u;
}

template <bool TRANS>
void launch_bits_dtype(const Problem &p, GemmArgs &a, uint16_t *side_out, hipStream_t s)
{
#define QLORA_CASE(B)                                   \
    case B:                                             \
        if (p.bf16) launch_tiles<B, true, TRANS>(a, side_out, s); \
        else launch_tiles<B, false, TRANS>(a, side_out, s);       \
        break
    switch (p.bits) {
        QLORA_CASE(2);
        QLORA_CASE(3);
        QLORA_CASE(4);
    default:
        if (p.bf16) launch_tiles<8, true, TRANS>(a, side_out, s);
        else launch_tiles<8, false, TRANS>(a, side_out, s);
        break;
    }
#undef QLORA_CASE
}

}  // namespace

// The arguments of a launch whose t (or u) is formed beside the GEMM: the adapter takes no part in the GEMM itself
static void take_side(GemmArgs &a, const void *side_w, float *side)
{
    a.side_w = (const uint16_t *)side_w;
    a.side = side;
    a.side_r = a.r;
    a.r = 0;
}

void launch_fwd_mfma(const Problem &p, const void *x, const uint32_t *packed, const void *scales, const uint8_t *zeros,
                     const void *t, const void *B, void *y, float *part, hipStream_t s, const void *A, void *t_out,
                     float *side)
{
    GemmArgs a{(const uint16_t *)x, packed, (const uint16_t *)scales, zeros, (const uint16_t *)t, (const uint16_t *)B,
               (uint16_t *)y, p.M, p.N, p.K, p.G, p.r, p.sc, 0, 0, group_magic(p.G), part, 1, 0, nullptr, 0.f,
               nullptr, nullptr, 0, 0};
    if (side) take_side(a, A, side);
    launch_bits_dtype<false>(p, a, (uint16_t *)t_out, s);
}

void launch_bwd_dx_mfma(const Problem &p, const void *dy, const uint32_t *packed, const void *scales,
                        const uint8_t *zeros, const void *u, const void *A, void *dx, float *part,
                        const uint32_t *keep, float keep_scale, hipStream_t s, const void *B, void *u_out, float *side)
{
    GemmArgs a{(const uint16_t *)dy, packed, (const uint16_t *)scales, zeros, (const uint16_t *)u, (const uint16_t *)A,
               (uint16_t *)dx, p.M, p.N, p.K, p.G, p.r, p.sc, 0, 0, group_magic(p.G), part, 1, 0,
               p.r > 0 ? (const uint8_t *)keep : nullptr, p.sc * keep_scale, nullptr, nullptr, 0, 0};
    if (side) take_side(a, B, side);
    launch_bits_dtype<true>(p, a, (uint16_t *)u_out, s);
}

}  // namespace qlora
