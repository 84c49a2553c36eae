// bf16 GEMM  C[M, N] = A[M, K] * W[N, K]^T  for gfx950 with fused epilogues.
//
// Shape of the problem.  A chunk has at most a few thousand rows (M = n_tokens) while N is the layer
// width, so the work per compute unit is small: about 44 K outputs for the gate/up projection of a
// 512-token chunk on 256 CUs.  The kernel therefore gives a CU one tall tile at a time, up to 256 or 288 rows by
// up to 256 columns, held entirely in accumulators (the register file of a CU is 512 KB), and picks the tile so that
// its grid fills whole rounds of CUs (pick_tall).  The larger the tile, the lower the L2 -> LDS traffic per flop.  Chunks of up to
// 128 rows take tiles of 32 to 128 rows, as narrow as one round of workgroups allows.
//
//   * Waves form a WM x WN grid over the tile; a wave owns BMB/WM row blocks x NB/WN column blocks of
//     32 x 32.  Measured at M = 512: eight waves (4 x 2, two per SIMD, 64 x 96 each) beat four waves of
//     128 x 96 (2 x 2) by 20 % although the latter read a third less from LDS: with one wave per SIMD
//     every wait of that wave idles the matrix pipe, with two the other wave's MFMAs cover it.
//     (The 16x16x32 form sustains only ~70 % of the 32x32x16 rate on this chip, measured.)
//   * K advances in stages of 32 through an LDS ring (as many slots as fit, at most 8) filled by direct global->LDS loads
//     (16 bytes per lane, no register staging).  A stage holds two K/16 sub-steps; the fragments of
//     one sub-step are read from LDS while the matrix cores work on the other.
//   * LDS rows are 64 bytes (32 bf16).  Four rows form a 256-byte super-row; chunk c of row r sits at
//     16-byte slot ((4*(r&3) + c) ^ ((r>>2)&3)) of super-row r>>2, so that 16 consecutive rows read at
//     one chunk column touch all 64 banks exactly once.
//   * Both operands are stored pre-tiled as [rows/32 row blocks][K/32 stages][2 KB], each 2 KB block being
//     the LDS image of its 32 rows x 32 columns, swizzle included (W at stage creation, activations by
//     the kernels that produce them).  A wave-wide load instruction then copies 1 KB of consecutive
//     bytes, which the L2 -> LDS path moves about three times faster than 16 pieces of 64 bytes, and a
//     workgroup streams each row block of W front to back in long sequential bursts.
//   * Workgroup ids are decoded so that the tiles sharing a slice of W run on the same XCD (same L2).
//   * The epilogues that write bf16 rows (QKV with rotary embedding and cache append, gate/up with SwiGLU) compute the
//     transposed product W A^T instead: the fragments are the same registers, only the MFMA's operand order changes,
//     and a lane then holds 16 output features of one token instead of 16 tokens of one feature.  With the weight
//     rows ordered for it at pack time a lane finishes its outputs alone (rotary partners, gate and up of a feature
//     sit in the same lane) and writes 16-byte pieces straight from registers.  The earlier epilogues went through a
//     wave-private LDS strip behind a workgroup barrier; measured at 512 rows: gate/up 85.8 -> 83.0 us, QKV unchanged
//     (its epilogue is bound by draining 16.7 MB of scattered 16-byte stores, with or without the strip).
//
// MFMA 32x32x16 bf16 operand layout (lane = 32*hh + c):
//   A: lane supplies A[m = c][k = 8*hh + e], e < 8;  B: lane supplies B[k = 8*hh + e][n = c];
//   D: lane holds D[m = 8*(i/4) + 4*hh + (i%4)][n = c] in register i < 16.
#include <cstdio>
#include <type_traits>
#include <utility>

#include "bf16_common.h"

namespace jup {
namespace {

constexpr int G_BK = 32;

constexpr int kLdsBudget = 160 * 1024;

// HALF: the last column block of the tile is half a block of W (see HalfTile)
template <int BMB, int NB, int WM, int WN, bool HALF = false>
struct Shape {
    static constexpr int BM = 32 * BMB;             // rows of the tile: 256 for prefill-sized chunks, 128, 64 or 32 for
                                                    // short ones (a short chunk is bound by streaming the weights:
                                                    // MFMAs on rows that do not exist would only slow that down)
    static constexpr int NBW = NB / WN;             // column blocks per wave
    static constexpr int MBW = BMB / WM;            // row blocks per wave
    static constexpr int EXTRA = BMB % WM;          // a row block more, of which every wave takes one column block
    static constexpr int WAVES = WM * WN;
    static constexpr int COLS = 32 * NB - (HALF ? 16 : 0);
    static constexpr int ROWS = BM + COLS;          // LDS rows per stage: A rows then W rows
    static constexpr int STAGE_BYTES = ROWS * 64;
    static constexpr int LOADERS = WAVES;           // every wave fetches its share of a stage between its MFMAs
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int NL = ROWS / 16;            // 1 KB load units (16 rows) per stage, dealt round-robin to the loading waves
    static constexpr int LPW = (NL + LOADERS - 1) / LOADERS;  // load instructions per stage of the waves that have the most
    static constexpr int REM = NL % LOADERS;        // loading waves below REM issue LPW loads, the others LPW - 1 (0: all LPW)
    static_assert(NB % WN == 0 && EXTRA <= 1, "tile does not split evenly over the waves");
    // as many ring slots as LDS holds (at most 8: the in-flight count must fit the 6-bit vmcnt)
    static constexpr int STAGES = kLdsBudget / STAGE_BYTES > 8 ? 8 : kLdsBudget / STAGE_BYTES;
    // tiles that chunks of up to 16 rows take: the factors of rows with partial sums of squares, behind the ring
    static constexpr bool ROW_SCALE = BMB <= 2;
    static constexpr int RING_BYTES = STAGES * STAGE_BYTES;
    static constexpr int LDS_BYTES = RING_BYTES + (ROW_SCALE ? kMaxProjectRows * 4 : 0);
    static_assert(STAGES >= 4 && (STAGES - 2) * LPW < 64, "ring depth");
};

__device__ inline f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// s_waitcnt with only the vector-memory counter constrained.
template <int N>
__device__ inline void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | 0x0F70);
}
__device__ inline void wait_lgkmcnt0() { __builtin_amdgcn_s_waitcnt(0xC07F); }  // lgkmcnt(0), others free

// Instruction-order hints.  A burst of LDS reads or of global->LDS loads keeps the wave's issue port busy
// for hundreds of cycles while the matrix pipe drains, so memory instructions are dealt out one (or two)
// after each MFMA.  Masks: 0x008 MFMA, 0x100 LDS read, 0x010 vector memory.
template <int MASK>
__device__ __forceinline__ void sched_one() {
    __builtin_amdgcn_sched_group_barrier(MASK, 1, 0);
}
template <int DS, int LO, int HI>
__device__ __forceinline__ void sched_mem_ops() {  // memory ops number LO..HI-1 of a half: LDS reads first
    if constexpr (LO < HI) {
        if constexpr (LO < DS) sched_one<0x100>();
        else sched_one<0x010>();
        sched_mem_ops<DS, LO + 1, HI>();
    }
}
// One half stage: M MFMAs with DS LDS reads and VM vector-memory loads spread evenly behind them.
template <int M, int DS, int VM, int m = 0>
__device__ __forceinline__ void sched_half() {
    if constexpr (m < M) {
        sched_one<0x008>();
        sched_mem_ops<DS, (DS + VM) * m / M, (DS + VM) * (m + 1) / M>();
        sched_half<M, DS, VM, m + 1>();
    }
}

// Waits until at most g of this wave's load groups (one group = the CNT loads of one stage) are still in
// flight; more than ST - 3 are never allowed to be.
template <int ST, int CNT>
__device__ __forceinline__ void wait_groups(int g) {
    if (g >= ST - 3) wait_vmcnt<(ST - 3) * CNT>();
    else if (g == 4) wait_vmcnt<(ST > 7 ? 4 : 0) * CNT>();
    else if (g == 3) wait_vmcnt<(ST > 6 ? 3 : 0) * CNT>();
    else if (g == 2) wait_vmcnt<(ST > 5 ? 2 : 0) * CNT>();
    else if (g == 1) wait_vmcnt<1 * CNT>();
    else wait_vmcnt<0>();
}

// Fragments of one K/16 sub-step of a wave: MB row blocks (the extra one last), NB column blocks.
template <int MB, int NB>
struct Frags {
    bf16x8 a[MB];
    bf16x8 b[NB];
};

// Tiles that end in half a column block.  Two neighbours share three blocks: the even one has the first and half of the second,
// the odd one the other half and the third.  A half is the packed rows 8 h .. 8 h + 7 and 16 + 8 h .. of the block, half of
// the registers of every lane of the epilogue, so that rotary partners stay together; LDS holds the 16 rows one after
// the other, and the MFMA has every row twice (rows c and c ^ 8 of its operand).
struct HalfTile {
    int full, half, h;  // blocks of W, and which half of the second
    __device__ __forceinline__ explicit HalfTile(int nt) : full(nt / 2 * 3 + nt % 2 * 2), half(nt / 2 * 3 + 1), h(nt & 1) {}
};

// The tile of row blocks mt * BMB .. and columns [n0, n_end) (K split: split).
// FACTOR: the results of a row may have to be multiplied by its 1 / rms.  A template parameter because on the tall tiles of
// long chunks, which never need it, the test alone cost the 512-row launches 1 %.
template <int BMB, int NB, int WM, int WN, int EPI, bool FACTOR, bool HALF = false>
__device__ __forceinline__ void gemm_tile(const GemmArgs& a, unsigned char* smem, int split, int mt, int n0, int n_end) {
    using S = Shape<BMB, NB, WM, WN, HALF>;
    static_assert(!HALF || (NB == 2 && WN == 2 && WM == 2 && BMB == 2 && EPI != EPI_PARTIAL), "the last column block belongs to waves of its own");
    constexpr int G_BM = S::BM;
    constexpr int NBW = S::NBW, MBW = S::MBW, EXTRA = S::EXTRA;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;  // wave owns row blocks [wm MBW, +MBW) x column blocks [wn NBW, +NBW)
    const int m0 = mt * G_BM;
    const int KT = a.kt_per_split;

    // ---- global -> LDS load slots of this wave --------------------------------------------------------
    // A stage is ROWS/4 super-rows of 256 bytes (4 rows of 64 bytes), A rows first, then W rows.  One load
    // instruction moves four super-rows: lane i's 16 bytes land at byte 16 i of the instruction's 1 KB.
    // Unit j of a stage = rows [16j, 16j+16) of the LDS image = 1 KB that is contiguous in the tiled operand
    // too (half a 2 KB block), so one load instruction is a wave-uniform base plus 16 bytes per lane.  Unit
    // j = q * LOADERS + wave belongs to that wave; HAS_LAST says whether its unit q = LPW-1 exists.
    const char* ubase[S::LPW];
    const int kt_total = a.K / G_BK;
    const unsigned lane16 = lane * 16;
    const HalfTile ht(HALF ? n0 / S::COLS : 0);
    // (of a unit of W: half a block is 512 bytes out of either KB of the block)
    const unsigned w_lane16 = HALF && wave == S::LOADERS - 2 ? lane16 + ht.h * 512 + (lane >> 5) * 512 : lane16;
#pragma unroll
    for (int q = 0; q < S::LPW; ++q) {
        const int j = min(q * S::LOADERS + wave, S::NL - 1);
        const u16* base;
        int blk;
        if (j < G_BM / 16) {
            blk = min(m0 / 32 + (j >> 1), (a.M + 31) / 32 - 1);  // blocks past M repeat the last one
            base = a.A;
        } else {
            blk = min(n0 / 32 + ((j - G_BM / 16) >> 1), a.N / 32 - 1);  // blocks past N repeat the last one
            if (HALF) blk = min(j - G_BM / 16 < 2 ? ht.full : ht.half, a.N / 32 - 1);
            base = a.W;
        }
        ubase[q] = uniform_ptr((const char*)(base + ((size_t)blk * kt_total + (size_t)split * KT) * 1024 + (j & 1) * 512));
    }
    // (the 64-row tiles and the four-wave 128-row tiles are the ones short chunks run; the eight-wave 128-row tiles serve
    // 512-row chunks, whose K loop does not afford the branch below: 2 us per launch, measured)
    constexpr bool kShortChunkTile = BMB <= 2 || (BMB == 4 && WM * WN == 4);
    const bool nt_weights = a.m_tiles == 1 && !a.shared_gpu;
    // Those tiles leave the rows past M out (LDS holds anything there, which reaches the accumulators of those rows alone): a CU
    // takes operands at about 50 GB/s, and 40 rows in a 64-row tile spent a fifth of that on rows that do not exist.  (A unit
    // past M keeps one lane, 16 bytes of its clamped block: every load has to count for the waits.)  Whole layers, before -> after
    // (same bits): 7B 40 rows 100.8 -> 96.0 us, 100 rows 135.0 -> 128.9, 5 rows 83.5 -> 82.5, 64 rows 103.6 -> 103.4; 13B 40 rows
    // 136.9 -> 131.4, 128 rows 182.4 -> 182.1.  (A ring of 16 stages instead of 8, now that a stage of few rows is short: 5 rows
    // 83.0 -> 85.6.)
    const unsigned ring = __builtin_amdgcn_readfirstlane(lds_byte_address(smem));
    unsigned long long lanes[S::LPW];
    if constexpr (kShortChunkTile) {
#pragma unroll
        for (int q = 0; q < S::LPW; ++q) {
            const int j = q * S::LOADERS + wave;
            lanes[q] = j < G_BM / 16 ? row_lanes(a.M, m0 + j * 16) : ~0ull;
        }
    }
    auto issue_one = [&](int q, int stage, int kt) {
        const char* at = uniform_ptr(ubase[q] + (size_t)kt * 2048);
        const int unit = q * S::LOADERS + wave;
        const auto* src = (const __attribute__((address_space(1))) void*)(at + (HALF ? w_lane16 : lane16));
        auto* dst = (__attribute__((address_space(3))) void*)(smem + stage * S::STAGE_BYTES + unit * 1024);
        // A chunk of up to 128 tokens alone on the chip streams every weight exactly once (one M tile): its weight units
        // are fetched with the non-temporal hint, so that the stream does not push the KV cache and the activations
        // out of L2 and the last-level cache.  Measured on the 7B shapes: gate/up at 5 rows 36.1 -> 32.5 us, the
        // attention launch behind the projections 15.0 -> 12.4 us, a 5-token call 6.59 -> 5.95 ms per 8 branches, 128-token
        // chunks +6 %.  Not for the tiles of longer chunks (the branch costs their K loop 2.5 % and a second M tile re-reads
        // the weights from L2) and not inside an overlapped call (the other chunks find the weights in the caches).
        // (which of the two a unit is folds to a constant where the waves divide the units of the rows)
        constexpr int ROW_UNITS = G_BM / 16;
        const bool rows = (q + 1) * S::LOADERS <= ROW_UNITS || (q * S::LOADERS < ROW_UNITS && unit < ROW_UNITS);
        if (kShortChunkTile && rows) load_to_lds_16(at, lane16, ring + stage * S::STAGE_BYTES + unit * 1024, lanes[q]);
        else if (kShortChunkTile && nt_weights) __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 2);
        else __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 0);
    };
    auto issue = [&](auto has_last, int stage, int kt) {
        constexpr int CNT = S::REM == 0 || decltype(has_last)::value ? S::LPW : S::LPW - 1;
#pragma unroll
        for (int q = 0; q < CNT; ++q) issue_one(q, stage, kt);
    };

    // Up to 16 rows that come with partial sums of squares: those are loaded ahead of the ring's first stages and added up
    // behind the K loop.
    constexpr bool ROW_SCALE = S::ROW_SCALE && EPI != EPI_PARTIAL;
    float* scale_of_row = (float*)(smem + S::RING_BYTES);
    RowScale<S::WAVES> sq;
    const bool scaled = ROW_SCALE && a.ssq;
    if (scaled) sq.begin(a.ssq, a.M, wave, lane, a.K);
    // 1 / rms of this lane's token in every row block of the wave, where the rows of A are not normalised
    float factor[MBW];
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb) factor[mb] = 1.0f;
    if (FACTOR && a.row_factor)
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) factor[mb] = a.row_factor[min(m0 + (wm * MBW + mb) * 32 + (lane & 31), a.M - 1)];

    // ---- LDS -> register fragment addresses -------------------------------------------------------------
    // Fragment row = 32*block + c (c = lane & 31), chunk = 2*ks + hh.  Block bases are multiples of 32,
    // so the swizzle term depends on the lane and on ks only: address = lane part + constant.
    const int c = lane & 31, hh = lane >> 5;
    int lane_off[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
        lane_off[ks] = (c >> 2) * 256 + ((((c & 3) << 2) + 2 * ks + hh) ^ ((c >> 2) & 3)) * 16;
    const int a_base = wm * MBW * 2048, b_base = G_BM * 64 + wn * NBW * 2048;
    int b_lane_off[2] = {lane_off[0], lane_off[1]};
    if (HALF && wn == 1)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
            b_lane_off[ks] = ((c >> 4) * 2 + ((c & 7) >> 2)) * 256 + ((((c & 3) << 2) + 2 * ks + hh) ^ (2 * ht.h + ((c & 7) >> 2))) * 16;
    // Tiles with an extra row block: the waves of a column range begin at different columns of it, and each multiplies the
    // extra rows by the columns it begins at (b[0]; more waves than columns: some for nothing).
    const int first_nb = EXTRA ? wm % NBW : 0;
    auto column = [&](int nb) { return EXTRA ? (nb + first_nb >= NBW ? nb + first_nb - NBW : nb + first_nb) : nb; };
    using F = Frags<MBW + EXTRA, NBW>;
    // Read number t of a sub-step, in the order the MFMAs need them: a[0], b[0], the other a, the other b, the extra a.
    constexpr int READS = MBW + NBW + EXTRA;
    auto load_frag_one = [&](F& f, int stage, int ks, int t) {
        const unsigned char* sb = smem + stage * S::STAGE_BYTES + lane_off[ks];
        if (t == 0) f.a[0] = *(const bf16x8*)(sb + a_base);
        else if (HALF) f.b[0] = *(const bf16x8*)(smem + stage * S::STAGE_BYTES + b_lane_off[ks] + b_base);
        else if (t == 1) f.b[0] = *(const bf16x8*)(sb + b_base + column(0) * 2048);
        else if (t < MBW + 1) f.a[t - 1] = *(const bf16x8*)(sb + a_base + (t - 1) * 2048);
        else if (t < MBW + NBW) f.b[t - MBW] = *(const bf16x8*)(sb + b_base + column(t - MBW) * 2048);
        else f.a[MBW + EXTRA - 1] = *(const bf16x8*)(sb + (BMB - 1) * 2048);
    };
    auto load_frags = [&](F& f, int stage, int ks) {
#pragma unroll
        for (int t = 0; t < READS; ++t) load_frag_one(f, stage, ks, t);
    };

    f32x16 acc[MBW][NBW], acc_extra;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_extra[r] = 0.f;
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mb][nb][r] = 0.f;


    // ---- prologue: fill all but one slot of the ring, fetch the first fragments -----------------------------
    constexpr int ST = S::STAGES;
    F f0, f1;
    // The whole K loop exists once per load count (waves with and without the last load unit), so that no
    // load sits under a condition: a branch inside the loop would also cut it into scheduling regions.
    auto k_loop = [&](auto has_last) {
    constexpr int CNT = S::REM == 0 || decltype(has_last)::value ? S::LPW : S::LPW - 1;  // loads per stage
#pragma unroll
    for (int s = 0; s < ST - 1; ++s)
        if (s < KT) issue(has_last, s, s);
    if (KT >= ST - 1) wait_vmcnt<(ST - 2) * CNT>();  // stage 0 landed, the others may be in flight
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    load_frags(f0, 0, 0);
    wait_lgkmcnt0();

    // Stage kt.  On entry f0 holds its sub-step 0.  The barrier at the top publishes stage kt+1 (whose
    // sub-step 0 is prefetched in the second half) and retires stage kt-1, which every wave finished
    // reading half a stage ago; that slot is refilled with stage kt+ST-1 right away.  The barrier falls
    // while the previous stage's last MFMAs are still in the pipe, and each half issues 2 + NB fragment
    // reads under 2 * NB MFMAs.
    //
    // STEADY stages (kt + ST - 1 < KT) have no conditions at all; the main loop runs ST of them per trip
    // with the ring slots as compile-time constants, so a trip is one straight run of instructions (taken
    // branches starve the MFMA pipe: the instruction buffer refills while nothing issues).
    // REFILL: the slot behind (pstage) is reloaded with stage kt+ST-1.  LAST: no stage follows (nothing is
    // prefetched and nothing waited for at the top).
    auto do_stage = [&](auto refill, auto last, int kt, int stage, int pstage, int nstage) {
        constexpr bool REFILL = decltype(refill)::value, LAST = decltype(last)::value;
        if (REFILL) {
            wait_vmcnt<(ST - 3) * CNT>();
            __builtin_amdgcn_s_barrier();
        } else if (!LAST) {
            wait_groups<ST, CNT>(KT - 1 - (kt + 1));  // stages issued after kt+1 may stay in flight
            __builtin_amdgcn_s_barrier();
        }
        // Memory instructions are dealt out between the MFMAs, and the compiler's scheduler is fenced at
        // every step: a burst of LDS reads or global->LDS loads would hold the wave's issue port while the
        // matrix pipe runs dry.  Fragment reads come first in a half, the global->LDS loads after them
        // (spreading the loads among the reads, or keeping the last MFMAs free of both, measured slower).
        constexpr int NM = MBW * NBW + EXTRA;
        constexpr int V1 = REFILL ? (CNT + 1) / 2 : 0;
        constexpr int V2 = REFILL ? CNT - V1 : 0;
        auto half = [&]<int... M>(std::integer_sequence<int, M...>, auto second) {
            constexpr bool SECOND = decltype(second)::value;
            constexpr int RD = SECOND && LAST ? 0 : READS;
            constexpr int V = SECOND ? V2 : V1;
            constexpr int TOT = RD + V;
            auto step = [&](auto mi) {
                constexpr int m = decltype(mi)::value;
                const F& use = SECOND ? f1 : f0;
                // QKV and gate/up compute the TRANSPOSED block (W A^T: the weight fragment as the MFMA's first operand),
                // so that a lane ends up with 16 output features of ONE token: see the epilogues
                constexpr bool X = m == MBW * NBW;
                constexpr int mb = X ? MBW : m % MBW, nb = X ? 0 : m / MBW;
                f32x16& sum = X ? acc_extra : acc[X ? 0 : mb][nb];
                if constexpr (EPI == EPI_PARTIAL) sum = mfma32(use.a[mb], use.b[nb], sum);
                else sum = mfma32(use.b[nb], use.a[mb], sum);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (TOT > 0) {
#pragma unroll
                    for (int t = TOT * m / NM; t < TOT * (m + 1) / NM; ++t) {
                        if (t >= RD) {
                            issue_one((SECOND ? V1 : 0) + t - RD, pstage, kt + ST - 1);
                        } else {
                            if (SECOND) load_frag_one(f0, nstage, 0, t);
                            else load_frag_one(f1, stage, 1, t);
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            (step(std::integral_constant<int, M>{}), ...);
        };
        half(std::make_integer_sequence<int, NM>{}, std::false_type{});
        half(std::make_integer_sequence<int, NM>{}, std::true_type{});
        // f0 (next stage) has had the last MFMAs to arrive; waiting here keeps the next stage's reads out of
        // the wait and leaves no LDS read of this wave outstanding at the barrier.
        wait_lgkmcnt0();
    };
    int kt = 0;
    for (; kt + 2 * ST - 1 <= KT; kt += ST) {  // ST refilling stages per trip, slots as compile-time constants
        [&]<int... I>(std::integer_sequence<int, I...>) {
            (do_stage(std::true_type{}, std::false_type{}, kt + I, I, (I + ST - 1) % ST, (I + 1) % ST), ...);
        }(std::make_integer_sequence<int, ST>{});
    }
    // The rest, with the slots as run-time values: the remaining refilling stages, the stages that only drain
    // the ring, and the last one.  One loop per kind (a single loop that branches between them makes the
    // compiler shuffle all accumulators at every merge).
    int stage = 0;
    auto next_slot = [&](int sl) { return sl + 1 == ST ? 0 : sl + 1; };
    auto prev_slot = [&](int sl) { return sl == 0 ? ST - 1 : sl - 1; };
    for (; kt + ST - 1 < KT; ++kt, stage = next_slot(stage))
        do_stage(std::true_type{}, std::false_type{}, kt, stage, prev_slot(stage), next_slot(stage));
    for (; kt + 1 < KT; ++kt, stage = next_slot(stage))
        do_stage(std::false_type{}, std::false_type{}, kt, stage, prev_slot(stage), next_slot(stage));
    if (kt < KT) do_stage(std::false_type{}, std::true_type{}, kt, stage, prev_slot(stage), next_slot(stage));
    };
    if constexpr (S::REM == 0) {
        k_loop(std::true_type{});
    } else {
        if (wave < S::REM) k_loop(std::true_type{});
        else k_loop(std::false_type{});
    }

    // ---- epilogues ---------------------------------------------------------------------------------------
    // Lane (c, hh) holds, for a block of rows row0 .. and columns col .., column col + c and rows row0 + 8*(i/4) + 4*hh + (i%4).
    constexpr int WROWS = 32 * MBW;  // rows of this wave
    const int nw0 = n0 + wn * NBW * 32;  // first column of this wave
    if constexpr (ROW_SCALE) {
            if (scaled) {
                sq.finish(scale_of_row, a.M, wave, lane, a.K, a.rms_eps);
                __syncthreads();
#pragma unroll
                for (int mb = 0; mb < MBW; ++mb) factor[mb] = scale_of_row[min(wm * WROWS + mb * 32 + c, kMaxProjectRows - 1)];
            }
    }

    if constexpr (EPI == EPI_PARTIAL) {
        static_assert(!EXTRA, "partial sums have no tile with an extra row block");
        const int row_base = m0 + wm * WROWS + 4 * hh;
        float* pbase = a.partial + (size_t)split * a.M * a.N + nw0 + c;
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) {
            if (nw0 + nb * 32 + c >= n_end) continue;
#pragma unroll
            for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int m = row_base + mb * 32 + 8 * (i >> 2) + (i & 3);
                    if (m < a.M) pbase[(size_t)m * a.N + nb * 32] = acc[mb][nb][i];
                }
        }
        return;
    }
    // (the arguments these read are copied into each of them: read through the reference or out of an enclosing scope between
    // stores they are read again for every block, under its condition, and the addresses made of them as well: QKV of 1536 rows of d_model
    // 512 17.2 us instead of 16.6)
    const int cols_end = HALF ? a.N : n_end;
    // Transposed block: lane (c, hh) holds token m = row c of the row block and the packed weight rows 8*(i/4) + 4*hh + (i%4)
    // of the 32-row block of W.  The pack kernel orders those rows so that a lane's registers 0..7 are the gate projections of 8
    // consecutive features and 8..15 their up projections (block nb = features 16 nb .. 16 nb + 15, lanes of half hh the
    // features 8 hh .. 8 hh + 7 of them).  A lane therefore finishes 8 outputs of one token by itself and stores them as
    // one 16-byte chunk of the tiled activation layout: no exchange between lanes, no LDS, no barrier.
    // (half a block: registers 0 .. 3 and 8 .. 11, features 4 h .. of those)
    auto swiglu_blocks = [&](auto half) __attribute__((always_inline)) {
        constexpr int PAIRS = decltype(half)::value ? 2 : 4;
        const int M = a.M, stages = a.N >> 6;
        u16* const act = a.act;
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) {
            const int col = HALF ? (PAIRS == 2 ? ht.half : ht.full) * 32 : nw0 + column(nb) * 32;
            if (col >= cols_end) continue;
            const int chunk = (col >> 4) + hh;  // 16-byte chunk of the output row: features 8 * chunk ..
#pragma unroll
            for (int mb = 0; mb < MBW + (EXTRA && nb == 0); ++mb) {
                const bool extra = mb == MBW;
                if (extra && wm >= NBW) continue;
                const int m = (extra ? m0 + (BMB - 1) * 32 : m0 + wm * WROWS + mb * 32) + c;
                if (m >= M) continue;
                const float f = FACTOR ? factor[mb] : 1.0f;
                const f32x16& sum = extra ? acc_extra : acc[extra ? 0 : mb][nb];
                std::conditional_t<PAIRS == 4, u32x4, u32x2> out;
#pragma unroll
                for (int e = 0; e < PAIRS; ++e) {
                    const float g0 = sum[2 * e] * f, g1 = sum[2 * e + 1] * f;
                    const float u0 = sum[8 + 2 * e] * f, u1 = sum[8 + 2 * e + 1] * f;
                    out[e] = pack_bf16x2(g0 * __builtin_amdgcn_rcpf(1.0f + __expf(-g0)) * u0,
                                         g1 * __builtin_amdgcn_rcpf(1.0f + __expf(-g1)) * u1);
                }
                *(decltype(out)*)(act + tiled_offset(m, chunk, stages) + (PAIRS == 2 ? 4 * ht.h : 0)) = out;
            }
        }
    };
    // Transposed block, as above.  A 32-row block of a Q or K head holds 16 rotary indices and their partners 64 further on,
    // ordered by the pack kernel so that a lane's registers 0..7 are the indices F .. F + 7 (F = 16 j + 8 hh for block j
    // of the head) and registers 8..15 their partners F + 64 ..: the lane rotates its 8 pairs and stores two 16-byte pieces.
    // A block of V holds 32 consecutive features, a lane 16 of them (16 hh ..).
    // (half a block: registers 0 .. 3 and 8 .. 11 are the indices F + 4 h .. and their partners)
    auto qkv_blocks = [&](auto half) __attribute__((always_inline)) {
        static_assert(!EXTRA || EPI != EPI_QKV, "QKV has no tile with an extra row block");
        constexpr int PAIRS = decltype(half)::value ? 2 : 4;
        const int M = a.M, d_model = a.d_model, n_heads = a.n_heads, layer = a.layer, pos0 = a.pos0;
        const KvView kv = a.kv;
        const BranchTable* branches = a.branches;
        u16* q_out = a.q_out;
        const float2* rope = a.rope;
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) {
            const int col = HALF ? (PAIRS == 2 ? ht.half : ht.full) * 32 : nw0 + column(nb) * 32;  // one (q|k|v, head, j) for all lanes
            if (col >= cols_end) continue;
            const int which = (col >= d_model) + (col >= 2 * d_model);
            const int in_model = col - which * d_model;
            const int head = in_model >> 7, j = (in_model & 127) >> 5;
            const int f_lo = (which == 2 ? 32 * j + 16 * hh : 16 * j + 8 * hh) + (PAIRS == 2 ? 4 * ht.h : 0);  // first feature of registers 0..7
            const int f_hi = which == 2 ? f_lo + 8 : f_lo + 64;                                                  // ... of registers 8..15
#pragma unroll
            for (int mb = 0; mb < MBW; ++mb) {
                const int m = m0 + wm * WROWS + mb * 32 + c;
                if (m >= M) continue;
                u16* dst;
                if (which == 0) {
                    dst = q_out + (size_t)m * d_model + head * 128;
                } else if (!branches) {
                    dst = kv_slot_bf16(kv, layer, which - 1, head, n_heads, pos0 + m);
                } else {  // row m is token t of branch b: that branch's cache and position
                    const int b = m / branches->n_tok, t = m - b * branches->n_tok;
                    dst = kv_slot_bf16(branches->kv[b], layer, which - 1, head, n_heads, branches->pos0[b] + t);
                }
                const float f = FACTOR ? factor[mb] : 1.0f;
                const f32x16& sum = acc[mb][nb];
                std::conditional_t<PAIRS == 4, u32x4, u32x2> lo, hi;
                if (which == 2) {
#pragma unroll
                    for (int e = 0; e < PAIRS; ++e) {
                        lo[e] = pack_bf16x2(sum[2 * e] * f, sum[2 * e + 1] * f);
                        hi[e] = pack_bf16x2(sum[8 + 2 * e] * f, sum[8 + 2 * e + 1] * f);
                    }
                } else {
                    const float4* rp = (const float4*)(rope + (size_t)m * 64 + f_lo);  // (cos, sin) pairs
#pragma unroll
                    for (int e = 0; e < PAIRS; ++e) {
                        const float4 cs = rp[e];  // (cos, sin) of indices f_lo + 2 e, f_lo + 2 e + 1
                        const float l0 = sum[2 * e] * f, l1 = sum[2 * e + 1] * f;
                        const float h0 = sum[8 + 2 * e] * f, h1 = sum[8 + 2 * e + 1] * f;
                        // lo' = lo cos - hi sin ; hi' = hi cos + lo sin
                        lo[e] = pack_bf16x2(l0 * cs.x - h0 * cs.y, l1 * cs.z - h1 * cs.w);
                        hi[e] = pack_bf16x2(h0 * cs.x + l0 * cs.y, h1 * cs.z + l1 * cs.w);
                    }
                }
                *(decltype(lo)*)(dst + f_lo) = lo;
                *(decltype(hi)*)(dst + f_hi) = hi;
            }
        }
    };
    auto blocks = [&](auto half) __attribute__((always_inline)) {
        if constexpr (EPI == EPI_QKV) qkv_blocks(half);
        else swiglu_blocks(half);
    };
    if (HALF && wn == 1) blocks(std::true_type{});
    else blocks(std::false_type{});
}

// REST: launches of several rounds of workgroups whose last round would leave much of the chip idle compute its columns in
// tiles of REST column blocks (and the same rows), those of the rounds before it in tiles of NB.
template <int BMB, int NB, int WM, int WN, int EPI, bool FACTOR, int REST = 0, bool HALF = false>
__global__ __launch_bounds__(64 * WM * WN) void gemm_bf16(const GemmArgs a) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    // Workgroup b runs on XCD b % 8.  Tiles are numbered so that each XCD owns one contiguous range of
    // them, M tiles fastest: the workgroups that read the same weight rows (all M tiles of an N tile) and
    // neighbouring N tiles (same activation rows) then share one L2.
    const bool rest = REST && (int)blockIdx.x >= a.wide_tiles;
    const int grid = REST ? (rest ? (int)gridDim.x - a.wide_tiles : a.wide_tiles) : (int)gridDim.x;
    const int block = REST && rest ? (int)blockIdx.x - a.wide_tiles : (int)blockIdx.x;
    const int q = grid >> 3, r = grid & 7;
    const int xcd = block & 7, local = block >> 3;
    const int tile = xcd * q + min(xcd, r) + local;
    const int grp = a.by_m.of(tile), mt = tile - grp * a.m_tiles;
    if constexpr (REST > 0) {
        if (rest) {
            const int n0 = a.n_tiles * a.n_stride + grp * 32 * REST;
            gemm_tile<BMB, REST, WM, WN, EPI, FACTOR>(a, smem, 0, mt, n0, min(n0 + 32 * REST, a.N));
            return;
        }
    }
    const int split = REST ? 0 : a.by_n.of(grp), nt = grp - split * a.n_tiles;
    const int n0 = nt * a.n_stride;
    gemm_tile<BMB, NB, WM, WN, EPI, FACTOR, HALF>(a, smem, split, mt, n0, min(n0 + a.n_stride, a.N));
}

// ---- host side: tiling policy and launch -----------------------------------------------------------------

constexpr int kCUs = 256;

int div_up(int x, int y) { return (x + y - 1) / y; }

// Row blocks of the tile for a chunk of M tokens.
int pick_row_blocks(int M) { return M > 128 ? 8 : M > 64 ? 4 : 2; }

// A launch in tiles of two widths: the N tiles of as many whole rounds of workgroups as tiles of nb column blocks fill, and the
// tiles of rest column blocks that the other columns take.
struct Rounds {
    int wide_n, rest_tiles;
};
Rounds rounds_of(int M, int N, int bmb, int nb, int rest) {
    const int m_tiles = div_up(M, 32 * bmb), wide_n = m_tiles * div_up(N, 32 * nb) / kCUs * kCUs / m_tiles;
    return {wide_n, m_tiles * div_up(max(N - wide_n * 32 * nb, 0), 32 * rest)};
}

template <int BMB, int NB, int WM, int WN, int REST, bool HALF>
constexpr int lds_bytes() {
    constexpr int wide = Shape<BMB, NB, WM, WN, HALF>::LDS_BYTES, rest = Shape<BMB, REST ? REST : NB, WM, WN>::LDS_BYTES;
    return wide > rest ? wide : rest;
}

template <int BMB, int NB, int WM, int WN, int EPI, bool FACTOR, int REST = 0, bool HALF = false>
hipError_t launch(GemmArgs a, hipStream_t s) {
    using S = Shape<BMB, NB, WM, WN, HALF>;
    a.n_stride = S::COLS;
    a.m_tiles = div_up(a.M, 32 * BMB);
    a.kt_per_split = a.K / G_BK / a.splits;
    int grid;
    if (REST) {
        const Rounds r = rounds_of(a.M, a.N, BMB, NB, REST);
        a.n_tiles = r.wide_n;
        a.wide_tiles = r.wide_n * a.m_tiles;
        grid = a.wide_tiles + r.rest_tiles;
    } else {
        a.n_tiles = div_up(a.N, a.n_stride);
        grid = a.m_tiles * a.n_tiles * a.splits;
    }
    a.by_m.set(a.m_tiles);
    a.by_n.set(a.n_tiles);
    constexpr int lds = lds_bytes<BMB, NB, WM, WN, REST, HALF>();
    hipLaunchKernelGGL((gemm_bf16<BMB, NB, WM, WN, EPI, FACTOR, REST, HALF>), dim3(grid), dim3(S::THREADS), lds, s, a);
    return hipGetLastError();
}

template <int BMB, int NB, int WM, int WN, int EPI, bool FACTOR, int REST = 0, bool HALF = false>
hipError_t configure_one() {
    return hipFuncSetAttribute((const void*)gemm_bf16<BMB, NB, WM, WN, EPI, FACTOR, REST, HALF>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes<BMB, NB, WM, WN, REST, HALF>());
}

}  // namespace

// Instantiations: (row blocks, column blocks, wave grid) per epilogue.  First the tall tiles of chunks of more than 128
// rows (kTallTiles below prices them), then the tiles of short chunks, narrow in N so that the grid is wide enough to
// keep every CU streaming weights, and those of chunks that share the GPU.
#define JUP_GEMM_TALL(X, EPI)                                                                              \
    X(8, 8, 4, 2, EPI) X(8, 6, 4, 2, EPI) X(8, 4, 4, 2, EPI) X(6, 8, 2, 4, EPI) X(6, 4, 2, 2, EPI)         \
    X(4, 8, 2, 4, EPI) X(4, 6, 4, 2, EPI) X(4, 4, 4, 2, EPI)
#define JUP_GEMM_SHAPES(X)                                                                                 \
    JUP_GEMM_TALL(X, EPI_QKV) X(6, 6, 2, 2, EPI_QKV) X(4, 3, 4, 1, EPI_QKV)                                \
    JUP_GEMM_TALL(X, EPI_SWIGLU) X(6, 6, 2, 2, EPI_SWIGLU) X(4, 3, 4, 1, EPI_SWIGLU) X(8, 3, 4, 1, EPI_SWIGLU) \
    JUP_GEMM_TALL(X, EPI_PARTIAL)                                                                          \
    X(9, 8, 4, 2, EPI_SWIGLU) X(9, 6, 4, 2, EPI_SWIGLU)                                                    \
    X(8, 1, 4, 1, EPI_QKV) X(8, 2, 4, 1, EPI_QKV) X(8, 3, 8, 1, EPI_QKV)                                   \
    X(4, 1, 4, 1, EPI_QKV) X(4, 2, 4, 1, EPI_QKV) X(2, 2, 2, 2, EPI_QKV)                                   \
    X(4, 1, 4, 1, EPI_SWIGLU) X(4, 2, 4, 1, EPI_SWIGLU)                                                    \
    X(8, 2, 4, 1, EPI_SWIGLU) X(4, 4, 4, 1, EPI_SWIGLU) X(2, 4, 2, 2, EPI_SWIGLU)                          \
    X(1, 3, 1, 3, EPI_SWIGLU) X(1, 4, 1, 4, EPI_SWIGLU) X(2, 3, 2, 3, EPI_SWIGLU) X(4, 6, 4, 1, EPI_SWIGLU) \
    X(2, 6, 2, 3, EPI_SWIGLU)                                                                              \
    X(4, 4, 4, 1, EPI_PARTIAL) X(2, 4, 2, 2, EPI_PARTIAL) X(2, 2, 2, 2, EPI_PARTIAL) X(4, 2, 4, 1, EPI_PARTIAL)
// Batches of more than 64 rows of branches of up to 16 tokens: rows with a factor (see FACTOR; the tiles of up to 64 rows
// all take one)
#define JUP_GEMM_FACTOR_SHAPES(X) \
    X(4, 1, 4, 1, EPI_QKV) X(4, 2, 4, 1, EPI_QKV) X(4, 1, 4, 1, EPI_SWIGLU) X(4, 2, 4, 1, EPI_SWIGLU)     \
    X(4, 3, 4, 1, EPI_SWIGLU) X(4, 4, 4, 1, EPI_SWIGLU)
// Tiles of two widths (see REST): the column blocks of the last round's behind the epilogue.
#define JUP_GEMM_REST_SHAPES(X) X(8, 8, 4, 2, EPI_SWIGLU, 6) X(8, 8, 4, 2, EPI_SWIGLU, 4)
// Tiles that end in half a column block (see HalfTile)
#define JUP_GEMM_HALF_SHAPES(X) X(2, 2, 2, 2, EPI_QKV) X(2, 2, 2, 2, EPI_SWIGLU)

hipError_t gemm_configure() {
    hipError_t e = hipSuccess;
    auto acc = [&](hipError_t r) { if (e == hipSuccess) e = r; };
#define X(BMB, NB, WM, WN, EPI) acc(configure_one<BMB, NB, WM, WN, EPI, BMB <= 2 && EPI != EPI_PARTIAL>());
    JUP_GEMM_SHAPES(X)
#undef X
#define X(BMB, NB, WM, WN, EPI) acc(configure_one<BMB, NB, WM, WN, EPI, true>());
    JUP_GEMM_FACTOR_SHAPES(X)
#undef X
#define X(BMB, NB, WM, WN, EPI, REST) acc(configure_one<BMB, NB, WM, WN, EPI, false, REST>());
    JUP_GEMM_REST_SHAPES(X)
#undef X
#define X(BMB, NB, WM, WN, EPI) acc(configure_one<BMB, NB, WM, WN, EPI, true, 0, true>());
    JUP_GEMM_HALF_SHAPES(X)
#undef X
    return e;
}

// ---- which instantiation serves a launch ------------------------------------------------------------------
struct TileShape {
    int bmb, nb, wm, wn;  // row blocks, column blocks, waves along M, waves along N
    int rest = 0;         // column blocks of the tiles of the last round, 0: as the others
    bool half = false;    // the last of the nb column blocks is half a block
};

namespace {

// Tiles of a chunk of more than 128 rows that has the chip to itself.  A launch is priced as rounds of workgroups (one
// workgroup per CU: the ring fills LDS) times what a round of the tile takes, and the cheapest tile (and number of K
// splits) wins.  The constants are fitted to a sweep of all tiles over 129 .. 2048 rows of the eight projections of the 7B
// and the 13B shapes (us on one MI355X; fit within 5 % on average; the pick costs 0.8 % more than the best measured
// tile on average and 6 % at worst).  What it replaced picked the width of a 256-row tile and nothing else; measured
// before -> after on the 7B shapes: QKV of 2048 rows 208 -> 175 us, of 539 rows (three 256-row tiles for 17 row blocks)
// 94 -> 59 us; gate/up of 539 rows 123 -> 104 us, of 320 rows 74 -> 59 us; down of 539 rows 69 -> 58 us with its share
// of the reduction; on the 13B shapes gate/up of 512 rows 136 -> 113 us, QKV 102 -> 76 us.
// What gate/up launches take against the model where tiles of 288 rows or two widths are a choice: full - less * 1024 / K (the clock
// falls under rounds of wide tiles and a long K loop).
struct Clock {
    float full, less;
    float factor(int K) const { return full - less * 1024.f / K; }
};
struct TileCost {
    TileShape t;
    int epilogues;            // 1 << EPI_*: what it is instantiated for
    float stage, round, qkv;  // us per K stage of 32, per round of workgroups, more per round with the QKV epilogue
    Clock clock = {1.0f, 0.0f};
};
constexpr int kWideEpi = 1 << EPI_QKV | 1 << EPI_SWIGLU, kAnyEpi = kWideEpi | 1 << EPI_PARTIAL;
constexpr TileCost kTallTiles[] = {
    {{8, 8, 4, 2}, kAnyEpi, 0.608f, 9.9f, 4.0f, {1.15f, 0.26f}}, {{8, 6, 4, 2}, kAnyEpi, 0.496f, 6.3f, 5.3f, {1.15f, 0.20f}},
    {{8, 4, 4, 2}, kAnyEpi, 0.386f, 5.5f, 2.6f}, {{6, 8, 2, 4}, kAnyEpi, 0.496f, 8.1f, 2.5f, {1.14f, 0.0f}},
    {{6, 4, 2, 2}, kAnyEpi, 0.282f, 7.5f, 2.0f, {0.97f, 0.0f}}, {{4, 8, 2, 4}, kAnyEpi, 0.401f, 5.4f, 2.2f, {1.02f, 0.0f}},
    {{4, 6, 4, 2}, kAnyEpi, 0.322f, 4.7f, 2.8f}, {{4, 4, 4, 2}, kAnyEpi, 0.230f, 4.1f, 2.0f},
    {{6, 6, 2, 2}, kWideEpi, 0.437f, 0.3f, 2.3f, {1.01f, -0.05f}}, {{4, 3, 4, 1}, kWideEpi, 0.196f, 4.9f, 1.4f},
    {{8, 3, 4, 1}, 1 << EPI_SWIGLU, 0.343f, 1.0f, 0.0f},
};
// Two more ways to fit gate/up.  288 rows: up to a row block or two more than whole 256-row tiles (the eight waves share the ninth
// row block's columns).  Measured: 539 rows 116.6 -> 92.7 us (two M tiles and one round of 230 workgroups instead of three M
// tiles and two rounds), on the 13B shapes 144 -> 133.  Not for QKV (539 rows: 79 us instead of 60; 1100 rows 110 instead of 114, the only
// gain) and the O / down projections, whose K splits fill the chip with any tile (down of 539 rows: 63.5 us instead of 59.2).
constexpr TileCost kTallTiles288[] = {
    {{9, 8, 4, 2}, 1 << EPI_SWIGLU, 0.720f, 10.0f, 0.0f, {1.13f, 0.33f}}, {{9, 6, 4, 2}, 1 << EPI_SWIGLU, 0.600f, 10.0f, 0.0f, {1.08f, 0.28f}},
};
// 256-row tiles of two widths: as many whole rounds of 256-column tiles as there are, and the last one of 192 or 128
// columns where those fill it better.  Measured, all rounds alike -> two widths: 2048 rows 293.8 -> 282.6 us, 1700 rows 281 ->
// 260, 1280 rows 193 -> 182; 13B 1024 rows 238 -> 228, 2048 rows 471 -> 443.  (QKV, whose column blocks are fewer: nothing
// gained at 1700 and 2048 rows of either.)
struct TwoWidths {
    TileShape t;
    Clock clock;
};
constexpr TwoWidths kTwoWidths[] = {{{8, 8, 4, 2, 6}, {1.18f, 0.33f}}, {{8, 8, 4, 2, 4}, {1.17f, 0.33f}}};
constexpr float kTwoWidthsUs = 3.0f;      // what such a launch has to be cheaper by
constexpr float kLaunchUs = 3.0f;
constexpr float kPartRound = 0.84f;       // a round that fills few CUs still takes this much of a full one
constexpr float kPartialUsPerByte = 1.0f / 5.2e6f;  // what the reduce + norm pass pays to read a partial sum back

struct TallPick {
    TileShape t;
    int splits;
};

float rounds(int wgs) {
    const int rest = wgs % kCUs;
    return (float)(wgs / kCUs) + (rest ? kPartRound + (1.f - kPartRound) * rest / kCUs : 0.f);
}

TallPick pick_tall(int epi, int M, int N, int K) {
    TallPick best{};
    float best_us = 0.f;
    const int stages = K / G_BK;
    auto round_us = [&](const TileCost& c, int splits) { return c.stage * (stages / splits) + c.round + (epi == EPI_QKV ? c.qkv : 0.f); };
    for (const TileCost& c : kTallTiles) {
        if (!(c.epilogues >> epi & 1)) continue;
        const int tiles = div_up(M, 32 * c.t.bmb) * div_up(N, 32 * c.t.nb);
        for (int splits = 1; splits <= (epi == EPI_PARTIAL ? 8 : 1); ++splits) {
            if (stages % splits || (splits > 1 && tiles * splits > kCUs)) continue;
            float us = kLaunchUs + rounds(tiles * splits) * round_us(c, splits);
            if (epi == EPI_PARTIAL) us += 4.f * M * N * splits * kPartialUsPerByte;
            if (best.splits == 0 || us < best_us) { best = {c.t, splits}; best_us = us; }
        }
    }
    if (epi != EPI_SWIGLU) return best;
    // The two other ways have to be cheaper by the model and with the clock in it.  Measured over 393 launches of 19 stages where the
    // model alone offers one of them: by the model alone 33 got slower than with the tiles above, 1025 to 1152 rows of the 7B
    // shapes most, 169 -> 179 us, where tiles of 192 x 192 hold the clock; with the clock none, and all of them run 1.080 times
    // as fast (1.082 with the best choice for each).
    const float plain_us = best_us;
    for (const TileCost& c : kTallTiles)
        if (c.t.bmb == best.t.bmb && c.t.nb == best.t.nb && c.t.wm == best.t.wm) best_us = plain_us * c.clock.factor(K);
    auto offer = [&](const TileShape& t, float us, const Clock& clock) {
        if (us < plain_us && us * clock.factor(K) < best_us) { best = {t, 1}; best_us = us * clock.factor(K); }
    };
    for (const TileCost& c : kTallTiles288)
        offer(c.t, kLaunchUs + rounds(div_up(M, 32 * c.t.bmb) * div_up(N, 32 * c.t.nb)) * round_us(c, 1), c.clock);
    for (const TwoWidths& w : kTwoWidths) {
        const TileShape& t = w.t;
        const int tiles = div_up(M, 32 * t.bmb) * div_up(N, 32 * t.nb);
        if (tiles < kCUs || tiles % kCUs == 0) continue;
        float wide = 0.f, rest = 0.f;
        for (const TileCost& c : kTallTiles) {
            if (c.t.bmb != t.bmb || c.t.wm != t.wm || c.t.wn != t.wn) continue;
            if (c.t.nb == t.nb) wide = round_us(c, 1);
            if (c.t.nb == t.rest) rest = round_us(c, 1);
        }
        const Rounds r = rounds_of(M, N, t.bmb, t.nb, t.rest);
        offer(t, kLaunchUs + kTwoWidthsUs + tiles / kCUs * wide + rounds(r.rest_tiles) * rest, w.clock);
    }
    return best;
}

}  // namespace

// The projections whose N (= d_model) alone cannot fill the chip are split along K; the fp32 partial sums are
// added up, in split order, by the reduce + norm kernel that follows.
namespace {
// splits for tiles of 32*nb columns: the largest count up to 8 that keeps the grid within one round of workgroups
// and divides the K stages evenly (powers of two on the 7B shapes; d = 5120 and FFN 13824 also allow 5, 3 and 6)
int splits_for(int M, int N, int K, int nb) {
    const int tiles = div_up(M, 32 * pick_row_blocks(M)) * div_up(N, 32 * nb);
    int splits = 1;
    for (int s = 2; s <= 8; ++s)
        if (tiles * s <= kCUs && (K / G_BK) % s == 0) splits = s;
    return splits;
}
}  // namespace

// Column blocks of the partial-sum tile.  Short chunks take 64-column tiles instead of 128 when the wide tile
// would leave a workgroup only a few K stages (fill and drain of its pipeline would dominate): half the
// splits, so half the partial sums to write and to read back.  Measured on the 7B shapes: 64-row chunks O
// 13.3 -> 12.5 us, down 23.0 -> 22.3 us, reduce + norm 8.2 -> 7.6 us; 128-row chunks O 18.2 -> 15.8 us (down,
// with 43 stages per workgroup, keeps the wide tile: 28.3 vs 29.5 us).
int gemm_partial_col_blocks(int M, int N, int K) {
    const int bmb = pick_row_blocks(M);
    const int stages_wide = K / G_BK / splits_for(M, N, K, 4);
    return stages_wide < (bmb == 2 ? 64 : 32) ? 2 : 4;
}

// shared: another chunk's kernels run beside this launch (overlapped multi-chunk call).  Filling the chip with one
// launch then matters less than the work per output: at most two splits (half or a quarter of the partial sums to
// write and read back, longer K loops per workgroup); the CUs a launch leaves free go to the other chunks.
// Measured on the 7B shapes, equal chunks on four lanes (see GemmArgs::shared_gpu): 4 x 512 tokens 274k -> 286k tokens/s, 8 x 256 tokens 204k -> 224k,
// 16 x 128 and 8 x 64 tokens +3-4 % (no split at all: -4 % there); alone on the chip the same cap costs 8 % (one
// launch then has to fill it).
int gemm_plan_splits(int M, int N, int K, bool shared) {
    if (M > 128 && !shared) return pick_tall(EPI_PARTIAL, M, N, K).splits;
    // beside other chunks' kernels: the widest tile of the chunk's row count (see launch_gemm_partial)
    const int nb = shared ? (pick_row_blocks(M) >= 8 ? 8 : 4) : gemm_partial_col_blocks(M, N, K);
    const int s = splits_for(M, N, K, nb);
    const int cap = shared ? 2 : 8;
    return s > cap ? cap : s;
}

namespace {
// Among the instantiated widths (in 32-column blocks) of the 256-row tile, the one with the least work on the
// busiest CU: rounds of workgroups x time of one tile.  A tile's time grows with its width plus a fixed part
// (pipeline fill and drain, epilogue, and the 256 rows of A it streams whatever its width) worth about two
// column blocks: without it many narrow tiles look cheapest, and they re-read A once per tile (measured at
// M = 2048: 1.66 GB fetched per launch and 445 us with 64-column tiles, against 325 us expected from M = 1024).
// Ties go to the wider tile.
int pick_blocks(int M, int N, const int* cands, int n_cands) {
    const int m_tiles = div_up(M, 256);
    int best = cands[0];
    long best_cost = -1;
    for (int i = 0; i < n_cands; ++i) {
        const int nb = cands[i];
        const long tiles = (long)m_tiles * div_up(N, 32 * nb);
        const long cost = div_up((int)tiles, kCUs) * (long)(32 * nb + 64);
        if (best_cost < 0 || cost <= best_cost) { best = nb; best_cost = cost; }
    }
    return best;
}
}  // namespace

namespace {

constexpr TileShape kHalfTile = {2, 2, 2, 2, 0, true};

TileShape pick_qkv(int M, int N, int K, bool shared_gpu) {
    const int bmb = pick_row_blocks(M);
    // 128-token chunks beside other chunks' kernels: 96-column tiles (half again as much work per workgroup; alone on
    // the chip 64 columns win, 24.0 vs 28.8 us at 64 rows).  Measured on four lanes: 13B shapes, 8 x 128 tokens
    // +2 %; 7B shapes, 16 x 128 tokens +0-1 %; 192 columns +4 % and -1 %; 64-token chunks no difference either way.
    if (shared_gpu && bmb == 4) return {4, 3, 4, 1};
    // 33 to 64 rows: tiles of one and a half column blocks where their grid is still one round of workgroups.  A CU takes rows and
    // weights at about 50 GB/s, and 64-column tiles leave a quarter of the CUs out on the 7B shapes (192 of 256).  Whole layers,
    // 64 -> 48 columns: 64 rows 7B 102.8 -> 101.8 us, d_model 2048 60.3 -> 59.8; 40 rows 95.6 -> 94.9, 56.9 -> 56.6.  Below 33 rows
    // nothing is gained (the rows weigh little), nor with fewer workgroups (d_model 1536: 53.1 -> 52.7 and 50.5 -> 50.5; 1024: 43.4 ->
    // 43.5 and 41.7 -> 42.4).
    if (M > 32 && M <= 64 && !shared_gpu && N % 96 == 0 && N / 48 >= kCUs / 2 && N / 48 <= kCUs) return kHalfTile;
    if (bmb == 2) return {2, 2, 2, 2};
    // Narrow stages: 32 columns where that is one round of workgroups.  A CU takes rows and weights at about 50 GB/s, so as few
    // columns each as there are CUs for.  Whole layers, 64 -> 32 columns: d_model 2048 (96 -> 192 workgroups) 128 rows 71.6 -> 69.5 us,
    // 65 rows 60.6 -> 57.8; 1536 61.8 -> 60.0, 53.5 -> 51.8; 1024 49.1 -> 47.8, 44.1 -> 42.8.
    if (bmb == 4 && div_up(N, 32) <= kCUs) return {4, 1, 4, 1};
    if (bmb == 4) return {4, 2, 4, 1};
    if (!shared_gpu) return pick_tall(EPI_QKV, M, N, K).t;
    static const int cands[] = {1, 2, 3};
    const int nb = pick_blocks(M, N, cands, 3);
    // Beside another chunk's kernels (overlapped multi-chunk call) half as many tiles of twice the width do the
    // same work in a quarter less CU time, and the other chunk uses the CUs they leave free: 76 us instead of 59 us
    // for this launch alone, but +1.7 % for the 4 x 512 prompt.
    if (nb == 3 && M > 256) return {8, 6, 4, 2};
    if (nb == 3) return {8, 3, 8, 1};  // 8 waves of 32 x 96: measured 1.3 % faster than 4 of 64 x 96
    if (nb == 2) return {8, 2, 4, 1};
    return {8, 1, 4, 1};
}

TileShape pick_swiglu(int M, int N, int K, bool shared_gpu) {
    const int bmb = pick_row_blocks(M);
    // Stages so narrow that 48-column tiles are one round of workgroups: those instead of 96 columns, for 33 to 64 rows, and for fewer
    // where the grid then fills three quarters of the chip.  Whole layers, 96 -> 48 columns: d_model 2048 (118 -> 235 workgroups)
    // 64 rows 59.4 -> 56.4 us, 40 rows 56.3 -> 53.3, 32 rows 54.4 -> 52.5, 16 rows 49.1 -> 48.2, 5 rows 45.1 -> 44.9; 1536 (88 -> 176) 52.6 ->
    // 51.4, 50.0 -> 49.3, 48.1 -> 48.0; 1024 (59 -> 118) 43.6 -> 43.1, 41.9 -> 41.8, 40.5 -> 41.0.
    const int halves = div_up(N, 48);
    if (M <= 64 && !shared_gpu && halves <= kCUs && (M > 32 || (M > 8 && halves > kCUs * 3 / 4))) return kHalfTile;
    // A short chunk is bound by streaming the weights, and every CU that streams adds bandwidth: the narrower
    // tile (96 columns) when its tiles still fit one round of workgroups (measured at 64 rows, N = 22016:
    // 230 workgroups 38.0 us, 172 workgroups of 128 columns 40.9 us, 344 of 64 columns 47.1 us).
    // Beside other chunks' kernels (overlapped multi-chunk call) the opposite holds: 192-column tiles, fewer and
    // longer-running workgroups, and the other chunks take the CUs they leave (64-token chunks +1.5 %, 128-token
    // chunks +2.5 %, the 13B shapes +4 % over 128 columns, which in turn beat 96 by 2-6 % there).
    if (shared_gpu && bmb == 2) return {2, 6, 2, 3};
    if (shared_gpu && bmb == 4) return {4, 6, 4, 1};
    const bool narrow = div_up(N, 96) <= kCUs;
    // Up to 32 rows: a tile of one row block (32 x 96 or 32 x 128, one wave per column block) leaves the fill path to the
    // weights; measured at 5 rows, N = 22016: 32.5 -> 31.5 us.  (The same for QKV and the O / down projections, on two
    // waves of 32 x 32: QKV 22.8 -> 23.4 us, O / down no different: they keep the 64-row tile.)
    if (bmb == 2 && M <= 32) return narrow ? TileShape{1, 3, 1, 3} : TileShape{1, 4, 1, 4};
    if (bmb == 2) return narrow ? TileShape{2, 3, 2, 3} : TileShape{2, 4, 2, 2};
    // 65 to 128 rows of narrow stages: the narrowest tile whose grid is one round of workgroups (see QKV).  Whole layers, 96 -> 64 ->
    // 32 columns: d_model 2048 (118, 176 workgroups) 128 rows 75.2 -> 71.7 us, 65 rows 62.9 -> 59.9; 1536 (88, 132) 64.0 -> 62.1,
    // 56.0 -> 53.7; 1024 (59, 88, 176) 51.9 -> 50.3 -> 49.1, 46.5 -> 45.0 -> 44.1.
    if (bmb == 4 && div_up(N, 32) <= kCUs) return {4, 1, 4, 1};
    if (bmb == 4 && div_up(N, 64) <= kCUs) return {4, 2, 4, 1};
    if (bmb == 4) return narrow ? TileShape{4, 3, 4, 1} : TileShape{4, 4, 4, 1};
    if (!shared_gpu) return pick_tall(EPI_SWIGLU, M, N, K).t;
    static const int cands[] = {2, 3, 4, 6};
    const int nb = pick_blocks(M, N, cands, 4);
    // beside other chunks' kernels: the widest tile (see pick_qkv); 256 x 256 over 256 x 192: +1.9 %
    if (nb == 6) return {8, 8, 4, 2};
    if (nb == 4) return {8, 4, 4, 2};
    if (nb == 3) return {8, 3, 4, 1};
    return {8, 2, 4, 1};
}

TileShape pick_partial(int M, int N, int K, bool shared_gpu) {
    const int bmb = pick_row_blocks(M);
    if (bmb == 8) return shared_gpu ? TileShape{8, 8, 4, 2}  // beside other chunks' kernels the widest tile (see pick_qkv)
                                    : pick_tall(EPI_PARTIAL, M, N, K).t;
    // (short chunks beside other chunks' kernels keep the 128-column tile: 64-token chunks +3 %, 128-token +5 %)
    const bool narrow = gemm_partial_col_blocks(M, N, K) == 2 && !shared_gpu;
    if (bmb == 2) return narrow ? TileShape{2, 2, 2, 2} : TileShape{2, 4, 2, 2};
    return narrow ? TileShape{4, 2, 4, 1} : TileShape{4, 4, 4, 1};
}

template <int EPI>
hipError_t dispatch(TileShape t, const GemmArgs& a, hipStream_t s) {
#define X(BMB, NB, WM, WN, E)                                                         \
    if constexpr (E == EPI)                                                           \
        if (t.bmb == BMB && t.nb == NB && t.wm == WM && t.wn == WN && !t.rest && !t.half) \
            return launch<BMB, NB, WM, WN, EPI, BMB <= 2 && EPI != EPI_PARTIAL>(a, s);
    JUP_GEMM_SHAPES(X)
#undef X
#define X(BMB, NB, WM, WN, E, REST)                                                           \
    if constexpr (E == EPI)                                                                   \
        if (t.bmb == BMB && t.nb == NB && t.wm == WM && t.wn == WN && t.rest == REST)         \
            return launch<BMB, NB, WM, WN, EPI, false, REST>(a, s);
    JUP_GEMM_REST_SHAPES(X)
#undef X
#define X(BMB, NB, WM, WN, E)                                                                 \
    if constexpr (E == EPI)                                                                   \
        if (t.bmb == BMB && t.nb == NB && t.wm == WM && t.wn == WN && t.half)                 \
            return launch<BMB, NB, WM, WN, EPI, true, 0, true>(a, s);
    JUP_GEMM_HALF_SHAPES(X)
#undef X
    return hipErrorInvalidConfiguration;  // a shape the pick functions name but the list above does not hold
}

// 65 to 128 rows with a factor: the tile that rows without one take.
template <int EPI>
hipError_t dispatch_factor(const GemmArgs& a, hipStream_t s) {
    if (a.M > kMaxSplitRows) return hipErrorInvalidValue;
    const TileShape t = EPI == EPI_QKV ? pick_qkv(a.M, a.N, a.K, false) : pick_swiglu(a.M, a.N, a.K, false);
#define X(BMB, NB, WM, WN, E)                                                         \
    if constexpr (E == EPI)                                                           \
        if (t.bmb == BMB && t.nb == NB && t.wm == WM && t.wn == WN) return launch<BMB, NB, WM, WN, EPI, true>(a, s);
    JUP_GEMM_FACTOR_SHAPES(X)
#undef X
    return hipErrorInvalidConfiguration;
}

}  // namespace

hipError_t launch_gemm_qkv(GemmArgs a, hipStream_t s) {
    a.splits = 1;
    if (a.row_factor && a.M > 64) return dispatch_factor<EPI_QKV>(a, s);
    return dispatch<EPI_QKV>(pick_qkv(a.M, a.N, a.K, a.shared_gpu), a, s);
}

hipError_t launch_gemm_swiglu(GemmArgs a, hipStream_t s) {
    a.splits = 1;
    if (a.row_factor && a.M > 64) return dispatch_factor<EPI_SWIGLU>(a, s);
    return dispatch<EPI_SWIGLU>(pick_swiglu(a.M, a.N, a.K, a.shared_gpu), a, s);
}

hipError_t launch_gemm_partial(GemmArgs a, hipStream_t s) {
    a.splits = gemm_plan_splits(a.M, a.N, a.K, a.shared_gpu);
    return dispatch<EPI_PARTIAL>(pick_partial(a.M, a.N, a.K, a.shared_gpu), a, s);
}

// The name of the launch a projection of M rows takes; jup_diag_kernel_name (jupiter_stage.h) has the forms.
void gemm_kernel_name(GemmKind kind, int M, int d_model, int d_ffn, bool shared_gpu, char* buf, size_t size) {
    TileShape t{};
    int epi = EPI_PARTIAL;
    switch (kind) {
        case GEMM_QKV: t = pick_qkv(M, 3 * d_model, d_model, shared_gpu); epi = EPI_QKV; break;
        case GEMM_GATE_UP: t = pick_swiglu(M, 2 * d_ffn, d_model, shared_gpu); epi = EPI_SWIGLU; break;
        case GEMM_O: t = pick_partial(M, d_model, d_model, shared_gpu); break;
        case GEMM_DOWN: t = pick_partial(M, d_model, d_ffn, shared_gpu); break;
    }
    if (epi == EPI_PARTIAL && M <= kMaxProjectRows && !shared_gpu) {
        snprintf(buf, size, "project_rows<bf16>");
        return;
    }
    char cols[24];
    if (t.rest) snprintf(cols, sizeof(cols), "%d+%d", t.nb, t.rest);
    else if (t.half) snprintf(cols, sizeof(cols), "%d.5", t.nb - 1);
    else snprintf(cols, sizeof(cols), "%d", t.nb);
    snprintf(buf, size, "gemm_bf16<%d,%s,%d,%d,%d>", t.bmb, cols, t.wm, t.wn, epi);
}

}  // namespace jup
