// Projections of a 4-bit stage (JUP_BF16_W4) for chunks and branches of more than 64 tokens, from 33 on where this is the faster
// kernel (w4_plan.h): C[M, N] = A[M, K] * W[N, K]^T on the packed codes and scales of w4_gemm.hip, whose kernel is built for
// decode-sized chunks (its waves read the rows from L2, 64 at a time, and expand the codes once per 64 rows).
//
//   * A wave owns 32 MB rows x 32 columns and every WK-th K group of its workgroup: its columns are its own, so the codes go
//     from global memory into registers and are expanded there, once per 32 MB rows; nothing of W passes through LDS.  The
//     rows are shared by the WN waves of a K share and come through an LDS ring of direct global->LDS loads, in stages of
//     one or half a group per share, one barrier per stage.
//   * v_mfma_f32_32x32x16_bf16 (operand layout: bf16_gemm.hip).  A group of 128 features is eight steps into a temporary
//     that then enters the sum times the column's scale: 16 vector instructions per 256 MFMA clocks and block.
//   * A code becomes the bf16 value (code - 8) / 16, exactly (cvt_off: a signed nibble / 16; 13 instructions for eight codes),
//     the sums are multiplied by 16 at the end.  No row sums of A are needed, as for the 128 + code form (seven instructions
//     and one more MFMA per step and 16 rows), which beside a 32-column wave would double the MFMAs.
//   * What bounds it is the waves' own instruction streams: a wave issues a vector instruction every 8 clocks, and a turn
//     (one group, 128 rows) is about 200 of them against 1024 clocks of MFMAs; two or three waves per SIMD overlap.  So the
//     loop is kept short: fragments of the next eight MFMAs are read and the codes of the next four steps expanded behind
//     the MFMAs, addresses are 32-bit offsets, and the tail of the loop is the loop itself with its loads pointed at one
//     cache line (the count of loads in flight then never depends on the turn).  Codes are asked for two turns ahead:
//     deeper (four, seven) measured 10 % slower, the unrolled loop no longer fits the instruction cache.
//
// Measured on the 7B shapes (us, kernel of w4_gemm.hip at 64 rows per pass -> this one; QKV, gate/up, O, down): 64 rows gate/up
// 34 -> 23 (the others stay there: 18, 9, 16); 128 rows 33 -> 23, 48 -> 35, 15 -> 11, 27 -> 22; 256 rows 52 -> 37, 89 -> 56, 27 ->
// 17, 49 -> 31; 512 rows 96 -> 62, 158 -> 108, 49 -> 25, 90 -> 50 (the bf16 kernels there: 56, 81, 25, 47).
#include <type_traits>
#include <utility>

#include "w4_plan.h"

namespace jup {
namespace {

constexpr int kLds = 160 * 1024;

template <int MB, int WN, int WK>
struct WideShape {
    static constexpr int WAVES = WN * WK, THREADS = 64 * WAVES;
    static constexpr int COLS = 32 * WN;                     // columns of the tile
    static constexpr int PARTS = MB * WK > 4 ? 2 : 1;        // stages per K group of 128
    static constexpr int PART_BYTES = 8192 / PARTS;          // of one row block and K share
    static constexpr int STAGE_BYTES = MB * WK * PART_BYTES;
    static constexpr int STAGES = 4 * STAGE_BYTES <= kLds ? 4 : 3;
    static constexpr int DEPTH = 2;
    static constexpr int UNITS = STAGE_BYTES / 1024;         // 1 KB loads per stage
    static constexpr int LOADS = (UNITS + WAVES - 1) / WAVES;
    // The queue of loads, which return in order.  At the start of stage st a wave asks for the rows of stage st + STAGES - 1 and,
    // where a turn begins, for the codes of the turn DEPTH further on; in front of the loop it asks for what the stages before 0
    // would have, in the same order.
    static constexpr int CODE_LOADS = 3;
    static constexpr bool rows_asked(int st) { return st >= 1 - STAGES; }
    static constexpr bool codes_asked(int st) { return st % PARTS == 0 && st / PARTS + DEPTH >= 0; }
    static constexpr int FIRST = -DEPTH * PARTS < 1 - STAGES ? -DEPTH * PARTS : 1 - STAGES;  // stage that asks first
    // Loads behind the rows of stage st when the stages before `until` have asked.
    static constexpr int behind(int st, int until) {
        int n = codes_asked(st + 1 - STAGES) ? CODE_LOADS : 0;
        for (int s = st + 2 - STAGES; s < until; ++s) n += LOADS + (codes_asked(s) ? CODE_LOADS : 0);
        return n;
    }
    // Stage st begins when the rows of stage st + 1 have landed: in the first stages no more loads are behind them than in any other.
    static constexpr int behind_next(int part) { return behind(PARTS * STAGES + part + 1, PARTS * STAGES + part); }
    static constexpr bool same_from_the_start() {
        for (int st = 0; st < PARTS * STAGES; ++st)
            if (behind(st + 1, st) != behind_next(st % PARTS)) return false;
        return true;
    }
    static_assert(same_from_the_start(), "a wait of the loop is too weak for its first stages");
    static constexpr int RED_STRIDE = COLS + 4;
    static constexpr int RED_BYTES = WK * 32 * RED_STRIDE * 4;
    static constexpr int LDS_BYTES = STAGES * STAGE_BYTES > RED_BYTES ? STAGES * STAGE_BYTES : RED_BYTES;
    static_assert(LDS_BYTES <= kLds && MB % 2 == 0, "ring");
};

__device__ inline f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }

template <int N>
__device__ inline void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit field");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | 0x0F70);
}

// Eight 4-bit codes of one dword as the bf16 values (code - 8) / 16, exactly, in two halves (elements 0, 1, 4, 5, then 2, 3, 6, 7).
struct Nibbles {
    unsigned x, y;  // one per byte: low, high
    __device__ __forceinline__ explicit Nibbles(unsigned w) : x(w), y(w >> 4) {
        asm("" : "+v"(x), "+v"(y));  // (else the bytes of y become bit fields of x, an instruction each)
    }
    static __device__ __forceinline__ float at(unsigned v, int byte) {
        return __builtin_amdgcn_cvt_off_f32_i4((int)((v >> (8 * byte)) & 0xffu));
    }
    __device__ __forceinline__ void first(u32x4& v) const { v[0] = pack_bf16x2(at(x, 0), at(x, 2)); v[2] = pack_bf16x2(at(x, 1), at(x, 3)); }
    __device__ __forceinline__ void second(u32x4& v) const { v[1] = pack_bf16x2(at(y, 0), at(y, 2)); v[3] = pack_bf16x2(at(y, 1), at(y, 3)); }
};

// fn(FROM), ..., fn(TO - 1), each number as a constant
template <int FROM, int TO>
__device__ __forceinline__ void static_for(auto fn) {
    [&]<int... K>(std::integer_sequence<int, K...>) __attribute__((always_inline)) {
        (fn(std::integral_constant<int, FROM + K>{}), ...);
    }(std::make_integer_sequence<int, TO - FROM>{});
}

template <int EPI, int MB, int WN, int WK, bool ONCE>
__global__ __launch_bounds__(64 * WN * WK) void gemm_w4_wide(const GemmArgs a) {
    using S = WideShape<MB, WN, WK>;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, hh = lane >> 5;
    const int wn = wave % WN, wk = wave / WN;
    int mt, grp;
    {
        const int q = gridDim.x >> 3, r = gridDim.x & 7;
        const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
        const int tile = xcd * q + min(xcd, r) + local;
        grp = a.by_m.of(tile);
        mt = tile - grp * a.m_tiles;
    }
    const int split = EPI == EPI_PARTIAL ? a.by_n.of(grp) : 0, nt = grp - split * a.n_tiles;
    const int m0 = mt * 32 * MB, n0 = nt * S::COLS;
    const int G = a.K / 128, KT = a.K / 32;
    const int gs0 = EPI == EPI_PARTIAL ? a.by_splits.of(split * G) : 0, gs1 = EPI == EPI_PARTIAL ? a.by_splits.of((split + 1) * G) : G;
    const int iters = (gs1 - gs0 + WK - 1) / WK;

    const char* const rows0 = uniform_ptr((const char*)a.A + (size_t)(m0 / 32) * KT * 2048);  // first row block of the tile
    // Rows: a stage is UNITS pieces of 1 KB, dealt to the waves.  A K share past the end of the range (last turn, count no
    // multiple of WK) repeats its last group, loads behind the last stage one cache line: the count of loads in flight is then
    // the same in every turn.
    const unsigned lane16 = lane * 16, ring0 = __builtin_amdgcn_readfirstlane(lds_byte_address(smem));
    unsigned row_at[S::LOADS];
    unsigned part_of[S::LOADS], part_of_last[S::LOADS];
#pragma unroll
    for (int q = 0; q < S::LOADS; ++q) {
        const int j = min(q * S::WAVES + wave, S::UNITS - 1);
        constexpr int PER_PART = S::PART_BYTES / 1024, PER_BLOCK = WK * PER_PART;
        const int k = j % PER_BLOCK / PER_PART;
        const int blk = min(j / PER_BLOCK, (a.M - 1) / 32 - m0 / 32);  // blocks past the chunk repeat its last one
        row_at[q] = (unsigned)blk * KT * 2048 + j % PER_PART * 1024 + lane16;
        part_of[q] = k * 8192;
        part_of_last[q] = min(k, gs1 - gs0 - 1 - (iters - 1) * WK) * 8192;
    }
    auto issue_rows = [&](int it, int part) __attribute__((always_inline)) {
        const int turn = min(it, iters - 1);
        const unsigned all = it < iters ? ~0u : 0u;
        const unsigned at = (unsigned)(gs0 + turn * WK) * 8192 + part * S::PART_BYTES;
        const unsigned slot = ring0 + (unsigned)(it * S::PARTS + part) % S::STAGES * S::STAGE_BYTES;
#pragma unroll
        for (int q = 0; q < S::LOADS; ++q) {
            const int j = min(q * S::WAVES + wave, S::UNITS - 1);
            const unsigned off = (row_at[q] & all) + (at + (turn == iters - 1 ? part_of_last[q] : part_of[q]));
            // (as text: beside the builtin, which the compiler takes for a flat access, it waits for every load in flight
            // in front of each use of a code or fragment.  Text it does not count: its wait for the next codes, all but the
            // youngest four or five loads, half a turn later drains most of the rows asked for in the same turn, so little more
            // than one stage of the ring is in flight)
            load_to_lds_16(rows0, off, slot + j * 1024);
        }
    };

    // Codes and scale of a group: eight dwords of eight codes (16 features each) of the lane's column.
    struct Codes {
        u32x4 w[2];
        float sc;
    };
    const int col_blk = min(nt * WN + wn, a.N / 32 - 1);  // 32-column block of the packed codes
    const int tile0 = min(n0, a.N - 32) >> 6;              // first of the tile's 64-column tiles of the packed codes
    const char* const codes0 = (const char*)a.W + (size_t)tile0 * G * 4096;
    const char* const scales0 = (const char*)a.w_scale + (size_t)tile0 * G * 256;
    const unsigned w_lane = (unsigned)((col_blk >> 1) - tile0) * G * 4096 + (col_blk & 1) * 2048 + (c >> 4) * 1024 + (16 * hh + (c & 15)) * 16;
    const unsigned s_lane = (unsigned)((col_blk >> 1) - tile0) * G * 256 + ((c & 15) * 4 + 2 * (col_blk & 1) + (c >> 4)) * 4;
    auto fetch_codes = [&](Codes& d, int it) __attribute__((always_inline)) {
        const unsigned g = min(gs0 + it * WK + wk, gs1 - 1);
        const unsigned at = (w_lane & (it < iters ? ~0u : 0u)) + g * 4096;
        d.w[0] = ONCE ? load_once_at<u32x4>(codes0, at) : load_at<u32x4>(codes0, at);
        d.w[1] = ONCE ? load_once_at<u32x4>(codes0, at + 512) : load_at<u32x4>(codes0, at + 512);
        d.sc = load_at<float>(scales0, s_lane + g * 256);
    };

    f32x16 acc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[mb][i] = 0.f;
    int lane_off[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) lane_off[ks] = (c >> 2) * 256 + ((((c & 3) << 2) + 2 * ks + hh) ^ ((c >> 2) & 3)) * 16;

    constexpr int ST = S::STAGES, PARTS = S::PARTS;
    constexpr int DEPTH = S::DEPTH, BUFS = DEPTH + 1;  // groups of codes on their way
    Codes buf[BUFS];
    static_for<S::FIRST, 0>([&](auto stage) __attribute__((always_inline)) {
        constexpr int st = decltype(stage)::value, asked = st + ST - 1;
        if constexpr (S::rows_asked(st)) issue_rows(asked / PARTS, asked % PARTS);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (S::codes_asked(st)) fetch_codes(buf[st / PARTS + DEPTH], st / PARTS + DEPTH);
        __builtin_amdgcn_sched_barrier(0);
    });

    // A chunk: two row blocks times four MFMA steps (64 features).  CHUNKS of them make a group, the first half of its features
    // for all row blocks, then the second.  Everything else is dealt out behind the eight MFMAs of a chunk: the fragments of
    // the next chunk, the codes of four steps expanded (four row blocks: in chunks 1 and 2), with four row blocks the sums of
    // a pair of them (pair 0 in chunk 3, pair 1 in chunk 0 of the next turn, when its MFMAs are done).
    constexpr int CHUNKS = MB, PAIRS = MB / 2;
    f32x16 t[MB];
    bf16x8 f[8];
    u32x4 b[MB == 2 ? 4 : 8];
    auto read_frag = [&](int it, auto chunk, auto k) __attribute__((always_inline)) {
        constexpr int CH = decltype(chunk)::value, KK = decltype(k)::value;
        constexpr int pair = CH % PAIRS, half = CH / PAIRS, s = KK >> 1, j = KK & 1;
        const int st = it * PARTS + (PARTS == 2 ? half : 0);
        const unsigned char* slot = smem + st % ST * S::STAGE_BYTES + wk * S::PART_BYTES;
        f[KK] = *(const bf16x8*)(slot + (2 * pair + j) * WK * S::PART_BYTES + (((PARTS == 1 ? 4 * half : 0) + s) >> 1) * 2048 + lane_off[s & 1]);
    };

    wait_vmcnt<S::behind(0, 0)>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");  // (no read of the ring in front of the barrier)
    static_for<0, 8>([&](auto k) __attribute__((always_inline)) { read_frag(0, std::integral_constant<int, 0>{}, k); });
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const Nibbles n(buf[0].w[s & 1][s >> 1]);
        n.first(b[s]);
        n.second(b[s]);
    }
    float sc = 0.f;
    if constexpr (MB == 4)
#pragma unroll
        for (int j = 2; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 16; ++i) t[j][i] = 0.f;

    auto iteration = [&](auto which, int it) __attribute__((always_inline)) {
        constexpr int B = decltype(which)::value;
        Codes& cur = buf[B];
        Codes& next = buf[(B + 1) % BUFS];
        Nibbles n(0);
        [&]<int... CHI>(std::integer_sequence<int, CHI...>) __attribute__((always_inline)) {
            ([&](auto chunk) __attribute__((always_inline)) {
                constexpr int CH = decltype(chunk)::value;
                constexpr int pair = CH % PAIRS, half = CH / PAIRS, part = PARTS == 2 ? half : 0;
                if constexpr (CH == 0 || (PARTS == 2 && CH == PAIRS)) {  // a stage begins
                    wait_vmcnt<S::behind_next(part)>();  // stage st + 1 has landed (its first fragments are read in this one)
                    __builtin_amdgcn_s_barrier();
                    issue_rows(it + (part + ST - 1) / PARTS, (part + ST - 1) % PARTS);
                    if (part == 0) fetch_codes(buf[(B + DEPTH) % BUFS], it + DEPTH);
                    __builtin_amdgcn_sched_barrier(0);
                }
                constexpr bool LAST = CH == CHUNKS - 1;
                constexpr bool OF_THIS = CH == (MB == 2 ? 0 : 1), OF_NEXT = CH == (MB == 2 ? 1 : 2);
                static_for<0, 8>([&](auto k) __attribute__((always_inline)) {
                    constexpr int K = decltype(k)::value, s = K >> 1, j = K & 1;
                    if constexpr (half == 0 && s == 0) {
#pragma unroll
                        for (int i = 0; i < 16; ++i) t[2 * pair + j][i] = 0.f;
                    }
                    t[2 * pair + j] = mfma32(f[K], __builtin_bit_cast(bf16x8, b[MB == 2 ? s : 4 * half + s]), t[2 * pair + j]);
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (LAST) read_frag(it + 1, std::integral_constant<int, 0>{}, k);
                    else read_frag(it, std::integral_constant<int, CH + 1>{}, k);
                    // two row blocks: the four steps' registers are free once their MFMAs are issued
                    if constexpr ((OF_THIS || OF_NEXT) && (MB == 4 || j == 1)) {
                        constexpr int at = OF_NEXT ? s : 4 + s;
                        u32x4& to = b[MB == 2 ? s : at];
                        if (MB == 2 || j == 0) {
                            n = Nibbles((OF_NEXT ? next : cur).w[at & 1][at >> 1]);
                            n.first(to);
                        }
                        if (j == 1) {
                            n.second(to);
                            asm volatile("" : "+v"(to));  // (here, not in front of its use: the codes' registers are wanted)
                        }
                    }
                    if constexpr (MB == 4 && (CH == 0 || CH == 3)) {
                        constexpr int from = CH == 0 ? 2 : 0;
#pragma unroll
                        for (int i = 4 * K; i < 4 * K + 4; ++i)
                            acc[from + i / 16][i % 16] = __builtin_fmaf(sc, t[from + i / 16][i % 16], acc[from + i / 16][i % 16]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
                // (a K share past the end of the range adds zero times the sum of a group that another share adds)
                if constexpr (CH == CHUNKS - 2) sc = gs0 + it * WK + wk < gs1 ? cur.sc : 0.f;
                if constexpr (MB == 2 && LAST) {
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[j][i] = __builtin_fmaf(sc, t[j][i], acc[j][i]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }(std::integral_constant<int, CHI>{}), ...);
        }(std::make_integer_sequence<int, CHUNKS>{});
    };
    int it = 0;
    auto turn = [&]<int... I>(std::integer_sequence<int, I...>) __attribute__((always_inline)) {
        return ((iteration(std::integral_constant<int, I>{}, it), ++it < iters) && ...);
    };
    while (turn(std::make_integer_sequence<int, BUFS>{})) {}

    wait_vmcnt<0>();  // (the last loads still write to the ring)
    if constexpr (MB == 4)
#pragma unroll
        for (int j = 2; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[j][i] = __builtin_fmaf(sc, t[j][i], acc[j][i]);

    // ---- sums of the K shares in order, then the epilogue, a row block at a time ----
    if constexpr (EPI == EPI_PARTIAL && WK == 1) {
        const int col = n0 + wn * 32 + c;
        if (col < a.N) {
            float* dst = a.partial + (size_t)split * a.M * a.N + col;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int m = m0 + mb * 32 + 8 * (i >> 2) + 4 * hh + (i & 3);
                    if (m < a.M) dst[(size_t)m * a.N] = 16.0f * acc[mb][i];
                }
        }
        return;
    }
    float* red = (float*)smem;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        if (m0 + mb * 32 >= a.M) break;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 16; ++i)
            red[(wk * 32 + 8 * (i >> 2) + 4 * hh + (i & 3)) * S::RED_STRIDE + wn * 32 + c] = acc[mb][i];
        __syncthreads();
        auto total4 = [&](int row, int col4) __attribute__((always_inline)) {
            f32x4 v = *(const f32x4*)(red + row * S::RED_STRIDE + col4);
#pragma unroll
            for (int k = 1; k < WK; ++k) v += *(const f32x4*)(red + (k * 32 + row) * S::RED_STRIDE + col4);
            return 16.0f * v;
        };
        if constexpr (EPI == EPI_PARTIAL) {
            for (int i = tid; i < 32 * S::COLS / 4; i += S::THREADS) {
                const int row = i / (S::COLS / 4), col = i % (S::COLS / 4) * 4, m = m0 + mb * 32 + row;
                if (m < a.M && n0 + col < a.N)
                    *(f32x4*)(a.partial + ((size_t)split * a.M + m) * a.N + n0 + col) = total4(row, col);
            }
        } else {
            for (int i = tid; i < 32 * S::COLS / 16; i += S::THREADS) {
                const int row = i / (S::COLS / 16), col = i % (S::COLS / 16) * 16, m = m0 + mb * 32 + row;
                const int pc = n0 + col;  // packed column of the block of 16
                if (m >= a.M || pc >= a.N) continue;
                f32x4 v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] = total4(row, col + 4 * k);
                if constexpr (EPI == EPI_SWIGLU) {
                    // even packed columns are gate rows, odd ones up rows: 8 outputs
                    u32x4 out;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const float g0 = v[k][0], u0 = v[k][1], g1 = v[k][2], u1 = v[k][3];
                        out[k] = pack_bf16x2(g0 * __builtin_amdgcn_rcpf(1.0f + __expf(-g0)) * u0,
                                             g1 * __builtin_amdgcn_rcpf(1.0f + __expf(-g1)) * u1);
                    }
                    *(u32x4*)(a.act + tiled_offset(m, pc >> 4, (a.N >> 1) >> 5)) = out;
                } else {
                    // rotary indices 8 u .. 8 u + 7 of a head and their partners 64 further on
                    const int which = (pc >= a.d_model) + (pc >= 2 * a.d_model), in = pc - which * a.d_model;
                    const int head = in >> 7, f = (in & 127) >> 1;
                    u32x4 lo, hi;
                    if (which == 2) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            lo[e] = pack_bf16x2(v[e >> 1][2 * (e & 1)], v[e >> 1][2 * (e & 1) + 1]);
                            hi[e] = pack_bf16x2(v[2 + (e >> 1)][2 * (e & 1)], v[2 + (e >> 1)][2 * (e & 1) + 1]);
                        }
                    } else {
                        const float4* rp = (const float4*)(a.rope + (size_t)m * 64 + f);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float4 cs = rp[e];
                            const float l0 = v[e >> 1][2 * (e & 1)], l1 = v[e >> 1][2 * (e & 1) + 1];
                            const float h0 = v[2 + (e >> 1)][2 * (e & 1)], h1 = v[2 + (e >> 1)][2 * (e & 1) + 1];
                            // (fused by hand: which product the compiler fuses differs between the shapes)
                            lo[e] = pack_bf16x2(__builtin_fmaf(l0, cs.x, -(h0 * cs.y)), __builtin_fmaf(l1, cs.z, -(h1 * cs.w)));
                            hi[e] = pack_bf16x2(__builtin_fmaf(h0, cs.x, l0 * cs.y), __builtin_fmaf(h1, cs.z, l1 * cs.w));
                        }
                    }
                    u16* dst;
                    if (which == 0) {
                        dst = a.q_out + (size_t)m * a.d_model + head * 128;
                    } else if (!a.branches) {
                        dst = kv_slot_bf16(a.kv, a.layer, which - 1, head, a.n_heads, a.pos0 + m);
                    } else {
                        const int b = m / a.branches->n_tok, tk = m - b * a.branches->n_tok;
                        dst = kv_slot_bf16(a.branches->kv[b], a.layer, which - 1, head, a.n_heads, a.branches->pos0[b] + tk);
                    }
                    *(u32x4*)(dst + f) = lo;
                    *(u32x4*)(dst + f + 64) = hi;
                }
            }
        }
    }
}

template <int EPI, int MB, int WN, int WK>
hipError_t launch(GemmArgs a, hipStream_t s) {
    using S = WideShape<MB, WN, WK>;
    a.n_tiles = (a.N + S::COLS - 1) / S::COLS;
    a.m_tiles = (a.M + 32 * MB - 1) / (32 * MB);
    a.by_m.set(a.m_tiles);
    a.by_n.set(a.n_tiles);
    a.by_splits.set(a.splits);
    const dim3 grid(a.n_tiles * a.m_tiles * a.splits);
    if (a.m_tiles == 1 && !a.shared_gpu)
        hipLaunchKernelGGL((gemm_w4_wide<EPI, MB, WN, WK, true>), grid, dim3(S::THREADS), S::LDS_BYTES, s, a);
    else
        hipLaunchKernelGGL((gemm_w4_wide<EPI, MB, WN, WK, false>), grid, dim3(S::THREADS), S::LDS_BYTES, s, a);
    return hipGetLastError();
}

template <int EPI>
hipError_t dispatch(const GemmArgs& a, hipStream_t s) {
    const WidePick p = wide_shape(EPI, a.n_tok, a.M, a.N, a.K);
    GemmArgs b = a;
    b.splits = p.splits;
#define X(MB, WN, WK) \
    if (p.c.mb == MB && p.c.wn == WN && p.c.wk == WK) return launch<EPI, MB, WN, WK>(b, s);
    JUP_WIDE_SHAPES(X)
#undef X
    return hipErrorInvalidConfiguration;
}
template <int EPI, int MB, int WN, int WK>
hipError_t configure_one() {
    using S = WideShape<MB, WN, WK>;
    hipError_t e = hipFuncSetAttribute((const void*)gemm_w4_wide<EPI, MB, WN, WK, true>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS_BYTES);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute((const void*)gemm_w4_wide<EPI, MB, WN, WK, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               S::LDS_BYTES);
}

}  // namespace

hipError_t launch_gemm_w4_wide(int epi, const GemmArgs& a, hipStream_t s) {
    if (a.M <= 0 || a.n_tok <= 0 || a.N % 64 || a.K % 128) return hipErrorInvalidValue;
    return epi == EPI_QKV ? dispatch<EPI_QKV>(a, s) : epi == EPI_SWIGLU ? dispatch<EPI_SWIGLU>(a, s) : dispatch<EPI_PARTIAL>(a, s);
}

hipError_t w4_wide_configure() {
    hipError_t e = hipSuccess;
    auto acc = [&](hipError_t r) { if (e == hipSuccess) e = r; };
#define X(MB, WN, WK) \
    acc(configure_one<EPI_QKV, MB, WN, WK>()); acc(configure_one<EPI_SWIGLU, MB, WN, WK>()); acc(configure_one<EPI_PARTIAL, MB, WN, WK>());
    JUP_WIDE_SHAPES(X)
#undef X
    return e;
}

}  // namespace jup
