// Projections of a stage whose matrices are stored as 4-bit codes (JUP_BF16_W4): C[M, N] = A[M, K] * W[N, K]^T with
// W[n][k] = scale[n][k / 128] * (code[n][k] - 8), for decode-sized chunks (Jupiter paper, Sec. V: a decoding step
// feeds a handful of tokens per sequence, so a projection is bound by streaming its weights; Sec. VI-A: the paper
// runs its models with INT4 weights).  The kernel streams the codes, a quarter of the bf16 bytes, straight from
// global memory into registers and expands them there:
//
//   * A wave owns 16 RG rows x 64 columns (RG = 1, 2 or 4 row groups: one expansion of the codes serves up to 64
//     rows) and a range of K; the eight waves of a workgroup split the workgroup's K range, add their sums through
//     LDS in a fixed order and run the epilogue.  No barrier inside the K loop and no LDS traffic for the operands:
//     every wave streams on its own.
//   * v_mfma_f32_16x16x32_bf16.  Operand layout (lane = 16 q + r): A: lane supplies A[m = r][k = 8 q + e], e < 8;
//     B: lane supplies B[k = 8 q + e][n = r]; D: lane holds D[m = 4 q + i][n = r] in register i < 4, so a lane's
//     four results share one column and take one scale.
//   * Codes are stored per (64-column tile, 128-K group, 16-column block) as 1 KB: lane (r, q) owns 16 bytes, dword
//     ks holding the eight codes of column r for k = 128 g + 32 ks + 8 q + e.  Inside a dword, nibble p < 4 is
//     element 2 p and nibble p + 4 is element 2 p + 1, each as code ^ 8 (code - 8 in two's complement):
//     ((w >> 4 j) & 0x000F000F) ^ 0x43084308 is then the bf16 pair (128 + code[2 j], 128 + code[2 j + 1]) -- two
//     instructions per two weights, exact (a bf16 mantissa holds 128..255 in steps of one).  and + xor are one instruction
//     only if at most one of the constants is a literal (W4Bits).
//   * The offset of 136 = 128 + 8 leaves through the row sums of A: sum_k A[m][k] (128 + c) - 136 sum_k A[m][k].
//     The row sums of a group come from one more MFMA per K step against a register of ones, and a group's
//     result enters the fp32 accumulator as scale * (t - 136 * rowsum): 4 FMAs per lane, group and column block.
//     Products of a bf16 value and an integer below 256 are exact in fp32, the sums round as any fp32 sum does.
//   * A (16 rows of the tiled activation layout per row group) is read from L2 with 16-byte loads, up to 1 KB per
//     wave and K step; lanes whose row lies past the chunk repeat its last row.
#include "w4_plan.h"

namespace jup {
namespace {

enum { W4_PACK_PLAIN = 0, W4_PACK_QKV = 1, W4_PACK_GATE_UP = 2 };

// Packed column -> (source matrix 0..2, source row).  QKV: a 16-column block of a Q or K head holds the rotary
// indices 8u..8u+7 in its lanes 0..7 and their partners 64 + 8u.. in lanes 8..15 (u = block within the head);
// V keeps the same order.  Gate/up: even packed columns are gate rows, odd ones up rows.
__device__ inline void w4_source(int mode, int pc, int rows_per, int& which, int& row) {
    if (mode == W4_PACK_QKV) {
        which = pc / rows_per;
        const int in = pc - which * rows_per;
        const int head = in >> 7, u = (in & 127) >> 4, r = in & 15;
        row = head * 128 + (r < 8 ? 8 * u + r : 64 + 8 * u + (r - 8));
    } else if (mode == W4_PACK_GATE_UP) {
        which = pc & 1;
        row = pc >> 1;
    } else {
        which = 0;
        row = pc;
    }
}

// One workgroup per (column tile, K group): 4 column blocks x 64 lanes.
__global__ __launch_bounds__(256) void pack_w4(unsigned char* __restrict__ dst, float* __restrict__ dst_scale,
                                               const unsigned char* __restrict__ c0, const unsigned char* __restrict__ c1,
                                               const unsigned char* __restrict__ c2, const float* __restrict__ s0,
                                               const float* __restrict__ s1, const float* __restrict__ s2, int K,
                                               int rows_per, int mode) {
    const int G = K / W4_GROUP;
    const int tile = blockIdx.x / G, g = blockIdx.x - tile * G;
    const int cg = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    int which, row;
    w4_source(mode, tile * W4_TILE_N + cg * 16 + r, rows_per, which, row);
    const unsigned char* src = (which == 0 ? c0 : which == 1 ? c1 : c2) + (size_t)row * (K / 2);
    u32x4 out;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        const int k = g * W4_GROUP + 32 * ks + 8 * q;  // eight codes = four bytes, low nibble first
        const unsigned w = *(const unsigned*)(src + k / 2);
        unsigned v = 0;
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            const int e = p < 4 ? 2 * p : 2 * (p - 4) + 1;
            v |= (((w >> (4 * e)) & 0xFu) ^ 8u) << (4 * p);
        }
        out[ks] = v;
    }
    *(u32x4*)(dst + (((size_t)tile * G + g) * 4 + cg) * 1024 + lane * 16) = out;
    if (q == 0) {
        const float* ss = which == 0 ? s0 : which == 1 ? s1 : s2;
        dst_scale[(((size_t)tile * G + g) * 16 + r) * 4 + cg] = ss[(size_t)row * G + g];
    }
}

// What a wave fetches for one K group: the codes of its four column blocks and their scales, and four A fragments
// per row group.
struct W4Codes {
    u32x4 w[4];
    f32x4 sc;
};
template <int RG>
struct W4Rows {
    bf16x8 a[RG][4];
};

template <int EPI, int RG, int WAVES, bool STREAM_ONCE>
// (up to 16 rows: 128 registers per lane, so that two workgroups share a CU and the widest grids take one round)
__global__ __launch_bounds__(64 * WAVES, RG == 1 ? 4 : 2) void gemm_w4(const GemmArgs a) {
    __shared__ float red[WAVES][16][W4_TILE_N];
    __shared__ float scale_of_row[16];  // 1 / rms of up to 16 rows that come with partial sums of squares
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, q = lane >> 4;
    const int tile = blockIdx.x, split = blockIdx.y, rg0 = blockIdx.z * RG;
    const int G = a.K / W4_GROUP;
    // K groups of this workgroup, then of this wave (floor division: the shares differ by at most one group)
    // (splits is a power of two: 64-bit and other divisions here were 300 scalar instructions in front of the first load)
    const int shift = EPI == EPI_PARTIAL ? __builtin_ctz(a.splits) : 0;
    const int ws0 = split * G >> shift, ws1 = (split + 1) * G >> shift;
    const int cnt = ws1 - ws0;
    const int g0 = ws0 + wave * cnt / WAVES, g1 = ws0 + (wave + 1) * cnt / WAVES;

    const int k_stages = a.K / 32;
    // Rows past the chunk repeat its last one (no extra cache lines); their results are dropped.  With 64 rows the vector
    // instructions beside the MFMAs are what bounds a wave: one instruction instead of two per expanded dword, no execution
    // masks and zero fills around the loads of rows took the passes of a 512-row call on the 7B shapes from 184 to 157 us
    // (gate/up), 110 to 96 (QKV) and 77 to 70 (O / down, mean), one row of eight layers from 424 to 416 us.  (Tried and slower:
    // rows and codes of a group through LDS, shared by all waves in step, 178 - 205 us for gate/up.)
    unsigned a_lane[RG];
#pragma unroll
    for (int j = 0; j < RG; ++j) a_lane[j] = 2 * (unsigned)tiled_offset(min(16 * (rg0 + j) + r, a.M - 1), q, k_stages);
    // (constant bases and 32-bit offsets: left to move the bases along, the compiler holds 64-bit addresses per lane)
    const char* wbase = uniform_ptr((const char*)a.W + (size_t)tile * G * 4096);
    const char* sbase = uniform_ptr((const char*)(a.w_scale + (size_t)tile * G * 64));
    const W4Bits bits;
    // STREAM_ONCE (one pass over the codes, up to 64 rows): every code is read exactly once, with the non-temporal hint,
    // so that the stream does not push the KV cache and the activations out of the caches (measured at 5 rows per call:
    // the attention launch behind the projections 15.0 -> 12.2 us, a step of 8 branches 3.96 -> 3.62 ms).  More rows
    // take several passes, which find the codes in L2, and inside an overlapped call the other chunks' launches find them
    // in the caches (as for the bf16 kernels: not measured separately for the codes).
    auto fetch_codes = [&](W4Codes& d, int g) __attribute__((always_inline)) {
#pragma unroll
        for (int cg = 0; cg < 4; ++cg) {
            const unsigned at = (unsigned)g * 4096 + lane * 16 + cg * 1024;
            d.w[cg] = STREAM_ONCE ? load_once_at<u32x4>(wbase, at) : load_at<u32x4>(wbase, at);
        }
        d.sc = load_at<f32x4>(sbase, (unsigned)g * 256 + r * 16);
    };
    auto fetch_rows = [&](W4Rows<RG>& d, int g) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < RG; ++j)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                d.a[j][ks] = load_at<bf16x8>((const char*)a.A, a_lane[j] + (unsigned)g * 8192 + ks * 2048);
    };

    f32x4 acc[RG][4];
#pragma unroll
    for (int j = 0; j < RG; ++j)
#pragma unroll
        for (int cg = 0; cg < 4; ++cg) acc[j][cg] = f32x4{0.f, 0.f, 0.f, 0.f};
    const u32x4 ones_bits = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
    const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_bits);

    auto compute = [&](const W4Codes& c, const W4Rows<RG>& d) {
        f32x4 rs[RG];
#pragma unroll
        for (int j = 0; j < RG; ++j) {
            rs[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) rs[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(d.a[j][ks], ones, rs[j], 0, 0, 0);
        }
        const f32x4 sc = c.sc;
#pragma unroll
        for (int cg = 0; cg < 4; ++cg) {
            f32x4 t[RG];
#pragma unroll
            for (int j = 0; j < RG; ++j) t[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {  // one expansion of the codes serves every row group
                const bf16x8 b = w4_expand(c.w[cg][ks], bits);
#pragma unroll
                for (int j = 0; j < RG; ++j) t[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(d.a[j][ks], b, t[j], 0, 0, 0);
                if (RG == 1 && (ks & 1)) __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int j = 0; j < RG; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[j][cg][i] = w4_group(acc[j][cg][i], sc[cg], t[j][i], rs[j][i]);
            // 64 rows: one column block's expansion at a time.  Free to overlap them the compiler takes 250 registers, two waves
            // of which are a whole SIMD: not even a one-wave kernel of another stream fits beside a workgroup then, it keeps
            // a CU to itself, and a grid of 256 workgroups (O, down) takes a second round.  228 as here: 64-row call of
            // eight layers beside such a kernel 879 -> 786 us, alone 776 -> 772.  (16 rows: half a block at a time, for the
            // same reason: four waves of 128 registers.)
            if (RG == 4) __builtin_amdgcn_sched_barrier(0);
        }
    };

    const bool scaled = RG == 1 && EPI != EPI_PARTIAL && a.ssq;  // (the barriers in front of the epilogue publish the factors)
    RowScale<WAVES> sq;
    if (scaled) sq.template begin<true>(a.ssq, a.M, wave, lane, a.K);
    if constexpr (RG <= 2) {
        // Two groups in flight per wave, codes (from HBM) and rows (from L2), in two sets of registers that take turns: a
        // set is filled again as soon as its products are issued.  (As one set that is copied to the other the loads of a
        // group only started when the group before had landed, one trip to HBM per group: gate/up of one row of the 7B
        // shapes 14.1 -> 12.8 us, QKV 9.1 -> 8.1, with the shorter way to the first load.)
        struct Group {
            W4Codes c;
            W4Rows<RG> r;
        };
        Group even, odd;
        auto fetch = [&](Group& d, int g) __attribute__((always_inline)) {
            fetch_codes(d.c, g);
            fetch_rows(d.r, g);
        };
        // (a path of its own for a wave's only group: the compiler counts the loads in flight path by path, and where they may or
        // may not be there it waits for all)
        auto factors = [&]() __attribute__((always_inline)) {
            if (scaled) sq.finish(scale_of_row, a.M, wave, lane, a.K, a.rms_eps);  // (behind the loop its registers would spill)
        };
        if (g0 + 1 >= g1) {
            if (g0 < g1) fetch(even, g0);
            factors();
            if (g0 < g1) compute(even.c, even.r);
        } else {
            int g = g0;
            fetch(even, g);
            __builtin_amdgcn_sched_barrier(0);
            fetch_codes(odd.c, g + 1);
            __builtin_amdgcn_sched_barrier(0);
            factors();  // (in front of the rows: their registers are not there yet)
            __builtin_amdgcn_sched_barrier(0);
            fetch_rows(odd.r, g + 1);
            __builtin_amdgcn_sched_barrier(0);
            for (; g + 3 < g1; g += 2) {  // (fences: left alone the scheduler puts both products in front of both fetches)
                compute(even.c, even.r);
                __builtin_amdgcn_sched_barrier(0);
                fetch(even, g + 2);
                __builtin_amdgcn_sched_barrier(0);
                compute(odd.c, odd.r);
                __builtin_amdgcn_sched_barrier(0);
                fetch(odd, g + 3);
                __builtin_amdgcn_sched_barrier(0);
            }
            compute(even.c, even.r);  // two or three are left
            if (g + 2 < g1) fetch(even, g + 2);
            compute(odd.c, odd.r);
            if (g + 2 < g1) compute(even.c, even.r);
        }
    } else {
        // 64 rows: a group's rows are asked for when its turn comes, behind the next group's codes.  Loads return in order, so its
        // products wait for those codes too: one trip to memory per group.  (Codes in two sets that take turns, asked for behind
        // the rows, would stay in flight through the group: 240 registers, not measured.)
        W4Codes cur, nxt;
        W4Rows<RG> rows;
        if (g0 < g1) fetch_codes(cur, g0);
        for (int g = g0; g < g1; ++g) {
            if (g + 1 < g1) fetch_codes(nxt, g + 1);
            fetch_rows(rows, g);
            __builtin_amdgcn_sched_barrier(0);  // all on their way before the first wait (gate/up of 512 rows: 157 us, else 168)
            compute(cur, rows);
            cur = nxt;
        }
    }

    // ---- per row group: sum over the waves (fixed order), then the epilogue, one output row per wave and pass ----
    static_assert(16 % WAVES == 0, "the epilogue deals the 16 rows of a row group to the waves");
    const int n = lane;                    // 64 lanes = the 64 columns of the tile
    const int col = tile * W4_TILE_N + n;  // packed column
#pragma unroll
    for (int j = 0; j < RG; ++j) {
        if (j > 0) __syncthreads();  // the sums of the row group before have been read
        float2 cs[16 / WAVES];       // rotary table of this wave's rows, on its way while the sums meet
        const int rr = col & 15, feature = rr < 8 ? ((col & 127) >> 4) * 8 + rr : 64 + ((col & 127) >> 4) * 8 + (rr - 8);
        if constexpr (EPI == EPI_QKV)
#pragma unroll
            for (int pass = 0; pass < 16 / WAVES; ++pass)
                cs[pass] = a.rope[(size_t)min(16 * (rg0 + j) + wave + WAVES * pass, a.M - 1) * 64 + (feature & 63)];
#pragma unroll
        for (int cg = 0; cg < 4; ++cg)
#pragma unroll
            for (int i = 0; i < 4; ++i) red[wave][4 * q + i][16 * cg + r] = acc[j][cg][i];
        __syncthreads();
#pragma unroll
        for (int pass = 0; pass < 16 / WAVES; ++pass) {
            const int m = wave + WAVES * pass;
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) v += red[w][m][n];
            const int row = 16 * (rg0 + j) + m;
            if (scaled) v *= scale_of_row[m];
            else if (EPI != EPI_PARTIAL && a.row_factor) v *= a.row_factor[min(row, a.M - 1)];
            if (EPI == EPI_PARTIAL) {
                if (row < a.M) a.partial[((size_t)split * a.M + row) * a.N + col] = v;
            } else if (EPI == EPI_SWIGLU) {
                const float up = dpp_move<0xB1>(v);  // the odd neighbour holds the up projection of the same output
                if (!(n & 1) && row < a.M) {
                    const int oc = col >> 1;  // output feature
                    a.act[tiled_offset(row, oc >> 3, (a.N >> 1) >> 5) + (oc & 7)] =
                        f2bf(v * __builtin_amdgcn_rcpf(1.0f + __expf(-v)) * up);
                }
            } else {  // EPI_QKV
                const float other = dpp_move<0x128>(v);  // rotary partner (lanes 0..7 <-> 8..15 of a 16-column block)
                const int which = (col >= a.d_model) + (col >= 2 * a.d_model);
                const int in = col - which * a.d_model;
                const int head = in >> 7;
                float out = v;
                if (which != 2) out = rr < 8 ? v * cs[pass].x - other * cs[pass].y : v * cs[pass].x + other * cs[pass].y;
                if (row < a.M) {
                    u16* dst;
                    if (which == 0) {
                        dst = a.q_out + (size_t)row * a.d_model + head * 128;
                    } else if (!a.branches) {
                        dst = kv_slot_bf16(a.kv, a.layer, which - 1, head, a.n_heads, a.pos0 + row);
                    } else {
                        const int b = row / a.branches->n_tok, t = row - b * a.branches->n_tok;
                        dst = kv_slot_bf16(a.branches->kv[b], a.layer, which - 1, head, a.n_heads,
                                           a.branches->pos0[b] + t);
                    }
                    dst[feature] = f2bf(out);
                }
            }
        }
    }
}

template <int EPI, int RG>
hipError_t launch_rg(GemmArgs a, hipStream_t s) {
    // Eight waves per workgroup split its K range, whatever the row count: the order in which the K shares are summed
    // is then the same for a branch submitted alone and batched with others, and the two give the same bits.  Measured
    // on the 7B shapes at 64 rows per pass (228 registers per lane, so eight waves per CU either way): two workgroups of
    // four waves per CU run gate/up 4-5 % faster (its 344 workgroups then fit one round instead of two) and QKV 40 %
    // slower than one of eight; at 5 rows 4, 8 and 16 waves measured within 5 % of each other.
    constexpr int WAVES = W4_WAVES;
    a.n_tiles = a.N / W4_TILE_N;
    a.m_tiles = (a.M + 16 * RG - 1) / (16 * RG);
    const dim3 grid(a.n_tiles, a.splits, a.m_tiles);
    if (a.m_tiles == 1 && !a.shared_gpu) hipLaunchKernelGGL((gemm_w4<EPI, RG, WAVES, true>), grid, dim3(64 * WAVES), 0, s, a);
    else hipLaunchKernelGGL((gemm_w4<EPI, RG, WAVES, false>), grid, dim3(64 * WAVES), 0, s, a);
    return hipGetLastError();
}
template <int EPI>
hipError_t launch_one(GemmArgs a, hipStream_t s) {
    const int rows = w4_rows(a.M, a.N, a.K, a.splits);
    return rows == 16 ? launch_rg<EPI, 1>(a, s) : rows == 32 ? launch_rg<EPI, 2>(a, s) : launch_rg<EPI, 4>(a, s);
}

}  // namespace

hipError_t launch_gemm_w4(int epi, GemmArgs a, hipStream_t s) {
    if (a.M <= 0 || a.n_tok <= 0 || a.N % W4_TILE_N || a.K % W4_GROUP) return hipErrorInvalidValue;
    if (w4_is_wide(epi, a.n_tok, a.N, a.K)) return launch_gemm_w4_wide(epi, a, s);
    if (epi == EPI_PARTIAL) {
        a.splits = w4_plan_splits(a.n_tok, a.N, a.K);
        return launch_one<EPI_PARTIAL>(a, s);
    }
    a.splits = 1;
    return epi == EPI_QKV ? launch_one<EPI_QKV>(a, s) : launch_one<EPI_SWIGLU>(a, s);
}

void launch_pack_w4_qkv(unsigned char* dst, float* dst_scale, const void* cq, const void* ck, const void* cv,
                        const float* sq, const float* sk, const float* sv, int d, hipStream_t s) {
    hipLaunchKernelGGL(pack_w4, dim3(3 * d / W4_TILE_N * (d / W4_GROUP)), dim3(256), 0, s, dst, dst_scale,
                       (const unsigned char*)cq, (const unsigned char*)ck, (const unsigned char*)cv, sq, sk, sv, d, d,
                       (int)W4_PACK_QKV);
}
void launch_pack_w4_gate_up(unsigned char* dst, float* dst_scale, const void* cg, const void* cu, const float* sg,
                            const float* su, int d, int f, hipStream_t s) {
    hipLaunchKernelGGL(pack_w4, dim3(2 * f / W4_TILE_N * (d / W4_GROUP)), dim3(256), 0, s, dst, dst_scale,
                       (const unsigned char*)cg, (const unsigned char*)cu, (const unsigned char*)nullptr, sg, su,
                       (const float*)nullptr, d, 0, (int)W4_PACK_GATE_UP);
}
void launch_pack_w4_plain(unsigned char* dst, float* dst_scale, const void* c, const float* sc, int n_rows, int k,
                          hipStream_t s) {
    hipLaunchKernelGGL(pack_w4, dim3(n_rows / W4_TILE_N * (k / W4_GROUP)), dim3(256), 0, s, dst, dst_scale,
                       (const unsigned char*)c, (const unsigned char*)nullptr, (const unsigned char*)nullptr, sc,
                       (const float*)nullptr, (const float*)nullptr, k, 0, (int)W4_PACK_PLAIN);
}

}  // namespace jup
