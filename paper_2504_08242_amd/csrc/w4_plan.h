// Which kernel, tile and split of K a projection of a 4-bit stage runs as: rows per workgroup of gemm_w4 (w4_gemm.hip, up to 64
// tokens), tile shapes of gemm_w4_wide (w4_wide.hip, longer chunks and branches), and the line between the two.  Host code
// only.
#pragma once

#include "bf16_common.h"

namespace jup {

constexpr int W4_GROUP = 128;   // input features per scale
constexpr int W4_TILE_N = 64;   // columns per workgroup of gemm_w4
constexpr int W4_WAVES = 8;     // ... and waves, which share the K groups of a split

// Rows per workgroup, by rounds of workgroups: one per CU with 64 or 32 rows, two with 16.  16 where that is one workgroup per
// CU, or where a wave has a single K group and two workgroups fit; then 32 (whose codes are expanded once for twice the
// rows); then 16 on two workgroups per CU; then 64.  Measured on one MI355X (us): QKV of d_model 1024, 64 rows, 64 -> 16 per
// workgroup 9.4 -> 4.7; of d_model 2048, 64 -> 32 12.7 -> 7.4; O of d_model 5120, 48 rows, 64 -> 16 12.1 -> 9.5; O of the 7B
// shapes, 32 rows (one group per wave), 32 -> 16 5.6 -> 4.9, but QKV of those (four groups) 12.2 -> 13.3.  Whatever the rows, a
// result's sums are the same.
inline int w4_rows(int M, int N, int K, int splits) {
    const int wgs = N / W4_TILE_N * splits, groups = (K / W4_GROUP + splits * W4_WAVES - 1) / (splits * W4_WAVES);
    const int at_16 = wgs * ((M + 15) / 16), at_32 = wgs * ((M + 31) / 32);
    if (M <= 16 || at_16 <= 256 || (groups == 1 && at_16 <= 512)) return 16;
    if (M <= 32 || at_32 <= 256) return 32;
    return at_16 <= 512 ? 16 : 64;
}

// Splits of K for the projections back to d_model (their N / 64 column tiles alone do not occupy the chip): as many
// as keep the grid within about one workgroup per CU, at most 8 (the reduce + norm pass sums up to 8 partial
// buffers), and no more than leave every wave a K group: with fewer groups than waves a split only adds partial sums
// (and ranges to add up: one row of six layers of d_model 1024 157 -> 148 us).  More than
// 16 tokens, whose rows weigh on the path from L2, spread over the CUs all the same.
inline int w4_plan_splits(int n_tok, int N, int K) {
    const int tiles = N / W4_TILE_N, G = K / W4_GROUP;
    int splits = 1;
    while (splits < 8 && tiles * splits * 2 <= 256 && splits * 2 * (n_tok <= kMaxProjectRows ? W4_WAVES : 1) <= G) splits *= 2;
    return splits;
}

// (row blocks, column blocks = waves that share a K share, K shares)
#define JUP_WIDE_SHAPES(X) X(2, 1, 4) X(2, 2, 4) X(2, 3, 4) X(4, 4, 2) X(4, 8, 1)

// A launch is priced as rounds of workgroups (one per CU) times what a round takes: turns of the loop and a fixed part.  The
// constants are fitted to 900 timings of these shapes (33 .. 1024 rows, the projections of stages of d_model 1024, 2048,
// 4096, 5120 and 8192, all numbers of splits): 5 % off on average; the pick costs 0.4 % more than the best shape measured
// on average and 10 % at worst.
struct WideCost {
    int mb, wn, wk;
    float turn, round, qkv;  // us; qkv: more per round with the QKV epilogue
};
constexpr WideCost kWide[] = {{2, 1, 4, 1.37f, 1.4f, 1.2f}, {2, 2, 4, 1.54f, 2.3f, 1.4f}, {2, 3, 4, 1.96f, 3.1f, 1.3f},
                              {4, 4, 2, 1.92f, 4.3f, 1.8f}, {4, 8, 1, 1.66f, 6.1f, 2.3f}};
constexpr int kWideCUs = 256;
constexpr float kLaunchUs = 3.0f, kPartRound = 0.7f;
constexpr float kPartialUsPerByte = 1.0f / 5.2e6f;  // what the reduce + norm pass pays to read a partial sum back

inline int ceil_div(int x, int y) { return (x + y - 1) / y; }

inline float rounds_of(int wgs) {
    const int rest = wgs % kWideCUs;
    return (float)(wgs / kWideCUs) + (rest ? kPartRound + (1.f - kPartRound) * rest / kWideCUs : 0.f);
}
inline float wide_cost(const WideCost& c, int epi, int M, int N, int K, int splits) {
    const int wgs = ceil_div(M, 32 * c.mb) * ceil_div(N, 32 * c.wn) * splits;
    const int turns = ceil_div(ceil_div(K / 128, splits), c.wk);
    return kLaunchUs + rounds_of(wgs) * (c.turn * turns + c.round + (epi == EPI_QKV ? c.qkv : 0.f)) +
           (epi == EPI_PARTIAL ? 4.f * M * N * splits * kPartialUsPerByte : 0.f);
}

struct WidePick {
    WideCost c;
    int splits;
    float us;
};
// The order of a sum is a matter of the K shares and splits, so these are picked for the tokens of one chunk or branch, and
// the rest of the shape for the rows of the launch: a branch has the same bits alone and batched with others.
inline WidePick wide_pick(int epi, int n_tok, int N, int K) {
    WidePick best{};
    for (const WideCost& c : kWide)
        for (int splits : {1, 2, 3, 4, 6, 8}) {
            if (splits > 1 && (epi != EPI_PARTIAL || splits > K / 128 ||
                               ceil_div(n_tok, 32 * c.mb) * ceil_div(N, 32 * c.wn) * splits > 2 * kWideCUs)) continue;
            const float us = wide_cost(c, epi, n_tok, N, K, splits);
            if (best.splits == 0 || us < best.us) best = {c, splits, us};
        }
    return best;
}
// The shape for a launch of M rows: K shares and splits as picked for n_tok of them.
inline WidePick wide_shape(int epi, int n_tok, int M, int N, int K) {
    WidePick t = wide_pick(epi, n_tok, N, K);
    const int wk = t.c.wk;
    t.us = wide_cost(t.c, epi, M, N, K, t.splits);
    for (const WideCost& c : kWide) {
        const float us = wide_cost(c, epi, M, N, K, t.splits);
        if (c.wk == wk && us < t.us) t = {c, t.splits, us};
    }
    return t;
}

// What a launch of w4_gemm.hip takes on 64 rows (rounds of 64-column tiles of w4_rows rows, eight waves that split a K range;
// fitted to the same stages within 10 %).
inline float cost_of_rows(int epi, int N, int K) {
    const int splits = epi == EPI_PARTIAL ? w4_plan_splits(64, N, K) : 1;
    const int rows = w4_rows(64, N, K, splits);
    const float groups = (float)ceil_div(ceil_div(K / 128, splits), 8);
    const float round = rows == 64 ? 3.3f * groups + (epi == EPI_PARTIAL ? 1.5f : 2.6f) : (rows == 32 ? 1.9f : 1.0f) * groups + 0.2f;
    return kLaunchUs + rounds_of(N / 64 * splits * (64 / rows) / (rows == 16 ? 2 : 1)) * round + (epi == EPI_PARTIAL ? 4.f * 64 * N * splits * kPartialUsPerByte : 0.f);
}

// More than 64 tokens: always (1.0 - 2.5 times as fast over the stages above).  33 .. 64 tokens: where it is the faster one alone,
// e.g. gate/up of the 7B shapes 32 -> 22 us, QKV of d_model 8192 58 -> 39 us, down of the 13B shapes 25 -> 19 us; not QKV of
// d_model 1024, 4.0 -> 7.1 us (0.95: it is 33 rows, too, that have to gain, which w4_gemm.hip does a tenth faster than 64).
// Up to 32 tokens the kernel of w4_gemm.hip takes half the time (QKV of the 7B shapes 14 us, here 18).
inline bool w4_is_wide(int epi, int n_tok, int N, int K) {
    if (n_tok <= 32) return false;
    return n_tok > 64 || wide_pick(epi, 64, N, K).us <= 0.95f * cost_of_rows(epi, N, K);
}
// Partial sums that the projections back to d_model leave to the reduce + norm pass.
inline int w4_partial_splits(int n_tok, int N, int K) {
    return w4_is_wide(EPI_PARTIAL, n_tok, N, K) ? wide_pick(EPI_PARTIAL, n_tok, N, K).splits : w4_plan_splits(n_tok, N, K);
}

}  // namespace jup
