// Projections back to d_model (output and down projection) for chunks of up to 16 rows and for batches of such chunks.
//
// A decode-sized layer is a chain of short launches, and two of the seven did nothing but add up the K splits of these
// projections and normalise a handful of rows: 4 - 5 us each for a few hundred KB.  Up to 16 rows project_rows finishes
// them in one launch, x += A W^T and with it everything the next projection needs of the norm that follows: a workgroup owns
// 16 output features and ALL of K (its eight waves split K and meet in LDS), so the sums are complete inside it: it adds
// the residual, writes the new residual stream and the rows bf16(x * g), and leaves the sum of squares of its 16 features.
// The norm's 1 / rms is a factor of the whole row and commutes with the projection: the next projection multiplies its
// results by it (RowScale in bf16_common.h adds up the d / 16 partial sums of squares of every row).
//
//   * 16 features per workgroup make d / 16 workgroups (256 for d = 4096: every CU), each streaming a contiguous 1 KB of
//     weights per wave and K step straight into registers, non-temporally (every weight is read once), a batch ahead.
//     The rows of A come from L2, 16 bytes per lane; rows past the chunk repeat its last one.
//   * At 16 rows a workgroup reads as many bytes of A as of bf16 weights, at 64 rows it would be four times as many and the
//     path from L2 bounds it (measured: O / down 14.9 / 34 us against 9.1 / 20.5 us + 4.8 us for each reduce + norm pass).
//     More rows (branches of up to 16 tokens in one call) keep K splits over workgroups, partial sums and the reduce + norm
//     pass: with bf16 weights, up to 128 rows, project_split below, tiles of 64 or 128 rows x 64 features through LDS; with
//     4-bit codes the kernel of w4_gemm.hip.
//   * Either way the MFMA, the ranges of K a sum is made of and the order they are added in are the same, whatever the row
//     count: a branch computes the same bits alone and batched with others.  bf16: MFMA 16x16x32, eight ranges, those of a
//     split added up first.  4-bit: the eight waves of every split.
//
// Measured on the 7B shapes at 5 rows (us, two K-split launches and two reduce + norm passes -> two launches): bf16
// 7.2 + 17.4 + 2 x 4.8 -> 7.7 + 17.4; 4-bit 3.7 + 9.2 + 2 x 4.3 -> 6.5 + 11.2, with four K groups in flight per wave and no division
// in front of them 5.6 + 9.9 (six 1 % slower, eight no different).  A whole call: 5 rows of eight bf16 layers
// 723 -> 681 us, one row of eight 4-bit layers 460 -> 416 us.  A batch of branches pays for the equal bits: 8 x 5 rows of two
// bf16 layers 203 -> 207 us.  Narrow stages, whose d / 16 workgroups leave CUs idle (64 of them for d = 1024, each walking all
// of K), gain more: their launches are short, and there are fewer.  Six layers, 1 / 16 rows, two launches and two passes -> two
// launches (with the first kernel of a call and the attention of short chunks as they are now): bf16 d = 1024 257 -> 198 /
// 263 -> 219 us, 2048 319 -> 273 / 346 -> 332, 4096 539 -> 496 / 585 -> 567; 4-bit d = 1024 202 -> 171 / 217 -> 186, 2048
// 224 -> 206 / 246 -> 223, 4096 332 -> 299 / 366 -> 332.
#include "bf16_common.h"

namespace jup {
namespace {

constexpr int kRowCols = 16;         // output features per workgroup of project_rows
constexpr int kRanges = 8;           // bf16: K ranges; 4-bit: K ranges per split
constexpr int kMaxRowSplits = 8;

// MFMA 16x16x32 (lane = 16 q + r): A: lane supplies A[m = r][k = 8 q + e], e < 8; B: B[k = 8 q + e][n = r];
// D: lane holds D[m = 4 q + i][n = r] in register i < 4.
__device__ inline f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

// bf16 weights, 16 features from feature f0 on, 16 rows, K range `range`: D = W A^T, a lane ends up with 4 features (4 q ..)
// of one row (r).
__device__ __forceinline__ f32x4 range_bf16(const RowArgs& a, int f0, int range, int lane) {
    constexpr int U = 8;  // K steps per batch; one batch is multiplied while the next is on its way
    const int r = lane & 15, q = lane >> 4;
    const int KT = a.K / 32;
    int s = range * KT / kRanges;
    const int s1 = (range + 1) * KT / kRanges;
    // a K step of 32 rows is a 2 KB block of the tiled layout, 16 rows are half of it (1 KB of consecutive bytes)
    const char* w_block = (const char*)a.W + (size_t)(f0 >> 5) * KT * 2048;
    const unsigned w_lane = 2 * (unsigned)tiled_offset((f0 & 16) + r, q, KT);
    const unsigned a_lane = 2 * (unsigned)tiled_offset(min(r, a.M - 1), q, KT);
    struct Batch {
        u32x4 w[U];
        bf16x8 a[U];
    };
    auto load = [&](Batch& b, int at, int u) __attribute__((always_inline)) {
        b.w[u] = load_once_at<u32x4>(w_block + (size_t)(at + u) * 2048, w_lane);
        b.a[u] = load_at<bf16x8>((const char*)a.A + (size_t)(at + u) * 2048, a_lane);
    };
    auto load_all = [&](Batch& b, int at) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) load(b, at, u);
    };
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const Batch& b, int u) __attribute__((always_inline)) {
        acc = mfma16(__builtin_bit_cast(bf16x8, b.w[u]), b.a[u], acc);
    };
    Batch even, odd;
    const int rem = (s1 - s) % U;  // the first, partial batch
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (u < rem) load(even, s, u);
    s += rem;
    if (s < s1) load_all(odd, s);
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (u < rem) multiply(even, u);
    while (s < s1) {
        if (s + U < s1) load_all(even, s + U);
#pragma unroll
        for (int u = 0; u < U; ++u) multiply(odd, u);
        s += U;
        if (s >= s1) break;
        if (s + U < s1) load_all(odd, s + U);
#pragma unroll
        for (int u = 0; u < U; ++u) multiply(even, u);
        s += U;
    }
    return acc;
}

// 4-bit codes (layout and arithmetic of w4_gemm.hip): a lane ends up with 4 rows (4 q ..) of one feature (r), whose scale it
// applies group by group.  The 8 x splits ranges are dealt to the eight waves, `splits` consecutive ones each; a range's sum
// goes to red[range] when its last group is done.
__device__ __forceinline__ void ranges_w4(const RowArgs& a, float (*red)[16 * kRowCols], int f0, int wave, int lane) {
    const int r = lane & 15, q = lane >> 4;
    const int G = a.K / 128;
    const int shift = __builtin_ctz(a.splits);  // (a power of two)
    auto first_group = [&](int R) {  // of range R: wave R % 8 of split R / 8
        const int split = R >> 3, ws0 = split * G >> shift, ws1 = (split + 1) * G >> shift;
        return ws0 + (R & 7) * (ws1 - ws0) / kRanges;
    };
    const int tile = f0 >> 6, cg = (f0 >> 4) & 3;  // 64-column tile of the packed codes, 16-column block in it
    const char* w_block = (const char*)a.W + ((size_t)tile * G * 4 + cg) * 1024;
    const char* s_block = (const char*)(a.w_scale + (size_t)tile * G * 64 + cg);
    const unsigned w_lane = lane * 16, s_lane = r * 16;
    const unsigned a_lane = 2 * (unsigned)tiled_offset(min(r, a.M - 1), q, a.K / 32);
    const u32x4 ones_bits = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
    const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_bits);
    const W4Bits bits;
    struct Group {
        u32x4 w;
        float sc;
        bf16x8 a[4];
    };
    auto load = [&](Group& d, int g) __attribute__((always_inline)) {
        d.w = load_once_at<u32x4>(w_block, w_lane + (unsigned)g * 4096);
        d.sc = load_at<float>(s_block, s_lane + (unsigned)g * 256);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            d.a[ks] = load_at<bf16x8>((const char*)a.A, a_lane + (unsigned)(4 * g + ks) * 2048);
    };
    // SETS groups in flight per wave, each set of registers filled again as soon as its products are issued.
    int g = first_group(wave * a.splits);
    const int g1 = first_group((wave + 1) * a.splits);
    int R = wave * a.splits, end = first_group(R + 1);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    auto close = [&]() __attribute__((always_inline)) {  // the sum of range R is complete
#pragma unroll
        for (int i = 0; i < 4; ++i) red[R][(4 * q + i) * kRowCols + r] = acc[i];
        acc = f32x4{0.f, 0.f, 0.f, 0.f};
        end = first_group(++R + 1);
    };
    auto multiply = [&](const Group& d, int at) __attribute__((always_inline)) {
        while (at == end) close();  // (ranges may be empty)
        f32x4 t = {0.f, 0.f, 0.f, 0.f}, rs = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            rs = mfma16(d.a[ks], ones, rs);
            t = mfma16(d.a[ks], w4_expand(d.w[ks], bits), t);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = w4_group(acc[i], d.sc, t[i], rs[i]);
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int SETS = 4;
    Group set[SETS];
    if (g1 - g < SETS) {
        // (a path of its own: the compiler counts the loads in flight path by path, and where they may or may not be there it
        // waits for all)
#pragma unroll
        for (int i = 0; i < SETS - 1; ++i)
            if (g + i < g1) load(set[i], g + i);
#pragma unroll
        for (int i = 0; i < SETS - 1; ++i)
            if (g + i < g1) multiply(set[i], g + i);
    } else {
#pragma unroll
        for (int i = 0; i < SETS; ++i) {
            load(set[i], g + i);
            __builtin_amdgcn_sched_barrier(0);
        }
        for (; g + 2 * SETS - 1 < g1; g += SETS) {
#pragma unroll
            for (int i = 0; i < SETS; ++i) {
                multiply(set[i], g + i);
                load(set[i], g + SETS + i);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        const int left = g1 - g;  // SETS to 2 SETS - 1
#pragma unroll
        for (int i = 0; i < SETS; ++i) {
            multiply(set[i], g + i);
            if (i + SETS < left) load(set[i], g + SETS + i);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < SETS - 1; ++i)
            if (i + SETS < left) multiply(set[i], g + SETS + i);
    }
    while (R < (wave + 1) * a.splits) close();
}

// x += eight range sums, PER of them to a split; HALVES: the two halves of a split are added up first
template <int PER, bool HALVES>
__device__ __forceinline__ void add_ranges(float4& x, const float (*red)[16 * kRowCols], int tid) {
    constexpr int HALF = HALVES && PER > 1 ? PER / 2 : PER;
    float4 p[kRanges];
#pragma unroll
    for (int w = 0; w < kRanges; ++w) p[w] = *(const float4*)&red[w][tid * 4];
    auto add = [](float4& to, const float4& v) { to.x += v.x; to.y += v.y; to.z += v.z; to.w += v.w; };
#pragma unroll
    for (int s = 0; s < kRanges; s += PER) {
#pragma unroll
        for (int h = s; h < s + PER; h += HALF) {
#pragma unroll
            for (int w = h + 1; w < h + HALF; ++w) add(p[h], p[w]);
            if (h > s) add(p[s], p[h]);
        }
        add(x, p[s]);
    }
}

template <bool W4>
__global__ __launch_bounds__(64 * kRanges) void project_rows(const RowArgs a) {
    extern __shared__ __attribute__((aligned(16))) float red_lds[];  // per range, [row][feature]
    float (*red)[16 * kRowCols] = (float (*)[16 * kRowCols])red_lds;
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // four features of one row per thread of the first wave: residual and gain are on their way while the products run
    const int row = tid >> 2, col = blockIdx.x * kRowCols + 4 * (tid & 3);
    const bool mine = tid < 64 && row < a.M;
    float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
    u32x2 g = {0, 0};
    if (mine) {
        x = *(const float4*)(a.x32 + (size_t)row * a.N + col);
        if (a.gain) g = *(const u32x2*)(a.gain + col);
    }
    if constexpr (W4) {
        ranges_w4(a, red, blockIdx.x * kRowCols, wave, lane);
    } else {
        const f32x4 acc = range_bf16(a, blockIdx.x * kRowCols, wave, lane);
        *(f32x4*)&red[wave][r * kRowCols + 4 * q] = acc;
    }
    __syncthreads();
    if (!mine) return;
    // sums of the splits, each added to the residual in turn
    if constexpr (W4) {
        for (int s = 0; s < a.splits; ++s) add_ranges<kRanges, false>(x, red + s * kRanges, tid);
    } else if (a.splits == 8) {
        add_ranges<1, true>(x, red, tid);
    } else if (a.splits == 4) {
        add_ranges<2, true>(x, red, tid);
    } else {
        add_ranges<4, true>(x, red, tid);
    }
    if (a.out) {  // the call's last projection: the stage's output
        u32x2 o;
        o[0] = pack_bf16x2(x.x, x.y);
        o[1] = pack_bf16x2(x.z, x.w);
        *(u32x2*)(a.out + (size_t)row * a.N + col) = o;
        return;
    }
    *(float4*)(a.x32 + (size_t)row * a.N + col) = x;
    u32x2 o;
    o[0] = pack_bf16x2(x.x * __uint_as_float(g[0] << 16), x.y * __uint_as_float(g[0] & 0xffff0000u));
    o[1] = pack_bf16x2(x.z * __uint_as_float(g[1] << 16), x.w * __uint_as_float(g[1] & 0xffff0000u));
    *(u32x2*)(a.xn + tiled_offset(row, col >> 3, a.N >> 5) + (col & 7)) = o;
    const float ss = sum_squares_16(x);  // (the four threads of a row are in or out together)
    if ((tid & 3) == 0) a.ssq[(size_t)row * (a.N / kRowCols) + blockIdx.x] = ss;
}

// Partial sums of batches, bf16 weights: a workgroup owns 32 RB rows x 64 features and the 8 / splits consecutive K ranges
// of its split; GROUPS = 2 groups of four waves take one half of them each (a wave 16 RB rows x 32 features) and add up at the
// end.  A group brings rows and weights through rings of its own in LDS, in pairs of K steps (the 32-row blocks of the tiled
// layout are LDS images), with one barrier per pair: 16 KB per pair and four pairs deep for up to 64 rows (RB = 2), 24 KB and
// three deep for more (RB = 4).  The launch is bound by streaming the weights as long as a pair's chain of wait, fragment reads
// and products stays short: with one group, whose chain nothing covers, the O / down launches took 9.9 / 23 us at 64 rows of
// the 7B shapes.  (RB = 4 with rows and weights in rings of their own, copied by different waves: rows one pair ahead and
// weights five 16 x 5 rows of two layers 264 -> 288 us, two and three ahead no difference.)
template <int RB>
struct SplitRing {
    static constexpr int STEP_BYTES = (RB + 2) * 2048;  // a K step: RB blocks of rows, two of weights
    static constexpr int PAIR_BYTES = 2 * STEP_BYTES;
    static constexpr int PAIRS = RB == 2 ? 4 : 3;
    static constexpr int LOADS = 2 * (RB / 2 + 1);      // per wave and pair
    static constexpr int BYTES = PAIRS * PAIR_BYTES;    // per group
};

// 1 KB per wave into LDS; NT: the weights, which are read once
template <bool NT>
__device__ __forceinline__ void load_unit(const char* uniform_base, unsigned lane_offset, unsigned lds) {
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt"
                     : : "v"(lane_offset), "s"(uniform_base), "s"(lds) : "memory", "m0");
    else load_to_lds_16(uniform_base, lane_offset, lds);
}

template <int GROUPS, int RB>
__global__ __launch_bounds__(256 * GROUPS) void project_split(const RowArgs a) {
    using R = SplitRing<RB>;
    extern __shared__ __attribute__((aligned(1024))) unsigned char ring[];
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const int wave8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = wave8 >> 2, wave = wave8 & 3, wm = wave & 1, wn = wave >> 1;
    const int KT = a.K / 32, split = blockIdx.y, per = kRanges / GROUPS >> __builtin_ctz(a.splits);  // ranges per group
    auto range_start = [&](int range) { return range * KT / kRanges; };
    auto count_of = [&](int g) { return range_start((split * GROUPS + g + 1) * per) - range_start((split * GROUPS + g) * per); };
    int range = (split * GROUPS + group) * per;
    const int first = range_start(range), count = count_of(group);  // K steps of this group
    const int pairs = (count + 1) / 2;
    const int rounds = GROUPS == 1 ? pairs : (max(count_of(0), count_of(1)) + 1) / 2;  // (the groups share the barriers)
    // A K step in LDS: RB 2 KB blocks of rows, two of weights.  Wave w copies half w & 1 of row blocks w >> 1, (w >> 1) + 2, ..
    // and the same half of weight block w >> 1.  Row blocks past the chunk repeat its last one.
    const char* a_src[RB / 2];
#pragma unroll
    for (int i = 0; i < RB / 2; ++i)
        a_src[i] = (const char*)a.A + ((size_t)min((wave >> 1) + 2 * i, (a.M - 1) >> 5) * KT + first) * 2048 + (wave & 1) * 1024;
    const char* w_src = (const char*)a.W + ((size_t)(blockIdx.x * 2 + (wave >> 1)) * KT + first) * 2048 + (wave & 1) * 1024;
    unsigned char* mine = ring + group * R::BYTES;
    const unsigned ring0 = __builtin_amdgcn_readfirstlane(lds_byte_address(mine));
    auto issue = [&](int pair) __attribute__((always_inline)) {  // R::LOADS loads per wave
        const unsigned dst = ring0 + (unsigned)pair % R::PAIRS * R::PAIR_BYTES + wave * 1024;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const size_t at = (size_t)min(2 * pair + h, count - 1) * 2048;
#pragma unroll
            for (int i = 0; i < RB / 2; ++i)
                load_unit<false>(uniform_ptr(a_src[i] + at), lane * 16, dst + h * R::STEP_BYTES + i * 4096);
            load_unit<true>(uniform_ptr(w_src + at), lane * 16, dst + h * R::STEP_BYTES + RB * 2048);
        }
    };
    for (int p = 0; p < R::PAIRS - 1 && p < pairs; ++p) issue(p);

    // fragment of 16 rows: chunk q of row r of the 16-row half
    unsigned off[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) off[h] = 2 * (unsigned)tiled_offset(16 * h + r, q, 1);
    f32x4 acc[2][RB], sum[2][RB];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < RB; ++j) acc[i][j] = sum[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto close_range = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < RB; ++j) {
                sum[i][j] += acc[i][j];
                acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
    };
    int boundary = range_start(range + 1) - first;
    for (int p = 0; p < rounds; ++p) {
        // pair p has landed when at most the loads of the pairs behind it are in flight (PAIRS - 2 of them, fewer at the end)
        if (R::PAIRS > 3 && p + 2 < pairs) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(2 * R::LOADS) : "memory");
        else if (p + 1 < pairs) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(R::LOADS) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();  // (every wave has read pair p - 1, whose slot is refilled now)
        if (p >= pairs) continue;
        if (p + R::PAIRS - 1 < pairs) issue(p + R::PAIRS - 1);
        const unsigned char* slot = mine + (unsigned)p % R::PAIRS * R::PAIR_BYTES;
        bf16x8 x[2][RB], w[2][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int j = 0; j < RB; ++j)
                x[h][j] = *(const bf16x8*)(slot + h * R::STEP_BYTES + ((wm * RB + j) >> 1) * 2048 + off[j & 1]);
#pragma unroll
            for (int i = 0; i < 2; ++i) w[h][i] = *(const bf16x8*)(slot + h * R::STEP_BYTES + (RB + wn) * 2048 + off[i]);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (2 * p + h < count) {
                while (2 * p + h == boundary) {  // (ranges may be empty)
                    close_range();
                    ++range;
                    boundary = range_start(range + 1) - first;
                }
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < RB; ++j) acc[i][j] = mfma16(w[h][i], x[h][j], acc[i][j]);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this wave has read the pair
    }
    close_range();
    if constexpr (GROUPS == 2) {  // the second group's sums through LDS
        __syncthreads();
        f32x4* other = (f32x4*)ring;
        const int t = threadIdx.x & 255;
#pragma unroll
        for (int i = 0; i < 2 * RB; ++i)
            if (group == 1) other[i * 256 + t] = sum[i / RB][i % RB];
        __syncthreads();
        if (group == 1) return;
#pragma unroll
        for (int i = 0; i < 2 * RB; ++i) sum[i / RB][i % RB] += other[i * 256 + t];
    }
    float* dst = a.partial + (size_t)split * a.M * a.N + blockIdx.x * 64 + wn * 32 + 4 * q;
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        const int row = wm * 16 * RB + 16 * j + r;
        if (row >= a.M) continue;
#pragma unroll
        for (int i = 0; i < 2; ++i) *(f32x4*)(dst + (size_t)row * a.N + 16 * i) = sum[i][j];
    }
}

bool bad(bool w4, const RowArgs& a, int rows) {
    return a.M < 1 || a.M > rows || a.N % 64 || a.N > 8192 || a.K % (w4 ? 128 : 32) || a.splits < 1 ||
           a.splits > kMaxRowSplits || (a.splits & (a.splits - 1)) || (!w4 && a.splits != row_splits(a.N));
}

}  // namespace

// As many splits (a divisor of the eight ranges) as keep the grid of 64-feature tiles within one round of workgroups (two up to
// the widest stage, 8192).
int row_splits(int N) {
    int splits = 2;
    while (splits < kRanges && N / 64 * splits * 2 <= 256) splits *= 2;
    return splits;
}

// 128 rows as long as a workgroup walks a quarter of K or less.  Measured against the partial-sum tiles that any other chunk
// takes (without the equal bits), batches of 72 to 128 rows, two layers: d = 1024 .. 4096 2 - 9 % faster (with the rest of the
// call), d = 5120 .. 8192, where two splits fill the chip, 3 - 5 % slower.
int max_split_rows(int N) { return row_splits(N) >= 4 ? kMaxSplitRows : 64; }

namespace {
template <int GROUPS, int RB>
hipError_t configure_split() {
    return hipFuncSetAttribute((const void*)project_split<GROUPS, RB>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               GROUPS * SplitRing<RB>::BYTES);
}

template <int GROUPS, int RB>
void run_split(const RowArgs& a, hipStream_t s) {
    hipLaunchKernelGGL((project_split<GROUPS, RB>), dim3(a.N / 64, a.splits), dim3(256 * GROUPS), GROUPS * SplitRing<RB>::BYTES, s, a);
}
}  // namespace

hipError_t rows_configure() {
    hipError_t e = configure_split<1, 2>();
    if (e == hipSuccess) e = configure_split<1, 4>();
    if (e == hipSuccess) e = configure_split<2, 2>();
    return e == hipSuccess ? configure_split<2, 4>() : e;
}

hipError_t launch_project_rows(bool w4, const RowArgs& a, hipStream_t s) {
    if (bad(w4, a, kMaxProjectRows)) return hipErrorInvalidValue;
    const int lds = (w4 ? a.splits : 1) * kRanges * 16 * kRowCols * 4;  // at most 64 KB
    hipLaunchKernelGGL(w4 ? project_rows<true> : project_rows<false>, dim3(a.N / kRowCols), dim3(64 * kRanges), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_project_split(const RowArgs& a, hipStream_t s) {
    if (bad(false, a, kMaxSplitRows)) return hipErrorInvalidValue;
    const bool two = a.splits < kRanges;  // one range per split leaves nothing to deal to a second group
    if (a.M <= 64) two ? run_split<2, 2>(a, s) : run_split<1, 2>(a, s);
    else two ? run_split<2, 4>(a, s) : run_split<1, 4>(a, s);
    return hipGetLastError();
}

}  // namespace jup
