"""Index arithmetic and plans of the kernels that the host compiler can run (no GPU needed)."""
import os
import shutil
import subprocess

import pytest

from paper_2504_08242_amd import build as jbuild

PROGRAM = r"""
#include <cstdio>
#include "bf16_common.h"
int main() {
    long bad = 0, n = 0;
    unsigned seed = 1;
    auto rnd = [&] { return seed = seed * 1664525u + 1013904223u; };
    auto check = [&](unsigned d, unsigned x) {
        if (d < 1 || d > 0x7fffffffu || x > 0x7fffffffu) return;
        jup::Quotient q;
        q.set((int)d);
        ++n;
        bad += q.of((int)x) != (int)(x / d);
    };
    for (unsigned d = 1; d < 70000; d += d < 600 ? 1 : 137)
        for (unsigned k : {0u, 1u, 2u, 3u, 255u, 256u, 65535u, 0x7fffffffu / d - 1, 0x7fffffffu / d})
            for (unsigned o : {0u, 1u, d - 1}) check(d, k * d + o);
    for (int i = 0; i < 4000000; ++i) check(rnd() >> (1 + rnd() % 31), rnd() >> 1);
    printf("%ld of %ld\n", bad, n);
    return bad != 0;
}
"""


BLOCKS = r"""
#include <cstdio>
#include <vector>
#include "bf16_common.h"
int main() {
    long bad = 0, n = 0;
    for (int heads : {1, 3, 8, 40})
        for (int blocks : {1, 2, 65535, 65536, 64 * 1024, 64 * 1025, 131070, 131071, 200001}) {
            const dim3 g = jup::chunk_grid(heads, blocks, 1);
            bad += g.y > 65535 || g.z != 1;
            std::vector<int> seen((size_t)heads * blocks);
            for (unsigned x = 0; x < g.x; ++x)
                for (unsigned y = 0; y < g.y; ++y) {
                    int head;
                    const int bq = jup::unfold_block(x, y, g.y, heads, head);
                    if ((int)x >= heads && bq >= blocks) continue;
                    if (head < 0 || head >= heads || bq >= blocks) ++bad;
                    else ++seen[(size_t)bq * heads + head];
                }
            for (int s : seen) n += 1, bad += s != 1;
        }
    printf("%ld of %ld\n", bad, n);
    return bad != 0;
}
"""


SHAPES = r"""
#include <cstdio>
#include "w4_plan.h"
int main() {
    struct { int d, f, n; } cases[] = {%s};
    for (auto c : cases) {
        struct { int epi, N, K; } projections[] = {{jup::EPI_QKV, 3 * c.d, c.d}, {jup::EPI_PARTIAL, c.d, c.d},
                                                   {jup::EPI_SWIGLU, 2 * c.f, c.d}, {jup::EPI_PARTIAL, c.d, c.f}};
        for (auto p : projections) {
            if (!jup::w4_is_wide(p.epi, c.n, p.N, p.K)) continue;
            const jup::WideCost t = jup::wide_shape(p.epi, c.n, c.n, p.N, p.K).c;
            printf("%%d,%%d,%%d,%%d\n", t.mb, t.wn, t.wk, p.epi);
        }
    }
#define X(MB, WN, WK) for (int epi = 0; epi < 3; ++epi) printf("built %%d,%%d,%%d,%%d\n", MB, WN, WK, epi);
    JUP_WIDE_SHAPES(X)
}
"""


LANES = r"""
#include <cstdio>
#include "bf16_common.h"
int main() {
    long bad = 0, n = 0;
    for (int M = 1; M <= 300; ++M)
        for (int first = 0; first < 320; first += 16) {
            const unsigned long long lanes = jup::row_lanes(M, first);
            for (int lane = 0; lane < 64; ++lane) {
                const int row = first + lane / 4;   // 16 bytes of a row of 64
                const bool brings_rows = row / 4 * 4 < M, keeps_count = first >= M && lane == 0;
                ++n, bad += (lanes >> lane & 1) != (brings_rows || keeps_count);
            }
            bad += lanes == 0;
        }
    printf("%ld of %ld\n", bad, n);
    return bad != 0;
}
"""


def run_on_the_host(program, tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not installed")
    src, exe = tmp_path / "program.hip", tmp_path / "program"
    src.write_text(program)
    flags = [f for f in jbuild.HIPCC_FLAGS if f not in ("-shared", "-c")]
    subprocess.run([hipcc, *flags, f"-I{jbuild.CSRC}", str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, stdout=subprocess.PIPE, text=True).stdout


def test_quotients_are_exact_for_every_index(tmp_path):
    """A multiplication and a compare instead of a division, against integer division."""
    assert run_on_the_host(PROGRAM, tmp_path).startswith("0 of")


def test_grid_of_chunk_attention_reaches_every_block_once(tmp_path):
    """Chunks and batches of branches with more query blocks than a grid's second dimension holds, and fewer.  Every
    launch uses this grid."""
    assert run_on_the_host(BLOCKS, tmp_path).startswith("0 of")
    source = open(os.path.join(jbuild.CSRC, "bf16_attention.hip")).read()
    launches = [l for l in source.splitlines() if "hipLaunchKernelGGL" in l and "chunk_attention_bf16" in l]
    assert len(launches) == 4 and all("chunk_grid(" in l for l in launches), launches


def test_masked_row_loads_bring_the_rows_of_the_chunk_and_keep_a_lane(tmp_path):
    """Loads of short-chunk tiles: every row of the chunk, no group of four rows past it, and never an empty mask (the waits of the ring
    count every load).  No other mask reaches such a load."""
    assert run_on_the_host(LANES, tmp_path).startswith("0 of")
    source = open(os.path.join(jbuild.CSRC, "bf16_gemm.hip")).read()
    masks = [l for l in source.splitlines() if "lanes[q] =" in l]
    assert len(masks) == 1 and masks[0].endswith("? row_lanes(a.M, m0 + j * 16) : ~0ull;"), masks
    for name in sorted(os.listdir(jbuild.CSRC)):
        if name.endswith((".h", ".hip")):
            lines = open(os.path.join(jbuild.CSRC, name)).read().splitlines()
            loads = [l for l in lines if "load_to_lds_16(" in l and "lanes" in l and "inline void" not in l]
            assert all(l.rstrip().endswith("lanes[q]);") for l in loads), (name, loads)
            assert sum("mov_b64 exec" in l for l in lines) == (name == "bf16_common.h"), name


def test_gpu_test_of_long_w4_chunks_runs_every_tile_shape(tmp_path):
    from test_gpu_tiles import W4_LONG_CHUNKS
    cases = ", ".join(f"{{{d}, {f}, {n}}}" for d, _, f, rows in W4_LONG_CHUNKS for n in rows)
    lines = run_on_the_host(SHAPES % cases, tmp_path).splitlines()
    built = {l.split()[1] for l in lines if l.startswith("built ")}
    assert len(built) == 15
    assert built == set(lines) - {l for l in lines if l.startswith("built ")}
