"""Which tiles the bf16 projections run on and what jup_diag_kernel_name calls them: the launch code itself on the host, with the
launch recorded instead of made (no GPU needed)."""
import collections

from test_tile_index import run_on_the_host

RECORDER = r"""
#include <cstdio>
#include <set>
#include <string>
#include "bf16_common.h"
struct Launched {
    int bmb, nb, wm, wn, epi, rest, half, grid;
    jup::GemmArgs a;
} launched;
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(kernel, blocks, threads, lds, stream, args) \
    launched = Launched{BMB, NB, WM, WN, EPI, REST, HALF, (int)(blocks).x, args}
#define hipGetLastError() hipSuccess
#define hipFuncSetAttribute(...) hipSuccess
#include "bf16_gemm.hip"

// Makes the launch of a projection of M rows; false where such rows take another kernel (row_gemm.hip).
bool launch(jup::GemmKind kind, int M, int d, int f, bool shared, const float* factor = nullptr) {
    jup::GemmArgs a{};
    a.M = M;
    a.N = kind == jup::GEMM_QKV ? 3 * d : kind == jup::GEMM_GATE_UP ? 2 * f : d;
    a.K = kind == jup::GEMM_DOWN ? f : d;
    a.shared_gpu = shared;
    a.row_factor = factor;
    launched = Launched{};
    if (kind == jup::GEMM_QKV) return jup::launch_gemm_qkv(a, nullptr) == hipSuccess;
    if (kind == jup::GEMM_GATE_UP) return jup::launch_gemm_swiglu(a, nullptr) == hipSuccess;
    return (M > jup::kMaxProjectRows || shared) && jup::launch_gemm_partial(a, nullptr) == hipSuccess;
}
std::string name(jup::GemmKind kind, int M, int d, int f, bool shared) {
    char buf[96];
    jup::gemm_kernel_name(kind, M, d, f, shared, buf, sizeof(buf));
    return buf;
}
constexpr jup::GemmKind kKinds[] = {jup::GEMM_QKV, jup::GEMM_O, jup::GEMM_GATE_UP, jup::GEMM_DOWN};
constexpr struct { int d, f; } kStages[] = {%s};
"""

NAMES = RECORDER + r"""
int main() {
    std::set<std::string> seen;
    const float factor = 1.f;
    for (auto st : kStages)
        for (int M = 1; M <= 2100; ++M)
            for (int shared = 0; shared < 2; ++shared)
                for (auto kind : kKinds) {
                    if (!launch(kind, M, st.d, st.f, shared)) continue;
                    const Launched l = launched;
                    char line[160];
                    snprintf(line, sizeof(line), "%%s|%%d,%%d,%%d,%%d,%%d rest %%d half %%d", name(kind, M, st.d, st.f, shared).c_str(), l.bmb, l.nb,
                             l.wm, l.wn, l.epi, l.rest, l.half);
                    if (seen.insert(line).second) puts(line);
                    // rows with a factor: the same tile
                    const bool wide = kind == jup::GEMM_QKV || kind == jup::GEMM_GATE_UP;
                    if (wide && !shared && M <= jup::kMaxSplitRows &&
                        (!launch(kind, M, st.d, st.f, false, &factor) || launched.bmb != l.bmb || launched.nb != l.nb ||
                         launched.half != l.half || launched.wm != l.wm))
                        printf("rows with a factor: %%d of %%d/%%d\n", M, st.d, st.f);
                    // every column has a tile, and the wide tiles of two widths lie in front of the others
                    const int wide_cols = l.a.n_tiles * l.a.n_stride, rest_wgs = l.rest ? l.grid - l.a.wide_tiles : 0;
                    const bool tiled = l.rest ? l.a.n_tiles > 0 && l.a.wide_tiles == l.a.n_tiles * l.a.m_tiles && wide_cols < l.a.N &&
                                                    rest_wgs %% l.a.m_tiles == 0 && wide_cols + rest_wgs / l.a.m_tiles * 32 * l.rest >= l.a.N
                                              : l.grid == l.a.m_tiles * l.a.n_tiles * l.a.splits && wide_cols >= l.a.N;
                    if (!tiled || l.a.m_tiles * 32 * l.bmb < M || (int)l.a.by_n.d != l.a.n_tiles) printf("columns: %%d of %%d/%%d\n", M, st.d, st.f);
                }
}
"""

PICKS = RECORDER + r"""
int main() {
    for (auto st : kStages)
        for (int M = %d; M < %d; M += %d)
            for (auto kind : kKinds) printf("%%d %%d %%d %%d %%s\n", st.d, st.f, M, (int)kind, name(kind, M, st.d, st.f, false).c_str());
}
"""
DISTINCT = RECORDER + r"""
int main() {
    std::set<std::string> names;
    for (auto st : kStages)
        for (int M = 129; M < 4097; ++M)
            for (auto kind : kKinds) names.insert(name(kind, M, st.d, st.f, false));
    for (const std::string& n : names) puts(n.c_str());
}
"""
KINDS = ["gemm_qkv", "gemm_o", "gemm_gate_up", "gemm_down"]


def stages(pairs):
    return ", ".join(f"{{{d}, {f}}}" for d, f in sorted(set(pairs)))


def picks(pairs, first, last, step, tmp_path):
    out = run_on_the_host(PICKS % (stages(pairs), first, last, step), tmp_path).split("\n")[:-1]
    return {(int(d), int(f), int(m), KINDS[int(k)]): name for d, f, m, k, name in (l.split(" ", 4) for l in out)}


def test_names_tell_the_kernels_apart(tmp_path):
    """Over widths and row counts, alone and beside other chunks: a name belongs to one instantiation and an instantiation to one
    name; every launch covers its rows and columns; a batch's rows with a factor take the tile of rows without."""
    pairs = [(256, 128), (512, 5632), (1024, 2816), (1536, 4224), (2048, 5632), (2816, 8192), (4096, 11008), (4352, 128), (5120, 13824), (5632, 128),
             (8192, 28672)]
    lines = run_on_the_host(NAMES % stages(pairs), tmp_path).splitlines()
    assert not (wrong := [l for l in lines if "|" not in l]), wrong[:10]
    tiles_of, names_of = collections.defaultdict(set), collections.defaultdict(set)
    for name, tile in (l.split("|") for l in lines):
        tiles_of[name].add(tile)
        names_of[tile].add(name)
    assert not (shared := {k: v for of in (tiles_of, names_of) for k, v in of.items() if len(v) > 1}), shared
    assert any("+" in name for name in tiles_of) and any(".5" in name for name in tiles_of)


HALF_TILES_END = [
    (2048, 5632, 32, "2,2,2,2", "2,1.5,2,2"), (2048, 5632, 33, "2,1.5,2,2", "2,1.5,2,2"), (2048, 5632, 64, "2,1.5,2,2", "2,1.5,2,2"),
    (2048, 5632, 65, "4,1,4,1", "4,2,4,1"), (2048, 5632, 8, "2,2,2,2", "1,3,1,3"), (2048, 5632, 9, "2,2,2,2", "2,1.5,2,2"),
    (2048, 4608, 24, "2,2,2,2", "1,3,1,3"), (2048, 4736, 24, "2,2,2,2", "2,1.5,2,2"),      # gate/up: 192 and 198 tiles
    (1792, 6144, 40, "2,2,2,2", "2,1.5,2,2"), (4096, 6272, 40, "2,1.5,2,2", "2,3,2,3"),     # 112 and 256; 256 and 262
    (4352, 128, 40, "2,2,2,2", "2,1.5,2,2"),                                                    # 272; 6
]


def test_rules_of_half_tiles_at_their_ends(tmp_path):
    got = picks([(d, f) for d, f, *_ in HALF_TILES_END], 1, 66, 1, tmp_path)
    for d, f, rows, qkv, gate_up in HALF_TILES_END:
        assert got[d, f, rows, "gemm_qkv"] == f"gemm_bf16<{qkv},0>", (d, f, rows)
        assert got[d, f, rows, "gemm_gate_up"] == f"gemm_bf16<{gate_up},2>", (d, f, rows)


GATE_UP_OF_LONG_CHUNKS = [   # (d_model, d_ffn, rows, tile): 288 rows and two widths where they measured faster, and only there
    (4096, 11008, 539, "9,6,4,2"), (4096, 11008, 1280, "8,8+6,4,2"), (4096, 11008, 2048, "8,8+6,4,2"), (5120, 13824, 2048, "8,8+4,4,2"),
    (1024, 11008, 1232, "8,8+6,4,2"), (5120, 13824, 800, "9,6,4,2"), (4096, 11008, 576, "9,6,4,2"),
    (4096, 11008, 1025, "6,6,2,2"), (4096, 11008, 1100, "6,6,2,2"), (4096, 11008, 1152, "6,6,2,2"),     # two widths: 169 -> 179 us
    (4096, 14336, 832, "6,6,2,2"), (5120, 13824, 912, "6,6,2,2"), (4096, 14336, 1850, "6,6,2,2"),
]


def test_gate_up_of_long_chunks_takes_the_measured_tile(tmp_path):
    got = picks([(d, f) for d, f, *_ in GATE_UP_OF_LONG_CHUNKS], 129, 2100, 1, tmp_path)
    wrong = [(d, f, rows, tile, name) for d, f, rows, tile in GATE_UP_OF_LONG_CHUNKS
             if (name := got[d, f, rows, "gemm_gate_up"]) != f"gemm_bf16<{tile},2>"]
    assert not wrong, wrong


def test_gpu_test_of_tall_tiles_runs_every_tile_of_its_stages(tmp_path):
    """A plan that leads one of those stages to another tile shows here; the comparison with the oracle does not depend on it."""
    from test_gpu_tiles import COVERED, TALL_TILES
    names = set(run_on_the_host(DISTINCT % stages((d, f) for d, _, f, *_ in TALL_TILES), tmp_path).splitlines())
    assert names == COVERED, names ^ COVERED
