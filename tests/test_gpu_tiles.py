"""GPU parity of kernels and launch rules at the sizes where they can go wrong (edges of tiles, remainders, the smallest
and largest of a range), against the CPU oracle; the bars of test_gpu_parity.py."""
import numpy as np
import pytest

from helpers import Pair
from paper_2504_08242_amd import binding as jb
from paper_2504_08242_amd import synth_inputs as si

pytestmark = pytest.mark.gpu


TALL_TILES = [
    (256, 2, 128, 129, {"gemm_gate_up": "8,3,4,1"}),
    (1024, 8, 128, 129, {"gemm_gate_up": "4,3,4,1"}),
    (1024, 8, 2816, 129, {"gemm_qkv": "4,3,4,1", "gemm_o": "4,4,4,2"}),
    (1024, 8, 2688, 257, {"gemm_gate_up": "4,4,4,2"}),
    (1024, 8, 4096, 961, {"gemm_gate_up": "8,4,4,2"}),
    (1024, 8, 2816, 1025, {"gemm_qkv": "4,4,4,2", "gemm_gate_up": "6,6,2,2", "gemm_down": "4,6,4,2"}),
    (1024, 8, 4096, 1297, {"gemm_gate_up": "6,8,2,4"}),
    (1024, 8, 2688, 2065, {"gemm_down": "8,4,4,2"}),
    (1536, 12, 4224, 607, {"gemm_gate_up": "4,6,4,2"}),
    (1536, 12, 4224, 897, {"gemm_qkv": "6,6,2,2"}),
    (1792, 14, 6272, 513, {"gemm_down": "4,8,2,4"}),
    (1792, 14, 128, 961, {"gemm_qkv": "4,6,4,2"}),
    (1792, 14, 128, 2321, {"gemm_qkv": "8,8,4,2"}),
    (2048, 16, 5632, 641, {"gemm_qkv": "6,4,2,2", "gemm_down": "6,4,2,2"}),
    (2048, 16, 5632, 1025, {"gemm_gate_up": "8,8,4,2", "gemm_down": "8,6,4,2"}),
    (2048, 16, 128, 1937, {"gemm_qkv": "8,6,4,2"}),
    (2304, 18, 6272, 257, {"gemm_gate_up": "6,4,2,2"}),
    (4096, 32, 11008, 639, {"gemm_qkv": "4,8,2,4", "gemm_gate_up": "4,8,2,4", "gemm_down": "6,8,2,4"}),
    (4096, 32, 11008, 893, {"gemm_qkv": "6,8,2,4", "gemm_gate_up": "8,6,4,2", "gemm_down": "8,8,4,2"}),
    (4352, 34, 128, 385, {"gemm_qkv": "8,4,4,2"}),
    (1536, 12, 11008, 539, {"gemm_gate_up": "9,6,4,2"}),     # a row block and 27 rows more than 256-row tiles hold
    (1024, 8, 8192, 1121, {"gemm_gate_up": "9,8,4,2"}),
    (1024, 8, 11008, 1239, {"gemm_gate_up": "8,8+6,4,2"}),   # tiles of two widths
    (1536, 12, 11008, 1755, {"gemm_gate_up": "8,8+4,4,2"}),
]
EPILOGUE = {"gemm_qkv": 0, "gemm_o": 1, "gemm_down": 1, "gemm_gate_up": 2}
# test_gemm_plan.py replays the plans: whatever other chunk lengths of these stages run is among them
COVERED = {f"gemm_bf16<{tile},{EPILOGUE[kernel]}>" for *_, tiles in TALL_TILES for kernel, tile in tiles.items()}


@pytest.mark.parametrize("d_model,n_heads,d_ffn,rows,tiles", TALL_TILES)
def test_bf16_tall_tiles(d_model, n_heads, d_ffn, rows, tiles):
    """Every tile of the projections of chunks above 128 rows, with a ragged last row block and a short prefix."""
    cfg = dict(si.LLAMA7B_STAGE, d_model=d_model, n_heads=n_heads, d_ffn=d_ffn, n_layers=1)
    p = Pair(cfg, "bf16", seed=rows, max_positions=rows + 7, max_chunk_tokens=rows)
    for kernel, tile in tiles.items():
        name = p.stage.kernel_name(jb.KERNEL_IDS[kernel], rows)
        assert name.startswith(f"gemm_bf16<{tile},"), (kernel, name)
    hidden = p.hidden(rows + 7)
    g, o = p.run_both(hidden, [7, rows])
    p.check(g[7:], o[7:], f"{rows} rows of d {d_model}")
    p.check(p.kv_gpu()[0], p.oracle.kv[0], "cache")


@pytest.mark.parametrize("rows", [1, 4, 5, 15, 17, 29, 33, 40, 61, 64, 65, 77, 100, 127])
def test_bf16_rows_that_do_not_exist(rows):
    """Tiles of up to 128 rows leave out the rows past the chunk: what LDS holds there reaches no row of the chunk.  Groups of four
    rows, halves of row blocks and whole blocks.  The first projection finds NaN there where a chunk of another cache left it,
    the later ones whatever kernels of the chunk itself did; test_tile_index.py has the masks."""
    cfg = dict(si.LLAMA7B_STAGE, d_model=512, n_heads=4, d_ffn=1408, n_layers=2)
    p = Pair(cfg, "bf16", seed=rows, max_positions=rows + 7, max_chunk_tokens=128)
    other = jb.KvCache(cfg, "bf16", 128)
    hidden = p.hidden(rows + 7)
    p.gpu_chunk(hidden[:7], 0)
    p.oracle.prefill_chunk(hidden[:7], 0)
    p.gpu_chunk(np.full((128 if rows > 64 else 64, cfg["d_model"]), np.nan, hidden.dtype), 0, other)
    p.check(p.gpu_chunk(hidden[7:], 7), p.oracle.prefill_chunk(hidden[7:], 7), f"{rows} rows")
    p.check(p.kv_gpu()[1], p.oracle.kv[1], "cache")


HALF_TILES = {   # (d_model, d_ffn, rows): tiles of QKV and gate/up
    (2048, 2816, 33): ("2,1.5,2,2", "2,1.5,2,2"), (2048, 4224, 47): ("2,1.5,2,2", "2,1.5,2,2"), (2048, 1408, 64): ("2,1.5,2,2", "2,1.5,2,2"),
    (4096, 256, 40): ("2,1.5,2,2", "2,1.5,2,2"), (512, 5632, 24): ("2,2,2,2", "2,1.5,2,2"), (512, 4864, 9): ("2,2,2,2", "2,1.5,2,2"),
}


@pytest.mark.parametrize("d_model,d_ffn,rows", HALF_TILES)
def test_bf16_tiles_of_half_column_blocks(d_model, d_ffn, rows):
    """48-column tiles of QKV (33 to 64 rows; 128 workgroups and 256, the ends of their range) and of gate/up (column blocks that
    are a multiple of three, one and two more; fewer rows on 203 and 235 workgroups) against the oracle, and a batch of
    branches against each of them alone, which runs on other tiles: the same bits."""
    import torch
    cfg = dict(si.LLAMA7B_STAGE, d_model=d_model, n_heads=d_model // 128, d_ffn=d_ffn, n_layers=1)
    p = Pair(cfg, "bf16", seed=rows, max_positions=rows + 7, max_chunk_tokens=64)
    n = 8 if rows % 8 == 0 else 3
    tok = rows // n
    names = [[p.stage.kernel_name(jb.KERNEL_IDS[k], m) for k in ("gemm_qkv", "gemm_gate_up")] for m in (rows, n * tok, tok)]
    for m, name in zip((rows, n * tok), names):
        assert name == [f"gemm_bf16<{tile},{e}>" for e, tile in zip((0, 2), HALF_TILES[d_model, d_ffn, rows])], m
    assert "1.5" not in names[2][0] + names[2][1], names[2]
    hidden = p.hidden(rows + 7)
    g, o = p.run_both(hidden, [7, rows])
    p.check(g[7:], o[7:], "chunk")
    p.check(p.kv_gpu()[0], p.oracle.kv[0], "cache")
    x = torch.from_numpy(hidden[7:7 + n * tok]).to("cuda:0", p.td)
    whole, alone = ([p.kv.fork(7, 7 + tok) for _ in range(n)] for _ in range(2))
    got = p.stage.prefill_branches(x, tok, [7] * n, whole)
    for b in range(n):
        assert torch.equal(p.stage.prefill_chunk(x[b * tok:(b + 1) * tok].contiguous(), 7, alone[b]), got.view(n, tok, -1)[b]), b
        assert torch.equal(alone[b].view(), whole[b].view()), b


@pytest.mark.parametrize("d_model,d_ffn,rows,tiles", [(1024, 2816, 65, ("4,1,4,1", "4,1,4,1")), (1024, 4096, 127, ("4,1,4,1", "4,1,4,1")),
                                                      (1024, 4224, 120, ("4,1,4,1", "4,2,4,1")), (2816, 8192, 72, ("4,2,4,1", "4,2,4,1")),
                                                      (1536, 8320, 96, ("4,1,4,1", "4,3,4,1"))])
def test_bf16_narrow_tiles_of_128_rows(d_model, d_ffn, rows, tiles):
    """65 to 128 rows: the narrowest tile whose grid is one round of workgroups, at the ends of its range, against the oracle, and
    a batch of branches (whose rows come with a factor) against each of them alone: the same bits."""
    import torch
    cfg = dict(si.LLAMA7B_STAGE, d_model=d_model, n_heads=d_model // 128, d_ffn=d_ffn, n_layers=2)
    p = Pair(cfg, "bf16", seed=rows, max_positions=rows + 7, max_chunk_tokens=128)
    for kernel, tile in zip(("gemm_qkv", "gemm_gate_up"), tiles):
        assert p.stage.kernel_name(jb.KERNEL_IDS[kernel], rows).startswith(f"gemm_bf16<{tile},"), kernel
    hidden = p.hidden(rows + 7)
    g, o = p.run_both(hidden, [7, rows])
    p.check(g[7:], o[7:], "chunk")
    p.check(p.kv_gpu()[1], p.oracle.kv[1], "cache")
    if rows % 8:
        return
    n, tok = 8, rows // 8
    x = torch.from_numpy(hidden[7:]).to("cuda:0", p.td)
    whole, alone = ([p.kv.fork(7, 7 + tok) for _ in range(n)] for _ in range(2))
    got = p.stage.prefill_branches(x, tok, [7] * n, whole)
    for b in range(n):
        assert torch.equal(p.stage.prefill_chunk(x[b * tok:(b + 1) * tok].contiguous(), 7, alone[b]), got.view(n, tok, -1)[b]), b
        assert torch.equal(alone[b].view(), whole[b].view()), b


@pytest.mark.parametrize("dtype,layers,rows", [("bf16", 1, 17), ("bf16", 2, 300), ("w4", 1, 70), ("w4", 2, 33), ("bf16", 1, 16)])
def test_hidden_states_in_place(dtype, layers, rows):
    """The residual stream begins in the input buffer: a call that overwrites it with its output, against one that does not."""
    import torch
    cfg = dict(si.LLAMA7B_STAGE, d_model=512, n_heads=4, d_ffn=1408, n_layers=layers)
    p = Pair(cfg, dtype, seed=rows, max_positions=rows, max_chunk_tokens=rows)
    hidden = p.hidden(rows)
    x = torch.from_numpy(hidden).to("cuda:0", p.td)
    apart = p.stage.prefill_chunk(x, 0, p.kv)
    p.check(apart.float().cpu().numpy(), p.oracle.prefill_chunk(hidden, 0), "apart")
    p.stage.prefill_chunk(x, 0, p.kv, x)
    assert torch.equal(x, apart)


@pytest.mark.parametrize("dtype,n_lanes,chunks,limit", [
    ("bf16", 2, [70, 3, 129, 64, 300], 300),     # together, as one group
    ("bf16", 2, [250] * 9, 250),                 # several groups
    ("bf16", 3, [1025, 30, 1100, 5], 1100),      # side by side
    ("bf16", 0, [100, 17, 5], 100),              # one after the other
    ("w4", 4, [1100, 65, 1026], 1100),           # the bf16 copy of a 4-bit stage, side by side
])
def test_chunks_in_place(dtype, n_lanes, chunks, limit):
    """Several chunks of one call whose output overwrites its input, against a call with an output of its own."""
    import torch
    cfg = dict(si.LLAMA7B_STAGE, d_model=512, n_heads=4, d_ffn=1408, n_layers=2)
    total = sum(chunks)
    p = Pair(cfg, dtype, seed=total, max_positions=total, max_chunk_tokens=limit, w4_expanded=dtype == "w4")
    if n_lanes:
        p.stage.enable_overlap(n_lanes)
    x = torch.from_numpy(p.hidden(total)).to("cuda:0", p.td)
    apart = p.stage.prefill_chunks(x, chunks, 0, p.kv)
    cache = p.kv.view().clone()
    p.stage.prefill_chunks(x, chunks, 0, p.kv, x)
    assert torch.equal(x, apart)
    assert torch.equal(p.kv.view(), cache)


@pytest.mark.parametrize("dtype,layers", [("bf16", 1), ("bf16", 2), ("w4", 2)])
@pytest.mark.parametrize("branches,n", [(8, 5), (3, 5), (3, 33)])   # rows with a late factor, row projections, rows of their own norm
def test_branches_and_trees_in_place(dtype, layers, branches, n):
    import torch
    cfg = dict(si.LLAMA7B_STAGE, d_model=512, n_heads=4, d_ffn=1408, n_layers=layers)
    p = Pair(cfg, dtype, seed=branches, max_positions=128, max_chunk_tokens=128)
    p.gpu_chunk(p.hidden(20), 0)
    x = torch.from_numpy(p.hidden(branches * n, tag=1)).to("cuda:0", p.td)
    parents = si.make_token_tree(min(64, branches * n), 3)
    tree = x[:len(parents)].clone()
    forks = [[p.kv.fork(20, 20 + n) for _ in range(branches)] for _ in range(2)]
    apart = p.stage.prefill_branches(x, n, [20] * branches, forks[0])
    p.stage.prefill_branches(x, n, [20] * branches, forks[1], x)
    assert torch.equal(x, apart)
    for a, b in zip(*forks):
        assert torch.equal(a.view(), b.view())
        a.destroy()
        b.destroy()
    apart = p.stage.prefill_tree(tree, 20, parents, p.kv)
    p.stage.prefill_tree(tree, 20, parents, p.kv, tree)
    assert torch.equal(tree, apart)


@pytest.mark.parametrize("n_lanes,chunks,limit", [
    (2, [70, 3, 0, 129, 64, 300], 300),     # one group: row counts that are no multiple of a row block
    (2, [250] * 9, 250),                    # more rows than the lanes' buffer holds: several groups
    (4, [768, 768, 600, 1], 768),           # more than 2048 rows: groups of about the same height
    (3, [1025, 30, 1100, 5], 1100),         # a chunk above 1024 tokens: the lanes
])
def test_bf16_chunks_in_one_call(n_lanes, chunks, limit):
    """The multi-chunk call with overlap enabled against the oracle, behind a cached prefix, on a cache that is a fork."""
    import torch
    cfg = dict(si.LLAMA7B_STAGE, d_model=1024, n_heads=8, d_ffn=2816, n_layers=2)
    total = sum(chunks)
    p = Pair(cfg, "bf16", seed=limit, max_positions=total + 40, max_chunk_tokens=limit)
    p.stage.enable_overlap(n_lanes)
    hidden = p.hidden(total + 40)
    p.gpu_chunk(hidden[:40], 0)
    p.oracle.prefill_chunk(hidden[:40], 0)
    fork = p.kv.fork(40, total + 40)
    x = torch.from_numpy(hidden[40:]).to("cuda:0", p.td)
    y = p.stage.prefill_chunks(x, chunks, 40, fork)
    assert len(fork) == total + 40
    want = p.oracle.prefill_chunk(hidden[40:], 40)
    p.check(y.float().cpu().numpy(), want, "hidden states")
    kv = fork.view().float().cpu().numpy()
    for l in range(cfg["n_layers"]):
        p.check(kv[l], p.oracle.kv[l][:, :, 40:total + 40], f"cache layer {l}")
    again = p.stage.prefill_chunks(x, chunks, 40, fork)
    assert torch.equal(again, y)


@pytest.mark.parametrize("dtype", ["bf16", "w4"])
@pytest.mark.parametrize("n,pos,shared", [
    (1, 0, 0), (1, 31, 17), (15, 33, 32), (16, 240, 100), (17, 255, 255), (31, 256, 1), (33, 500, 490), (64, 700, 333),
    (5, 1100, 1024), (16, 2300, 0), (17, 2300, 2299),   # several key ranges per query block
    (65, 40, 0), (129, 700, 64), (256, 1, 0), (300, 5, 5),
])
def test_short_attention(dtype, n, pos, shared):
    """Query blocks of 16 and 32 rows (chunks of up to 64 tokens; some longer ones on key quarters beside them), partial blocks,
    key counts around a tile and around a second key range, forks whose border falls inside a tile, and the tree mask against
    the oracle."""
    cfg = dict(si.LLAMA7B_STAGE, d_model=256, n_heads=2, d_ffn=128, n_layers=1)
    p = Pair(cfg, dtype, seed=n + pos, max_positions=pos + n, max_chunk_tokens=max(n, 512))
    hidden = p.hidden(pos + n)
    p.run_both(hidden[:shared], [min(512, shared - i) for i in range(0, shared, 512)] or [0])
    kv = p.kv.fork(shared, pos + n) if shared else p.kv
    for lo in range(shared, pos, 512):
        h = hidden[lo:min(pos, lo + 512)]
        p.gpu_chunk(h, lo, kv)
        p.oracle.prefill_chunk(h, lo)
    h = hidden[pos:]
    first = p.gpu_chunk(h, pos, kv)
    p.check(first, p.oracle.prefill_chunk(h, pos), "chunk")
    assert np.array_equal(p.gpu_chunk(h, pos, kv), first)
    if n <= 64:
        parents = si.make_token_tree(n, 3)
        p.check(p.gpu_tree(h, pos, parents, kv), p.oracle.prefill_tree(h, parents, pos), "tree")


@pytest.mark.parametrize("d_model,n_heads,d_ffn", [
    (256, 2, 128),       # fewer K steps than ranges: some are empty
    (2304, 18, 1408),    # ranges of unequal length, four splits
    (5120, 40, 3456),    # two splits
])
@pytest.mark.parametrize("dtype", ["bf16", "w4"])
def test_row_projections(dtype, d_model, n_heads, d_ffn):
    """Output and down projections of calls of up to 16 rows and of batches of such branches (17 to 64 rows), two layers deep
    (the norm between them is a factor of the rows): against the oracle, and a branch has the same bits alone, batched within
    16 rows and batched beyond."""
    import torch
    cfg = dict(si.LLAMA7B_STAGE, d_model=d_model, n_heads=n_heads, d_ffn=d_ffn, n_layers=2)
    p = Pair(cfg, dtype, seed=d_model, max_positions=48, max_chunk_tokens=64)
    for n in (1, 15, 16, 17):
        g, o = p.run_both(p.hidden(20 + n, tag=n), [20, n])
        p.check(g, o, f"{n} rows")
        p.check(p.kv_gpu()[:, :, :, :20 + n], p.oracle.kv[:, :, :, :20 + n], f"cache, {n} rows")
    for branches, n in ((3, 5), (16, 1), (9, 2), (2, 9), (11, 3), (4, 16)):
        h = p.hidden(branches * n, tag=100 + n).reshape(branches, n, d_model)
        alone = [p.gpu_chunk(h[b], 20) for b in range(branches)]
        kvs = [p.kv.fork(20, 40) for _ in range(branches)]
        y = p.stage.prefill_branches(torch.from_numpy(h.reshape(-1, d_model)).to("cuda:0", p.td), n, [20] * branches, kvs)
        y = y.float().cpu().numpy().reshape(branches, n, d_model)
        for b in range(branches):
            assert np.array_equal(y[b], alone[b]), (branches, n, b)
        for kv in kvs:
            kv.destroy()


@pytest.mark.parametrize("n,branches", [(65, 3), (100, 2), (128, 4), (129, 2), (200, 3), (256, 2), (300, 2)])
@pytest.mark.parametrize("pos", [20, 1975, 2100])   # 1975: a second key range for 64 queries that the first 32 alone do not reach
def test_attention_of_long_branches_alone_and_batched(n, branches, pos):
    """Branches of more than 64 tokens: alone (32-query workgroups up to 128 tokens) and batched (64-query workgroups) the
    attention has the same bits, on a stage whose projections do not depend on the rows of the launch (4-bit codes)."""
    import torch
    cfg = dict(si.LLAMA7B_STAGE, d_model=256, n_heads=2, d_ffn=128, n_layers=1)
    p = Pair(cfg, "w4", seed=n, max_positions=pos + n, max_chunk_tokens=max(branches * n, 512))
    prefix = p.hidden(pos)
    for lo in range(0, pos, 512):
        p.gpu_chunk(prefix[lo:lo + 512], lo)
    h = p.hidden(branches * n, tag=1).reshape(branches, n, 256)
    alone = [p.gpu_chunk(h[b], pos) for b in range(branches)]
    kvs = [p.kv.fork(pos, pos + n) for _ in range(branches)]
    y = p.stage.prefill_branches(torch.from_numpy(h.reshape(-1, 256)).to("cuda:0", p.td), n, [pos] * branches, kvs)
    assert np.array_equal(y.float().cpu().numpy().reshape(branches, n, 256), np.stack(alone))


@pytest.mark.parametrize("one_call", [False, True])
@pytest.mark.parametrize("n", [1, 5, 16, 17, 33, 64, 65, 128, 129, 300, 1100])
def test_attention_of_peaked_rows_returns_the_value(n, one_call):
    """Every query sees only itself: queries and keys are 4 times the normalised rows, so its own score lies some 170 above
    all others.  The value row must come back exactly, whatever that score is: the largest probability takes no rounding.
    Values and output projection are the identity, the rest of the layer adds nothing, and the residual is too small to
    show."""
    d = 256
    cfg = dict(si.LLAMA7B_STAGE, d_model=d, n_heads=2, d_ffn=128, n_layers=1, rms_eps=0.0)
    layers = si.make_layers(cfg, seed=n, bf16=True)
    eye = np.eye(d, dtype=np.float32)
    layers[0].update(wq=4 * eye, wk=4 * eye, wv=eye, wo=eye, w_down=np.zeros((d, 128), np.float32), g_attn=np.ones(d, np.float32))
    p = Pair(cfg, "bf16", seed=n, max_positions=4 * n, max_chunk_tokens=n, layers_np=layers)
    h = p.hidden(4 * n) * np.float32(2.0 ** -50)
    if one_call:   # several chunks as one group, or (above 1024 tokens) beside each other
        import torch
        p.stage.enable_overlap(2)
        y = p.stage.prefill_chunks(torch.from_numpy(h).to("cuda:0", p.td), [n] * 4, 0, p.kv).float().cpu().numpy()
    else:
        y = np.concatenate([p.gpu_chunk(h[i:i + n], i) for i in range(0, 4 * n, n)])
    v = p.kv_gpu()[0, 1].transpose(1, 0, 2).reshape(4 * n, d)
    assert np.abs(v).max() > 1.0
    assert np.array_equal(y, v)


@pytest.mark.parametrize("d_model,n_heads,d_ffn", [(256, 2, 128), (2304, 18, 1408), (4096, 32, 11008), (5120, 40, 3456)])
@pytest.mark.parametrize("dtype", ["bf16", "w4"])
def test_batched_branches_of_more_than_64_rows_have_the_bits_they_have_alone(dtype, d_model, n_heads, d_ffn):
    """Batches of 65 to 128 rows (bf16 stages wider than 4096: up to 64) of branches of up to 16 tokens (row projections alone,
    partial sums of the same ranges batched, the norm's factor on either side); 4-bit codes at any row count and branch length."""
    import torch
    cfg = dict(si.LLAMA7B_STAGE, d_model=d_model, n_heads=n_heads, d_ffn=d_ffn, n_layers=2)
    p = Pair(cfg, dtype, seed=d_model, max_positions=160, max_chunk_tokens=320)
    p.gpu_chunk(p.hidden(20), 0)
    cases = [(13, 5), (16, 5), (5, 16), (6, 16), (7, 14), (8, 16), (16, 8)]
    if dtype == "bf16" and d_model > 4096:
        cases = [(12, 5), (8, 8), (4, 16)]
    codes = [(9, 16), (16, 16), (4, 17), (3, 33), (4, 64), (5, 64), (2, 65), (2, 130)]
    for branches, n in cases + (codes if dtype == "w4" else []):
        h = p.hidden(branches * n, tag=100 + n).reshape(branches, n, d_model)
        alone = [p.gpu_chunk(h[b], 20) for b in range(branches)]
        bits = p.kv.view()[:, :, :, 20:20 + n].clone()   # of the last branch
        kvs = [p.kv.fork(20, 20 + n) for _ in range(branches)]
        y = p.stage.prefill_branches(torch.from_numpy(h.reshape(-1, d_model)).to("cuda:0", p.td), n, [20] * branches, kvs)
        y = y.float().cpu().numpy().reshape(branches, n, d_model)
        assert np.array_equal(y, np.stack(alone)), (branches, n)
        assert torch.equal(kvs[-1].view(), bits), (branches, n)
        for kv in kvs:
            kv.destroy()


# test_tile_index.py replays the plans: every (row blocks, column blocks, K shares) of gemm_w4_wide with every epilogue is among them
W4_LONG_CHUNKS = [
    (256, 2, 128, [33, 65, 129]),               # fewer K groups than K shares
    (768, 6, 896, [64, 200, 513]),              # groups no multiple of the shares, column tiles past the matrix
    (1024, 8, 2816, [33, 65, 257, 384, 1024]),  # up to six K splits
    (2304, 18, 1408, [129, 513, 1024]),
    (4096, 32, 11008, [64]),                    # gate/up alone on gemm_w4_wide
    (5120, 40, 3456, [40, 200, 1024]),
]


@pytest.mark.parametrize("d_model,n_heads,d_ffn,rows", W4_LONG_CHUNKS)
def test_w4_projections_of_long_chunks(d_model, n_heads, d_ffn, rows):
    """4-bit codes, more than 32 tokens: rows on and beside the edges of the tiles of 64 and 128 rows, every tile shape with every
    epilogue, against the oracle, behind a cached prefix; the same bits twice."""
    cfg = dict(si.LLAMA7B_STAGE, d_model=d_model, n_heads=n_heads, d_ffn=d_ffn, n_layers=1)
    p = Pair(cfg, "w4", seed=d_model + 1, max_positions=max(rows) + 5, max_chunk_tokens=max(rows))
    for n in rows:
        p.kv.reset()
        p.oracle.reset()
        h = p.hidden(n + 5)
        p.gpu_chunk(h[:5], 0)
        y = p.gpu_chunk(h[5:], 5)
        want = p.oracle.prefill_chunk(h, 0)
        p.check(y, want[5:], f"{n} rows")
        p.check(p.kv_gpu()[:, :, :, :n + 5], p.oracle.kv[:, :, :, :n + 5], f"cache, {n} rows")
        assert np.array_equal(p.gpu_chunk(h[5:], 5), y), n


@pytest.mark.parametrize("rows", [1280, 1281])
def test_attention_of_long_chunks_around_one_round_of_workgroups(rows):
    """64-query workgroups, 320 and 336 of them, with a ragged last tile, behind a cached prefix: on a stage whose call stays in the
    last-level cache (one barrier per round), and, to the bit, on one with more layers that goes through 340 MB (320 of them: K
    and V parts of a tile apart)."""
    cfg = dict(si.LLAMA7B_STAGE, d_model=2048, n_heads=16, d_ffn=128, n_layers=2)
    p = Pair(cfg, "bf16", seed=rows, max_positions=rows + 471, max_chunk_tokens=rows)
    hidden = p.hidden(rows + 471)
    g, o = p.run_both(hidden, [471, rows])
    p.check(g[471:], o[471:], f"{rows} rows")
    long = Pair(dict(cfg, n_layers=7), "bf16", seed=rows, layers_np=p.layers_np + p.layers_np[:1] * 5, max_positions=rows + 471,
                max_chunk_tokens=rows)
    long.gpu_chunk(hidden[:471], 0)
    long.gpu_chunk(hidden[471:], 471)
    assert np.array_equal(long.kv_gpu()[:2], p.kv_gpu())


@pytest.mark.parametrize("d_model,n_heads,d_ffn,dtype,n_lanes,chunks,tiles", [
    # two chunks a second lane's scratch cannot hold together: side by side
    (1024, 8, 2816, "bf16", 2, [1024, 1024, 1000], {}),
    # short chunks between long ones: the tiles of short chunks that share the GPU
    (1024, 8, 2816, "bf16", 4, [1100, 64, 100, 300, 1050, 33, 128, 5],
     {("gemm_gate_up", 64): "2,6,2,3", ("gemm_gate_up", 100): "4,6,4,1", ("gemm_qkv", 100): "4,3,4,1", ("gemm_o", 33): "2,4,2,2",
      ("gemm_down", 128): "4,4,4,1", ("gemm_qkv", 1100): "8,2,4,1", ("gemm_o", 300): "8,8,4,2"}),
    (256, 2, 1024, "bf16", 3, [2065, 129, 1030], {("gemm_qkv", 129): "8,1,4,1", ("gemm_gate_up", 2065): "8,3,4,1"}),
    (512, 4, 2048, "bf16", 2, [1297, 300, 2065], {("gemm_gate_up", 1297): "8,4,4,2", ("gemm_gate_up", 2065): "8,8,4,2"}),
    (768, 6, 128, "bf16", 2, [1809, 769], {("gemm_qkv", 1809): "8,6,4,2", ("gemm_gate_up", 769): "8,2,4,1"}),
    (5632, 44, 128, "bf16", 2, [1025, 129], {("gemm_qkv", 129): "8,3,8,1"}),
    (1024, 8, 2816, "w4", 2, [1024, 1024], {}),                   # the bf16 copy of a 4-bit stage
    (1024, 8, 2816, "w4", 4, [1100, 65, 300, 1026], {}),
])
def test_chunks_beside_each_other(d_model, n_heads, d_ffn, dtype, n_lanes, chunks, tiles):
    """Chunks of one call on several streams: against the oracle, behind a cached prefix; three times the same bits (a chunk
    that did not wait for the cache entries of the one before would show as a run-to-run difference)."""
    import torch
    cfg = dict(si.LLAMA7B_STAGE, d_model=d_model, n_heads=n_heads, d_ffn=d_ffn, n_layers=2 if d_model <= 1024 else 1)
    total = sum(chunks)
    p = Pair(cfg, dtype, seed=total, max_positions=total + 70, max_chunk_tokens=max(chunks), w4_expanded=dtype == "w4")
    p.stage.enable_overlap(n_lanes)
    for (kernel, rows), tile in tiles.items():
        name = p.stage.kernel_name(jb.KERNEL_IDS[kernel], rows, True)
        assert name.startswith(f"gemm_bf16<{tile},"), (kernel, rows, name)
    hidden = p.hidden(total + 70)
    p.gpu_chunk(hidden[:70], 0)
    want = p.oracle.prefill_chunk(hidden, 0)
    x = torch.from_numpy(hidden[70:]).to("cuda:0", p.td)
    y = p.stage.prefill_chunks(x, chunks, 70, p.kv).clone()
    kv = p.kv.view().clone()
    p.check(y.float().cpu().numpy(), want[70:], "hidden states")
    p.check(kv.float().cpu().numpy(), p.oracle.kv, "cache")
    for _ in range(3):
        assert torch.equal(p.stage.prefill_chunks(x, chunks, 70, p.kv), y)
        assert torch.equal(p.kv.view(), kv)
