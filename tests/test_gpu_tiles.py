"""GPU parity of kernels and launch rules at the sizes where they can go wrong (edges of tiles, remainders, the smallest
and largest of a range), against the CPU oracle; the bars of test_gpu_parity.py."""
import numpy as np
import pytest

from helpers import Pair
from paper_2504_08242_amd import binding as jb
from paper_2504_08242_amd import synth_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_model,n_heads,d_ffn,rows,tiles", [
    (1024, 8, 2816, 129, {"gemm_qkv": "4,3,4,1", "gemm_o": "4,4,4,2"}),
    (1024, 8, 2816, 1025, {"gemm_qkv": "4,4,4,2", "gemm_gate_up": "6,6,2,2", "gemm_down": "4,6,4,2"}),
    (1536, 12, 4224, 607, {"gemm_gate_up": "4,6,4,2"}),
    (1536, 12, 4224, 897, {"gemm_qkv": "6,6,2,2"}),
    (2048, 16, 5632, 641, {"gemm_qkv": "6,4,2,2", "gemm_down": "6,4,2,2"}),
    (2048, 16, 5632, 1025, {"gemm_gate_up": "8,8,4,2", "gemm_down": "8,6,4,2"}),
    (4096, 32, 11008, 639, {"gemm_qkv": "4,8,2,4", "gemm_gate_up": "4,8,2,4", "gemm_down": "6,8,2,4"}),
    (4096, 32, 11008, 893, {"gemm_qkv": "6,8,2,4", "gemm_gate_up": "8,6,4,2", "gemm_down": "8,8,4,2"}),
])
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
