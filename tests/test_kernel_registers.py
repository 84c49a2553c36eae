"""What the compiler makes of kernels where it matters, from its own listing (no GPU needed): registers of the kernels whose workgroups
must leave room on a SIMD, address arithmetic of the QKV epilogue."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2504_08242_amd import build as jbuild


def test_4_bit_projections_leave_room_for_a_wave_of_another_stream(tmp_path):
    """Two waves of gemm_w4 share the 512 registers per lane of a SIMD (eight waves per workgroup, one workgroup per CU above 16
    rows).  With all 512 taken, a one-wave kernel beside the call keeps a CU to itself and a grid of one workgroup per CU
    takes a second round: at least 32 stay free."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not installed")
    out = tmp_path / "w4_gemm.s"
    subprocess.run([hipcc, *jbuild.HIPCC_FLAGS, "-S", "--offload-device-only", os.path.join(jbuild.CSRC, "w4_gemm.hip"), "-o", out],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    used = {}
    name = None
    for line in out.read_text().splitlines():
        if m := re.match(r"\s+\.name:\s+(\S*gemm_w4\S*)$", line):
            name = m.group(1)
        elif (m := re.match(r"\s+\.vgpr_count:\s+(\d+)$", line)) and name:
            used[name] = int(m.group(1))
            name = None
    assert len(used) == 18, sorted(used)   # three epilogues, 16 / 32 / 64 rows, codes read once or again
    for name, n in used.items():
        waves = 4 if "ELi1ELi8E" in name else 2          # per SIMD: two workgroups up to 16 rows, else one
        assert waves * ((n + 7) // 8 * 8) <= 512 - 32, (name, n)


def test_qkv_epilogue_makes_the_addresses_of_a_column_block_once(tmp_path):
    """Behind the K loop a column block has one query, key or value head for all its row blocks: its 64-bit cache address is made per
    block (in two forms), not again for every row block, and two neighbouring members of the arguments come with one load."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not installed")
    out = tmp_path / "bf16_gemm.s"
    subprocess.run([hipcc, *jbuild.HIPCC_FLAGS, "-S", "--offload-device-only", os.path.join(jbuild.CSRC, "bf16_gemm.hip"), "-o", out],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    kernels, lines = {}, None
    for line in out.read_text().splitlines():
        if m := re.match(r"_ZN\S*gemm_bf16ILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi0E\S*:", line):
            kernels[line] = lines = []
            columns = int(m.group(2)) // int(m.group(4))   # blocks of a wave
        elif re.match(r"\.Lfunc_end\d+:", line) and lines is not None:
            last = max(i for i, l in enumerate(lines) if "v_mfma" in l)
            wide = sum("s_mul_hi_u32" in l for l in lines[last:])
            assert wide <= 2 * columns, (wide, columns, list(kernels)[-1])
            lines = None
        elif lines is not None:
            lines.append(line)
    assert len(kernels) == 19, len(kernels)
    common = open(os.path.join(jbuild.CSRC, "bf16_common.h")).read()
    assert re.search(r"int n_stride;.*\n\s+int kt_per_split;", common)
