"""What the waits of kernels with direct global->LDS loads leave in flight, from the compiler's own listing of every instantiation
(no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2504_08242_amd import build as jbuild

SLOTS = 4   # of the ring: the rows of SLOTS - 1 stages are asked for in front of the loop
STAGES = 24  # of the loop that are walked: at least four rounds of its body


def listing(tmp_path, source, kernel):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not installed")
    out = tmp_path / "listing.s"
    subprocess.run([hipcc, *jbuild.HIPCC_FLAGS, "-S", "--offload-device-only", os.path.join(jbuild.CSRC, source), "-o", out],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    kernels, name = {}, None
    for line in out.read_text().splitlines():
        line = line.split(";")[0].strip()
        if m := re.match(rf"(_ZN\S*{kernel}\S*):$", line):
            kernels[name := m.group(1)] = []
        elif re.match(r"\.Lfunc_end\d+:$", line):
            name = None
        elif name and line and (not line.startswith(".") or line.endswith(":")):
            kernels[name].append(line)
    return kernels


def loop_path(lines):
    """The instructions from the kernel's entry through the prologue's barrier and those of STAGES stages, along the branches that
    stay in the loop (the way out of it waits for everything)."""
    labels = {l[:-1]: i for i, l in enumerate(lines) if l.endswith(":")}
    todo = [(0, [], 0)]
    while todo:
        i, path, barriers = todo.pop()
        while i < len(lines) and barriers <= STAGES:
            op, *args = lines[i].split()
            i += 1
            if op == "s_endpgm" or (barriers and op == "s_waitcnt" and "vmcnt(0)" in lines[i - 1]):
                break
            if op == "s_branch":
                i = labels[args[0]]
            elif op.startswith("s_cbranch"):
                todo.append((labels[args[0]], list(path), barriers))
            elif not op.endswith(":"):
                path.append(lines[i - 1])
                barriers += op == "s_barrier"
        if barriers > STAGES:
            return path
    raise AssertionError("no path through the loop")


def unlanded(path):
    """Replays the queue of loads (they return in order): the barriers behind whose wait some row of the stage they publish may
    still be in flight, as (barrier, loads in flight too many).  Barrier b publishes stage b.  Since the last load
    or barrier the loosest wait counts: tighter ones may be the compiler's, who does not know the row loads."""
    queue, rows, barriers = [], 0, [i for i, l in enumerate(path) if l == "s_barrier"]
    first = path[:barriers[0]]
    per_stage, rest = divmod(sum(l.startswith("global_load_lds") for l in first), SLOTS - 1)
    assert per_stage and not rest
    late, allowed = [], []
    for i, line in enumerate(path):
        if m := re.match(r"s_waitcnt.*vmcnt\((\d+)\)", line):
            allowed.append(int(m.group(1)))
        if line.startswith("global_load_lds"):
            allowed = []
            queue.append(rows // per_stage)
            rows += 1
        elif re.match(r"(global|buffer|flat|scratch)_(load|store|atomic)", line):
            assert line.startswith("global_load"), line
            allowed = []
            queue.append(None)
        elif line == "s_barrier":
            assert allowed, path[i - 4:i + 1]
            stage = barriers.index(i)
            behind = len(queue) - 1 - max(j for j, s in enumerate(queue) if s == stage)
            if max(allowed) > behind:
                late.append((stage, max(allowed) - behind))
            allowed = []
    assert rows // per_stage >= STAGES and not rows % per_stage
    return late


def test_rows_of_a_stage_have_landed_when_its_barrier_opens(tmp_path):
    kernels = listing(tmp_path, "w4_wide.hip", "gemm_w4_wide")
    assert kernels
    late = {name: found for name, lines in kernels.items() if (found := unlanded(loop_path(lines)))}
    assert not late, late


def test_loader_waves_of_chunk_attention_wait_for_tiles_only(tmp_path):
    """Between its loads a loader wave waits in front of its barriers (K and V parts apart: for all but one or both parts of the
    next tile) and nowhere else.  The compiler, who does not know these loads, adds waits of its own where a register is still
    the target of a load on some way to the loop; in the loop they hold up the tiles in every round."""
    kernels = listing(tmp_path, "bf16_attention.hip", "chunk_attention_bf16")
    assert len(kernels) == 4, sorted(kernels)
    for name, lines in kernels.items():
        loads = [i for i, l in enumerate(lines) if l.startswith("global_load_lds")]
        waits = {int(m.group(1)) for l in lines[loads[0]:loads[-1]] if (m := re.match(r"s_waitcnt.*vmcnt\((\d+)\)", l))}
        assert waits <= ({0, 8, 16} if "Lb1" in name else {0}), (name, waits)
