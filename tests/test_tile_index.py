"""Quotients of the tile index (a multiplication and a compare instead of a division) against integer division (no GPU needed)."""
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


def test_quotients_are_exact_for_every_index(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not installed")
    src, exe = tmp_path / "quotient.hip", tmp_path / "quotient"
    src.write_text(PROGRAM)
    flags = [f for f in jbuild.HIPCC_FLAGS if f not in ("-shared", "-c")]
    subprocess.run([hipcc, *flags, f"-I{jbuild.CSRC}", str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, stdout=subprocess.PIPE, text=True).stdout
    assert out.startswith("0 of"), out
