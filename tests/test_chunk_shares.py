"""How the pair-once kernels cut a block's tiles into chunks (chunk_begin), on the
host: every tile in one chunk, no chunk empty or longer than its bound."""

import os
import shutil
import subprocess

import pytest

from paper_0904_3659_amd import build as B

PROGRAM = r"""
#include "pair_once.hpp"
#include <cstdio>
int main()
{
    using namespace nbody;
    for (int C = 1; C <= 220; ++C)
        for (int U = 1; U <= 4200; U += U < 600 ? 1 : 97) {
            int longest = 0;
            if (chunk_begin(U, C, 0) != 0 || chunk_begin(U, C, C) != U) return printf("ends U=%d C=%d\n", U, C), 1;
            for (int c = 0; c < C; ++c) {
                const int t = chunk_begin(U, C, c + 1) - chunk_begin(U, C, c);
                if (t < (U >= C ? 1 : 0)) return printf("empty U=%d C=%d c=%d\n", U, C, c), 1;
                if (t > longest) longest = t;
            }
            SymPlan pl;
            pl.C = C;
            pl.G = U - 1;
            if (longest > longest_chunk(pl, 1)) return printf("bound U=%d C=%d %d\n", U, C, longest), 1;
        }
    puts("ok");
    return 0;
}
"""


def test_chunks(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    source = tmp_path / "chunks.hip"
    source.write_text(PROGRAM)
    exe = tmp_path / "chunks"
    subprocess.run(["hipcc", "-O1", "-std=c++17", f"--offload-arch={B.ARCH}", "-w", "-I", B.CSRC, str(source),
                    "-o", str(exe)], check=True, capture_output=True, timeout=300)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout
