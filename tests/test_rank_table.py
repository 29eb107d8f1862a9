"""The rank table of the level-by-level forms, made by the lanes of one
wavefront, stepped on the CPU and compared with the binomials it holds, up to
the most photons a vector may have."""
import math
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include <vector>
#include "pq_common.h"
int main(int argc, char** argv) {
    const int m = atoi(argv[1]), n = atoi(argv[2]);
    int P = 1;
    while (P < m) P *= 2;
    std::vector<uint32_t> G((size_t)(n + 1) * P);
    for (size_t e = 0; e < G.size(); ++e) G[e] = e % P == 0 ? 0u : 0xffffffffu;
    pq::RankLane x[64] = {};
    for (int s = 0; s < pq::rank_table_steps(m, n); ++s) {
        uint32_t left[64];
        for (int l = 0; l < 64; ++l) left[l] = l ? x[l - 1].v : 0u;
        for (int l = 0; l < 64; ++l) pq::rank_table_step(x[l], l, left[l], s, m, n, P, G.data());
    }
    for (int r = 0; r <= n; ++r)
        for (int q = 0; q < m; ++q) printf("%u\n", G[(size_t)r * P + q]);
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("rank")
    src, exe = d / "rank.cpp", d / "rank"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "paper_2403_04006_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True)
    return str(exe)


@pytest.mark.parametrize("m,n", [(1, 1), (1, 64), (2, 1), (2, 62), (2, 63), (2, 64), (3, 64), (4, 63), (8, 64), (9, 48),
                                 (16, 10), (32, 4), (64, 5)])
def test_rank_table_holds_the_binomials(program, m, n):
    got = [int(v) for v in subprocess.run([program, str(m), str(n)], check=True, capture_output=True, text=True).stdout.split()]
    want = [0 if q == 0 else math.comb(r + q - 1, r) for r in range(n + 1) for q in range(m)]
    assert max(want) < 2**32 - 1
    assert got == want
