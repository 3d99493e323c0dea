"""The FP32 step reads a fixed number of words from every row of a tile's slot list,
however few slots the rows have: every such read stays inside the workspace that the
layout asks for, whatever the plan."""
import os
import shutil
import subprocess

import pytest

import paper_1803_07491_amd as P

PKG = os.path.dirname(os.path.abspath(P.__file__))
ROOT = os.path.dirname(PKG)

PROGRAM = r"""
#include <cstdio>
#include "tiles.h"
using namespace bop;
int main()
{
    long plans = 0, past = 0, bad = 0;
    for (int rows = 1; rows <= 40; ++rows)
        for (int deg = 1; deg <= 20; ++deg)
            for (int dtype : {(int)BOP_F64, (int)BOP_F32, (int)BOP_BF16, (int)BOP_F16})
                for (int no : {5, 9})
                    for (int tiles : {1, 2, 7})
                        for (int batch = 1; batch <= tiles; ++batch)
                            for (int n_max : {1, 2, 9}) {
                                bop_plan p{};
                                p.n_atoms = rows;
                                p.n_orb = no;
                                p.n_max = n_max;
                                p.dtype = dtype;
                                p.n_tiles = tiles;
                                p.batch_tiles = batch;
                                p.rows_cap = rows;
                                p.deg_max = deg;
                                p.chunk_rows = 64;
                                for (int k = 0; k <= n_max / 2; ++k) p.rows_k[k] = rows;
                                const Layout L = make_layout(p, 1);
                                const size_t record = L.tiles + L.tile_stride * (size_t)(tiles - 1);
                                const size_t end = record + 4ull * (2 * rows + (size_t)(rows - 1) * deg + SLOTS_HELD);
                                ++plans;
                                past += end > record + L.tile_stride;
                                bad += end > L.bytes || L.x < L.tiles + L.tile_stride * tiles ||
                                       L.x_stride * (batch >= 2 ? 2 * (size_t)batch : 4) < 4ull * SLOTS_HELD;
                            }
    std::printf("%ld %ld %ld\n", plans, past, bad);
    return 0;
}
"""


def test_slot_words_stay_inside_the_workspace(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "layout.hip", tmp_path / "layout"
    src.write_text(PROGRAM)
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                           "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                           str(src), "-o", str(exe)], stderr=subprocess.DEVNULL)
    plans, past, bad = map(int, subprocess.check_output([str(exe)]).split())
    assert plans > 10000
    assert past > 0            # the layouts that the reads leave the records of are among them
    assert bad == 0
