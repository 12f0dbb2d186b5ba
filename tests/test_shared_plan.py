"""Kernels that AUTO takes for another one by price, in every form that it gives them: the mid-M kernel that shares its rows
(csrc/shared_plan.h) and the tiled kernels' 128-column workgroups (tiles::slim in csrc/tile_plan.h).  The rules of csrc/auto_plan.h
are compiled by themselves."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

import oracle
from paper_2508_06753_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "%s/paper_2508_06753_amd/csrc/auto_plan.h"
#include <stdio.h>
using namespace w2;
int main()
{
    int a16, G, gated, field, value;
    long long M, K, N, cap;
    while (scanf("%%d %%lld %%lld %%lld %%d %%d %%lld %%d %%d", &a16, &M, &K, &N, &gated, &G, &cap, &field, &value) == 9) {
        w2_tuning_t tn = {};
        int* const fields[] = {&tn.midm_min_m, &tn.midm_max_m, &tn.gemv_max_m, &tn.midm_cbw, &tn.splitk, &tn.splitk_min_tiles,
                               &tn.tiled_bm, &tn.tiled_bn, &tn.tiled_kw, &tn.tiled_wd};
        *fields[field] = value;
        const route::Problem p = {M, K, N, (N + 15) / 16, K / 256, G, gated != 0, cap};
        const route::Instead r = a16 ? route::a16(p, tn).instead : route::a8(p, tn).instead;
        const shared::Plan s = r.shared;
        if (r.to_shared) printf("1 %%d %%d %%d %%d %%d\n", s.rt, s.cj, s.sh, shared::k_ranges(a16, G, s.rt, s.cj, s.sh), shared::range_lds(s.rt, s.cj, s.sh));
        else if (r.to_slim) printf("2 %%d %%d 0 0 0\n", r.slim.ri, r.slim.splits);
        else printf("0 0 0 0 0 0\n");
    }
}
"""
# one problem for every (rows int8 0 / bf16 1, row tiles, blocks per wave, waves across the columns, exact dequant, group size) that AUTO
# gives: (rows, M, K, N, gated, G), without a workspace.  Seven 256-k tiles to a K range where AUTO gives the form so many (every buffer
# and weight register used again, the bias settled twice), mostly ranges of unequal length, ragged rows and columns
SHARED_FORMS = [(0, 50, 10496, 4104, 0, 64), (0, 62, 9216, 4104, 0, 128), (0, 27, 9216, 9752, 0, 128), (0, 76, 8448, 4104, 0, 128),
                (0, 31, 7168, 14424, 0, 128), (0, 72, 6400, 6536, 0, 64), (0, 124, 6400, 4104, 0, 128), (0, 30, 2304, 16424, 0, 64),
                (0, 29, 6656, 17256, 0, 128), (0, 63, 3584, 11680, 1, 64), (0, 115, 4352, 4128, 1, 128), (0, 28, 3840, 20488, 0, 128),
                (0, 62, 2304, 12296, 0, 64), (0, 115, 3584, 6152, 0, 128), (0, 24, 3840, 24584, 0, 128), (0, 90, 768, 8224, 1, 64),
                (0, 86, 3584, 10248, 0, 128), (0, 31, 3584, 28696, 0, 128), (0, 137, 7424, 5472, 1, 128), (0, 30, 7424, 24584, 0, 128),
                (0, 127, 5632, 9728, 1, 64), (0, 116, 5632, 8224, 1, 128), (0, 31, 6400, 38688, 1, 64), (0, 19, 5632, 32776, 0, 128),
                (0, 25, 3840, 40968, 0, 128), (0, 88, 3328, 32808, 0, 128), (0, 31, 3840, 53512, 0, 64), (0, 18, 3840, 49160, 0, 128),
                (0, 67, 1792, 20488, 0, 128), (0, 40, 6400, 5448, 0, 64), (0, 37, 4864, 5448, 0, 128), (0, 46, 9216, 8200, 0, 64),
                (0, 39, 9216, 8200, 0, 128), (0, 47, 8448, 10752, 1, 64), (0, 47, 8448, 10752, 1, 128), (0, 130, 5888, 5560, 0, 64),
                (0, 132, 5632, 5448, 0, 128), (0, 129, 4352, 7064, 0, 64), (0, 133, 3840, 6808, 0, 128), (0, 132, 3840, 8200, 0, 64),
                (0, 140, 3840, 8184, 0, 128), (0, 142, 3584, 9816, 0, 64), (0, 132, 3840, 9528, 0, 128), (0, 141, 5632, 9704, 0, 64),
                (0, 132, 7424, 9544, 0, 128), (0, 136, 3840, 10920, 0, 64), (0, 138, 5632, 10904, 0, 128), (0, 143, 3840, 13720, 0, 64),
                (0, 136, 3840, 13608, 0, 128), (0, 129, 1792, 16392, 0, 64), (0, 131, 3840, 16328, 0, 128), (0, 136, 1792, 19048, 0, 64),
                (0, 142, 3840, 19048, 0, 128), (0, 52, 4352, 6152, 0, 64), (0, 49, 7168, 5088, 1, 128), (0, 101, 7424, 5448, 0, 64),
                (0, 109, 7424, 5448, 0, 128), (0, 99, 7424, 6344, 0, 64), (0, 107, 7424, 6152, 0, 128), (0, 103, 5632, 8200, 0, 64),
                (0, 122, 5632, 8200, 0, 128), (0, 127, 3840, 10344, 0, 64), (0, 125, 3840, 10248, 0, 128), (0, 98, 3840, 12296, 0, 64),
                (0, 97, 3840, 12296, 0, 128), (0, 115, 2560, 14344, 0, 64), (0, 111, 2560, 14344, 0, 128), (0, 123, 5888, 13000, 0, 64),
                (0, 102, 5888, 12296, 0, 128), (0, 102, 3840, 16392, 0, 64), (0, 97, 3840, 16408, 0, 128), (0, 116, 3840, 20504, 0, 64),
                (0, 100, 3840, 20504, 0, 128), (0, 121, 1792, 24584, 0, 64), (0, 115, 1792, 24584, 0, 128), (0, 99, 1792, 28680, 0, 64),
                (0, 108, 2048, 32008, 0, 128), (1, 51, 2304, 4088, 0, 128), (1, 60, 2816, 4104, 0, 64), (1, 20, 5120, 11560, 0, 128),
                (1, 85, 2304, 4128, 1, 64), (1, 30, 5120, 14840, 0, 128), (1, 89, 2560, 6152, 0, 64), (1, 79, 4352, 6152, 0, 128),
                (1, 31, 3840, 45448, 0, 64), (1, 27, 4352, 20536, 0, 128), (1, 31, 4352, 27992, 0, 64), (1, 31, 3840, 24616, 0, 128),
                (1, 31, 2304, 32408, 0, 64), (1, 28, 2560, 28680, 0, 128), (1, 89, 7424, 10488, 0, 128), (1, 27, 5632, 32800, 1, 64),
                (1, 29, 5632, 32776, 0, 128), (1, 32, 4864, 49112, 0, 128), (1, 30, 3840, 49312, 1, 64), (1, 30, 3840, 49240, 0, 128),
                (1, 33, 3072, 5448, 0, 64), (1, 34, 3072, 5448, 0, 128), (1, 68, 6656, 5448, 0, 64), (1, 69, 6656, 5448, 0, 128),
                (1, 46, 8960, 16232, 0, 64), (1, 46, 8960, 16360, 0, 128), (1, 131, 5632, 5448, 0, 64), (1, 140, 5632, 5464, 0, 128),
                (1, 129, 3840, 6808, 0, 64), (1, 131, 3840, 6808, 0, 128), (1, 137, 3840, 8200, 0, 64), (1, 139, 3840, 8168, 0, 128),
                (1, 143, 3840, 10088, 0, 64), (1, 135, 3840, 9528, 0, 128), (1, 140, 7424, 9560, 0, 64), (1, 143, 7424, 9528, 0, 128),
                (1, 139, 5632, 10904, 0, 64), (1, 139, 5632, 10888, 0, 128), (1, 134, 3840, 13624, 0, 64), (1, 142, 3840, 13608, 0, 128),
                (1, 141, 3840, 16328, 0, 64), (1, 135, 3840, 16344, 0, 128), (1, 131, 3840, 19048, 0, 64), (1, 130, 3840, 19048, 0, 128),
                (1, 97, 3072, 4088, 0, 64), (1, 106, 3072, 4088, 0, 128), (1, 49, 7168, 10264, 0, 64), (1, 57, 7168, 10248, 0, 128),
                (1, 63, 8448, 14728, 0, 64), (1, 63, 8960, 13928, 0, 128), (1, 121, 5632, 8200, 0, 64), (1, 103, 5632, 8200, 0, 128),
                (1, 113, 3840, 10248, 0, 64), (1, 108, 3840, 10248, 0, 128), (1, 126, 3840, 12296, 0, 64), (1, 99, 3840, 12296, 0, 128),
                (1, 125, 3584, 14344, 0, 64), (1, 99, 3584, 14344, 0, 128), (1, 126, 7424, 12664, 0, 64), (1, 124, 7424, 12296, 0, 128),
                (1, 124, 5632, 16392, 0, 64), (1, 100, 5632, 16408, 0, 128), (1, 105, 3840, 20488, 0, 64), (1, 116, 3840, 20488, 0, 128),
                (1, 119, 3840, 24664, 0, 64), (1, 117, 3840, 24584, 0, 128), (1, 113, 19712, 28808, 0, 64), (1, 116, 3840, 28712, 0, 128)]
# and short ones: down to one tile in a range, fewer than there are buffers
SHORT_RUNS = [(0, 49, 768, 5992, 0, 128), (0, 24, 2560, 12208, 0, 128), (0, 65, 3072, 4912, 0, 128),
              (0, 17, 4608, 12304, 0, 128), (0, 49, 768, 9016, 0, 128), (0, 28, 1280, 18616, 0, 64),
              (0, 49, 768, 10272, 1, 128), (0, 17, 1280, 20488, 0, 128), (0, 65, 768, 8200, 0, 128),
              (0, 17, 768, 24592, 0, 128), (0, 65, 768, 8224, 1, 128), (0, 32, 768, 24672, 1, 128),
              (0, 65, 4096, 8672, 1, 128), (0, 20, 4608, 26080, 1, 128), (0, 97, 768, 8224, 1, 128),
              (0, 20, 1280, 32776, 0, 128), (0, 32, 768, 48328, 0, 128), (0, 65, 768, 16408, 0, 128),
              (0, 17, 768, 49168, 0, 128), (0, 65, 768, 20488, 0, 128), (0, 33, 768, 5464, 0, 128),
              (0, 33, 768, 10936, 0, 64), (0, 33, 768, 13144, 0, 128), (0, 33, 768, 16408, 0, 64),
              (0, 33, 768, 16416, 1, 128), (0, 65, 768, 12304, 0, 64), (0, 65, 768, 12320, 1, 128),
              (0, 33, 4608, 24608, 1, 64), (0, 33, 768, 32776, 0, 128), (0, 36, 1024, 46024, 0, 64),
              (0, 65, 768, 24592, 0, 128), (0, 65, 768, 28696, 0, 64), (0, 49, 1792, 7456, 0, 128),
              (0, 49, 768, 10288, 0, 64), (0, 49, 768, 12320, 1, 128), (0, 97, 768, 8200, 0, 64),
              (0, 49, 768, 16416, 1, 128), (0, 97, 768, 12304, 0, 64), (0, 97, 768, 14344, 0, 128),
              (0, 49, 3072, 24608, 1, 64), (0, 97, 768, 16408, 0, 128), (0, 97, 768, 20488, 0, 64),
              (0, 97, 768, 20488, 0, 128), (0, 97, 768, 28696, 0, 64), (1, 33, 2560, 4096, 0, 128),
              (1, 49, 1280, 5128, 0, 64), (1, 17, 2560, 15488, 1, 128), (1, 17, 1280, 17320, 0, 64),
              (1, 17, 1280, 21016, 0, 128), (1, 17, 1280, 24592, 0, 64), (1, 17, 1280, 24608, 1, 128),
              (1, 24, 3584, 30424, 0, 128), (1, 17, 768, 40072, 0, 128), (1, 24, 1024, 40984, 0, 128),
              (1, 17, 1024, 49168, 0, 128), (1, 33, 2560, 5464, 0, 64), (1, 33, 768, 10936, 0, 128),
              (1, 33, 768, 16240, 0, 64), (1, 33, 768, 16408, 0, 128), (1, 33, 768, 21688, 0, 64),
              (1, 33, 768, 26152, 0, 128), (1, 65, 1280, 12320, 1, 64), (1, 33, 5120, 24640, 1, 128),
              (1, 33, 768, 32800, 1, 64), (1, 33, 768, 40984, 0, 128), (1, 33, 768, 50992, 0, 64),
              (1, 65, 768, 31744, 0, 128), (1, 49, 2560, 4128, 1, 64), (1, 49, 768, 9160, 0, 128),
              (1, 49, 768, 14008, 0, 64), (1, 97, 768, 8200, 0, 128), (1, 49, 768, 16416, 1, 64),
              (1, 97, 768, 12304, 0, 128), (1, 97, 768, 12320, 1, 64), (1, 97, 4096, 12320, 1, 128),
              (1, 97, 768, 16408, 0, 64), (1, 97, 768, 20488, 0, 128), (1, 113, 1536, 24592, 0, 64),
              (1, 113, 2560, 28696, 0, 128)]
# long runs of K in few ranges: 77 tiles in one, 38 and 39 in two
LONG_RUNS = [(0, 112, 19712, 24600, 0, 128), (0, 140, 19712, 7256, 0, 64), (1, 144, 19712, 6560, 1, 64), (1, 131, 19712, 5664, 1, 128)]

# and one for every (rows, group size, row tiles, K in parts or not) of the 128-column workgroups, with nine tiles to a part (eight in one):
# (rows, M, K, N, gated, G, fp32 copies of the output that the workspace holds)
SLIM_FORMS = [(0, 245, 2304, 1048, 0, 64, 0), (0, 322, 7424, 1320, 0, 64, 16), (0, 194, 2304, 8232, 0, 64, 0),
              (0, 323, 4864, 2792, 0, 64, 16), (0, 163, 2304, 10888, 0, 64, 0), (0, 258, 7424, 2904, 0, 64, 16),
              (0, 193, 2304, 10936, 0, 64, 0), (0, 326, 7424, 2696, 0, 64, 16), (0, 749, 2304, 10824, 0, 64, 0),
              (0, 252, 8192, 8328, 0, 64, 16), (0, 241, 2304, 1032, 0, 128, 0), (0, 323, 9728, 1048, 0, 128, 16),
              (0, 197, 2304, 8264, 0, 128, 0), (0, 395, 7168, 1544, 0, 128, 16), (0, 161, 2304, 10952, 0, 128, 0),
              (0, 258, 7424, 2728, 0, 128, 16), (0, 194, 2304, 10984, 0, 128, 0), (0, 335, 7168, 2744, 0, 128, 16),
              (0, 812, 2304, 9272, 0, 128, 0), (0, 339, 10240, 4216, 0, 128, 16), (1, 263, 2304, 1032, 0, 64, 0),
              (1, 292, 8192, 2088, 0, 64, 16), (1, 197, 2304, 8280, 0, 64, 0), (1, 386, 7936, 2064, 0, 64, 16),
              (1, 242, 2304, 8296, 0, 64, 0), (1, 568, 9472, 1048, 0, 64, 16), (1, 193, 2304, 10968, 0, 64, 0),
              (1, 297, 9472, 2616, 0, 64, 16), (1, 226, 2560, 11224, 0, 64, 0), (1, 869, 9472, 1112, 0, 64, 16),
              (1, 260, 2304, 1032, 0, 128, 0), (1, 303, 7936, 2072, 0, 128, 16), (1, 194, 2304, 8232, 0, 128, 0),
              (1, 394, 5376, 3080, 0, 128, 16), (1, 243, 2304, 8232, 0, 128, 0), (1, 595, 9472, 1048, 0, 128, 16),
              (1, 197, 2304, 11160, 0, 128, 0), (1, 991, 7168, 1032, 0, 128, 16), (1, 227, 2560, 10904, 0, 128, 0),
              (1, 890, 9472, 1112, 0, 128, 16)]
SLIM_SHORT_RUNS = [(0, 163, 768, 11624, 0, 128, 0), (0, 167, 1280, 12384, 1, 64, 16), (0, 193, 256, 8208, 0, 128, 16),
                   (0, 242, 2304, 1184, 0, 64, 16), (0, 249, 2816, 1080, 0, 128, 16), (0, 257, 6400, 1888, 1, 128, 16),
                   (0, 265, 512, 1272, 0, 64, 0), (0, 269, 5376, 1040, 0, 128, 16), (0, 270, 512, 1288, 0, 128, 0),
                   (0, 329, 768, 6544, 0, 128, 0), (0, 330, 512, 10808, 0, 64, 0), (0, 334, 6400, 1904, 0, 128, 16),
                   (0, 335, 5888, 2208, 1, 64, 16), (0, 339, 2560, 1032, 0, 64, 16), (0, 356, 6400, 1344, 0, 64, 16),
                   (0, 395, 256, 2952, 0, 64, 0), (0, 482, 256, 14304, 1, 64, 0), (0, 723, 256, 10816, 0, 128, 0),
                   (1, 193, 512, 11040, 1, 128, 16), (1, 204, 512, 10976, 1, 64, 0), (1, 258, 1536, 1112, 0, 128, 16),
                   (1, 259, 2560, 1576, 0, 64, 16), (1, 263, 512, 8416, 0, 64, 16), (1, 263, 3072, 1056, 1, 64, 16),
                   (1, 276, 2560, 1304, 0, 128, 16), (1, 280, 256, 1096, 0, 64, 0), (1, 294, 256, 1056, 0, 128, 0),
                   (1, 309, 1536, 1056, 0, 64, 16), (1, 322, 2560, 1360, 0, 128, 16), (1, 329, 512, 6768, 0, 128, 16),
                   (1, 378, 5376, 1416, 0, 64, 16), (1, 449, 256, 2912, 1, 64, 16), (1, 467, 256, 2824, 0, 128, 16),
                   (1, 474, 5376, 1056, 1, 128, 16), (1, 518, 2560, 1192, 0, 128, 16), (1, 534, 3328, 1176, 0, 64, 16),
                   (1, 722, 256, 13136, 0, 64, 16), (1, 746, 256, 10864, 0, 128, 0)]


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("shared_plan")
    (d / "p.cpp").write_text(PROGRAM % ROOT)
    subprocess.run(["g++", "-O1", "-std=c++17", "-o", str(d / "p"), str(d / "p.cpp")], check=True)

    def ask(problems, cap=0, field=0, value=0):
        """cap: copies of the output that the workspace holds, for all or each
        -> (1, rt, cj, sh, K ranges, bytes of local memory of one): rows shared; (2, row tiles, parts of K, ...): 128 columns; (0, ...)"""
        caps = cap if isinstance(cap, list) else [cap] * len(problems)
        text = "".join("{} {} {} {} {} {} {} {} {}\n".format(*p, c, field, value) for p, c in zip(problems, caps))
        out = subprocess.run([str(d / "p")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, l.split())) for l in out.splitlines()]

    return ask


GRID = [(xt, M, K, N, g, G) for xt in (0, 1) for M in (1, 8, 9, 16, 17, 32, 33, 48, 49, 64, 65, 100, 144, 145, 300)
        for K in (512, 768, 1280, 2048, 4096, 5120, 8192, 12288, 20480, 20736) for N in list(range(2048, 57344, 1312)) + [4080, 4096, 28672]
        for g in (0, 1) if not (g and N % 32) for G in (64, 128)]


def test_shapes_fit_the_kernel(routes):
    taken = slim = 0
    for cap in (0, 8):
        for (xt, M, K, N, g, G), (to, rt, cj, sh, ks, lds) in zip(GRID, routes(GRID, cap)):
            assert to != 1 or (17 <= M <= 144 and N > 4080 and 768 <= K <= 20480)
            if to == 2:
                slim += 1
                assert M >= 33 and 4 <= rt <= 8 and 1 <= cj <= max(1, min(8, cap, K // 512)) and (cj == 1 or cj * M * N * 4 <= 64 << 20)
            if to == 1:
                taken += 1
                assert 2 <= rt <= min(4, -(-M // 16)) and cj in (1, 2) and 2 <= sh <= 8 and not (g and cj * sh % 2)
                assert 1 <= ks <= 8 and ks * sh <= 16 and ks * lds + rt * 64 <= 160 * 1024
                # room for every load of every wave in four buffers, and for the waves' partial results
                assert lds >= 4 * -(-2 * rt // sh) * sh * 1024 and lds >= sh * rt * 16 * (cj * 16 + 4) * 4
    assert taken > 2000 and slim > 2000


# a field of w2_tuning_t and a value of it: midm_min_m, midm_max_m, gemv_max_m, midm_cbw, splitk, splitk_min_tiles, tiled_bm, tiled_bn,
# tiled_kw, tiled_wd
@pytest.mark.parametrize("field,value", [(0, 5), (1, 1), (1, 16), (1, 256), (2, 8), (3, 4), (4, 2), (5, 1024), (6, 64), (7, 256), (8, 2), (9, 8)])
def test_not_where_the_caller_says(routes, field, value):
    # which rows the mid-M or the decode kernel gets, what a launch shape is to be, how many tiles a part of K has
    assert not any(r[0] for cap in (0, 16) for r in routes(GRID[::7], cap, field, value))


def test_the_workspace_asked_for_holds_the_parts(routes):
    # whatever AUTO cuts into parts over 128-column workgroups where there is room, it does in the room that w2_workspace_size reports
    # (behind the int8 rows and their scales)
    from paper_2508_06753_amd import binding as w2
    problems = [(xt, M, K, N, g, G) for xt in (0, 1) for M in (33, 46, 62, 96, 132, 255, 310, 392, 669, 851, 1300) for K in (256, 2816, 6656, 8960, 16384, 24832)
                for N in (1024, 1576, 2056, 3488, 3808, 6240, 11104, 23872, 49248) for g in (0, 1) if not (g and N % 32) for G in (64, 128)]
    quant = lambda M, K: ((M * K + 15) // 16 * 16 + 4 * M + 255) // 256 * 256
    room = [(w2.workspace_size(M, K, N, G, a16=bool(xt)) - (0 if xt else quant(M, K))) // (4 * M * N) for xt, M, K, N, _, G in problems]
    parts = 0
    for p, there, reported in zip(problems, routes(problems, 16), routes(problems, room)):
        if there[0] == 2:
            assert there == reported, p
            parts += there[2] > 1
    assert parts > 200


def test_sides_of_autos_lines(routes):
    # of the problems that the mid-M kernel and another one are compared on, which AUTO gives to a third
    from paper_2508_06753_amd import binding as w2
    from test_gpu_parity import AUTO_SIDES, AUTO_SIDES_SHARED
    for path, M, K, N in AUTO_SIDES:
        p = [(int(path == "a16"), M, K, N, 0, 128)]
        cap = w2.workspace_size(M, K, N, 128, a16=path == "a16") // (4 * M * N)
        assert routes(p, cap)[0][0] == ((path, M, K, N) in AUTO_SIDES_SHARED)
        assert routes(p, cap, 1, 1)[0][0] == 0                               # (the "other" side, midm_max_m = 1: the plain tiled kernel)


def drawn(n, seed, rows, tiles, cols):
    rng, out = np.random.default_rng(seed), []
    log = lambda lo, hi: int(np.exp(rng.uniform(np.log(lo), np.log(hi + 1))))
    for _ in range(n):
        g = int(rng.random() < 0.35)
        step = 32 if g else 8
        out.append((int(rng.integers(2)), log(*rows), 256 * log(*tiles), log(*cols) // step * step, g, int(rng.choice([64, 128]))))
    return out


def test_every_form_is_run(routes):
    def forms(problems):
        return {(p[0],) + r[1:4] + (p[0] == 0 and p[1] <= 32, p[5]) for p, r in zip(problems, routes(problems)) if r[0] == 1}

    given = forms(SHARED_FORMS)
    assert len(given) == len(SHARED_FORMS) and given >= forms(GRID) and given >= forms(drawn(80000, 1, (17, 144), (3, 80), (4088, 57344)))
    assert all(r[0] == 1 for r in routes(SHORT_RUNS))
    ranges = [(p[2] // 256 // min(r[4], p[2] // 256), r) for p, r in zip(SHARED_FORMS + LONG_RUNS, routes(SHARED_FORMS + LONG_RUNS))]
    assert all(r[0] == 1 for _, r in ranges) and sum(t >= 7 for t, _ in ranges) >= 120 and [t for t, _ in ranges[-4:]] == [77, 38, 38, 38]


def test_every_slim_form_is_run(routes):
    def forms(problems, caps):
        return {(p[0], p[5], q[1], q[2] > 1): p[2] // 256 // q[2] for p, q in zip(problems, routes(problems, caps)) if q[0] == 2}

    given = forms([p[:6] for p in SLIM_FORMS], [p[6] for p in SLIM_FORMS])
    some = [p for p in GRID if p[1] >= 33] + drawn(40000, 2, (33, 1100), (1, 40), (1024, 30000))
    assert len(given) == len(SLIM_FORMS) == 40 and all(given.keys() >= forms(some, [cap] * len(some)).keys() for cap in (0, 16))
    assert min(given.values()) >= 8
    assert all(r[0] == 2 for r in routes([p[:6] for p in SLIM_SHORT_RUNS], [p[6] for p in SLIM_SHORT_RUNS]))


@pytest.mark.gpu
@pytest.mark.parametrize("xt,M,K,N,gated,G", SHARED_FORMS + SHORT_RUNS + LONG_RUNS)
def test_every_form(xt, M, K, N, gated, G):
    run_form(xt, M, K, N, gated, G, 0)


@pytest.mark.gpu
@pytest.mark.parametrize("xt,M,K,N,gated,G,cap", SLIM_FORMS + SLIM_SHORT_RUNS)
def test_every_slim_form(xt, M, K, N, gated, G, cap):
    run_form(xt, M, K, N, gated, G, cap)


def problem(M, K, N, G, cap):
    from paper_2508_06753_amd import binding as w2
    g = torch.Generator(device="cuda").manual_seed(M + K + N)
    codes = torch.randint(0, 4, (K, N), dtype=torch.uint8, device="cuda", generator=g)
    ws = torch.empty(cap * M * N * 4, dtype=torch.uint8, device="cuda") if cap else None
    return w2, g, codes, ws


def run_form(xt, M, K, N, gated, G, cap):
    # all columns are computed; the oracle has the first 8 and the last 8 pairs of column blocks (a widest workgroup) and 4 between
    # (128-column workgroups: 4 of each), in whole pairs; bf16 rows lie in a wider matrix of NaNs, none of which may be read as part of
    # a row.  Plain or gated, and again with a bias (not aligned) and the other epilogues into a wider matrix, whose rest has to stay
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from test_gpu_parity import bf16_bits, check_epilogue, dev
    w2, g, codes, ws = problem(M, K, N, G, cap)
    rng = np.random.default_rng(M + K + N)
    scales = torch.empty((K // G, N), device="cuda").uniform_(0.005, 0.05, generator=g).to(torch.bfloat16)
    packed = w2.prepack(codes, scales, G)
    e = 4 if N < 4080 or M > 144 else 8
    pairs = np.unique(np.concatenate([np.arange(e), rng.choice(np.arange(e, N // 32 - e), 4, replace=False), np.arange(N // 32 - e, N // 32)]))
    cols = (pairs[:, None] * 32 + np.arange(32)).reshape(-1)
    if not gated:
        cols = np.concatenate([cols, np.arange(N // 32 * 32, N)])
    at = torch.from_numpy(cols).cuda()
    cs, ss = codes[:, at].cpu().numpy(), scales[:, at].contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
    X = synth.make_activations(M, K, seed=M + K)
    bias = torch.randn(N + 1, device="cuda", generator=g).to(torch.bfloat16)[1:]
    bs = bias[at].view(torch.int16).cpu().numpy().view(np.uint16)
    if xt == 0:
        oq, osx, _ = oracle.quantize_rows(X, G)
        _, y64 = oracle.matmul_a8(cs, ss, G, 0, oq, osx)
        mag = oracle.a8_term_magnitude(cs, ss, G, 0, oq, osx)
        call = lambda **kw: w2.matmul_a8_epi(packed, K, N, G, dev(oq), dev(osx), workspace=ws, **kw)
    else:
        Xb = synth.f32_to_bf16_bits(X)
        wide = torch.full((M + 1, K + 24), float("nan"), dtype=torch.bfloat16, device="cuda")
        wide[:M, 8:K + 8] = dev(Xb).view(torch.bfloat16)
        _, y64, mag = oracle.matmul_a16(cs, ss, G, 0, Xb)
        call = lambda **kw: w2.matmul_a16_epi(packed, K, N, G, wide[:M, 8:K + 8], workspace=ws, **kw)
    out = (pairs[:, None] * 16 + np.arange(16)).reshape(-1) if gated else cols
    n_out = N // 2 if gated else N
    for act, b in ((w2.ACT_SILU_MUL if gated else w2.ACT_NONE, None), (w2.ACT_SILU_MUL if gated else w2.ACT_SILU, bias)):
        Y = call(act=act, bias=b)
        check_epilogue(np.ascontiguousarray(bf16_bits(Y)[:, out]), y64, mag, None if b is None else bs, act, f"xt={xt} M={M} K={K} N={N} G={G} act={act}")
        big = torch.full((M, n_out + 40), 7.0, dtype=torch.bfloat16, device="cuda")
        call(act=act, bias=b, out=big[:, :n_out])
        assert torch.equal(big[:, :n_out].contiguous().view(torch.int16), Y.view(torch.int16)), "not deterministic"
        assert (big[:, n_out:] == 7.0).all(), "columns past the last were written"


@pytest.mark.gpu
@pytest.mark.parametrize("xt,M,K,N,gated,G,cap", [p + (0,) for p in SHARED_FORMS + SHORT_RUNS + LONG_RUNS] +
                         SLIM_FORMS + SLIM_SHORT_RUNS)
def test_every_form_holds_exact_group_sums(xt, M, K, N, gated, G, cap):
    # Each column takes one group, with a scale of 1 (the others 0): the output is that group's sum of products, an integer, rounded
    # to bf16 once.  Even rows hold -1, 0, 1 (the integer itself, below 256), odd ones the whole range of the type's integers.
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w2, g, codes, ws = problem(M, K, N, G, cap)
    groups = torch.arange(N, device="cuda") * 7 % (K // G)
    scales = torch.zeros((K // G, N), dtype=torch.bfloat16, device="cuda")
    scales[groups, torch.arange(N, device="cuda")] = 1.0
    packed = w2.prepack(codes, scales, G)
    X = torch.randint(-127, 128, (M, K), dtype=torch.int8, device="cuda", generator=g)
    X[::2] = X[::2].remainder(3) - 1
    want = torch.empty((M, N), dtype=torch.float64, device="cuda")
    for k in range(K // G):
        own = (groups == k).nonzero().reshape(-1)
        want[:, own] = X[:, k * G:(k + 1) * G].double() @ (codes[k * G:(k + 1) * G, own].double() - 2)
    if xt == 0:
        Y = w2.matmul_a8(packed, K, N, G, X, torch.ones(M, device="cuda"), workspace=ws)
    else:
        Y = w2.matmul_a16(packed, K, N, G, X.to(torch.bfloat16), workspace=ws)
    assert torch.equal(Y, want.to(torch.float32).to(torch.bfloat16))         # (exact in fp32, so rounded once)
