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
# one problem for every (rows int8 0 / bf16 1, row tiles, blocks per wave, waves across the columns, exact dequant) that AUTO gives:
# (rows, M, K, N, gated, G), without a workspace
SHARED_FORMS = [(0, 49, 768, 5992, 0, 128), (0, 24, 2560, 12208, 0, 128), (0, 65, 3072, 4912, 0, 128),
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

# and one for every (rows, group size, row tiles, K in parts or not) of the 128-column workgroups: (rows, M, K, N, gated, G, fp32 copies of
# the output that the workspace holds).  Eight row tiles of int8 rows are never in parts.
SLIM_FORMS = [(0, 163, 768, 11624, 0, 128, 0), (0, 167, 1280, 12384, 1, 64, 16), (0, 193, 256, 8208, 0, 128, 16),
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


def test_every_form_is_run(routes):
    def forms(problems):
        return {(p[0],) + r[1:4] + (p[0] == 0 and p[1] <= 32,) for p, r in zip(problems, routes(problems)) if r[0] == 1}

    assert all(r[0] == 1 for r in routes(SHARED_FORMS)) and forms(SHARED_FORMS) >= forms(GRID)


def test_every_slim_form_is_run(routes):
    def forms(problems):
        r = [routes([p[:6]], p[6])[0] for p in problems]
        return {(p[0], p[5], q[1], q[2] > 1) for p, q in zip(problems, r) if q[0] == 2}

    grid = [p for p in GRID if p[1] >= 33] + [(xt, M, K, N, 0, G) for xt in (0, 1) for M in (280, 335, 482, 534, 746) for K in (256, 2816, 6400)
                                              for N in range(1040, 16000, 520) for G in (64, 128)]
    found = {(p[0], p[5], r[1], r[2] > 1) for cap in (0, 16) for p, r in zip(grid, routes(grid, cap)) if r[0] == 2}
    assert len(forms(SLIM_FORMS)) == len(SLIM_FORMS) and forms(SLIM_FORMS) >= found and len(found) > 30


@pytest.mark.gpu
@pytest.mark.parametrize("xt,M,K,N,gated,G", SHARED_FORMS)
def test_every_form(xt, M, K, N, gated, G):
    run_form(xt, M, K, N, gated, G, 0)


@pytest.mark.gpu
@pytest.mark.parametrize("xt,M,K,N,gated,G,cap", SLIM_FORMS)
def test_every_slim_form(xt, M, K, N, gated, G, cap):
    run_form(xt, M, K, N, gated, G, cap)


def run_form(xt, M, K, N, gated, G, cap):
    # all columns are computed; the oracle has the first 8 and the last 8 pairs of column blocks (a widest workgroup) and 8 between,
    # in whole pairs; bf16 rows lie in a wider matrix of NaNs, none of which may be read as part of a row
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_06753_amd import binding as w2
    from test_gpu_parity import bf16_bits, check_epilogue, dev
    rng = np.random.default_rng(M + K + N)
    g = torch.Generator(device="cuda").manual_seed(M + K + N)
    codes = torch.randint(0, 4, (K, N), dtype=torch.uint8, device="cuda", generator=g)
    scales = torch.empty((K // G, N), device="cuda").uniform_(0.005, 0.05, generator=g).to(torch.bfloat16)
    packed = w2.prepack(codes, scales, G)
    pairs = np.unique(np.concatenate([np.arange(8), rng.choice(np.arange(8, N // 32 - 8), 8, replace=False), np.arange(N // 32 - 8, N // 32)]))
    cols = (pairs[:, None] * 32 + np.arange(32)).reshape(-1)
    if not gated:
        cols = np.concatenate([cols, np.arange(N // 32 * 32, N)])
    at = torch.from_numpy(cols).cuda()
    cs, ss = codes[:, at].cpu().numpy(), scales[:, at].contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
    X = synth.make_activations(M, K, seed=M + K)
    act = w2.ACT_SILU_MUL if gated else w2.ACT_NONE
    ws = torch.empty(cap * M * N * 4, dtype=torch.uint8, device="cuda") if cap else None
    if xt == 0:
        oq, osx, _ = oracle.quantize_rows(X, G)
        _, y64 = oracle.matmul_a8(cs, ss, G, 0, oq, osx)
        mag = oracle.a8_term_magnitude(cs, ss, G, 0, oq, osx)
        call = lambda: w2.matmul_a8_epi(packed, K, N, G, dev(oq), dev(osx), act=act, workspace=ws)
    else:
        Xb = synth.f32_to_bf16_bits(X)
        wide = torch.full((M + 1, K + 24), float("nan"), dtype=torch.bfloat16, device="cuda")
        wide[:M, 8:K + 8] = dev(Xb).view(torch.bfloat16)
        _, y64, mag = oracle.matmul_a16(cs, ss, G, 0, Xb)
        call = lambda: w2.matmul_a16_epi(packed, K, N, G, wide[:M, 8:K + 8], act=act, workspace=ws)
    Y = call()
    assert torch.equal(Y.view(torch.int16), call().view(torch.int16)), "not deterministic"
    out = (pairs[:, None] * 16 + np.arange(16)).reshape(-1) if gated else cols
    check_epilogue(np.ascontiguousarray(bf16_bits(Y)[:, out]), y64, mag, None, act, f"xt={xt} M={M} K={K} N={N} G={G} act={act}")
