"""The tiled kernels' launch shapes: csrc/tile_plan.h compiled by itself, and on the GPU a problem for every tile height."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from paper_2508_06753_amd import synth

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "%s/paper_2508_06753_amd/csrc/tile_plan.h"
#include <stdio.h>
using namespace w2::tiles;
int main()
{
    char what;
    int kind, f1, f2, f3;
    long long M, N, n_kt, cap;
    while (scanf(" %%c %%d %%lld %%lld %%lld %%lld %%d %%d %%d", &what, &kind, &M, &N, &n_kt, &cap, &f1, &f2, &f3) == 9) {
        if (what == 'a') {                                   // the whole choice for w2a8: kind is G, the forced tiled_bm, tiled_bn, splitk
            w2_tuning_t tune = {};
            tune.tiled_bm = f1;
            tune.tiled_bn = f2;
            tune.splitk = f3;
            const A8Shape s = a8_shape(kind, M, N, n_kt, cap, tune);
            printf("%%d %%d %%d %%.9g\n", 16 * s.ri, s.bn, s.splits, s.us);
        } else if (what == 't') {
            const Shape s = pick((Kind)kind, M, N, n_kt, cap, f1, f2);
            printf("%%d %%d 0 %%.9g\n", s.ri, s.splits, s.us);
        } else {
            const Shape64 s = pick64(kind, M, N, n_kt, cap, f1, f2, f3);
            printf("%%d %%d %%d %%.9g\n", s.bn, s.kw, s.splits, s.us);
        }
    }
}
"""

# Problems that the library's own choice runs in every tile height, without and with K split across workgroups (given the
# workspace that w2_workspace_size asks for): (path, G, K, N, M, ri, split).  Rows one past a whole tile, ragged columns.
HEIGHTS = [("a8", 128, 4096, 6712, 257, 4, False), ("a8", 128, 8192, 1504, 321, 4, True),
           ("a8", 128, 768, 10184, 769, 5, False), ("a8", 128, 8192, 1752, 257, 5, True),
           ("a8", 128, 1024, 8944, 641, 6, False), ("a8", 128, 8192, 2248, 257, 6, True),
           ("a8", 128, 512, 11424, 513, 7, False), ("a8", 128, 8192, 5472, 321, 7, True),
           ("a8", 64, 768, 3984, 257, 4, False), ("a8", 64, 8192, 1256, 401, 4, True),
           ("a8", 64, 512, 10928, 321, 5, False), ("a8", 64, 8192, 1752, 257, 5, True),
           ("a8", 64, 512, 10928, 401, 6, False), ("a8", 64, 8192, 2248, 257, 6, True),
           ("a8", 64, 512, 9440, 577, 7, False), ("a8", 64, 8192, 2744, 321, 7, True), ("a8", 64, 8192, 8200, 241, 8, True),
           ("a16", 128, 512, 264, 257, 4, False), ("a16", 64, 2048, 264, 257, 4, True),
           ("a16", 64, 512, 10928, 321, 5, False), ("a16", 128, 2048, 3240, 257, 5, True),
           ("a16", 128, 512, 10928, 401, 6, False), ("a16", 64, 2048, 3240, 321, 6, True),
           ("a16", 64, 512, 9440, 577, 7, False), ("a16", 128, 4096, 4232, 289, 7, True)]
KINDS = {("a8", 128): 0, ("a8", 64): 1, ("a16", 128): 2, ("a16", 64): 2}


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("tile_plan")
    (d / "p.cpp").write_text(PROGRAM % ROOT)
    subprocess.run(["g++", "-O1", "-std=c++17", "-o", str(d / "p"), str(d / "p.cpp")], check=True)

    def ask(lines):
        text = "".join("{} {} {} {} {} {} {} {} {}\n".format(*l) for l in lines)
        out = subprocess.run([str(d / "p")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(float(v) if i == 3 else int(v) for i, v in enumerate(l.split())) for l in out.splitlines()]

    return ask


SHAPES = [(K, N) for K in (256, 512, 2304, 4096, 28672) for N in (8, 264, 1032, 28672, 57344)]
ROWS = (1, 33, 64, 65, 130, 257, 1000, 4096, 1 << 20)


def test_tall_tiles(plans):
    ask = [("t", kind, M, N, K // 256, cap, ri, forced, 0) for kind in (0, 1, 2) for K, N in SHAPES for M in ROWS
           for cap in (0, 1, 3, 16) for ri, forced in ((0, 0), (8, 0), (0, 1), (0, 3), (8, 16))]
    for (_, _, M, N, n_kt, cap, ri, forced, _), (got, splits, _, us) in zip(ask, plans(ask)):
        assert got in ((ri,) if ri else (4, 5, 6, 7, 8)) and us < 1e30
        assert 1 <= splits <= max(1, min(cap, n_kt))                         # every range holds a tile, every part has room
        if forced:
            assert splits == max(1, min(forced, cap, n_kt))
        else:
            assert splits == 1 or (splits <= 8 and 2 * splits <= n_kt and splits * M * N * 4 <= 64 << 20)


def test_narrow_64_row_tiles(plans):
    ask = [("n", G, M, N, K // 256, cap, bn, kw, forced) for G in (64, 128) for K, N in SHAPES for M in ROWS for cap in (0, 1, 3, 16)
           for bn, kw, forced in ((0, 0, 0), (128, 0, 0), (64, 0, 0), (0, 2, 0), (0, 4, 3), (0, 0, 1), (128, 1, 16))]
    for (_, _, M, N, n_kt, cap, bn, kw, forced), (b, k, s, _) in zip(ask, plans(ask)):
        assert b == bn if bn else b in (64, 128)
        assert k in (1, 2, 4) and (not kw or k <= kw)
        assert 1 <= s <= max(1, min(cap, 16, n_kt)) and (k == 1 or n_kt % (k * s) == 0)
        if forced:
            assert s == max(1, min(forced, cap, n_kt))
        else:
            assert s == 1 or (s * M * N * 4 <= 16 << 20 and n_kt // (s * k) >= 2)
        if b == 64 and not bn:
            assert k == 4 and s == 1 and -(-M // 64) * -(-N // 64) <= 256


def test_forced_tiles(plans):
    # a forced width and height are what runs, whatever the price says of K ranges; parts only as far as there is room
    ask = [("a", G, M, N, K // 256, cap, bm, bn, forced) for G in (64, 128) for K, N in SHAPES for M in ROWS for cap in (0, 1, 3, 16)
           for bm, bn, forced in ((128, 128, 0), (128, 128, 3), (128, 256, 0), (128, 256, 16), (128, 0, 0), (64, 64, 0), (64, 128, 0), (64, 256, 0),
                                  (64, 0, 0), (0, 64, 0), (0, 128, 2))]
    for (_, G, _, _, n_kt, cap, bm, bn, forced), (rows, width, splits, _) in zip(ask, plans(ask)):
        assert rows == (128 if bm == 128 else 0)                             # (0: the 64-row kernel)
        assert width == bn if bn else width in ((128, 256) if bm == 128 else (64, 128, 256))
        assert 1 <= splits <= max(1, min(cap, n_kt))
        assert splits == 1 or not (bm == 128 and width == 128 and G == 64)    # (the whole K there)


def test_groups_of_64_on_narrow_grids(plans):
    # 64-row tiles, measured 8 to 10 % faster than the tall ones whose price is 2 to 3 % lower; tall ones where the price is clear
    low = [("a", 64, M, N, K // 256, 0, 0, 0, 0) for M, K, N in ((506, 27648, 5440), (1257, 26112, 1728), (597, 18432, 3584))]
    tall = [("a", 64, 257, 1752, 32, 16, 0, 0, 0), ("a", 64, 321, 2744, 32, 16, 0, 0, 0)]
    assert [r[0] for r in plans(low)] == [0] * 3 and all(r[0] for r in plans(tall))


def test_heights_are_the_librarys_choice(plans):
    ask = [("t", KINDS[p, G], M, N, K // 256, 16, 0, 0, 0) for p, G, K, N, M, _, _ in HEIGHTS]
    for case, (ri, splits, _, us) in zip(HEIGHTS, plans(ask)):
        assert ri == case[5] and (splits > 1) == case[6], (case, ri, splits)
    narrow = [("n", G, M, N, K // 256, 16, 0, 0, 0) for p, G, K, N, M, _, _ in HEIGHTS]
    for case, tall, low in zip(HEIGHTS, plans(ask), plans(narrow)):           # (all below 400 tiles of 64 x 256, or wide ones)
        assert case[0] == "a16" or -(-case[4] // 64) * -(-case[3] // 256) >= 400 or tall[3] < low[3], case


@pytest.mark.gpu
@pytest.mark.parametrize("gated", [False, True])
@pytest.mark.parametrize("path,G,K,N,M,ri,split", HEIGHTS)
def test_tile_heights(path, G, K, N, M, ri, split, gated):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_06753_amd import binding as w2
    from test_gpu_parity import bf16_bits, check_epilogue, check_y, dev
    if gated:
        N -= N % 32
    act = w2.ACT_SILU_MUL if gated else w2.ACT_NONE
    codes, scales, X = synth.make_problem(M, K, N, G, 0, seed=M + K + N)
    packed = w2.prepack(dev(codes), dev(scales), G, 0)
    ws = torch.empty(max(16, w2.workspace_size(M, K, N, G, a16=path == "a16")), dtype=torch.uint8, device="cuda")
    # whole pairs of column blocks: the first, the last, and some between; the oracle takes these columns of every row
    pairs = np.unique(np.concatenate([[0, N // 32 - 1], np.random.default_rng(M).choice(N // 32, 4)]))
    cols = (pairs[:, None] * 32 + np.arange(32)[None, :]).reshape(-1)
    if not gated:
        cols = np.unique(np.concatenate([cols, np.arange(N - 8, N)]))
    cs, ss = np.ascontiguousarray(codes[:, cols]), np.ascontiguousarray(scales[:, cols])
    if path == "a16":
        Xb = synth.f32_to_bf16_bits(X)
        Y = w2.matmul_a16_epi(packed, K, N, G, dev(Xb).view(torch.bfloat16), act=act, workspace=ws)
        Yo, y64, mag = oracle.matmul_a16(cs, ss, G, 0, Xb)
    else:
        xq, sx, _ = w2.quantize_rows(dev(X), G)
        Y = w2.matmul_a8_epi(packed, K, N, G, xq, sx, act=act, workspace=ws)
        oq, osx, _ = oracle.quantize_rows(X, G)
        Yo, y64 = oracle.matmul_a8(cs, ss, G, 0, oq, osx)
        mag = oracle.a8_term_magnitude(cs, ss, G, 0, oq, osx)
    what = f"{path} {16 * ri}-row tiles M={M} K={K} N={N} G={G}"
    if gated:
        ocols = (pairs[:, None] * 16 + np.arange(16)[None, :]).reshape(-1)
        check_epilogue(np.ascontiguousarray(bf16_bits(Y)[:, ocols]), y64, mag, None, act, what)
    else:
        check_y(np.ascontiguousarray(bf16_bits(Y)[:, cols]), Yo, y64, mag, what)


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(129, 4608, 288), (256, 1024, 1056)])
def test_forced_width_groups_of_64_with_a_workspace(M, K, N):
    # 128-row tiles of 128 columns, groups of 64: K is never cut into ranges there, so that room for partial results
    # changes nothing, bit for bit
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_06753_amd import binding as w2
    from test_gpu_parity import bf16_bits, check_y, dev
    codes, scales, X = synth.make_problem(M, K, N, 64, 0, seed=M + K + N)
    packed = w2.prepack(dev(codes), dev(scales), 64, 0)
    xq, sx, _ = w2.quantize_rows(dev(X), 64)
    ws = torch.empty(8 * M * N * 4, dtype=torch.uint8, device="cuda")
    tune = {"tiled_bm": 128, "tiled_bn": 128}
    Y, Z = (bf16_bits(w2.matmul_a8(packed, K, N, 64, xq, sx, variant=w2.VARIANT_TILED, workspace=w, tune=tune)) for w in (ws, None))
    assert np.array_equal(Y, Z)
    oq, osx, _ = oracle.quantize_rows(X, 64)
    Yo, y64 = oracle.matmul_a8(codes, scales, 64, 0, oq, osx)
    check_y(Y, Yo, y64, oracle.a8_term_magnitude(codes, scales, 64, 0, oq, osx), f"128 x 128 tiles M={M} K={K} N={N} G=64")
