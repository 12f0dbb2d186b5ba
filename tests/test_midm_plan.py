"""The mid-M kernel's launch shapes, on the host: csrc/midm_plan.h compiled by itself."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "%s/paper_2508_06753_amd/csrc/midm_plan.h"
#include <stdio.h>
int main()
{
    int xt, gated, cbw, splitk, G;
    long long M, n_cb, n_kt, cap;
    while (scanf("%%d %%lld %%lld %%lld %%d %%d %%lld %%d %%d", &xt, &M, &n_cb, &n_kt, &gated, &cbw, &cap, &splitk, &G) == 9) {
        if (M == 0) {                                        // (rows that no call has: the registers' table; gated: with parts)
            printf("%%d\n", w2::midm::simd_waves(w2::midm::kind_of(xt, G), (int)n_cb, (int)n_kt, gated != 0));
            continue;
        }
        w2_tuning_t tune = {};
        tune.midm_cbw = cbw;
        tune.splitk = splitk;
        const w2::midm::Plan p = w2::midm::plan(xt, M, n_cb, n_kt, gated != 0, cap, tune, nullptr, G);
        printf("%%d %%d %%d %%d %%d\n", p.rt, p.cj, p.ks, p.sh, p.sp);
    }
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("midm_plan")
    (d / "p.cpp").write_text(PROGRAM % ROOT)
    subprocess.run(["g++", "-O1", "-std=c++17", "-o", str(d / "p"), str(d / "p.cpp")], check=True)

    def ask(problems):
        """problems: (rows int8 0 / bf16 1, M, K, N, gated, midm_cbw[, copies of the output that fit, splitk[, G]])
        -> (rt, cj, ks, sh, sp) each"""
        text = "".join("{} {} {} {} {} {} {} {} {}\n".format(xt, M, (N + 15) // 16, K // 256, g, cbw, *(more + [0, 0, 128][len(more):]))
                       for xt, M, K, N, g, cbw, *more in problems)
        out = subprocess.run([str(d / "p")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, l.split())) for l in out.splitlines()]

    return ask


SHAPES = [(K, N) for K in (256, 512, 2304, 4096, 8192, 14336, 23040, 28672) for N in (8, 16, 48, 1024, 1376, 1408, 1488, 6144, 8192, 28672)]
ROWS = (1, 5, 16, 17, 33, 64, 65, 99, 173, 241, 256)


def test_shapes_fit_the_kernel(plans):
    problems = [(xt, M, K, N, g, cbw, cap, splitk) for xt in (0, 1) for K, N in SHAPES for M in ROWS for g in (0, 1)
                if not (g and N % 32) for cbw in (0, 2, 4, 8) for cap, splitk in ((0, 0), (1, 3), (2, 3), (16, 0), (16, 1), (16, 16))]
    for (xt, M, K, N, g, cbw, cap, splitk), (rt, cj, ks, sh, sp) in zip(problems, plans(problems)):
        assert 1 <= rt <= min((M + 15) // 16, 4) and cj in ((1, 2, 4) if rt == 1 else (2, 4))
        assert ks >= 1 and 1 <= sp <= max(1, min(cap, 16)) and ks * sp <= K // 256     # every range holds a tile
        assert splitk == 0 or sp == max(1, min(splitk, cap, K // 256))
        assert sh in (1, 2) and (sh == 1 or xt == 0)
        assert ks * sh <= (16 if rt == 1 and cj <= 2 else 8)
        assert not g or cj * sh >= 2
        assert not cbw or cj * sh == (cbw if xt == 0 else min(cbw, 4))
        stage, red = rt * 2048 * sh, sh * rt * 16 * (cj * 16 + 4) * 4
        assert ks * max(stage, red) + rt * 64 <= 160 * 1024


def test_row_stream_limit(plans):
    # int8 rows: no shape of one or two column blocks per workgroup where all workgroups together would read more than
    # 172 MB of rows; just below, that shape may win.  (The sizes that the GPU tests run on either side.)
    def streamed(M, K, N, p):
        return -(-((N + 15) // 16) // (p[1] * p[3])) * M * K

    problems = [(0, M, K, N, 0, 0) for K, N in SHAPES for M in ROWS]
    for (_, M, K, N, _, _), p in zip(problems, plans(problems)):
        assert p[1] * p[3] > 2 or streamed(M, K, N, p) <= 172000000, (M, K, N, p)
    for M, N in ((241, 672), (256, 640)):
        below, above = plans([(0, M, 32768, N, 0, 0), (0, M, 32768, N + 32, 0, 0)])
        assert below[1] * below[3] == 2 and above[1] * above[3] == 4, (M, below, above)
    # two column blocks are not replaced by one, which reads twice as much
    (p,) = plans([(0, 173, 23040, 1488, 0, 0)])
    assert streamed(173, 23040, 1488, p) < 110000000


def test_k_across_workgroups(plans):
    # only with room for two copies of the output, on a deep K, for a grid that all fits the chip at once
    problems = [(xt, M, K, N, 0, 0, cap, 0) for xt in (0, 1) for K, N in SHAPES for M in ROWS for cap in (0, 1, 2, 5, 16)]
    split = 0
    for (xt, M, K, N, _, _, cap, _), (rt, cj, ks, sh, sp) in zip(problems, plans(problems)):
        if sp > 1:
            split += 1
            wgs = -(-((N + 15) // 16) // (cj * sh)) * -(-M // (16 * rt))
            assert cap >= 2 and K >= (20480 if xt == 0 else 8192) and wgs * sp <= (256 if xt == 0 or wgs <= 128 else 512)
            assert ks * sp <= K // 512
    assert split > 50


def test_odd_widths(plans):
    # three or five column blocks per wave: only above 512 blocks, where the busiest CU then has no more blocks to do than with
    # two or four; in pairs (an even number per workgroup) for the gated epilogue; never with K split across workgroups
    def busiest(blocks, width, bands):
        return -(-(-(-blocks // width) * bands) // 256) * width

    problems = [(xt, M, K, N, g, 0, cap, 0) for xt in (0, 1) for K in (768, 1280, 2048, 5120) for N in range(7968, 36000, 544)
                for M in (3, 16, 31, 33, 49, 64, 96, 240) for g in (0, 1) for cap in (0, 16)]
    odd = set()
    for (xt, M, K, N, g, _, _, _), (rt, cj, ks, sh, sp) in zip(problems, plans(problems)):
        if cj not in (3, 5):
            continue
        blocks, bands = -(-N // 16), -(-M // (16 * rt))
        assert blocks > 512 and sp == 1 and bands <= 4 and not (g and sh == 1) and not (rt == 4 and cj == 5)
        assert ks * sh <= 8 and ks * max(rt * 2048 * sh, sh * rt * 16 * (cj * 16 + 4) * 4) + rt * 64 <= 160 * 1024
        assert busiest(blocks, cj * sh, bands) <= min(busiest(blocks, 2 * sh, bands), busiest(blocks, 4 * sh, bands))
        odd.add((xt, cj, sh))
    assert odd >= {(0, 3, 1), (0, 3, 2), (1, 3, 1), (1, 3, 2), (1, 5, 1), (1, 5, 2)}
    # the sizes that the GPU tests run
    for p, want in (((0, 64, 1024, 8776, 0, 0), (1, 3, 4, 1)), ((0, 16, 2048, 22432, 1, 0), (1, 3, 4, 2)),
                    ((0, 96, 768, 11560, 0, 0), (2, 3, 3, 1)), ((0, 48, 768, 21928, 0, 0), (3, 3, 3, 1)),
                    ((0, 96, 2048, 10912, 1, 0), (3, 3, 4, 2)), ((1, 32, 1280, 17928, 0, 0), (1, 3, 4, 1)),
                    ((1, 16, 2048, 8760, 0, 0), (1, 3, 8, 1)), ((1, 32, 1024, 23200, 1, 0), (2, 3, 4, 2)),
                    ((1, 31, 2048, 16392, 0, 0), (2, 5, 8, 1)), ((1, 96, 1536, 8264, 0, 0), (3, 5, 6, 1)),
                    ((1, 96, 1536, 19360, 1, 0), (3, 5, 4, 2)), ((1, 64, 1280, 18336, 1, 0), (4, 3, 2, 2)), ((0, 64, 4096, 8200, 0, 0), (2, 5, 8, 1)),
                    ((1, 64, 768, 18952, 0, 0), (4, 3, 3, 1))):
        (got,) = plans([p])
        assert got == want + (1,), (p, got)


def test_every_odd_form_is_run(plans):
    # the GPU tests' list has every (rows, row tiles, blocks, waves to a range, exact dequant) of three and five blocks that the
    # planner gives over a grid of sizes, in both group sizes
    from test_gpu_parity import MIDM_ODD_FORMS

    def forms(problems):
        return {(p[0], rt, cj, sh, p[0] == 0 and p[1] <= 32) for p, (rt, cj, _, sh, _) in zip(problems, plans(problems)) if cj in (3, 5)}

    grid = [(xt, M, K, N, g, 0, 0, 0, G) for xt in (0, 1) for M in (5, 9, 16, 17, 31, 33, 40, 49, 64, 96, 97, 128, 192)
            for K in (512, 768, 1024, 2048, 3072, 5120, 8192, 10240, 14336) for N in range(8192, 57344, 416) for g in (0, 1) for G in (64, 128)]
    run = [{(p, G): forms([p + (0, 0, 0, G)]) for p in MIDM_ODD_FORMS} for G in (64, 128)]
    for r in run:
        assert all(r.values())                               # each is what it is there for
        have = set().union(*r.values())
        assert len(have) == len(MIDM_ODD_FORMS) == 32 and have >= forms(grid)


def test_pairs_of_one_block(plans):
    # int8 rows: two waves of one column block each on one K range, on narrow grids of short launches
    for M, K, N in ((57, 1536, 4672), (77, 2560, 3360), (210, 1024, 1600), (169, 2560, 1632)):
        assert plans([(0, M, K, N, int(N % 32 == 0), 0)]) == [(1, 1, 2, 2, 1)]


def test_groups_of_64_take_more_registers(plans):
    # bf16 rows, groups of 64: one row tile x 2 blocks holds four waves a SIMD where groups of 128 hold five, and parts of one
    # row tile x 4 blocks three: no second round that the price does not know of, no parts that do not run at once
    assert plans([(1, 22, 1280, 18496, 0, 0, 16, 0, G) for G in (128, 64)]) == [(1, 2, 4, 1, 1), (2, 2, 4, 1, 1)]
    for M, K, N in ((7, 27648, 12896), (8, 22784, 13184), (3, 26624, 14240)):
        assert [p[4] for p in plans([(1, M, K, N, 0, 0, 16, 0, G) for G in (128, 64)])] == [2, 1]


def test_uneven_waves_fill_a_simd(plans):
    # (rows, M, K, N): measured 20 to 40 % slower in 5, 6, 9 or 10 waves, of which a CU runs fewer workgroups than its registers
    # would hold
    problems = [(1, 71, 1536, 8384), (1, 18, 1536, 42944), (1, 51, 2560, 2848), (1, 22, 2560, 5664), (0, 79, 2560, 2112), (0, 57, 2560, 3552)]
    for (xt, M, K, N), (rt, cj, ks, sh, sp) in zip(problems, plans([p + (0, 0) for p in problems])):
        wgs, waves = -(-((N + 15) // 16) // (cj * sh)) * -(-M // (16 * rt)), ks * sh
        per_simd = plans([(xt, 0, 256 * cj, 16 * rt, 0, 0)])[0][0]
        assert wgs <= 256 * max(1, per_simd // -(-waves // 4)) or waves <= 4, (M, K, N, waves)


READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def test_simd_waves_are_those_of_the_built_kernels(plans, tmp_path):
    # the planner's table against the registers of what was compiled
    lib = os.path.join(ROOT, "paper_2508_06753_amd", "libw2mm.so")
    if not (os.path.exists(lib) and os.path.exists(READELF)):
        pytest.skip("no built library or no llvm-readelf")
    data, magic, regs, at = open(lib, "rb").read(), b"__CLANG_OFFLOAD_BUNDLE__", {}, -1
    while (at := data.find(magic, at + 1)) >= 0:             # (one bundle per source file)
        (n,), p = struct.unpack_from("<Q", data, at + len(magic)), at + len(magic) + 8
        if n > 8:
            continue                                         # (the text itself, in a string)
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name, p = data[p + 24:p + 24 + idlen], p + 24 + idlen
            if b"gfx950" in name and b"midm_kernel" in (code := data[at + off:at + off + size]):
                (tmp_path / "code").write_bytes(code)
                notes = subprocess.run([READELF, "--notes", str(tmp_path / "code")], capture_output=True, text=True).stdout
                for m in re.finditer(r"\.name:\s+\S*midm_kernelILi(\d)ELi(\d+)ELi(\d)ELi(\d)ELi(\d)ELb(\d)ELi(\d)E.*?\.vgpr_count:\s+(\d+)",
                                     notes, re.S):
                    regs[tuple(map(int, m.groups()[:7]))] = int(m[8])
    assert len(regs) > 200
    # (xt, G, rt, cj, waves to a range, exact dequant, 0 whole / 1 parts / 2 the test-only export)
    keys = [k for k in regs if k[6] < 2]
    for k, (table,) in zip(keys, plans([(k[0], 0, 256 * k[3], 16 * k[2], k[6], 0, 0, 0, k[1]) for k in keys])):
        waves = min(8, 512 // (-(-regs[k] // 8) * 8))
        assert waves - 2 <= table <= waves, (k, regs[k])     # (pairs of one block with the exact dequant: six of eight)
