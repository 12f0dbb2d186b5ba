"""AUTO's choice of kernel and the launch shapes that it hands on: csrc/auto_plan.h compiled by itself."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "%s/paper_2508_06753_amd/csrc/auto_plan.h"
#include <stdio.h>
using namespace w2;
static bool same(const midm::Plan& a, const midm::Plan& b) { return a.rt == b.rt && a.cj == b.cj && a.ks == b.ks && a.sh == b.sh && a.sp == b.sp; }
int main()
{
    int a16, G, gated;
    long long M, K, N, cap;
    while (scanf("%%d %%lld %%lld %%lld %%d %%d %%lld", &a16, &M, &K, &N, &G, &gated, &cap) == 7) {
        const w2_tuning_t tn = {};
        const route::Problem p = {M, K, N, (N + 15) / 16, K / 256, G, gated != 0, cap};
        double us = 0, tiled_us;
        const midm::Plan m = M <= 256 ? route::midm_shape(a16, p, tn, &us) : midm::Plan{};
        int variant, fallback = 0;
        bool as_planned, low = false;
        if (!a16) {
            const route::A8 r = route::a8(p, tn);
            const tiles::A8Shape t = route::a8_tiled_shape(p, tn);
            variant = r.variant; fallback = r.fallback; tiled_us = t.us; low = t.ri == 0;
            as_planned = (!r.has_midm || same(r.midm, m)) &&
                         (!r.has_tiled || (r.tiled.ri == t.ri && r.tiled.bn == t.bn && r.tiled.kw == t.kw && r.tiled.splits == t.splits));
        } else {
            const route::A16 r = route::a16(p, tn);
            const tiles::Shape t = route::a16_tiled_shape(p, tn);
            variant = r.gemv_first ? W2_VARIANT_GEMV : r.to_midm ? W2_VARIANT_MIDM : W2_VARIANT_TILED;
            fallback = r.to_midm ? W2_VARIANT_MIDM : W2_VARIANT_TILED; tiled_us = t.us;
            as_planned = (!r.has_midm || same(r.midm, m)) && (!r.has_tiled || (r.tiled.ri == t.ri && r.tiled.splits == t.splits));
        }
        printf("%%d %%d %%d %%.9g %%.9g %%.9g\n", variant, fallback, (int)as_planned, us, tiled_us, route::tiled_share(a16, m, low));
    }
}
"""
TILED, MIDM, SMALLM, GEMV = 3, 4, 2, 6


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("auto_plan")
    (d / "p.cpp").write_text(PROGRAM % ROOT)
    subprocess.run(["g++", "-O1", "-std=c++17", "-o", str(d / "p"), str(d / "p.cpp")], check=True)

    def ask(problems):
        """problems: (rows int8 0 / bf16 1, M, K, N, G, gated, copies of the output that fit)
        -> (kernel, the next one, shapes as planned, price of the mid-M kernel, of the tiled ones, margin) each"""
        text = "".join("{} {} {} {} {} {} {}\n".format(*p) for p in problems)
        out = subprocess.run([str(d / "p")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(v) if i < 3 else float(v) for i, v in enumerate(l.split())) for l in out.splitlines()]

    return ask


PROBLEMS = [(a16, M, K, N, G, g, cap) for a16 in (0, 1) for K in (256, 1024, 2048, 4096, 5120, 8192, 14336, 28672)
            for N in (8, 1024, 2048, 6144, 8192, 10240, 12288, 28672, 57344) for G in (64, 128) for g in (0, 1) if not (g and N % 32)
            for cap in (0, 1, 2, 16) for M in (1, 4, 5, 8, 9, 12, 16, 17, 32, 33, 48, 64, 65, 96, 100, 128, 129, 192, 240, 256, 257, 4096)]


def test_kernels_take_their_rows(routes):
    for (a16, M, *_), (kernel, then, *_) in zip(PROBLEMS, routes(PROBLEMS)):
        for k in (kernel, then):
            assert k in ((TILED, MIDM, GEMV) if a16 else (TILED, MIDM, SMALLM, GEMV))
            assert k != GEMV or M <= 32
            assert k != MIDM or 3 <= M <= 256
            assert k != SMALLM or M <= 16
        assert then != GEMV


def test_prices_decide_and_shapes_are_handed_on(routes):
    # from 33 rows on the tiled kernels come first where they are cheaper by the margin, priced or skipped because the mid-M
    # kernel is cheaper than any launch of them; what was priced is what is launched
    cheaper = 0
    for (a16, M, K, N, G, g, cap), (kernel, then, as_planned, midm, tiled, margin) in zip(PROBLEMS, routes(PROBLEMS)):
        assert as_planned
        if 32 < M <= 256:
            if tiled < margin * midm:
                assert kernel == TILED
                cheaper += 1
            elif M <= 48:                                                    # (within the mid-M kernel's range everywhere)
                assert kernel == MIDM
    assert cheaper > 50


def test_sides_of_the_line(routes):
    # graph-timed on both kernels: tiled 6 to 14 % faster, where one share for all shapes kept the mid-M kernel; mid-M 1 to 5 %
    # faster (eight K ranges, priced high), or 10 % (64-row tiles, priced low); tiled with room for its K ranges only
    tiled = [(0, 127, 26880, 9664, 128, 0, 16), (0, 121, 27648, 11648, 128, 0, 16), (0, 126, 25600, 10112, 128, 0, 16),
             (1, 226, 13312, 6688, 64, 0, 16), (1, 128, 24576, 6144, 128, 0, 16), (1, 225, 12800, 6912, 64, 0, 16)]
    midm = [(0, 103, 24832, 6976, 128, 0, 16), (0, 80, 29440, 8192, 128, 0, 16), (0, 77, 26624, 7360, 128, 0, 16),
            (1, 100, 28672, 4096, 128, 0, 16), (0, 101, 7680, 33408, 128, 0, 16)] + [p[:6] + (0,) for p in tiled]
    assert [r[0] for r in routes(tiled)] == [TILED] * len(tiled)
    assert [r[0] for r in routes(midm)] == [MIDM] * len(midm)
