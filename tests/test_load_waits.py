"""The kernels that count their loads to local memory: what a barrier lets through has landed.  The order in which a wave issues its
loads, walked with the kernels' own counts (csrc/tall_waits.h and csrc/shared_plan.h, compiled by themselves); vector memory operations complete in order."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "%s/paper_2508_06753_amd/csrc/shared_plan.h"
#include "%s/paper_2508_06753_amd/csrc/tall_waits.h"
#include <stdio.h>
using namespace w2;
int main()
{
    for (int pair = 0; pair < 2; ++pair)
        for (int np = 1; np <= 4; ++np) {
            printf("%%d %%d %%d %%d", tall::ahead(pair), tall::at_start(pair, np), tall::weights(false, 2), tall::weights(true, 2));
            for (int t = 0; t < 4; ++t) printf(" %%d %%d", tall::behind(pair, t, np, 0), tall::behind(pair, t, np, 1));
            printf("\n");
        }
    for (int ch : {2, 4})
        for (int rt = 2; rt <= 4; ++rt)
            for (const auto& s : shared::SHAPES)
                for (int h = 0; h < ch; ++h)
                    printf("%%d %%d %%d %%d %%d %%d\n", ch, shared::BUFS, shared::loads(rt, s[1]), s[0], h, shared::under_way(h, ch, shared::loads(rt, s[1]), s[0]));
}
"""


@pytest.fixture(scope="module")
def counts(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("load_waits")
    (d / "p.cpp").write_text(PROGRAM % (ROOT, ROOT))
    subprocess.run(["g++", "-O1", "-std=c++17", "-o", str(d / "p"), str(d / "p.cpp")], check=True)
    lines = [tuple(map(int, l.split())) for l in subprocess.run([str(d / "p")], capture_output=True, text=True, check=True).stdout.splitlines()]
    counts = {(pair, np_): lines[4 * pair + np_ - 1] for pair in (0, 1) for np_ in (1, 2, 3, 4)}
    counts["shared"] = {}
    for ch, bufs, nj, cj, h, n in lines[8:]:
        counts["shared"].setdefault((ch, bufs, nj, cj), {})[h] = n
    return counts


class Wave:
    def __init__(self):
        self.issued, self.landed = [], 0

    def load(self, what, n):
        self.issued += [what] * n

    def wait(self, left):
        self.landed = max(self.landed, len(self.issued) - left)

    def has(self, what):
        return what not in self.issued[self.landed:]


def tall(counts, pair, np_, per_tile, counted, issued, stages=48):
    # -> whether every stage that a barrier lets a wave read has landed
    ahead, start, _, _, *by_stage = counts[pair, np_]
    w, ok = Wave(), True
    w.load("weights", issued)
    for s in range(ahead):
        w.load(s, np_)
    w.wait(start)
    ok &= all(w.has(s) for s in range(3 if pair else 2))
    for it in range(stages):
        t = it % per_tile
        if t == 0:
            w.load("weights", issued)
        w.load(it + ahead, np_)
        if not pair or t & 1:
            base, one = by_stage[2 * t:2 * t + 2]
            w.wait(base + (one - base) * counted)
            ok &= all(w.has(s) for s in range(it + 1, it + (4 if pair else 3)))
    return ok


@pytest.mark.parametrize("pair", [0, 1])
@pytest.mark.parametrize("np_", [1, 2, 3, 4])
def test_tall_tiles(counts, pair, np_):
    product, export = counts[pair, np_][2:4]
    for per_tile in (2, 4):
        assert tall(counts, pair, np_, per_tile, product, 4)
        # an export issues as many as the compiler leaves of them
        assert all(tall(counts, pair, np_, per_tile, export, n) for n in range(5))
        # (the walk sees a count that is too high)
        assert not tall(counts, pair, np_, per_tile, product, 2) and not tall(counts, pair, np_, per_tile, product + 1, 4)


def shared(bufs, ch, nj, cj, counts, tiles=12):
    w, ok = Wave(), True
    for c in range(bufs - 1):
        w.load(c, nj)
    for i in range(2):                                       # two tiles of weights in flight
        w.load("weights", 2 * cj)
    for c in range(tiles * ch):
        w.wait(counts[c % ch])
        ok &= w.has(c)
        w.load(c + bufs - 1, nj)
        if c % ch == ch - 1:
            w.load("weights", 2 * cj)
    return ok


def test_shared_rows(counts):
    for (ch, bufs, nj, cj), n in counts["shared"].items():
        assert max(n.values()) < 64                          # (what a wait can count)
        assert shared(bufs, ch, nj, cj, n)
        assert not any(shared(bufs, ch, nj, cj, {**n, h: n[h] + 1}) for h in n)
    assert len(counts["shared"]) == 12
