"""The mid-M kernel's launch shapes, on the host: csrc/midm_plan.h compiled by itself."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "%s/paper_2508_06753_amd/csrc/midm_plan.h"
#include <stdio.h>
int main()
{
    int xt, gated, cbw;
    long long M, n_cb, n_kt;
    while (scanf("%%d %%lld %%lld %%lld %%d %%d", &xt, &M, &n_cb, &n_kt, &gated, &cbw) == 6) {
        w2_tuning_t tune = {};
        tune.midm_cbw = cbw;
        const w2::midm::Plan p = w2::midm::plan(xt, M, n_cb, n_kt, gated != 0, tune);
        printf("%%d %%d %%d %%d\n", p.rt, p.cj, p.ks, p.sh);
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
        """problems: (rows int8 0 / bf16 1, M, K, N, gated, midm_cbw) -> (rt, cj, ks, sh) each"""
        text = "".join(f"{xt} {M} {(N + 15) // 16} {K // 256} {int(g)} {cbw}\n" for xt, M, K, N, g, cbw in problems)
        out = subprocess.run([str(d / "p")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, l.split())) for l in out.splitlines()]

    return ask


SHAPES = [(K, N) for K in (256, 512, 2304, 4096, 8192, 14336, 23040, 28672) for N in (8, 16, 48, 1024, 1376, 1408, 1488, 6144, 8192, 28672)]
ROWS = (1, 5, 16, 17, 33, 64, 65, 99, 173, 241, 256)


def test_shapes_fit_the_kernel(plans):
    problems = [(xt, M, K, N, g, cbw) for xt in (0, 1) for K, N in SHAPES for M in ROWS for g in (0, 1) if not (g and N % 32)
                for cbw in (0, 2, 4, 8)]
    for (xt, M, K, N, g, cbw), (rt, cj, ks, sh) in zip(problems, plans(problems)):
        assert 1 <= rt <= min((M + 15) // 16, 4) and cj in ((1, 2, 4) if rt == 1 else (2, 4))
        assert 1 <= ks <= K // 256 and sh in (1, 2) and (sh == 1 or xt == 0)
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
