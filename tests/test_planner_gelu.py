"""What GELU costs in the planner's table for long sums, where that table begins, and which layers get its tiles: asked on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")

PROGRAM = r"""
#include <cstdio>
#include "kernels.h"
using namespace eclip;
int main()
{
    int v[7];
    while (std::scanf("%d %d %d %d %d %d %d", v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6) == 7) {
        GemmTraits t;
        t.lean = true;
        t.even_cu = v[6];
        t.copied = v[4] != 0;
        t.gelu = v[5] != 0;
        const GemmPlan p = conv_gemm_plan(v[0], v[1], v[2], v[3], (size_t)16 << 20, t);
        std::printf("%d %d %d %.6f\n", p.kind, p.variant, p.kind == 0 ? p.splits : p.nw, p.cost);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("gelu")
    src, obj, exe = (str(tmp / n) for n in ("p.cpp", "p.o", "p"))
    pkg = os.path.join(ROOT, "paper_2506_12598_amd")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-c", "-I", os.path.join(pkg, "csrc"),
                    "-I", os.path.join(ROOT, "include"), src, "-o", obj], check=True, capture_output=True)
    subprocess.run(["hipcc", obj, "-o", exe, os.path.join(pkg, "libeclip.so"), "-Wl,-rpath," + pkg], check=True, capture_output=True)

    def run(problems):
        """[(M, N, K, CUs, copied form, GELU[, CUs an undealt launch can count on])] -> [((kind, variant, slices or wavefronts), us)]"""
        text = "".join(" ".join(str(int(v)) for v in (*p, 0)[:7]) + "\n" for p in problems)
        lines = [s.split() for s in subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()]
        return [(tuple(int(v) for v in f[:3]), float(f[3])) for f in lines]
    return run


GRID = [(m, n, k, c) for m in (512, 640, 768, 1005, 1536, 2048, 3072) for n in (768, 1024, 2304, 3072, 4096) for k in (768, 1024, 1536, 3072) for c in range(48, 257, 16)]


def test_gelu_is_free_on_no_tile(plan):
    plain, gelu = plan([p + (1, 0) for p in GRID]), plan([p + (1, 1) for p in GRID])
    for p, (a, us_a), (b, us_b) in zip(GRID, plain, gelu):
        assert us_b > us_a + 0.05, (p, a, b)                           # the cheapest measured: 0.24 us on average
    # the tiles of which many share a compute unit are among those that stay
    assert {b[1] for (a, _), (b, _) in zip(plain, gelu) if a == b and b[0] == 0} & {22, 23, 26}
    assert any(b[0] == 1 for b, _ in gelu)


@pytest.mark.parametrize("m,n,k,cus,small,large", [(768, 3072, 768, 256, 26, 20)])       # us with GELU 12.5, 10.6
def test_gelu_does_not_draw_layers_to_small_tiles(plan, m, n, k, cus, small, large):
    (_, v, _), _ = plan([(m, n, k, cus, 1, 1)])[0]
    assert v != small and v == large


def test_sums_and_rows_where_the_table_begins(plan):
    for inside, outside in (((512, 4096, 768, 64), (511, 4096, 768, 64)), ((1536, 4096, 768, 64), (1536, 4096, 736, 64))):
        (_, a), (_, b), (_, c), (_, d) = plan([inside + (1, 0), inside + (1, 1), outside + (1, 0), outside + (1, 1)])
        assert b > a and c == d


def test_tiles_that_have_fast_forms_only(plan):
    wide = [p + (1, g) for p in GRID for g in (0, 1)]
    assert {v for (kind, v, _), _ in plan(wide) if kind == 0} >= {29, 30, 31}
    small = [(m, n, k, c, 1, g) for m, n, k in ((511, 4096, 1024), (384, 4096, 1024), (1536, 4096, 736), (3072, 1024, 256)) for c in (48, 64, 96, 128) for g in (0, 1)]
    for problems in ([p[:4] + (0, p[5]) for p in wide], small):        # layers whose address form they lack; layers below the table
        assert not {v for (kind, v, _), _ in plan(problems) if kind == 0} & {29, 30, 31}


@pytest.mark.parametrize("m,n,k,cus,even", [(1024, 4096, 1024, 176, 96), (3072, 4096, 1024, 192, 128), (3072, 4096, 1024, 208, 160)])      # us 29.8, 17.3; 47.8, 30.4; 46.9, 30.4
def test_no_two_workgroups_on_a_unit_where_launches_are_dealt(plan, m, n, k, cus, even):
    assert plan([(m, n, k, cus, 1, 0, even)])[0][0][1] not in (29, 30, 31)
    dealt = [p[:3] + (c, 1, g, e) for p in GRID for c, e in ((144, 32), (160, 64), (176, 96), (192, 128), (208, 160), (224, 192)) for g in (0, 1)]
    rows, cols = {29: 128, 30: 128, 31: 192}, {29: 256, 30: 192, 31: 128}
    for p, ((kind, v, _), _) in zip(dealt, plan(dealt)):
        assert kind != 0 or v not in rows or -(-p[0] // rows[v]) * -(-p[1] // cols[v]) <= p[6], p


@pytest.mark.parametrize("m,n,k,cus,slow,best", [
    # us on the tile that looks cheaper by its tiles per compute unit, us on the best one
    (3072, 3072, 768, 96, 29, 25), (2720, 3072, 768, 96, 29, 25), (3072, 2304, 768, 96, 30, 29),       # 65.0, 41.5; 54.0, 37.8; 53.8, 35.8
    (3072, 3072, 1536, 128, 30, 25),                                                                   # 67.5, 59.3
])
def test_blocks_that_one_xcd_has_more_of_are_priced(plan, m, n, k, cus, slow, best):
    (kind, v, _), _ = plan([(m, n, k, cus, 1, 0)])[0]
    assert kind == 0 and v != slow and v in (best, 24)                 # 24 is next to 25 in all of them
