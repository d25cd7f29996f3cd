"""Rules that choose a launch on the host, called directly: a small program around the library and its headers, built once."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")

PROGRAM = r"""
#include <cstdio>
#include "gemm_tile.h"
using namespace eclip;
int main()
{
    char what;
    int v[8];
    while (std::scanf(" %c", &what) == 1) {
        if (what == 'a') {                                   // addressing form: KH KW Cin K-step loop
            std::scanf("%d %d %d %d %d", v, v + 1, v + 2, v + 3, v + 4);
            GemmDev d{};
            d.KH = v[0]; d.KW = v[1]; d.Cin = v[2]; d.K = v[0] * v[1] * v[2];
            std::printf("%d\n", gemm_amode(d, v[3], v[4]));
        } else if (what == 'p') {                            // plan of a problem: M N K compute-units
            std::scanf("%d %d %d %d", v, v + 1, v + 2, v + 3);
            const GemmPlan p = conv_gemm_plan(v[0], v[1], v[2], v[3], (size_t)16 << 20);
            std::printf("%d %d %d %.6f\n", p.kind, p.variant, p.splits, p.cost);
        } else if (what == 's') {                            // shape of a first layer that reads the caller's planes: M N K compute-units
            std::scanf("%d %d %d %d", v, v + 1, v + 2, v + 3);
            GemmPlan p{};
            std::printf("%d\n", conv_gemm_plan_stem(v[0], v[1], v[2], v[3], 0, 1e9, &p) ? p.variant : -1);
        } else if (what == 'w') {                            // cost of a wave-split-K shape with 4 wavefronts: M N K compute-units shape
            std::scanf("%d %d %d %d %d", v, v + 1, v + 2, v + 3, v + 4);
            std::printf("%.6f\n", conv_wsk_cost_estimate(v[0], v[1], v[2], v[3], v[4], 4));
        }
    }
}
"""
GENERAL, UNIFORM, MATRIX = range(3)
PINGPONG, BDIRECT, DMA = 2, 3, 4


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, obj, exe = str(d / "rules.hip"), str(d / "rules.o"), str(d / "rules")
    open(src, "w").write(PROGRAM)
    pkg = os.path.join(ROOT, "paper_2506_12598_amd")
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-c", "-I", os.path.join(pkg, "csrc"),
                    "-I", os.path.join(ROOT, "include"), src, "-o", obj], check=True, capture_output=True)
    subprocess.run(["hipcc", obj, "-o", exe, os.path.join(pkg, "libeclip.so"), "-Wl,-rpath," + pkg], check=True, capture_output=True)

    def ask(line):
        return subprocess.run([exe], input=line, capture_output=True, text=True, check=True).stdout.split()
    return ask


@pytest.mark.parametrize("loop", [PINGPONG, BDIRECT, DMA])
@pytest.mark.parametrize("kh,kw,cin,bk,form", [
    (1, 1, 128, 64, MATRIX), (1, 1, 96, 64, GENERAL), (3, 3, 64, 64, UNIFORM), (3, 3, 96, 64, GENERAL), (3, 3, 96, 32, UNIFORM),
    (4, 8, 64, 64, UNIFORM),                                  # 32 taps: the last window whose taps fit a word of bits
    (3, 11, 64, 64, None), (7, 7, 512, 32, None),             # more: a limit of the kernel that keeps those bits, and of no other
])
def test_addressing_form(rules, kh, kw, cin, bk, loop, form):
    want = (GENERAL if loop == DMA else UNIFORM) if form is None else form
    assert rules(f"a {kh} {kw} {cin} {bk} {loop}\n") == [str(want)]


@pytest.mark.parametrize("m,n,k,n_cu,variant,cost", [
    (1536, 4096, 1024, 96, 3, 8.784 + 32 * 0.568 * 1.15),                               # 96 tiles of 256 x 256, one per CU
    (1536, 1024, 4096, 96, 20, 4.272 + 64 * 0.337 * 1.15),                              # 96 tiles of 128 x 128
])
def test_a_tile_is_priced_as_its_row_of_the_table_says(rules, m, n, k, n_cu, variant, cost):
    # fixed cost + K steps x cost per step, slower by 15 % on a full GPU, and nothing on top that the fit does not contain
    got = rules(f"p {m} {n} {k} {n_cu}\n")
    assert got[:3] == ["0", str(variant), "1"]
    assert float(got[3]) == pytest.approx(cost, abs=1e-4)


@pytest.mark.parametrize("n_cu", [64, 96, 128, 160, 192, 256])
@pytest.mark.parametrize("m,n,k", [(12544, 64, 392), (3 * 12544, 32, 72), (25088, 64, 392), (50176, 64, 72), (12 * 6400, 64, 392)])
def test_first_layer_takes_the_shape_whose_loop_is_cheapest(rules, m, n, k, n_cu):
    # wave-split-K shapes are compared by the cost of their loops; the price against other kernels only decides whether one is taken
    shapes = [0, 1, 5]
    cost = [float(c) for c in rules("".join(f"w {m} {n} {k} {n_cu} {v}\n" for v in shapes))]
    assert rules(f"s {m} {n} {k} {n_cu}\n") == [str(shapes[cost.index(min(cost))])]
