"""What the planner makes of small shares, of shares whose shader engines hold unequal numbers of compute units, and of layers that only some
kernels take in their fast form: called directly on the host."""
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
    char what;
    int v[8];
    while (std::scanf(" %c", &what) == 1) {
        const int n = what == 'f' ? 4 : what == 'e' ? 5 : what == 's' ? 8 : 6;
        for (int i = 0; i < n; ++i) std::scanf("%d", v + i);
        if (what == 'e') {                                   // n_cu and the enabled CUs of the four shader engines
            CuShare cu{v[0], SeDeal()};
            int lo = 255;
            for (int q = 0; q < 4; ++q) {
                const uint32_t c = (uint32_t)v[1 + q];
                if (c == 0) continue;
                cu.deal.se_caps |= c << (8 * q);
                cu.deal.slots++;
                if (c > cu.deal.level) cu.deal.level = c;
                if ((int)c < lo) lo = (int)c;
            }
            if ((int)cu.deal.level == lo) cu.deal.level = 0;
            std::printf("%d\n", cu.even_cu());
        } else if (what == 's') {                            // two layers: M N K and lean form of each; 1 when they share a launch on 256 CUs
            GemmTraits t;
            GemmPlan own[2], pl[2];
            for (int k = 0; k < 2; ++k) {
                t.lean = v[4 * k + 3] >= 0;
                own[k] = conv_gemm_plan(v[4 * k], v[4 * k + 1], v[4 * k + 2], 256, (size_t)16 << 20, t);
            }
            std::printf("%d\n", (int)conv_gemm_plan_pair(own[0], v[0], v[1], v[2], v[3], own[1], v[4], v[5], v[6], v[7], 256, &pl[0], &pl[1]));
        } else if (what == 'f') {                            // KH KW Cin Cout
            std::printf("%d\n", (int)conv_gemm_is_copied(v[0], v[1], v[2], v[3]));
        } else {                                             // p or c (the copied tiles' fast form): M N K n_cu even_cu lean
            GemmTraits t;
            t.even_cu = v[4];
            t.lean = v[5] != 0;
            t.copied = what == 'c';
            const GemmPlan p = conv_gemm_plan(v[0], v[1], v[2], v[3], (size_t)16 << 20, t);
            std::printf("%d %.4f %d %d\n", p.kind, p.cost, p.variant, p.nw);
        }
    }
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    d = tmp_path_factory.mktemp("plans")
    src, obj, exe = str(d / "plans.hip"), str(d / "plans.o"), str(d / "plans")
    open(src, "w").write(PROGRAM)
    pkg = os.path.join(ROOT, "paper_2506_12598_amd")
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-c", "-I", os.path.join(pkg, "csrc"),
                    "-I", os.path.join(ROOT, "include"), src, "-o", obj], check=True, capture_output=True)
    subprocess.run(["hipcc", obj, "-o", exe, os.path.join(pkg, "libeclip.so"), "-Wl,-rpath," + pkg], check=True, capture_output=True)

    def ask(line):
        return subprocess.run([exe], input=line, capture_output=True, text=True, check=True).stdout.split()
    return ask


@pytest.mark.parametrize("n_cu,engines,even", [
    (256, (8, 8, 8, 8), 256), (160, (5, 5, 5, 5), 160), (128, (8, 8, 0, 0), 128),                   # nothing to deal
    (144, (8, 8, 1, 1), 32), (160, (8, 8, 2, 2), 64), (160, (2, 2, 8, 8), 64), (192, (8, 8, 4, 4), 128), (240, (8, 8, 7, 7), 224),
    (88, (0, 8, 0, 3), 48),
])
def test_cus_an_undealt_launch_can_count_on(plans, n_cu, engines, even):
    assert plans(f"e {n_cu} " + " ".join(map(str, engines)) + "\n") == [str(even)]


@pytest.mark.parametrize("m,n,k,n_cu,even", [
    # us on wave-split-K, us on the dealt tile
    (128, 3072, 768, 144, 32), (128, 3072, 768, 160, 64),             # 12.5, 6.9; 9.8, 6.2
    (384, 1024, 1024, 144, 32), (384, 1024, 1024, 160, 64),           # 12.4, 7.1; 10.7, 6.4
    (1005, 768, 3072, 192, 128), (1176, 128, 1152, 144, 32),          # 25.1, 14.3; 22.0, 8.0
])
def test_layers_that_fill_an_uneven_share_take_a_dealt_tile(plans, m, n, k, n_cu, even):
    assert plans(f"p {m} {n} {k} {n_cu} {even} 1\n")[0] == "0"


@pytest.mark.parametrize("lean", [0, 1])
@pytest.mark.parametrize("m,n,k", [(49, 512, 512), (128, 768, 768), (784, 128, 512), (3136, 64, 576), (1005, 768, 3072)])
def test_an_uneven_share_never_looks_cheaper_than_an_even_one(plans, m, n, k, lean):
    even, uneven, fewer = (float(plans(f"p {m} {n} {k} {c} {e} {lean}\n")[1]) for c, e in ((192, 192), (192, 128), (144, 32)))
    assert even <= uneven <= fewer


@pytest.mark.parametrize("m,n,k,n_cu", [(64, 2304, 768, 64), (3136, 64, 576, 96)])      # 7.5 -> 6.6 us, 6.3 -> 5.5
def test_a_second_round_of_32x64_tiles_of_8_wavefronts_is_not_free(plans, m, n, k, n_cu):
    kind, _, variant, nw = plans(f"p {m} {n} {k} {n_cu} 0 1\n")
    assert (kind, variant, nw) != ("1", "1", "8")


def test_even_share_is_the_default(plans):
    for m, n, k in ((128, 3072, 768), (1536, 1024, 4096), (49, 2048, 512)):
        assert plans(f"p {m} {n} {k} 160 0 1\n") == plans(f"p {m} {n} {k} 160 160 1\n")


@pytest.mark.parametrize("kh,kw,cin,cout,copied", [
    (1, 1, 1024, 4096, 1), (1, 1, 1032, 4096, 0), (1, 1, 1024, 4092, 0), (3, 3, 96, 2048, 1), (3, 3, 72, 2048, 0), (4, 8, 64, 64, 1), (7, 7, 64, 2048, 0),
])
def test_which_layers_the_copied_tiles_take_in_their_fast_form(plans, kh, kw, cin, cout, copied):
    assert plans(f"f {kh} {kw} {cin} {cout}\n") == [str(copied)]


@pytest.mark.parametrize("what,k,variant,fixed,step", [
    ("c", 1024, 17, 9.7, 0.515), ("c", 4096, 17, 9.7, 0.515),
    ("p", 1024, 3, 8.784, 0.568), ("p", 2048, 17, 10.9, 0.512),      # general address form or ragged columns: the copied tile from 1056 on
])
def test_256x256_tiles_are_picked_and_priced_by_one_table(plans, what, k, variant, fixed, step):
    # 96 tiles of 256 x 256, one per CU
    kind, cost, v, _ = plans(f"{what} 1536 4096 {k} 96 0 1\n")
    assert (kind, v) == ("0", str(variant))
    assert float(cost) == pytest.approx(fixed + k / 32 * step * 1.15, abs=1e-3)


def test_short_sums_stay_on_the_ping_pong_tiles(plans):
    for k in (128, 256):
        assert plans(f"c 1536 4096 {k} 96 0 1\n")[2] != "17"


ROWS, ROWS_TAIL, WINDOW, GENERAL = 0, 1, 2, -1


@pytest.mark.parametrize("a,b,shared", [
    ((784, 128, 72, ROWS_TAIL), (784, 128, 2304, WINDOW), 0),      # the general kernel's price: no lean form serves both
    ((784, 128, 72, ROWS_TAIL), (784, 128, 64, ROWS), 1),          # short sums: it pays all the same
    ((784, 128, 64, ROWS), (784, 128, 2304, WINDOW), 1), ((784, 128, 576, WINDOW), (784, 128, 2304, WINDOW), 1),
    ((784, 128, 72, ROWS_TAIL), (784, 128, 72, ROWS_TAIL), 1),
])
def test_two_layers_are_priced_on_the_kernel_that_would_run_both(plans, a, b, shared):
    ask = lambda p, q: plans("s " + " ".join(map(str, p + q)) + "\n")
    assert ask(a, b) == ask(b, a) == [str(shared)]
