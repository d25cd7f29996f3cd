"""Which layers the lean form of the wave-split-K kernel takes, and the reciprocals it divides with: called directly on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")

PROGRAM = r"""
#include <cstdio>
#include "gemm_common.h"
using namespace eclip;
static GemmDev layer(const int *v)
{
    GemmDev d{};
    d.KH = v[0]; d.KW = v[1]; d.stride = v[2]; d.pad = v[3]; d.Cin = v[4]; d.N = v[5]; d.ldy = v[6]; d.nchw_c = v[7];
    d.K = d.KH * d.KW * d.Cin;
    return d;
}
int main()
{
    char what;
    while (std::scanf(" %c", &what) == 1) {
        int v[16];
        const int n = what == 'p' ? 16 : 8;
        if (what == 'd') {                                       // n / d for the n where a reciprocal can be off by one
            unsigned d, bad = 0;
            std::scanf("%u", &d);
            const Magic m = magic_of(d);
            for (unsigned long long q = 0; q * d < (1ull << 31); q += q < 1000 ? 1 : q / 97)
                for (long long e = -1; e <= 1; ++e) {
                    const long long x = (long long)(q * d) + e;
                    if (x < 0 || x >= (1ll << 31)) continue;
                    bad += (unsigned)(((unsigned long long)(unsigned)(2 * x) * m.mul) >> 32 >> m.shift) != (unsigned)x / d;
                }
            const unsigned top = 0x7fffffffu;
            bad += (unsigned)(((unsigned long long)(2 * top) * m.mul) >> 32 >> m.shift) != top / d;
            std::printf("%u\n", bad);
            continue;
        }
        for (int i = 0; i < n; ++i) std::scanf("%d", v + i);
        if (what == 'p') std::printf("%d\n", wsk_lean_pair_form(layer(v), layer(v + 8)));
        else std::printf("%d\n", wsk_lean_form(layer(v)));
    }
}
"""
ROWS, ROWS_TAIL, WINDOW, GENERAL = 0, 1, 2, -1


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    d = tmp_path_factory.mktemp("forms")
    src, obj, exe = str(d / "forms.hip"), str(d / "forms.o"), str(d / "forms")
    open(src, "w").write(PROGRAM)
    pkg = os.path.join(ROOT, "paper_2506_12598_amd")
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-c", "-I", os.path.join(pkg, "csrc"),
                    "-I", os.path.join(ROOT, "include"), src, "-o", obj], check=True, capture_output=True)
    subprocess.run(["hipcc", obj, "-o", exe, os.path.join(pkg, "libeclip.so"), "-Wl,-rpath," + pkg], check=True, capture_output=True)

    def ask(line):
        return [int(v) for v in subprocess.run([exe], input=line, capture_output=True, text=True, check=True).stdout.split()]
    return ask


LAYERS = [
    # KH KW stride pad Cin N ldy planes
    ((1, 1, 1, 0, 64, 64, 64, 0), ROWS), ((1, 1, 1, 0, 72, 64, 64, 0), ROWS_TAIL), ((1, 1, 1, 0, 8, 4, 4, 0), ROWS_TAIL),
    ((1, 1, 2, 0, 64, 64, 64, 0), WINDOW), ((1, 1, 2, 0, 72, 64, 64, 0), GENERAL), ((1, 1, 1, 1, 64, 64, 64, 0), WINDOW),
    ((3, 3, 1, 1, 32, 32, 256, 0), WINDOW), ((3, 3, 1, 1, 48, 32, 32, 0), GENERAL),
    ((1, 31, 1, 0, 32, 32, 32, 0), WINDOW), ((4, 8, 1, 0, 32, 32, 32, 0), GENERAL),      # a run of up to 31 taps is one mask instruction
    ((1, 1, 1, 0, 64, 10, 10, 0), GENERAL), ((1, 1, 1, 0, 64, 12, 12, 0), ROWS),         # four channels per thread
    ((7, 7, 2, 3, 8, 64, 64, 3), GENERAL),                                               # reads the caller's planes
]


def test_form_of_a_layer(forms):
    assert forms("".join("f " + " ".join(map(str, v)) + "\n" for v, _ in LAYERS)) == [w for _, w in LAYERS]


def test_form_of_two_layers_in_one_launch(forms):
    for a, fa in LAYERS:
        for b, fb in LAYERS:
            want = fa if fa == fb else WINDOW if {fa, fb} == {ROWS, WINDOW} else GENERAL
            assert forms("p " + " ".join(map(str, a + b)) + "\n") == [want], (a, b)


def test_reciprocals_divide_exactly(forms):
    ds = [1, 2, 3, 5, 7, 8, 13, 49, 56, 96, 112, 196, 784, 3136, 12544, 50176, 65535, 65537, 1 << 20, (1 << 30) - 1, 1 << 30, (1 << 31) - 1]
    assert forms("".join(f"d {d}\n" for d in ds)) == [0] * len(ds)
