"""When an expansion, the depthwise layer and the pointwise layer behind it share a launch: the rule on sizes and compute units, both sides of each of its lines,
and the switch that overrides it.  Asked on the host."""
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
    int v[8];
    while (std::scanf("%d %d %d %d %d %d %d %d", v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6, v + 7) == 8) {
        ExpDwPlan p{0, 0, 0};
        const bool one = expdw_plan(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], &p);
        std::printf("%d %d %d %d\n", (int)one, p.kmax, p.tn, p.nw);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("expdw")
    src, obj, exe = (str(tmp / n) for n in ("p.cpp", "p.o", "p"))
    pkg = os.path.join(ROOT, "paper_2506_12598_amd")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-c", "-I", os.path.join(pkg, "csrc"),
                    "-I", os.path.join(ROOT, "include"), src, "-o", obj], check=True, capture_output=True)
    subprocess.run(["hipcc", obj, "-o", exe, os.path.join(pkg, "libeclip.so"), "-Wl,-rpath," + pkg], check=True, capture_output=True)

    def run(b, side, cin, c, n, stride, cus, switch=None):
        """Side of the output image; (one launch, (K steps held, tiles of 16 output channels, wavefronts))."""
        env = {k: v for k, v in os.environ.items() if k != "ECLIP_EXPDW"}
        if switch is not None:
            env["ECLIP_EXPDW"] = switch
        got = subprocess.run([exe], input=f"{b} {side} {side} {cin} {c} {n} {stride} {cus}\n", env=env, capture_output=True, text=True, check=True).stdout.split()
        return bool(int(got[0])), tuple(int(x) for x in got[1:])
    return run


# batch, output side, channels in, hidden, out, stride, CUs: workgroups per CU in the comments
TAKEN = [
    (3, 56, 24, 144, 24, 1, 128), (8, 56, 24, 144, 24, 1, 32),              # 4.6, 49
    (3, 112, 16, 64, 16, 1, 384), (8, 56, 16, 96, 24, 2, 256),              # 6.1, 6.1: stride 2 was refused from 4 on
    (3, 28, 32, 64, 128, 1, 64), (1, 56, 32, 64, 128, 2, 128),              # two columns: 4.6, 3.06
    (3, 14, 32, 256, 256, 1, 64), (8, 7, 32, 192, 320, 1, 64),              # four: 3.0; five: 2.5
    (3, 14, 64, 384, 64, 1, 192), (8, 14, 64, 384, 64, 1, 32), (8, 14, 64, 384, 64, 2, 64),       # 0.25, 4, 2
    (8, 14, 64, 384, 96, 1, 256), (3, 14, 96, 576, 96, 1, 96), (8, 7, 96, 192, 192, 1, 256),      # 0.5, 0.5, 0.25 in two columns
    (3, 28, 32, 384, 64, 1, 64),                                            # three slices: 2.3
]
LEFT = [
    (8, 56, 32, 256, 256, 1, 64), (1, 112, 32, 192, 512, 1, 64),            # four and eight columns, 98 and 98: each repeats the expansion
    (1, 14, 32, 64, 576, 1, 256), (8, 112, 32, 64, 128, 2, 64),             # nine columns; two, 196
    (8, 112, 16, 64, 24, 1, 64), (8, 56, 16, 96, 24, 2, 128),               # 98 with half of the wavefronts idle; 12.3 at stride 2
    (8, 112, 24, 144, 24, 1, 64),                                           # 98: beyond what was timed
    (1, 14, 32, 192, 64, 2, 256), (8, 28, 64, 256, 64, 1, 64), (8, 28, 64, 256, 64, 2, 128),      # 0.06, 6.1, 3.06
    (1, 14, 64, 384, 96, 1, 256), (8, 14, 64, 384, 96, 1, 96), (3, 14, 96, 576, 96, 1, 128),      # 0.06, 1.3, 0.375
    (8, 14, 96, 576, 320, 1, 256), (8, 7, 96, 576, 352, 1, 256), (8, 14, 32, 416, 32, 1, 32),     # three slices in two columns; three columns; four slices
    (1, 14, 104, 128, 32, 1, 256), (1, 14, 32, 96, 32, 3, 256),             # no kernel: input channels, stride
]


@pytest.mark.parametrize("sizes", TAKEN)
def test_taken(ask, sizes):
    assert ask(*sizes)[0]


@pytest.mark.parametrize("sizes", LEFT)
def test_left_apart(ask, sizes):
    assert not ask(*sizes)[0]


@pytest.mark.parametrize("cin,n,form", [(32, 32, (1, 2, 4)), (32, 33, (1, 4, 4)), (33, 64, (3, 4, 8)), (96, 65, (3, 10, 8))])
def test_form_by_channels(ask, cin, n, form):
    assert ask(1, 28, cin, 96, n, 1, 64)[1] == form


@pytest.mark.parametrize("sizes,own", [(TAKEN[0], True), (LEFT[0], False)])
def test_the_switch(ask, sizes, own):
    assert ask(*sizes, switch="1")[0] and not ask(*sizes, switch="0")[0]
    for no_choice in ("", "x", "2", "-1"):
        assert ask(*sizes, switch=no_choice) == ask(*sizes) and ask(*sizes)[0] == own


def test_the_switch_cannot_take_what_no_kernel_serves(ask):
    assert not ask(1, 14, 104, 128, 32, 1, 256, switch="1")[0] and not ask(1, 14, 32, 96, 32, 3, 256, switch="1")[0]
