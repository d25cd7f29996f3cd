"""Which layers the 3 x 3 patch kernel takes, in which shapes, and where the planner leaves a layer to the dealt tiles: asked on the host."""
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
    int B, H, W, Cin, N, stride, ldx, cu, even;
    while (std::scanf("%d %d %d %d %d %d %d %d %d", &B, &H, &W, &Cin, &N, &stride, &ldx, &cu, &even) == 9) {
        GemmTraits t;
        t.conv3 = conv3_takes(3, 3, stride, 1, H, W, Cin, N, ldx);
        t.B = B; t.Ho = (H - 1) / stride + 1; t.Wo = (W - 1) / stride + 1; t.Cin = Cin; t.stride = stride;
        t.even_cu = even;
        int shapes = 0, bad = 0;
        for (int v = 0; t.conv3 && v < CONV3_VARIANTS; ++v)
            for (int nw = 1; nw <= 32; ++nw) {
                if (!conv3_launchable(v, nw, t, N)) continue;
                ++shapes;
                int th, tw, bn;
                conv3_tile(v, &th, &tw, &bn);
                const long tiles = conv3_tiles(v, B, t.Ho, t.Wo, N);
                bad += conv3_lds_bytes(v, nw, stride, Cin) > CONV3_MAX_LDS || N % bn || tiles * th * tw * bn < (long)B * t.Ho * t.Wo * N || nw * 64 > 1024;
            }
        const GemmPlan p = conv_gemm_plan((long)B * t.Ho * t.Wo, N, 9l * Cin, cu, 0, t);
        std::printf("%d %d %d %d\n", (int)t.conv3, shapes > 0, bad, p.kind);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("conv3")
    src, obj, exe = (str(tmp / n) for n in ("p.cpp", "p.o", "p"))
    pkg = os.path.join(ROOT, "paper_2506_12598_amd")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-c", "-I", os.path.join(pkg, "csrc"),
                    "-I", os.path.join(ROOT, "include"), src, "-o", obj], check=True, capture_output=True)
    subprocess.run(["hipcc", obj, "-o", exe, os.path.join(pkg, "libeclip.so"), "-Wl,-rpath," + pkg], check=True, capture_output=True)
    return lambda *v: [int(x) for x in subprocess.run([exe], input=" ".join(map(str, v)), capture_output=True, text=True, check=True).stdout.split()]


@pytest.mark.parametrize("case,taken,shapes,kind", [
    ((1, 28, 28, 128, 128, 1, 128, 128, 128), 1, 1, 2),
    ((1, 7, 7, 512, 512, 1, 512, 256, 256), 1, 1, 2),
    ((8, 56, 56, 64, 64, 1, 64, 64, 64), 1, 1, None),
    ((1, 28, 28, 32, 32, 1, 32, 128, 128), 1, 0, None),          # one slice: no number of wavefronts
    ((1, 28, 28, 72, 64, 1, 72, 128, 128), 0, 0, None),          # channels that are no whole slices
    ((1, 28, 28, 64, 40, 1, 64, 128, 128), 0, 0, None),          # output channels that are no whole blocks
    ((1, 28, 28, 64, 64, 3, 64, 128, 128), 0, 0, None),
    ((1, 28, 28, 64, 64, 1, 32768, 128, 128), 0, 0, None),       # pixel pitch beyond 16 bits
    ((1, 4096, 8, 64, 64, 1, 64, 128, 128), 0, 0, None),
    ((1, 5, 5, 4096, 64, 1, 4096, 128, 128), 1, 0, None),        # more slices than four per wavefront
    ((3, 28, 28, 128, 128, 1, 128, 192, 128), 1, 1, 0),          # an uneven share with many tiles
    ((1, 28, 28, 128, 128, 1, 128, 192, 128), 1, 1, 2),
])
def test_what_is_taken(ask, case, taken, shapes, kind):
    got = ask(*case)
    assert got[:3] == [taken, shapes, 0]
    assert (got[3] != 2 if not shapes else True) and (kind is None or got[3] == kind)
