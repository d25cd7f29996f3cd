"""When an expansion, a depthwise and a pointwise layer sum in one launch as they do apart: asked on the host."""
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
    while (std::scanf("%d %d %d %d %d %d %d", v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6) == 7) {       // input, hidden, output channels; kind, splits, lean; wk
        const GemmPlan e{v[3], 0, v[4], 1, 4, 0};
        std::printf("%d\n", (int)expdw_sums_as_apart(v[0], v[1], v[2], e, v[5] != 0, DwPwPlan{2, v[6], 1}));
    }
    ExpDwPlan p;
    std::printf("%d %d\n", (int)expdw_plan(3, 28, 28, 32, 192, 32, 1, 64, &p, true), (int)expdw_plan(3, 28, 28, 32, 192, 32, 1, 64, &p, false));
    return 0;
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("sums")
    src, obj, exe = (str(tmp / n) for n in ("p.cpp", "p.o", "p"))
    pkg = os.path.join(ROOT, "paper_2506_12598_amd")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-c", "-I", os.path.join(pkg, "csrc"),
                    "-I", os.path.join(ROOT, "include"), src, "-o", obj], check=True, capture_output=True)
    subprocess.run(["hipcc", obj, "-o", exe, os.path.join(pkg, "libeclip.so"), "-Wl,-rpath," + pkg], check=True, capture_output=True)
    return lambda text, **env: subprocess.run([exe], input=text, capture_output=True, text=True, check=True, env={**os.environ, **env}).stdout.split()


@pytest.mark.parametrize("cin,c,n,kind,splits,lean,wk,same", [
    (32, 144, 24, 0, 1, 1, 4, 1), (32, 144, 24, 1, 1, 1, 4, 1), (32, 144, 24, 1, 1, 0, 4, 1),       # one step of the expansion has no order
    (32, 144, 24, 0, 2, 1, 4, 0), (32, 144, 24, 2, 1, 1, 4, 0),                                     # slices of K, another kernel
    (32, 192, 24, 0, 1, 1, 8, 0), (32, 128, 24, 0, 1, 1, 8, 1), (32, 64, 24, 0, 1, 1, 2, 1), (32, 64, 24, 0, 1, 1, 1, 0), (32, 32, 24, 0, 1, 1, 1, 1),
    (40, 384, 64, 1, 1, 1, 8, 1), (96, 384, 96, 1, 1, 1, 8, 1), (64, 384, 64, 1, 1, 1, 4, 0), (64, 128, 64, 1, 1, 1, 4, 1), (64, 136, 64, 1, 1, 1, 4, 0),
    (64, 384, 64, 0, 1, 1, 8, 0), (64, 384, 64, 1, 1, 0, 8, 0),                                     # a running sum, the general kernel
])
def test_same_sums(ask, cin, c, n, kind, splits, lean, wk, same):
    assert ask(f"{cin} {c} {n} {kind} {splits} {lean} {wk}\n")[0] == str(same)


def test_other_sums_are_left_apart_but_for_the_switch(ask):
    assert ask("") == ["1", "0"]
    assert ask("", ECLIP_EXPDW="1") == ["1", "1"] and ask("", ECLIP_EXPDW="0") == ["0", "0"]
