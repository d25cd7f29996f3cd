"""The switches of the fused depthwise + pointwise kernel and of the grouped patch kernel: forms that exist are taken, other values leave the choice to the
planner.  Asked on the host."""
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
    DwPwPlan p{0, 0, 0};
    const bool one = dwpw_plan(37632, 32, 16, DT_F16, 128, &p);
    GConvArgs a{};
    a.B = 1; a.H = a.W = a.Ho = a.Wo = 56; a.Cin = a.Cout = 128; a.KH = a.KW = 3; a.stride = a.pad = 1; a.groups = 32;
    std::printf("%d %d %d %d %d", (int)one, p.tn, p.wk, p.wm, gconv3_blocks(a, 8, 128));
    return 0;
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("switches")
    src, obj, exe = (str(tmp / n) for n in ("p.cpp", "p.o", "p"))
    pkg = os.path.join(ROOT, "paper_2506_12598_amd")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-c", "-I", os.path.join(pkg, "csrc"),
                    "-I", os.path.join(ROOT, "include"), src, "-o", obj], check=True, capture_output=True)
    subprocess.run(["hipcc", obj, "-o", exe, os.path.join(pkg, "libeclip.so"), "-Wl,-rpath," + pkg], check=True, capture_output=True)

    def run(**env):
        keep = {k: v for k, v in os.environ.items() if k not in ("ECLIP_DWPW", "ECLIP_GCONV3")}
        return [int(x) for x in subprocess.run([exe], env={**keep, **env}, capture_output=True, text=True, check=True).stdout.split()]
    return run


@pytest.mark.parametrize("value,plan", [("1,1", (1, 1, 4)), ("2,2", (2, 2, 2)), ("4,4", (4, 4, 1)), ("1,8", (1, 8, 1)), ("0,0", None),
                                        ("2,0", "own"), ("3,4", "own"), ("2,16", "own"), ("-1,4", "own"), ("x", "own"), ("", "own")])
def test_depthwise_and_pointwise(ask, value, plan):
    own, got = ask()[:4], ask(ECLIP_DWPW=value)[:4]
    assert own[0] == 1
    if plan is None:
        assert got[0] == 0
    else:
        assert got == (own if plan == "own" else [1, *plan])


@pytest.mark.parametrize("value,blocks", [("0", 0), ("1", 1), ("2", 2), ("4", 4), ("3", None), ("-1", None), ("8", None), ("x", None), ("", None)])
def test_blocks_of_the_grouped_form(ask, value, blocks):
    own = ask()[4]
    assert own in (1, 2, 4)
    assert ask(ECLIP_GCONV3=value)[4] == (own if blocks is None else blocks)
