"""The patch kernels wait for their copies into LDS by the number of fetches issued behind them.  The number is written by hand: here it is compared with what
the compiler issued, in every kernel of the built object."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OBJ = os.path.join(ROOT, "paper_2506_12598_amd", "_build", "k_conv3.hip.o")
OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
pytestmark = pytest.mark.skipif(not (os.path.exists(OBJ) and os.path.exists(OBJDUMP)), reason="needs the object file of the build")


def fetches_behind_the_copies(code):
    """(fetches issued behind the last copy into LDS, the number the first wait behind it allows); None: no copy."""
    copies = [i for i, line in enumerate(code) if re.match(r"buffer_load_\w+ .*\blds\b", line)]
    if not copies:
        return None
    fetches = 0
    for line in code[copies[-1] + 1:]:
        wait = re.match(r"s_waitcnt .*vmcnt\((\d+)\)", line)
        if wait:
            return fetches, int(wait.group(1))
        fetches += bool(re.match(r"(buffer|global|flat)_load_", line))
    return fetches, None


def test_what_is_counted():
    code = ["buffer_load_dwordx4 v1, s[0:3], 0 offen lds", "buffer_load_dwordx4 v[2:5], v1, s[0:3], 0 offen", "s_waitcnt lgkmcnt(0)", "buffer_load_dwordx2 v[6:7], v1, s[0:3], 0 offen"]
    assert fetches_behind_the_copies(code + ["s_waitcnt vmcnt(2)"]) == (2, 2)
    assert fetches_behind_the_copies(code[:3] + ["s_waitcnt vmcnt(2) lgkmcnt(0)"]) == (1, 2)
    assert fetches_behind_the_copies(code) == (2, None) and fetches_behind_the_copies(code[1:]) is None


def test_the_patch_kernels(tmp_path):
    obj = str(tmp_path / "k.o")
    shutil.copy(OBJ, obj)
    subprocess.run([OBJDUMP, "--offloading", obj], check=True, capture_output=True, cwd=tmp_path)
    device = [f for f in os.listdir(tmp_path) if f.endswith("gfx950")]
    assert len(device) == 1
    text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(tmp_path / device[0])], check=True, capture_output=True, text=True).stdout
    kernels, name = {}, None
    for line in text.splitlines():
        m = re.match(r"[0-9a-f]+ <(\w+)>:", line)
        if m:
            name = m.group(1)
            kernels[name] = []
        elif name and line.startswith("\t"):
            kernels[name].append(line.strip())
    got = {n: fetches_behind_the_copies(code) for n, code in kernels.items() if "conv" in n}
    # 2 types x 2 strides x (6 shapes x (4 wavefront counts + 2 of several slices) - 1) and x 2 widths x 3 patches of the grouped form
    assert len(got) == 2 * 2 * (6 * 6 - 1) + 2 * 2 * 2 * 3
    for n, v in got.items():
        assert v and v[1] and v[0] >= v[1], (n, v)
