"""The patch kernels that take a max-pool along are compiled apart: what their objects hold, and their counted waits."""
import os
import re
import shutil
import subprocess

import pytest

from test_counted_waits import OBJ, OBJDUMP, ROOT, fetches_behind_the_copies

POOLING = os.path.join(ROOT, "paper_2506_12598_amd", "_build", "k_conv3.hip.p.o")
pytestmark = pytest.mark.skipif(not (os.path.exists(OBJ) and os.path.exists(POOLING) and os.path.exists(OBJDUMP)), reason="needs the object files of the build")


def _kernels(path, tmp_path):
    obj = str(tmp_path / "k.o")
    shutil.copy(path, obj)
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
    return kernels


def test_the_pooling_forms_stand_apart(tmp_path):
    # a launch without a pool runs no instruction of one: the exchange between the lanes of a window is in the pooling forms, all of them, and nowhere else
    (tmp_path / "p").mkdir()
    plain, pooling = _kernels(OBJ, tmp_path), _kernels(POOLING, tmp_path / "p")
    swaps = {n: any(re.match(r"v_permlane(16|32)_swap", line) for line in code) for kernels in (plain, pooling) for n, code in kernels.items() if "conv" in n}
    assert not any(swaps[n] for n in plain if "conv" in n) and all(swaps[n] for n in pooling if "conv" in n)
    got = {n: fetches_behind_the_copies(code) for n, code in pooling.items() if "conv" in n}
    assert len(got) == 2 * 2 * (6 * 6 - 1)
    for n, v in got.items():
        assert v and v[1] and v[0] >= v[1], (n, v)
