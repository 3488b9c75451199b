"""Hazards of the built device code that no output shows reliably, looked for in its disassembly
(the library of this repository, built from csrc): direct-to-LDS loads and their wait states."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2510_02345_amd as cm

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel symbol: its instructions in order}"""
    cm.lib()
    d = tmp_path_factory.mktemp("device_code")
    lib = shutil.copy(cm.binding.lib_path(), d)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=d, check=True, capture_output=True)
    out = {}
    for f in sorted(os.listdir(d)):
        if "gfx950" not in f:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", os.path.join(d, f)], check=True, capture_output=True,
                              text=True).stdout
        ins = None
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(.+)>:$", line)
            if m:
                ins = out.setdefault(m.group(1), [])
            elif ins is not None and line.startswith("\t"):
                ins.append(line.split("//")[0].strip())
    assert any("gemm_kernel" in n for n in out)
    return out


def _to_lds(i):
    return i.startswith("global_load_lds") or (i.startswith("buffer_load") and i.endswith(" lds"))


def test_a_wait_state_between_m0_and_the_load_that_uses_it(kernels):
    n = 0
    for name, ins in kernels.items():
        for a, b in zip(ins, ins[1:]):
            if _to_lds(b):
                n += 1
                assert not re.match(r"s_\w+ m0,", a), (name, a, b)
    assert n > 100
