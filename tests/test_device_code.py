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


def _waits_for_lds(i):
    return i.startswith("s_waitcnt") and "lgkmcnt(0)" in i


# The loops that refill a stage of LDS behind a bare barrier: the stage was read an iteration ago, and the
# barrier is passed only with those reads completed, wherever the compiler puts the products.
@pytest.mark.parametrize("kernel", ["route_rows_lds_kernel", "t1_rows_kernel", "gemm_thin_kernel", "cmp_stream_kernel"])
def test_lds_reads_are_complete_before_a_stage_is_refilled(kernels, kernel):
    n = 0
    for name, ins in kernels.items():
        if kernel not in name:
            continue
        for at, i in enumerate(ins):
            if i != "s_barrier":
                continue
            # the instructions that run into the barrier from above
            near = ins[max(at - 6, 0):at]
            near = near[max((j + 1 for j, w in enumerate(near) if w.startswith("s_branch")), default=0):]
            if any(re.fullmatch(r"s_waitcnt vmcnt\(\d+\)", w) for w in near):   # the wait for the stage's loads
                n += 1
                assert any(_waits_for_lds(w) for w in near), (name, near)
    assert n


def test_t1_rows_shares_its_expert_table_behind_a_barrier(kernels):
    # wavefront 0 writes the table that all four read: a barrier of its own before the first stage's loads
    found = [ins for name, ins in kernels.items() if "t1_rows_kernel" in name]
    assert found
    for ins in found:
        written = max(at for at, i in enumerate(ins[:ins.index(next(filter(_to_lds, ins)))]) if i.startswith("ds_write_b32"))
        shuffles = [at for at, i in enumerate(ins) if at > written and i.startswith("ds_bpermute")]
        # the six shuffles that join the tile's needs come right behind the table
        assert "s_barrier" in ins[written:shuffles[5]]
