"""Hazards of the built device code that no output shows reliably, looked for in its disassembly
(the library of this repository, built from csrc): direct-to-LDS loads and their wait states; and registers that a kernel
spills, from its metadata."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2510_02345_amd as cm

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    cm.lib()
    d = tmp_path_factory.mktemp("device_code")
    lib = shutil.copy(cm.binding.lib_path(), d)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=d, check=True, capture_output=True)
    return [os.path.join(d, f) for f in sorted(os.listdir(d)) if "gfx950" in f]


@pytest.fixture(scope="module")
def kernels(code_objects):
    """{kernel symbol: its instructions in order}"""
    out = {}
    for f in code_objects:
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], check=True, capture_output=True, text=True).stdout
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


# The same of the weight stream of 64 tokens a pass, whose weights go to registers: a chunk's tokens are written by all four
# wavefronts ahead of the barrier, and the other buffer has been read there.  And behind the last two barriers, those of the last
# chunks, no more weights are loaded (non-temporal), which nothing would use.
def test_wide_weight_stream(kernels):
    found = [ins for name, ins in kernels.items() if re.search("skinny_base_kernelILi[0-9]ELi64E", name)]
    assert found
    for ins in found:
        mfma = [at for at, i in enumerate(ins) if i.startswith("v_mfma")]
        loads = [at for at, i in enumerate(ins) if i.startswith("global_load") and i.endswith(" nt")]
        chunks = [at for at, i in enumerate(ins) if i == "s_barrier" and loads[0] < at < mfma[-1]]
        assert len(chunks) == 4 and loads[-1] < chunks[-2]
        for at in chunks:
            assert any(_waits_for_lds(w) for w in ins[at - 6:at]), ins[at - 6:at]


def test_t1_rows_shares_its_expert_table_behind_a_barrier(kernels):
    # wavefront 0 writes the table that all four read: a barrier of its own before the first stage's loads
    found = [ins for name, ins in kernels.items() if "t1_rows_kernel" in name]
    assert found
    for ins in found:
        written = max(at for at, i in enumerate(ins[:ins.index(next(filter(_to_lds, ins)))]) if i.startswith("ds_write_b32"))
        shuffles = [at for at, i in enumerate(ins) if at > written and i.startswith("ds_bpermute")]
        # the six shuffles that join the tile's needs come right behind the table
        assert "s_barrier" in ins[written:shuffles[5]]


def test_up_projection_with_its_panels_in_memory_spills_nothing(code_objects):
    # K*r > 128: operands fetched ahead would wait in registers, of which the 256 x 256 tile has none to spare
    found = {}
    for f in code_objects:
        notes = subprocess.run([READELF, "--notes", f], check=True, capture_output=True, text=True).stdout
        for kernel in notes.split("- .agpr_count")[1:]:
            name = re.search(r"\.name:\s+(\S+)", kernel).group(1)
            m = re.search(r"gemm_kernel.*EpiFusedUpILi(\d+)ELi([12])ELb0E", name)
            if m:
                found[m.groups()] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel).group(1))
    assert set(found) == {(r, k) for r in ("4", "8", "16", "32") for k in "12"}
    assert not any(found.values()), found
