"""Properties of the built library's device code that no run on a GPU would reliably show, read from the
disassembly of the code objects that were compiled here."""
import os
import re
import subprocess

import pytest

from paper_2603_06350_amd import binding as B
from paper_2603_06350_amd import build

LLVM = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.hipcc()))), "llvm", "bin")
if not os.path.isdir(LLVM):
    LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    if not os.path.exists(B.lib_path()):
        build.build()
    folder = tmp_path_factory.mktemp("code")
    copy = folder / "lib.so"
    copy.write_bytes(open(B.lib_path(), "rb").read())
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", str(copy)], cwd=folder, check=True,
                   capture_output=True)
    found = sorted(str(p) for p in folder.iterdir() if p.name.endswith("gfx950") and p.stat().st_size)
    assert len(found) >= 5
    return found


def test_every_barrier_of_the_ffn_kernels_waits_for_the_wave_s_lds_reads(code_objects):
    # after the barrier another wave, or a load that writes LDS directly, overwrites what was read before it
    barriers, bad = 0, []
    for path in code_objects:
        text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", path], check=True,
                              capture_output=True, text=True).stdout
        name, settled = "", False
        for line in text.splitlines():
            head = re.match(r"^[0-9a-f]+ <(\S+)>:", line)
            if head:                              # a function, or a label inside one
                name = head.group(1) if head.group(1).startswith("_Z") else name
                settled = False
                continue
            op = line.split("//")[0].split()
            if not op or "ffn_" not in name:
                continue
            if op[0] == "s_barrier":
                barriers += 1
                if not settled:
                    bad.append(name)
            elif op[0] == "s_waitcnt":
                settled = settled or "lgkmcnt(0)" in line
            elif op[0].startswith("ds_") or "branch" in op[0]:
                settled = False
    assert barriers > 50
    assert not bad, f"{len(bad)} of {barriers} barriers, in {sorted(set(bad))}"


def test_the_ffn_kernels_spill_no_scalar_registers(code_objects):
    # a spilled scalar is a lane of a vector register, read back inside the K loops
    spills = {}
    for path in code_objects:
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", path], check=True, capture_output=True,
                               text=True).stdout
        for name, count in re.findall(r"\.name:\s+(\S+).*?\.sgpr_spill_count:\s+(\d+)", notes, re.S):
            if "ffn_" in name:
                spills[name] = int(count)
    assert len(spills) > 10
    assert not any(spills.values()), {k: v for k, v in spills.items() if v}
