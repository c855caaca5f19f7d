"""CPU checks of the built GPU code (the library's own code object, as the
compiler left it): what the sources ask for and no test on a GPU can show."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2109_11083_amd import binding as B

LLVM = "/opt/rocm/llvm/bin"
pytestmark = pytest.mark.skipif(not os.path.exists(f"{LLVM}/llvm-objdump"), reason="no LLVM tools")


@pytest.fixture(scope="module")
def code_object(tmp_path_factory):
    d = tmp_path_factory.mktemp("code")
    so = shutil.copy(B.LIB_PATH, d / "lib.so")
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", so], check=True, capture_output=True, cwd=d)
    found = [f for f in sorted(d.iterdir()) if "gfx950" in f.name]
    for f in found:
        syms = subprocess.run([f"{LLVM}/llvm-readelf", "-sW", f], check=True, capture_output=True, text=True).stdout
        if "k_sort" in syms:
            names = sorted(set(re.findall(r"FUNC\s.*\s(_Z\S+)$", syms, re.M)))
            return f, names
    raise AssertionError("no gfx950 code object with the library's kernels")


def test_blocks_count_themselves_done_after_every_waves_stores(code_object):
    """A block of the sort or rebuild in one launch counts itself done by one
    thread, whose release waits for the stores of its own wave alone: the
    barrier before it must find every wave's stores complete."""
    f, names = code_object
    kernels = [n for n in names if re.search(r"k_sort|k_rebuild", n)]
    assert len(kernels) >= 5  # k_sort and k_rebuild of four tile configurations
    text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", "--no-leading-addr",
                           "--disassemble-symbols=" + ",".join(kernels), f],
                          check=True, capture_output=True, text=True).stdout
    for body in text.split("Disassembly of section")[-1].split(">:")[1:]:
        ins = [ln.split("//")[0].strip() for ln in body.splitlines() if ln.startswith("\t")]
        counts = [k for k, i in enumerate(ins) if i.startswith("buffer_wbl2")]
        assert counts
        for k in counts:
            barrier = max(j for j in range(k) if ins[j].startswith("s_barrier"))
            before = ins[max(barrier - 3, 0):barrier]
            assert any(re.match(r"s_waitcnt .*vmcnt\(0\)", i) for i in before), (before, ins[barrier:k + 1])


def test_search_and_plain_steps_keep_their_registers(code_object):
    """No scratch in the list search, in any launch form, nor in the force kernel of a
    plain step of one simulation."""
    f, _ = code_object
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", f], check=True, capture_output=True, text=True).stdout
    found = dict(re.findall(r"\.name:\s+(\S+).*?\.private_segment_fixed_size: (\d+)", notes, re.S))
    # (k_force<kStepFused = 1 or kDpdForce = 4, ., ., no sample, ...>)
    kernels = [n for n in found if re.search(r"k_neighbors|k_rebuild|k_sort|k_forceILi[14]ELb[01]ELb[01]ELb0E", n)]
    assert len(kernels) >= 12
    assert [n for n in kernels if int(found[n])] == []
