"""What the compiler made of the kernels: the metadata of the code object inside the built library."""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2503_23186_amd import cnnk

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels():
    """{demangled name without arguments: (vector registers, spilled registers, bytes of scratch a lane)}"""
    out = {}
    with tempfile.TemporaryDirectory() as d:
        lib = os.path.join(d, "lib.so")
        os.symlink(cnnk.LIB_PATH, lib)
        subprocess.run([LLVM + "/llvm-objdump", "--offloading", lib], cwd=d, check=True, capture_output=True)
        for f in sorted(os.listdir(d)):
            if "gfx950" not in f:
                continue
            notes = subprocess.run([LLVM + "/llvm-readelf", "--notes", os.path.join(d, f)], check=True, capture_output=True, text=True).stdout
            for k in notes.split("- .agpr_count")[1:]:
                value = lambda key: re.search(r"\.%s:\s+(\S+)" % key, k).group(1)
                out[value("name")] = tuple(int(value(x)) for x in ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size"))
    names = subprocess.run(["c++filt"], input="\n".join(out), capture_output=True, text=True, check=True).stdout.splitlines()
    clean = [n.replace("(anonymous namespace)::", "").replace("void ", "").split("(")[0] for n in names]
    return dict(zip(clean, out.values()))


def test_small_tiles_leave_the_registers_to_as_many_workgroups_as_lds_holds(kernels):
    """64 x 64 tiles of one group of wavefronts: 24 or 48 KB of LDS, six or three workgroups to a CU.  A workgroup has one
    wavefront on each SIMD, so 64 registers leave room for eight; and there is no kernel that walks several such tiles."""
    small = {n: v for n, v in kernels.items()
             if re.match(r"gemm_kernel<false, (true|false), \d, 1, 1, 64, 128, 3, 1\b", n) or re.match(r"conv_gemm_kernel<Tile<false, (true|false), 1, 1, 2, \d+, \d+, 3, 1\b", n)}
    assert len(small) == 13
    for name, (registers, spilled, scratch) in small.items():
        assert registers <= 64 and spilled == 0 and scratch == 0, name


def test_classifier_head_keeps_its_registers(kernels):
    """1024 threads to a workgroup: 128 registers are the most, 64 let a CU hold two workgroups.  Nothing spills, also with the
    features of a 2048-wide row in registers."""
    head = {n: v for n, v in kernels.items() if n.startswith("logits_softmax_kernel<")}
    assert len(head) == 6
    for name, (registers, spilled, scratch) in head.items():
        assert spilled == 0 and scratch == 0 and registers <= (128 if ", 4>" in name else 64), (name, registers)
