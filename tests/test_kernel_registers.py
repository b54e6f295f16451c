"""The register use of the built forward kernels, from the notes of their code objects.

The ring kernel runs at 4 waves per SIMD, which leaves 128 VGPRs.  A few registers spilled
outside its loop cost nothing; with 11 and more in it every slice goes to memory and back.
"""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2401_13660_amd", "libmbscan.so")
LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
MAX_SPILLS = 6

pytestmark = pytest.mark.skipif(not os.path.exists(os.path.join(LLVM, "llvm-readelf")), reason="needs the ROCm LLVM tools")


@pytest.fixture(scope="module")
def spills(tmp_path_factory):
    """{mangled kernel name: spilled VGPRs}"""
    if not os.path.exists(LIB):
        from __graft_entry__ import build
        build()
    at = tmp_path_factory.mktemp("co")
    fat, code = str(at / "fat"), str(at / "code")
    for cmd in ([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", LIB, str(at / "lib")],
                [f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={fat}", f"--output={code}",
                 "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"]):
        subprocess.run(cmd, check=True, capture_output=True)
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout
    names = re.findall(r"\.symbol:\s+(\S+)\.kd", notes)
    counts = [int(n) for n in re.findall(r"\.vgpr_spill_count:\s+(\d+)", notes)]
    assert len(names) == len(counts)
    return dict(zip(names, counts))


def test_ring_kernel_keeps_its_registers(spills):
    ring = {n: c for n, c in spills.items() if "scan_fwd_ring" in n}
    # fp32 / bf16 in x out, gate, softplus, plain / checkpoints / positions
    assert len(ring) == 48
    assert {n: c for n, c in ring.items() if c > MAX_SPILLS} == {}
