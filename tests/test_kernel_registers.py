"""Register spills of the built hop kernels, from the library's own kernel
metadata: the throughput forms run at a fixed budget of wavefronts per SIMD, and
what does not fit goes through scratch memory."""
import os
import re
import subprocess

import pytest

from paper_1611_00298_amd import _lib

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


@pytest.fixture(scope="module")
def spills(tmp_path_factory):
    """VGPR spill count of every k_hop<...>, by its template arguments (P, DAG, HOP, MF, DENSE, BLK, IO, LAT)."""
    tools = [os.path.join(LLVM, t) for t in ("llvm-objdump", "llvm-readelf")]
    if not all(map(os.path.exists, tools)) or not os.path.exists(_lib.LIB_PATH):
        pytest.skip("needs the built library and the LLVM tools of ROCm")
    d = tmp_path_factory.mktemp("kernels")
    os.symlink(os.path.abspath(_lib.LIB_PATH), d / "lib.so")
    subprocess.run([tools[0], "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    out = {}
    for f in sorted(d.glob("lib.so.*gfx*")):
        notes = subprocess.run([tools[1], "--notes", f], check=True, capture_output=True, text=True).stdout
        for kernel in notes.split("  - .agpr_count")[1:]:
            name = re.search(r"\.name:\s+(\S*k_hopI\S+)", kernel)
            if name:
                args = tuple(int(v) for v in re.findall(r"L[ib](\d+)E", name.group(1)))
                out[args] = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel).group(1))
    return out


def test_throughput_hops(spills):
    assert spills
    for (P, dag, hop, mf, dense, blk, io, lat), n in spills.items():
        if not lat and io == 0:
            # FP64 hops: 3 wavefronts per SIMD, 8 registers over (12 cost the block form 4 %); all others fit
            assert n <= (8 if P == 0 and hop and not dense else 0), (P, dag, hop, mf, dense, blk)
