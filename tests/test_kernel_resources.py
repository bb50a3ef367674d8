"""What the compiler made of the kernels, read from the built library's own metadata."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2604_18396_amd import build

LLVM = "/opt/rocm/llvm/bin"


def kernels(tmp_path):
    """{kernel symbol: {field: value}} of the library's gfx950 code object."""
    for tool in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf"):
        if not shutil.which(os.path.join(LLVM, tool)):
            pytest.skip(f"{tool} is not installed")
    if not os.path.exists(build.LIB):
        build.build()
    bundle, code = str(tmp_path / "bundle"), str(tmp_path / "code")
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={bundle}", build.LIB, os.devnull], check=True)
    subprocess.run([f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={bundle}", f"--output={code}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout
    out = {}
    for part in notes.split("  - .agpr_count")[1:]:
        fields = dict(re.findall(r"^ {4}\.(\w+): +(\S+)$", part, re.M))
        out[fields["name"]] = fields
    return out


def test_step_kernels_keep_everything_in_registers(tmp_path):
    """A value of the one-launch step kernel that is spilled to scratch memory is read back behind the weight
    prefetch its wavefront has in flight (loads return in order): twelve such words per block made a
    backbone token of the 8B shape at 4096 positions 3.6 % longer."""
    steps = {n: f for n, f in kernels(tmp_path).items() if "k_step_persistent" in n}
    assert len(steps) == 12
    for name, f in steps.items():
        assert int(f["private_segment_fixed_size"]) == 0 and int(f["vgpr_spill_count"]) == 0, (name, f)


def test_block_end_of_a_batched_step_takes_no_more_registers_than_it_did(tmp_path):
    """The sums of partial results are shared with the prefill's row kernels: a branch that only those need made
    this one 18 registers larger and slower, in every block of every batched step."""
    (f,) = [f for n, f in kernels(tmp_path).items() if "k_bd_block_end" in n]
    assert int(f["vgpr_count"]) <= 124 and int(f["private_segment_fixed_size"]) == 0, f
