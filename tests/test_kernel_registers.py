"""Vector registers of the built library's own kernels, where a few more cost a wave per SIMD and no result shows it."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2210_08804_amd import binding

LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    """The library's code objects."""
    d = tmp_path_factory.mktemp("objects")
    lib = shutil.copy(binding.LIB_PATH, d)
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", lib], check=True, capture_output=True)
    return [os.path.join(d, f) for f in sorted(os.listdir(d)) if "gfx950" in f]


@pytest.fixture(scope="module")
def metadata(objects):
    """By kernel name, what the code objects say of it."""
    found = {}
    for f in objects:
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", f], check=True, capture_output=True, text=True).stdout
        for kernel in notes.split(".agpr_count:")[1:]:
            found[re.search(r"\.name:\s*(\S+)", kernel)[1]] = kernel
    return found


@pytest.fixture(scope="module")
def vgprs(metadata):
    return {name: int(re.search(r"\.vgpr_count:\s*(\d+)", kernel)[1]) for name, kernel in metadata.items()}


@pytest.mark.parametrize("lru", [0, 1])
@pytest.mark.parametrize("kpw", [8, 16])
@pytest.mark.parametrize("W", [1, 2, 4, 8])
def test_inserts_of_long_rows_keep_four_waves(vgprs, W, kpw, lru):
    """512 registers per SIMD lane, 128 for each of four waves."""
    name = f"insert_kernelILi{W}ELi{kpw}ELb1ELb{lru}E"
    mine = [v for k, v in vgprs.items() if name in k]
    assert len(mine) == 1 and mine[0] <= 128


@pytest.mark.parametrize("lng", [0, 1])
@pytest.mark.parametrize("kpw", [16, 64])
@pytest.mark.parametrize("W", [1, 2, 4, 8, 16, 32, 64])
def test_updates_keep_four_waves(vgprs, W, kpw, lng):
    name = f"update_kernelILi{W}ELi{kpw}ELb{lng}E"
    mine = [v for k, v in vgprs.items() if name in k]
    assert len(mine) == 1 and mine[0] <= 128


@pytest.mark.parametrize("lng", [0, 1])
@pytest.mark.parametrize("kpw", [16, 64])
@pytest.mark.parametrize("W", [1, 2, 4, 8, 16, 32, 64])
def test_updates_keep_their_registers_out_of_memory(metadata, W, kpw, lng):
    """Held to four waves they may not need more than 128: what does not fit goes to scratch memory, in the middle of the copy of rows."""
    mine = [v for k, v in metadata.items() if f"update_kernelILi{W}ELi{kpw}ELb{lng}E" in k]
    assert len(mine) == 1
    assert re.search(r"\.vgpr_spill_count:\s*(\d+)", mine[0])[1] == "0"
    assert re.search(r"\.private_segment_fixed_size:\s*(\d+)", mine[0])[1] == "0"


@pytest.mark.parametrize("lng", [0, 1])
@pytest.mark.parametrize("kpw", [16, 64])
@pytest.mark.parametrize("W", [2, 8, 64])
def test_updates_do_not_wait_for_keys_in_front_of_their_barrier(metadata, objects, W, kpw, lng):
    """A wait for the keys there is for wave 0 also one for its count of the work-group, and the others wait for wave 0.  (What the
    kernels do in front of the barrier is the same for all sets; three widths are looked at.)"""
    name, = [k for k in metadata if f"update_kernelILi{W}ELi{kpw}ELb{lng}E" in k and not k.endswith(".kd")]
    for f in objects:
        text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", f"--disassemble-symbols={name}", f], check=True, capture_output=True, text=True).stdout
        if "s_barrier" in text:
            assert "vmcnt" not in text[:text.index("s_barrier")]
            return
    raise AssertionError(f"no object has {name}")
