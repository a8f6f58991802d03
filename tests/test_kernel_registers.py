"""What the rules of a launch take for granted about the built kernels' registers, read from the library's own notes."""
import os
import re
import shutil
import subprocess

import pytest

READELF, OBJDUMP = "/opt/rocm/llvm/bin/llvm-readelf", "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> {field: number} of every kernel of the library"""
    if not (os.path.exists(READELF) and os.path.exists(OBJDUMP)):
        pytest.skip("no binary tools")
    from paper_2206_04746_amd import binding
    tmp = tmp_path_factory.mktemp("notes")
    lib = shutil.copy(binding.LIB_PATH, tmp / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=tmp, check=True, capture_output=True)
    found = {}
    for obj in sorted(tmp.glob("lib.so.*gfx950")):
        notes = subprocess.run([READELF, "--notes", str(obj)], check=True, capture_output=True, text=True).stdout
        for entry in re.split(r"\n  - \.a", notes)[1:]:
            name = re.search(r"\.symbol:\s+(\S+)\.kd", entry)
            if name:
                found[name[1].strip("'")] = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\n", ".a" + entry)}
    return found


def of(kernels, pattern):
    some = {n: f for n, f in kernels.items() if re.search(pattern, n)}
    assert some, pattern
    return some


def test_contraction_blocks_of_eight_waves_fit_a_compute_unit_twice(kernels):
    some = of(kernels, r"encode_contract_kernelILi\d+ELi\dELb\dELi8E")
    assert len(some) == 24                    # 1, 2 or 4 steps; 6 or 8 planes; floats or bytes; chains or none
    for name, f in some.items():              # 16 waves on four SIMDs of 512 registers a lane each
        assert f["vgpr_count"] <= 128 and f["agpr_count"] == 0, (name, f)


def test_cosines_are_finished_by_eight_waves_a_simd(kernels):
    for name, f in of(kernels, "cosine_finish_kernel|online_weights_kernel").items():
        assert f["vgpr_count"] <= 64 and f["private_segment_fixed_size"] == 0, (name, f)


def test_passes_of_online_training_by_samples_do_not_spill(kernels):
    for name, f in of(kernels, r"online_spread_kernelILi\dELb0E").items():    # (in batches 18 and 49 registers do)
        assert f["private_segment_fixed_size"] == 0 and f["vgpr_count"] <= 128, (name, f)


def test_whole_block_walk_of_online_training_does_not_spill(kernels):
    for name, f in of(kernels, "online_wide_kernel").items():
        assert f["private_segment_fixed_size"] == 0 and f["vgpr_count"] <= 256, (name, f)
