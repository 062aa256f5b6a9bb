"""Registers of kernels whose speed hangs on how many waves a SIMD holds, read from the metadata of the built library (no GPU)."""
import shutil
import struct
import subprocess

import pytest

from paper_2406_18139_amd import lookm

READELF = shutil.which("llvm-readelf") or shutil.which("llvm-readelf", path="/opt/rocm/llvm/bin")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def registers(tmp_path_factory):
    """{mangled kernel name: (vector registers, bytes of scratch, spilled scalar registers)} over the gfx950 code objects of the library."""
    if not READELF:
        pytest.skip("no llvm-readelf")
    lookm.lib()
    blob, found, at = lookm.LIB_PATH.read_bytes(), {}, 0
    while (at := blob.find(MAGIC, at)) >= 0:
        n, p = struct.unpack_from("<Q", blob, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(n):
            offset, size, length = struct.unpack_from("<3Q", blob, p)
            target = blob[p + 24:p + 24 + length].decode()
            p += 24 + length
            if "gfx950" in target and size:
                path = tmp_path_factory.mktemp("co") / "code.elf"
                path.write_bytes(blob[at + offset:at + offset + size])
                name = scratch = spilled = None
                for line in subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout.splitlines():
                    key, _, value = line.strip().partition(":")
                    value = value.strip()
                    if key == ".name" and value.startswith("_Z"):
                        name = value
                    elif key == ".private_segment_fixed_size":
                        scratch = int(value)
                    elif key == ".sgpr_spill_count":
                        spilled = int(value)
                    elif key == ".vgpr_count":
                        found[name] = (int(value), scratch, spilled)
        at += len(MAGIC)
    assert found
    return found


# 512 registers a lane of a SIMD, allotted in eights: 168 for three waves, 128 for four
@pytest.mark.parametrize("kernel,limit", [("k_score_anyILi1EtLi3ELi4EE", 168), ("k_score_anyILi2EtLi3ELi4EE", 168),     # bf16, 72 to 96 wide
                                          ("k_nearest_anyItLi3ELi4EE", 168),
                                          ("k_score_anyILi1EtLi2ELi4EE", 128), ("k_score_anyILi2EtLi2ELi4EE", 128),     # bf16, 40 to 64 wide
                                          ("k_nearest_anyItLi2ELi4EE", 128),
                                          ("k_score_anyILi1EfLi4ELi2EE", 128), ("k_score_anyILi2EfLi4ELi2EE", 168),     # fp32, 56 and 64 wide
                                          ("k_score_anyILi1EfLi8ELi2EE", 256), ("k_score_anyILi2EfLi8ELi2EE", 256),     # 104 to 128: two waves
                                          ("k_nearest_foldILi1EE", 128), ("k_nearest_foldILi2EE", 128), ("k_nearest_foldILi4EE", 128)])
def test_waves_per_simd(registers, kernel, limit):
    counts = [v for k, v in registers.items() if kernel in k]
    assert len(counts) == 1
    assert counts[0][0] <= limit and counts[0][1] == 0, counts


@pytest.mark.parametrize("kernel", ["k_score_anyILi1EfLi12ELi1EE", "k_score_anyILi2EfLi12ELi1EE",       # fp32 wider than 128: one wave
                                    "k_score_anyILi1EfLi16ELi1EE", "k_score_anyILi2EfLi16ELi1EE"])
def test_scalar_registers_of_a_single_wave(registers, kernel):
    """Where one wave has a SIMD to itself nothing hides the reloads of what the loop over the blocks keeps in scalar registers; a
    few that are spilled lie outside it."""
    counts = [v for k, v in registers.items() if kernel in k]
    assert len(counts) == 1
    assert counts[0][2] <= 16, counts
