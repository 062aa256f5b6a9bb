"""Registers of kernels whose speed hangs on how many waves a SIMD holds, read from the metadata of the built library (no GPU)."""
import shutil
import struct
import subprocess

import pytest

from paper_2406_18139_amd import lookm

READELF, OBJDUMP = (shutil.which(tool) or shutil.which(tool, path="/opt/rocm/llvm/bin") for tool in ("llvm-readelf", "llvm-objdump"))
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """Files of the library's gfx950 code objects."""
    lookm.lib()
    blob, found, at = lookm.LIB_PATH.read_bytes(), [], 0
    while (at := blob.find(MAGIC, at)) >= 0:
        n, p = struct.unpack_from("<Q", blob, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(n):
            offset, size, length = struct.unpack_from("<3Q", blob, p)
            target = blob[p + 24:p + 24 + length].decode()
            p += 24 + length
            if "gfx950" in target and size:
                path = tmp_path_factory.mktemp("co") / "code.elf"
                path.write_bytes(blob[at + offset:at + offset + size])
                found.append(path)
        at += len(MAGIC)
    assert found
    return found


@pytest.fixture(scope="module")
def registers(code_objects):
    """{mangled kernel name: (vector registers, bytes of scratch, spilled scalar registers)}."""
    if not READELF:
        pytest.skip("no llvm-readelf")
    found = {}
    for path in code_objects:
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
    assert found
    return found


# 512 registers a lane of a SIMD, allotted in eights: 168 for three waves, 128 for four
@pytest.mark.parametrize("kernel,limit", [("k_score_anyILi1EtLi3ELi4EE", 168), ("k_score_anyILi2EtLi3ELi4EE", 168),     # bf16, 72 to 96 wide
                                          ("k_nearest_anyItLi3ELi4EE", 168),
                                          ("k_score_anyILi1EtLi2ELi4EE", 128), ("k_score_anyILi2EtLi2ELi4EE", 128),     # bf16, 40 to 64 wide
                                          ("k_nearest_anyItLi2ELi4EE", 128),
                                          ("k_score_anyILi1EfLi4ELi2EE", 128), ("k_score_anyILi2EfLi4ELi2EE", 168),     # fp32, 56 and 64 wide
                                          ("k_score_anyILi5EfLi4ELi2EE", 128), ("k_score_anyILi6EfLi4ELi2EE", 168),     # .. remainders by subtraction
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


@pytest.mark.parametrize("kernel", ["k_score_anyILi1EfLi%dELi2EE", "k_score_anyILi2EfLi%dELi2EE", "k_nearest_anyIfLi%dELi2EE"])
@pytest.mark.parametrize("steps", [1, 3])
def test_no_remainders_of_dims_that_are_not_there(registers, code_objects, kernel, steps):
    """fp32 widths of an odd number of 16-dim steps: the missing half of the last pair of steps is zeros, and no dot instruction works
    out its remainders.  Eight of them a step and row, two rows of the strip and two of a block (24 products a pair of steps; a
    loop that the compiler peels holds those twice)."""
    if not OBJDUMP:
        pytest.skip("no llvm-objdump")
    name = [k for k in registers if kernel % steps in k]
    assert len(name) == 1
    text = "".join(subprocess.run([OBJDUMP, "-d", f"--disassemble-symbols={name[0]}", str(path)], capture_output=True, text=True,
                                  check=True).stdout for path in code_objects)
    blocks = text.count("v_mfma_f32_16x16x32_bf16") / (24 * ((steps + 1) // 2))
    assert blocks in (1, 2) and text.count("v_dot2") == 2 * 8 * steps * (1 + blocks)
