"""Registers of the compiled kernels, from the code object that the build left: the wide blocks of 32
rows must fit 168 registers, three blocks per compute unit, without spilling any of them (a spill
inside their K loop cost 12 % of a decoding stack in groups of 128); so must the blocks of up to 8 rows, whose
call is a chain of trips to memory that spills lengthen."""
import os
import re
import subprocess

import pytest

from paper_2604_18655_amd import build

BIN = "/opt/rocm/llvm/bin/"


def kernels(tmp_path):
    bundle, elf = os.path.join(build.OBJ, "layer_kernels.co"), str(tmp_path / "layer_kernels.elf")
    if not os.path.exists(bundle) or not os.path.exists(BIN + "llvm-readelf"):
        pytest.skip("no code object from a build here")
    subprocess.run([BIN + "clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                    "--input=" + bundle, "--output=" + elf], check=True, capture_output=True)
    notes = subprocess.run([BIN + "llvm-readelf", "--notes", elf], capture_output=True, text=True, check=True).stdout
    out = {}
    for block in re.split(r"\n\s*- \.agpr_count:", notes)[1:]:
        field = lambda key: re.search(r"\.%s:\s+(\S+)" % key, block).group(1)  # noqa: E731
        out[field("name")] = (int(field("vgpr_count")), int(field("vgpr_spill_count")))
    return out


def test_wide_blocks_of_32_rows_fit_their_registers(tmp_path):
    wide = {name: v for name, v in kernels(tmp_path).items() if re.search(r"wide_kernelILi\dELi2E", name)}
    assert wide
    for name, (registers, spilled) in wide.items():
        assert registers <= 168 and spilled == 0, (name, registers, spilled)


def test_blocks_of_up_to_8_rows_fit_their_registers(tmp_path):
    rows8 = [v for name, v in kernels(tmp_path).items() if "layer_kernelILi1ELi8E" in name]
    assert rows8
    for registers, spilled in rows8:
        assert registers <= 168 and spilled == 0, (registers, spilled)
