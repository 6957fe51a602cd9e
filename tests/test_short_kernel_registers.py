"""Wide blocks of eight waves (short launches): two of them share a compute unit, which 128 registers without spills and
half its LDS allow; a spill there lengthened calls that read many adapters by a quarter."""
import os
import re
import subprocess

import pytest

from paper_2604_18655_amd import build

BIN = "/opt/rocm/llvm/bin/"


def test_two_blocks_of_eight_waves_fit_a_compute_unit(tmp_path):
    bundle, elf = os.path.join(build.OBJ, "wide_short_kernels.co"), str(tmp_path / "kernels.elf")
    if not os.path.exists(bundle) or not os.path.exists(BIN + "llvm-readelf"):
        pytest.skip("no code object from a build here")
    subprocess.run([BIN + "clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                    "--input=" + bundle, "--output=" + elf], check=True, capture_output=True)
    notes = subprocess.run([BIN + "llvm-readelf", "--notes", elf], capture_output=True, text=True, check=True).stdout
    seen = 0
    for block in re.split(r"\n\s*- \.agpr_count:", notes)[1:]:
        field = lambda key: re.search(r"\.%s:\s+(\S+)" % key, block).group(1)  # noqa: E731
        assert "wide_short_kernel" in field("name")
        assert int(field("vgpr_count")) <= 128 and int(field("vgpr_spill_count")) == 0, block
        assert int(field("group_segment_fixed_size")) <= 80 * 1024
        seen += 1
    assert seen == 6
