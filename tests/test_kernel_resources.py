"""What the compiler gave kernels whose speed depends on it, from the metadata of the library as it is built: the dense pass of the batched scan
over up to 64 coordinates keeps everything in registers (its slab loop waited for its scores' stores wherever operands went through
scratch memory), and workgroups of the exact redo are few enough in registers that a compute unit holds four of them."""
import os
import re
import subprocess

import pytest

from test_matrix_operand_waits import LIB, device_code

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel: (registers a lane, scratch bytes a lane)}"""
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf not available")
    if not os.path.exists(LIB):
        from paper_2605_17415_amd import build
        build.build_library(verbose=False)
    found = {}
    for i, code in enumerate(device_code(LIB)):
        unit = tmp_path_factory.mktemp("unit") / f"{i}.o"
        unit.write_bytes(code)
        notes = subprocess.run([READELF, "--notes", str(unit)], capture_output=True, text=True).stdout
        for entry in notes.split("  - .agpr_count:")[1:]:
            name, = re.findall(r"\n    \.name: +(\S+)", entry)
            scratch, = re.findall(r"\n    \.private_segment_fixed_size: +(\d+)", entry)
            registers, = re.findall(r"\n    \.vgpr_count: +(\d+)", entry)
            found[name] = int(registers), int(scratch)
    return found


def test_dense_pass_of_few_coordinates_uses_no_scratch(kernels):
    forms = {k: v for k, v in kernels.items() if re.search(r"k_batch_denseILi64ELi\dELb\d", k)}
    assert len(forms) == 10
    assert not {k: v for k, v in forms.items() if v[1]}


def test_four_workgroups_of_the_redo_fit_a_compute_unit(kernels):
    """512 threads each: 8 wavefronts a SIMD, which 64 registers allow (5 and 8 bits with a table in LDS take more)."""
    forms = {k: v for k, v in kernels.items() if re.search(r"k_list_scanILi[234]ELb\dELb1ELb0E", k)}
    assert len(forms) == 6
    assert not {k: v for k, v in forms.items() if v[0] > 64 or v[1]}
