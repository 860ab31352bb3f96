"""The static check of test_asm_hazards.py on the other kernels that issue loads from inline assembly: the row pass, the
forms of the scoring passes for runs and query groups, and the plain attention kernel."""
import os
import re
import shutil

import pytest

from test_asm_hazards import _assembly_of, check_function, kernels_of

# file, kernel name, instantiations (row pass: two head dimensions; attention: also four workgroup shapes)
CHECKED = [("colmass_bf16.hip", "rowlse_bf16_kernel", 2), ("colmass_bf16.hip", "rowlse_runs_bf16_kernel", 2),
           ("colmass_bf16.hip", "colmass_runs_bf16_kernel", 2), ("colmass_bf16.hip", "colmass_groups_bf16_kernel", 2),
           ("colmass_bf16.hip", "colmass_groups_runs_bf16_kernel", 2), ("attn_bf16_group.hip", "attn_bf16_group_kernel", 8)]


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
@pytest.mark.parametrize("source,kernel,count", CHECKED)
def test_no_instruction_touches_an_assembly_issued_load_in_flight(source, kernel, count):
    found = 0
    for name, lines in kernels_of(_assembly_of(source), kernel):
        found += 1
        bad = check_function(lines)
        assert not bad, "%s: %d hazards, first: line %d `%s` touches %s" % (name, len(bad), bad[0][0], bad[0][1], bad[0][2])
    assert found == count


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
def test_two_wave_blocks_come_four_to_a_compute_unit():
    """Groups of 64 rows at D = 128: 160 KB of LDS for four workgroups, two waves' registers (with three they are slower than
    without the software pipeline)."""
    text = _assembly_of("attn_bf16_group.hip")
    at = text.index("attn_bf16_group_kernelILi128ELi2ELi1E")
    lds = int(re.search(r"; LDSByteSize: (\d+)", text[at:]).group(1))
    registers = int(re.search(r"; TotalNumVgprs: (\d+)", text[at:]).group(1))
    assert 4 * lds <= 160 * 1024 and registers <= 256
