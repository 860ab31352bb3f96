"""Static check of the generated code of the fp32 kernels (no GPU needed): a vector instruction reads a matrix instruction's result 19 issue
slots after it at the earliest (32x32x2 fp32; fewer for the bf16 one), and the compiler, which fills them with no-ops where it has to,
does not look into inline assembly.  So no assembly-written instruction may read such a result sooner, nor overwrite what a matrix instruction may
still be adding to."""
import os
import re
import shutil

import pytest

from test_asm_hazards import _assembly_of, kernels_of, regs_of

SLOTS = 20


def early_reads(lines):
    """(line number, instruction, slots since the matrix instruction) in the order of the text."""
    written, added_to, at, in_asm, bad = {}, {}, 0, False, []
    for no, raw in lines:
        if "#ASMSTART" in raw or "#ASMEND" in raw:
            in_asm = "#ASMSTART" in raw
            continue
        ins = raw.split(";")[0].strip()
        if not ins or ins.startswith(".") or ins.endswith(":"):
            continue
        op, _, rest = ins.partition(" ")
        operands = [regs_of(o) for o in rest.split(",")]
        nops = re.match(r"s_nop (\d+)", ins)
        at += int(nops.group(1)) + 1 if nops else 1
        if in_asm and op.startswith("v_") and "mfma" not in op:
            late = [at - written[r] - 1 for o in operands[1:] for r in o if r in written]
            late += [at - added_to[r] - 1 for r in operands[0] if r in added_to]
            if late and min(late) < SLOTS:
                bad.append((no, ins, min(late)))
        for r in operands[0]:
            written.pop(r, None)
            if "mfma" in op:
                written[r] = at
        for r in operands[3] if "mfma" in op else ():
            added_to[r] = at
    return bad


@pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")
@pytest.mark.parametrize("source,kernel,count", [("attn_f32.hip", "attn_f32_kernel", 4), ("attn_f32.hip", "attn_f32_split_kernel", 6), ("colmass_f32.hip", "score_f32_kernel", 12)])
def test_no_assembly_reads_a_matrix_result_early(source, kernel, count):
    found = 0
    for name, lines in kernels_of(_assembly_of(source), kernel):
        found += 1
        bad = early_reads(lines)
        assert not bad, (name, bad[:3])
    assert found == count
