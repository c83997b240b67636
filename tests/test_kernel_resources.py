"""What the kernels' sources and builds have to keep."""
import os
import re

import paper_2603_12646_amd as fa


def test_exchanges_write_no_register_in_an_asm_block_alone():
    """An exchange between lanes takes both registers in with a value: the compiler then waits for a matrix product that still
    writes them.  Only the dot product that starts a sum (its operands are the probabilities, behind all products) has an
    output of its own."""
    src = os.path.join(os.path.dirname(fa.LIB_PATH), "csrc", "fa_kernels.hip")
    with open(src) as f:
        outputs = [line.strip() for line in f if re.search(r'"=&?v"', line)]
    assert all("v_dot2_f32_f16" in line for line in outputs), outputs
