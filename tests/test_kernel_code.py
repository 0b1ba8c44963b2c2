"""What the compiler made of the kernels (built library, no GPU)."""
import re

from kernel_code import instructions

# A buffer access whose base address is in vector registers is wrapped in a loop over the different values that the lanes hold.
LOOP_OVER_VALUES = r"s_xor_b64 exec, exec, [^\n]*\n[^\n]*s_cbranch_execnz"


def test_base_addresses_are_in_scalar_registers():
    loops = instructions(lambda body: len(re.findall(LOOP_OVER_VALUES, body)))
    assert len(loops) > 500 and any("ArithS, 13" in k for k in loops)
    assert not {k: n for k, n in loops.items() if n}
