"""What the compiler made of the kernels (built library, no GPU)."""
import re

from kernel_code import instructions, registers

# A buffer access whose base address is in vector registers is wrapped in a loop over the different values that the lanes hold.
LOOP_OVER_VALUES = r"s_xor_b64 exec, exec, [^\n]*\n[^\n]*s_cbranch_execnz"


def test_base_addresses_are_in_scalar_registers():
    loops = instructions(lambda body: len(re.findall(LOOP_OVER_VALUES, body)))
    assert len(loops) > 500 and any("ArithS, 13" in k for k in loops)
    assert not {k: n for k, n in loops.items() if n}


def test_single_key_decryption_has_room():
    """It adds up no shares: its registers are not those of the kernels that do."""
    spilled = {k: v[1] for k, v in registers().items() if k.startswith("k_decrypt<")}
    assert len(spilled) == 30                       # five ring degrees on six back-ends
    # N = 2^14 (16 coefficients per thread): sums and accumulators of 24 spilled registers at most
    assert not {k: n for k, n in spilled.items() if n > (24 if ", 14, 4," in k else 0)}


def test_receivers_sums_have_room():
    """Key switching adds up two polynomials of every member next to the receiver's key."""
    spilled = {k: v[1] for k, v in registers().items() if k.startswith("k_convert_combine_decode<")}
    assert len(spilled) == 34
    # N = 2^14: two sums of 32 registers, accumulators of 48; as many again for the quotients of ArithS and ArithB, and for loads in pairs
    # (launches of up to 64 workgroups, not on doubles and 32-bit words)
    pairs = [k for k in spilled if ", 14, 4," in k and k.endswith("false>")]
    assert len(pairs) == 4
    assert not {k: n for k, n in spilled.items() if n > ((110 if k in pairs else 80 if re.search("Arith[SB]", k) else 40) if ", 14, 4," in k else 0)}


def test_finish_has_room():
    """Sum, shares and combine of a round in one kernel: what it spills is written and read again for every limb.  (Before the sums were
    read in pairs: 0, 0, 13, 13, 9, 20; 32-bit words keep one, the lane's offset, out of the loop.)"""
    limit = {"Arith32": 1, "ArithF": 0, "ArithS": 13, "ArithB": 13, "ArithP": 9, "ArithQ": 16}
    spilled = {k: v[1] for k, v in registers().items() if k.startswith("k_finish<")}
    assert len(spilled) == 27
    # ArithP at N = 1024 takes two passes of other sizes and 14
    assert not {k: n for k, n in spilled.items() if n > limit[re.search(r"Arith\w", k).group(0) if "Arith32" not in k else "Arith32"] + 5 * ("ArithP, 10" in k)}


def test_encryption_by_components_has_room():
    """A workgroup that makes one component of a ciphertext keeps nothing of the other (24 to 41 registers were spilled for it)."""
    spilled = {k: v[1] for k, v in registers().items() if k.startswith("k_encrypt_components<")}
    assert len(spilled) >= 50
    assert not {k: n for k, n in spilled.items() if n > (0 if ", 14, 3," in k else 16)}


def test_combines_of_few_members_have_room():
    """N = 2^14 on doubles and 32-bit words: as many coefficients per thread as fit, so the loops over members decide."""
    spilled = {k: v[1] for k, v in registers().items() if re.match(r"k_combine(_decode)?<Engine<Arith(F|32), 14, 4.*, true>", k)}
    assert len(spilled) == 4 and not any(spilled.values()), spilled


def test_wide_stores_have_no_scalar_offset():
    """Such a store may find its registers overwritten by the next instruction, and the compiler does not keep that one away."""
    stores = instructions(lambda body: re.findall(r"buffer_store_dwordx[34] [^\n/]*", body))
    assert sum(len(v) for v in stores.values()) > 500
    scalar = {k: [s for s in v if not re.search(r"s\[\d+:\d+\], 0( |$)", s)] for k, v in stores.items()}
    assert not {k: v[:2] for k, v in scalar.items() if v}
