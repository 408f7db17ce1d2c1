"""The one-pass kernel of width 576 keeps its accumulators in accumulation registers that it names itself.  What the compiler
must not do for that to hold is looked up in the assembly of the file: touch those registers outside the kernel's own statements,
spill, or write an operand of a product with a vector instruction less than two wait states before it (the products carry no
wait states of their own)."""
import re
import subprocess

import pytest

from paper_2505_11580_amd import build as B

NAME = "fipa_bf16_attn_fwd_576.hip"


@pytest.fixture(scope="module")
def assembly():
    import os
    cmd = [B.HIPCC] + B.FLAGS + B.PER_FILE.get(NAME, []) + ["-S", "--offload-device-only", os.path.join(B.CSRC, NAME), "-o", "-"]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    return res.stdout.split("\n")


def registers(text):
    """The vector registers that an operand names."""
    m = re.match(r"v\[(\d+):(\d+)\]$", text)
    if m:
        return set(range(int(m.group(1)), int(m.group(2)) + 1))
    m = re.match(r"v(\d+)$", text)
    return {int(m.group(1))} if m else set()


def test_no_accumulation_register_outside_the_named_statements(assembly):
    inside = False
    for line in assembly:
        if "ASMSTART" in line:
            inside = True
        elif "ASMEND" in line:
            inside = False
        code = line.split(";")[0].strip()
        if inside or not code or code.startswith("."):
            continue
        assert not re.search(r"\ba\[\d+:\d+\]|\ba\d+\b|accvgpr|scratch_", code), code


def test_no_spills(assembly):
    counts = [int(m.group(1)) for m in (re.search(r"\.vgpr_spill_count:\s*(\d+)", x) for x in assembly) if m]
    assert len(counts) >= 4 and not any(counts), counts


def test_operands_of_the_products_are_two_wait_states_old(assembly):
    products, recent = 0, []  # of the last instructions: (registers written by the vector unit, wait states)
    for line in assembly:
        code = line.split(";")[0].strip()
        if code.endswith(":") and not code.startswith("."):
            recent = []  # (a kernel; a label inside one: whatever came before it in the text is looked at)
        if not code or code.startswith((".", "#")) or code.endswith(":"):
            continue
        op, _, rest = code.partition(" ")
        args = [a.strip() for a in re.split(r",(?![^\[]*\])", rest)]
        if op.startswith("v_mfma"):
            if args[0].startswith("a["):
                products += 1
                used = registers(args[1]) | registers(args[2])
                states = 0
                for written, wait in reversed(recent):
                    if states >= 2:
                        break
                    assert not (written & used), code
                    states += wait
            recent.append((set(), 1))
        elif op == "s_nop":
            recent.append((set(), 1 + int(args[0])))
        else:
            recent.append((registers(args[0]) if op.startswith("v_") and args else set(), 1))
        recent = recent[-4:]
    assert products == 4 * 2 * 32, products  # four kernels, two steps with products
