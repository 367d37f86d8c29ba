"""The prefill kernel names its accumulators (a0 ..) in inline assembly, where the compiler inserts no idle slots and knows
of no owner.  What it relies on is checked here in the assembly that the build's own flags produce."""
import os
import re
import subprocess

import pytest

from paper_2403_08058_amd import build


def _registers(token):
    m = re.match(r"([va])\[(\d+):(\d+)\]$", token)
    if m:
        return {(m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}
    m = re.match(r"([va])(\d+)$", token)
    return {(m.group(1), int(m.group(2)))} if m else set()


def _operands(line):
    return [o.strip() for o in re.split(r",\s*(?![^\[]*\])", line.split(None, 1)[1])]


def _is_product(line):
    """A matrix instruction of the source's assembly: it adds into accumulation registers (the compiler's own do not)."""
    return line.startswith("v_mfma") and _operands(line)[0].startswith("a[")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "prefill.s")
    cmd = [build.hipcc(), *build.COMMON, *build.SOURCES["prefill.hip"], "--offload-device-only", "-S",
           os.path.join(build.CSRC, "prefill.hip"), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True)
    with open(out) as f:
        text = f.read()
    found = {}
    for m in re.finditer(r"^(_Z\S*prefill_kernel\S*):[^\n]*\n(.*?)\.Lfunc_end", text, re.S | re.M):
        lines = [ln.split(";")[0].strip() for ln in m.group(2).split("\n")]
        found[m.group(1)] = [ln for ln in lines if ln and not (ln.startswith(".") and not ln.startswith(".LBB"))]
    assert len(found) == 4                       # wide or small tiles, clustered or dense
    return found


def test_products_are_two_slots_behind_their_operands(kernels):
    """A vector instruction's result needs two idle slots before a matrix instruction reads it."""
    for name, lines in kernels.items():
        seen = 0
        for i, line in enumerate(lines):
            if not _is_product(line):
                continue
            seen += 1
            ops = _operands(line)
            reads = set().union(*(_registers(o) for o in ops[1:4]))
            slots, j = 0, i - 1
            while j >= 0 and slots < 2:
                before = lines[j]
                j -= 1
                if before.startswith(".LBB"):
                    continue
                if before.startswith("s_nop"):
                    slots += int(before.split()[1], 0) + 1
                    continue
                if before.startswith("v_") and not before.startswith(("v_mfma", "v_cmp")):
                    dst = _operands(before)
                    written = _registers(dst[0]) | (_registers(dst[1]) if before.startswith(("v_permlane", "v_swap")) else set())
                    assert not (written & reads), f"{name}: '{before}' too close to '{line}'"
                slots += 1
        assert seen >= 64, name


def test_accumulators_have_one_owner(kernels):
    """The named accumulation registers are written by zeroing, by a rescaling's read-multiply-write and by the products, and
    read by those and by the output: nothing of the compiler's goes there, and no read comes without the idle slots after
    the products.  No kernel uses scratch memory."""
    for name, lines in kernels.items():
        named = set()
        for line in lines:
            if _is_product(line):
                named |= _registers(_operands(line)[0])
        assert named == {("a", i) for i in range(len(named))} and len(named) in (64, 128, 256), name
        for i, line in enumerate(lines):
            assert not line.startswith("scratch_"), f"{name}: {line}"
            if line.startswith("v_accvgpr_mov"):
                assert not (named & (_registers(_operands(line)[0]) | _registers(_operands(line)[1]))), f"{name}: {line}"
            if line.startswith("v_accvgpr_write"):
                ops = _operands(line)
                if not named & _registers(ops[0]):
                    continue
                if ops[1] != "0":                # the write of a rescaling: read, multiply, write of one register
                    assert lines[i - 1].startswith("v_mul_f32") and lines[i - 2].startswith("v_accvgpr_read"), f"{name}: {line}"
                    assert _operands(lines[i - 2])[1] == ops[0], f"{name}: {line}"
            if line.startswith("v_accvgpr_read") and named & _registers(_operands(line)[1]):
                slots, j = 0, i - 1
                while j >= 0 and slots < 19:     # a product's sixteen passes and the write behind them
                    before = lines[j]
                    j -= 1
                    if before.startswith(".LBB"):
                        continue
                    assert not (before.startswith("v_mfma") and _registers(_operands(before)[0]) & _registers(_operands(line)[1])), \
                        f"{name}: '{line}' too close to '{before}'"
                    slots += int(before.split()[1], 0) + 1 if before.startswith("s_nop") else 1
