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
    """A matrix instruction of the source's assembly.  The compiler's own ones multiply bf16."""
    return line.startswith("v_mfma_f32_32x32x16_f16")


def _accumulators(line):
    """All accumulation registers that a line names, wherever it names them."""
    return {("a", i) for m in re.finditer(r"\ba(?:(\d+)|\[(\d+):(\d+)\])", line)
            for i in range(int(m.group(1) or m.group(2)), int(m.group(1) or m.group(3)) + 1)}


# named registers, and zeroed ones (a clustered kernel zeroes those of one and of two members), by streams, waves and density
EXPECTED = {(1, 4, 0): (128, 64 + 128), (2, 4, 0): (256, 128 + 256), (1, 4, 1): (64, 64), (1, 8, 1): (64, 64)}


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
    assert len(found) == 5                       # wide or small tiles, clustered or dense, few keys
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


def _slots_behind_products(lines, i, register, name):
    """No product that writes `register` less than a product's sixteen passes and the write behind them before line i."""
    slots, j = 0, i - 1
    while j >= 0 and slots < 19:
        before = lines[j]
        j -= 1
        if before.startswith(".LBB"):
            continue
        assert not (before.startswith("v_mfma") and register in _registers(_operands(before)[0])), \
            f"{name}: '{lines[i]}' too close to '{before}'"
        slots += int(before.split()[1], 0) + 1 if before.startswith("s_nop") else 1


def test_accumulators_have_one_owner(kernels):
    """The named accumulation registers are written by zeroing, by a rescaling's read-multiply-write and by the products, and
    read by those and by the output.  No other instruction names one, be it a load, a copy or an operand, and no read or
    zero comes without the idle slots after the products.  No kernel uses scratch memory."""
    for name, lines in kernels.items():
        streams, waves, dense = (int(x) for x in re.search(r"prefill_kernelILi(\d)ELi(\d)ELb(\d)E", name).groups())
        n_named, n_zeroed = EXPECTED[streams, waves, dense]
        named = {("a", i) for i in range(n_named)}
        zeroed, scaled, output, products = [], [], 0, set()
        for i, line in enumerate(lines):
            assert not line.startswith("scratch_"), f"{name}: {line}"
            hit = _accumulators(line) & named
            if not hit:
                continue
            ops = _operands(line)
            if _is_product(line):                # a whole tile, added into; operands in ordinary registers
                first = min(i for _, i in hit)
                tile = f"a[{first}:{first + 15}]"
                assert first % 16 == 0 and ops[0] == ops[3] == tile and not _accumulators(ops[1] + ops[2]), f"{name}: {line}"
                products.add(first)
            elif line.startswith("v_accvgpr_write") and ops[1] == "0":
                zeroed.append(ops[0])
                _slots_behind_products(lines, i, ("a", int(ops[0][1:])), name)
            elif line.startswith("v_accvgpr_write"):     # the write of a rescaling: read, multiply, write of one register
                assert lines[i - 1].startswith("v_mul_f32") and lines[i - 2].startswith("v_accvgpr_read"), f"{name}: {line}"
                value = _operands(lines[i - 2])[0]
                assert _operands(lines[i - 2])[1] == ops[0] and ops[1] == value, f"{name}: {line}"
                assert _operands(lines[i - 1])[0] == value and value in _operands(lines[i - 1])[1:], f"{name}: {line}"
                scaled.append(int(ops[0][1:]))
            else:
                assert line.startswith("v_accvgpr_read") and hit == _accumulators(ops[1]), f"{name}: {line}"
                _slots_behind_products(lines, i, ("a", int(ops[1][1:])), name)
                output += 1
        assert products == set(range(0, n_named, 16)), name
        assert len(zeroed) == n_zeroed and set(zeroed) == {f"a{i}" for i in range(n_named)}, name
        assert output - len(scaled) == n_zeroed, name
        for first in products:                   # rescaled together, behind either block of a tile or wherever that code went
            assert len({scaled.count(i) for i in range(first, first + 16)}) == 1 and scaled.count(first) >= 2, name


@pytest.mark.parametrize("planted", [
    "ds_read_b128 a[0:3], v5", "buffer_load_dwordx4 a[60:63], v1, s[0:3], 0 offen", "v_accvgpr_mov_b32 a3, a70",
    "v_accvgpr_mov_b32 a70, a3", "v_accvgpr_write_b32 a5, v9", "v_accvgpr_write_b32 a5, 0", "v_accvgpr_read_b32 v9, a5",
    "v_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]", "v_mfma_f32_32x32x16_bf16 v[0:15], a[60:63], v[4:7], v[0:15]",
    "v_mfma_f32_32x32x16_f16 a[0:15], a[4:7], v[4:7], a[0:15]", "v_mfma_f32_32x32x16_f16 a[8:23], v[0:3], v[4:7], a[8:23]",
    "scratch_store_dword off, v0, s32"])
def test_another_owner_is_noticed(kernels, planted):
    """A line of the compiler's that takes a named register, put into the text of each kernel."""
    for name, lines in kernels.items():
        with pytest.raises(AssertionError):
            test_accumulators_have_one_owner({name: lines[:40] + [planted] + lines[40:]})
