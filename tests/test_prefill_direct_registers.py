"""The kernel that converts the values itself, held to what test_prefill_registers asks of the others, and its waits: the
requests it counts on are in the order it counts them in."""
import os
import re
import subprocess

import pytest

import test_prefill_registers as R
from paper_2403_08058_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "prefill.s")
    cmd = [build.hipcc(), *build.COMMON, *build.SOURCES["prefill.hip"], "--offload-device-only", "-S",
           os.path.join(build.CSRC, "prefill.hip"), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True)
    with open(out) as f:
        text = f.read()
    found = {}
    for m in re.finditer(r"^_Z\S*prefill_direct_kernelILb(\d)E\S*:[^\n]*\n(.*?)\.Lfunc_end", text, re.S | re.M):
        lines = [ln.split(";")[0].strip() for ln in m.group(2).split("\n")]
        # by the name of the kernel with the same accumulators
        found[f"prefill_kernelILi1ELi4ELb{m.group(1)}E"] = [ln for ln in lines if ln and not (ln.startswith(".") and not ln.startswith(".LBB"))]
    assert len(found) == 2
    return found


def test_products_are_two_slots_behind_their_operands(kernels):
    R.test_products_are_two_slots_behind_their_operands(kernels)


def test_accumulators_have_one_owner(kernels):
    R.test_accumulators_have_one_owner(kernels)


def test_key_requests_are_older_than_the_waits_allow(kernels):
    """Before the barrier behind a tile, at most N requests may be left, and the last N requests are loads of values to
    registers: keys on their way to LDS are older.  Both in blocks that a wave multiplies and in those it only prepares."""
    for name, lines in kernels.items():
        waits = [i for i, ln in enumerate(lines) if re.match(r"s_waitcnt vmcnt\((4|8|16)\) lgkmcnt\(0\)$", ln) and lines[i + 1] == "s_barrier"]
        assert len(waits) >= (3 if "Lb1" in name else 6), name
        for i in waits:
            n = int(re.search(r"vmcnt\((\d+)\)", lines[i]).group(1))
            seen, j = 0, i - 1
            while seen < n:
                assert j >= 0, f"{name}: only {seen} requests before '{lines[i]}'"
                ln = lines[j]
                if ln.startswith(("buffer_load", "global_load")):
                    assert not ln.endswith("lds"), f"{name}: '{ln}' within the last {n} requests before '{lines[i]}'"
                    seen += 1
                j -= 1
