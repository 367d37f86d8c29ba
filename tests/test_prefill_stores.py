"""The prefill kernels' 16-byte stores: a vector instruction that writes a store's data registers has to stay two slots behind it."""
import os
import re
import subprocess

import pytest

import test_prefill_registers as R
from paper_2403_08058_amd import build


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "prefill.s")
    cmd = [build.hipcc(), *build.COMMON, *build.SOURCES["prefill.hip"], "--offload-device-only", "-S",
           os.path.join(build.CSRC, "prefill.hip"), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True)
    with open(out) as f:
        text = [ln.split(";")[0].strip() for ln in f]
    return [ln for ln in text if ln and not ln.startswith(".")]


def clobbered(lines):
    """(store, writer) pairs in which an instruction less than two slots behind a store of more than 8 bytes writes its data."""
    found = []
    for i, store in enumerate(lines):
        if not re.match(r"(buffer|global)_store_dwordx[34]", store):
            continue
        data, slots = R._registers(R._operands(store)[0 if store.startswith("buffer") else 1]), 0
        for behind in lines[i + 1:i + 3]:
            if slots >= 2:
                break
            if behind.startswith("v_") and not behind.startswith("v_cmp") and data & R._registers(R._operands(behind)[0]):
                found.append((store, behind))
            slots += int(behind.split()[1], 0) + 1 if behind.startswith("s_nop") else 1
    return found


def test_data_of_a_store_outlives_it_by_two_slots(lines):
    stores = [ln for ln in lines if ln.startswith("buffer_store_dwordx4")]
    assert len(stores) >= 7 * 16                 # every kernel writes its rows so
    assert all(re.search(r"\], 0 offen", ln) for ln in stores), "no scalar offset"
    assert clobbered(lines) == []


def test_a_store_that_loses_its_data_is_noticed():
    assert clobbered(["buffer_store_dwordx4 v[4:7], v3, s[12:15], s36 offen", "v_mul_f32_e32 v4, v12, v9"])
    assert clobbered(["buffer_store_dwordx4 v[4:7], v3, s[12:15], 0 offen", "s_nop 0", "v_accvgpr_read_b32 v5, a4"])
    assert not clobbered(["buffer_store_dwordx4 v[4:7], v3, s[12:15], 0 offen", "s_nop 1", "v_mul_f32_e32 v4, v12, v9"])
