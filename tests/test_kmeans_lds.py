"""LDS of the k-means launches, static and dynamic together, over all accepted sizes: 64 KB unless the kernel has asked for
more, and what it has asked for otherwise."""
import os
import re
import subprocess

import launch_log
from paper_2403_08058_amd import build


def _static_lds(tmp_path):
    out = str(tmp_path / "kmeans.s")
    subprocess.run([build.hipcc(), *build.COMMON, *build.SOURCES["kmeans.hip"], "--offload-device-only", "-S",
                    os.path.join(build.CSRC, "kmeans.hip"), "-o", out], check=True, capture_output=True)
    with open(out) as f:
        text = f.read()
    return {name: int(size) for size, name in re.findall(r"\.group_segment_fixed_size:\s*(\d+)(?:(?!\.group_segment).)*?\.name:\s*(\S+)", text, re.S)}


def test_lds_of_every_accepted_size(tmp_path):
    fixed = _static_lds(tmp_path)
    assert len(fixed) >= 8 and max(fixed.values()) > 0
    got = launch_log.run(tmp_path, """
        worst = {}
        for F in (1, 4, 9, 16, 20, 25, 30, 33, 36, 49, 55, 64):
            for H in range(1, 257):
                for k in range(1, H + 1):
                    if k * F > 7168 or L.chai_assign_clusters(P, 1, H, F, k, P, 50, P, P, P, None, None) != 0:
                        continue
                    for name, grid, block, lds, leave in launches():
                        key = name + " " + str(leave)
                        if lds > worst.get(key, (0,))[0]:
                            worst[key] = (lds, H, F, k)
        result = worst
    """)
    assert len(got) >= 8
    for key, (dynamic, H, F, k) in got.items():
        name, leave = key.split(" ")
        assert dynamic + fixed[name] <= max(64 * 1024, int(leave)) and int(leave) + fixed[name] <= 160 * 1024, (name, H, F, k, dynamic, fixed[name])
