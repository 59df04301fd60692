"""The vector accumulates keep the resident waves that they are held to: the compiler's
report of registers and spills for gfx950 (no GPU needed)."""
import os
import re
import subprocess

from paper_2604_17155_amd import build

WAVES = {0: 7, 1: 7, 2: 6, 3: 6, 4: 5, 8: 4, 16: 4}  # channels: waves per SIMD


def test_accumulate_occupancy(tmp_path):
    cmd = [build._hipcc(), *build.HIPCC_FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage",
           "-c", os.path.join(build.CSRC, "k_accum.hip"), "-o", str(tmp_path / "k.o")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    seen = set()
    for block in r.stderr.split("Function Name: ")[1:]:
        m = re.match(r"_ZN3gsc12k_accumulateILi(\d+)E", block)
        if not m:
            continue
        ch = int(m[1])
        waves = int(re.search(r"Occupancy \[waves/SIMD\]: (\d+)", block)[1])
        spills = int(re.search(r"VGPRs Spill: (\d+)", block)[1])
        assert waves >= WAVES[ch] and spills == 0, (ch, waves, spills)
        seen.add(ch)
    assert seen == set(WAVES)
