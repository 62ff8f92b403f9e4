"""The persistent line kernel with the version-3 equilibria at region 128: its
chunks are short, so registers that the compiler spills show in its time (300
uneven lines, 200 steps, 12 per block: 3.6 ms at 44 spilled, 3.1 at none)."""

import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "native", "line_instance.hip")


def test_no_register_is_spilled(tmp_path):
    r = subprocess.run(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "--offload-device-only", "-c", SRC, "-o",
                        str(tmp_path / "k.o"), "-Rpass-analysis=kernel-resource-usage"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    name = re.findall(r"Function Name: (\S+)", r.stderr)
    spills = [int(v) for v in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]
    assert len(name) == len(spills) and all(s == 0 for n, s in zip(name, spills) if "persistent" in n), (name, spills)
    assert any("persistent" in n for n in name)
