"""The flux-limited step with the version-3 equilibria is the kernel with the
most values live at once (five rows of neighbours, sixteen exponentials); how
many of its registers the compiler spills decides its speed (2048 x 2048: 397
us per step at 126, 444 at 222)."""

import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "native", "limited_instance.hip")


def test_few_registers_are_spilled(tmp_path):
    r = subprocess.run(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "--offload-device-only", "-c", SRC, "-o",
                        str(tmp_path / "k.o"), "-Rpass-analysis=kernel-resource-usage"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    spills = [int(v) for v in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]
    assert len(spills) == 1 and spills[0] <= 126, spills
