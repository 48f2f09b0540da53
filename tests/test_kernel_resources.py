"""What the compiler reports for kernels whose working set has to stay in registers: the units
are compiled with the library's own flags (device code only) and no lane may have scratch memory."""
import os
import re
import subprocess

import pytest

from paper_1601_06274_amd import build


def _scratch(source, tmp_path):
    """{mangled kernel name: scratch bytes per lane} of a unit."""
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc is not installed")
    flags = [f for f in build.FLAGS if f != "--offload-compress"]
    r = subprocess.run([build.HIPCC, *flags, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                        os.path.join(build.CSRC, source), "-o", str(tmp_path / "unit.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return {k: int(v) for k, v in re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+)", r.stderr, re.S)}


@pytest.mark.parametrize("source,n", [("cost_volume.hip", 20), ("flow.hip", 16)])
def test_strip_differences_in_registers(source, n, tmp_path):
    strips = {k: v for k, v in _scratch(source, tmp_path).items() if "sad_strip_kernel" in k}
    assert len(strips) == n  # 2 cost types x vector widths x window radii
    assert not any(strips.values()), strips
