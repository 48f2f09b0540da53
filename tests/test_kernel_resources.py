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


RULE = """
#include <cstdio>
#include "pipe_rule.h"
using namespace dm;
int main() {
    const Tile tiles[] = {{8, 4}, {16, 4}, {32, 3}, {32, 4}, {64, 3}, {64, 4}};
    for (int K = 5; K <= 256; ++K)
        for (const Tile& t : tiles) {
            if (t.G * t.LPL < K || (t.G > 8 && t.G * t.LPL >= 2 * K)) continue;
            for (int T = 3; T < 40; T = 3 * T)
                for (int form = 0; form < 3; ++form) {  // columns, FP32 rows, FP16 rows
                    const bool scan = T > 3, theta = form > 0, f16 = form == 2;
                    const Tile d = scan ? t : window_tile(K);
                    std::printf("%d %d %d %d %d %d %d %d %d\\n", K, d.LPL, t.LPL, t.G * t.LPL == K, T, form,
                                pipe_vec(K, d.LPL, theta, f16), pipe_per_cu(d, t, scan, T, K, theta, f16),
                                pipe_lds_count(d.LPL, theta));
                }
        }
}
"""


def test_pipelines_are_resident(tmp_path):
    """The workgroups per CU up to which the pipelined sweeps are taken: never more than LDS
    holds, nor, for 3 and more labels a lane by single accesses (whose one-wave kernel is as
    fast from a second round on), more than the registers of the half-step kernels hold."""
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc is not installed")
    src = tmp_path / "rule.cpp"
    src.write_text(RULE)
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, str(src), "-o", str(tmp_path / "rule")], check=True)
    out = subprocess.run([str(tmp_path / "rule")], capture_output=True, text=True, check=True).stdout
    rows = [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    assert len(rows) > 2000
    held = {}
    for lpl in (3, 4):
        for scan in (0, 1):
            flags = [f for f in build.FLAGS if f != "--offload-compress"]
            defs = ["-DDM_PIPE_G=64", f"-DDM_PIPE_L={lpl}", f"-DDM_PIPE_SCAN={scan}"]
            cmd = [build.HIPCC, *flags, *defs, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                   os.path.join(build.CSRC, "dmm_pipe.hip"), "-o", str(tmp_path / f"pipe{lpl}{scan}.o")]
            held[lpl, scan] = subprocess.Popen(cmd, stderr=subprocess.PIPE, text=True)
    for key, proc in held.items():
        report = proc.communicate()[1]
        assert proc.returncode == 0, report
        # half-step kernels that access label by label: <64, labels, type, false, theta, message, 0>
        found = re.findall(r"Function Name: (_ZN2dm11pipe_kernel\S+Lb0ELb([01])ELi[023]ELi0E\S+).*?"
                           r"Occupancy \[waves/SIMD\]: (\d+)", report, re.S)
        assert len(found) == (3 if key[1] else 6), [f[0] for f in found]
        held[key] = min(int(occ) * 4 // 3 for _, _, occ in found)  # workgroups of three waves
    for K, lpl, t_lpl, full, T, form, vec, per_cu, lds in rows:
        assert 0 <= per_cu <= lds, (K, T, form)
        assert full or per_cu >= 1, (K, T, form)
        if lpl >= 3 and not vec:
            assert per_cu <= held[lpl, T > 3], (K, T, form)
