"""Register allocation of device kernels that fit the registers only at the occupancy they are compiled
for: compiled for gfx950 (no GPU needed), they must not use scratch memory."""
import re
import subprocess

import pytest

from paper_2510_00193_amd import build
from paper_2510_00193_amd.codegen.emit import write_level


@pytest.mark.parametrize("level", [12, 14])
def test_pair_gradients_of_one_part_stay_in_registers(level, tmp_path):
    write_level(level, str(tmp_path))
    unit = tmp_path / "unit.hip"
    lines = ['#include "mtp_device.h"', f'#include "mtp_L{level}.inc"', '#include "mtp_level_impl.h"']
    for ncheb in (0, 8):
        for lanes in (1, 2):
            lines.append(f"template __global__ void mtp::k_backward<Lv{level}, 0, double, false, {ncheb}, false, {lanes}>("
                         "mtp::SysArgs, int, int, const double*, long, double*, double*, double*, double*);")
    unit.write_text("\n".join(lines) + "\n")
    cmd = [build.HIPCC, *build.FLAGS, f"-I{tmp_path}", "--offload-device-only", "-Rpass-analysis=kernel-resource-usage",
           "-c", str(unit), "-o", str(tmp_path / "unit.o")]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", res.stderr)]
    assert scratch == [0] * 4
