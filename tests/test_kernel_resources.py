"""Device kernels compiled for gfx950 (no GPU needed): those that fit the registers only at the occupancy
they are compiled for must not use scratch memory, and the copy of list rows to LDS must stay short."""
import re
import subprocess

import pytest

from paper_2510_00193_amd import build
from paper_2510_00193_amd.codegen.emit import write_level


def _compile(tmp_path, level, kernels, *options):
    """stderr and output of the device compilation of explicit kernel instantiations."""
    write_level(level, str(tmp_path))
    unit, out = tmp_path / "unit.hip", tmp_path / "unit.out"
    lines = ['#include "mtp_device.h"', f'#include "mtp_L{level}.inc"', '#include "mtp_level_impl.h"']
    unit.write_text("\n".join(lines + [f"template __global__ void mtp::{k};" for k in kernels]) + "\n")
    cmd = [build.HIPCC, *build.FLAGS, f"-I{tmp_path}", "--offload-device-only", *options, str(unit), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    return res.stderr, out


@pytest.mark.parametrize("level", [12, 14])
def test_pair_gradients_of_one_part_stay_in_registers(level, tmp_path):
    args = "mtp::SysArgs, int, int, const double*, long, double*, double*, double*, double*"
    kernels = [f"k_backward<Lv{level}, 0, double, false, {ncheb}, false, {lanes}>({args})"
               for ncheb in (0, 8) for lanes in (1, 2)]
    log, _ = _compile(tmp_path, level, kernels, "-Rpass-analysis=kernel-resource-usage", "-c")
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", log)]
    assert scratch == [0] * len(kernels)


def test_row_stage_selects_nothing_per_entry(tmp_path):
    """Whether a read might pass the end of the list is one test per wave: the smallest binary32 moment
    kernel, whose code is mostly the stage, holds few selects (5 when written, 102 with a test per read)."""
    _, asm = _compile(tmp_path, 2, ["k_moments<Lv2, 0, float, false, 8, false, 1>(mtp::SysArgs, int, int, float*, long)"],
                      "-S")
    assert asm.read_text().count("v_cndmask_b32") < 32


def test_waves_of_small_launches_take_a_simd_each(tmp_path):
    """The forms for launches of at most one wave per SIMD hold all its registers (more than 256), so that
    no second wave is placed beside one while other SIMDs idle; the other forms leave room for two."""
    moments, gradients = "(mtp::SysArgs, int, int, double*, long)", "(mtp::SysArgs, int, int, const double*, long, " \
        "double*, double*, double*, double*)"
    kernels = [f"{name}<Lv12, 0, double, false, 7, false, 1, {alone}>{args}"
               for name, args in (("k_moments", moments), ("k_backward", gradients)) for alone in ("true", "false")]
    _, asm = _compile(tmp_path, 12, kernels, "-S")
    vgprs = [int(x) for x in re.findall(r"\.amdhsa_next_free_vgpr (\d+)", asm.read_text())]
    assert [v > 256 for v in vgprs] == [True, False] * 2, vgprs
