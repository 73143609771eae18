"""The wave programs of level 18, which the default build leaves out: cut and emitted by the same rules
as those of levels 16 and 20, against the one-lane programs on the host."""
import shutil

import pytest

from test_codegen_waves import test_wave_programs_match_the_one_lane_programs as check_waves


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_wave_programs_of_level_18(tmp_path):
    check_waves(tmp_path, 18)
