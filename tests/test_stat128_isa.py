"""The statistics kernel of large shares at head size 128 reads its fragments like the others (test_wave_isa.py)."""
import os
import subprocess

from paper_2301_08984_amd import build as B
from test_wave_isa import pending_read_violations


def test_no_register_is_touched_between_a_read_and_its_wait(tmp_path):
    out = os.path.join(tmp_path, "k.s")
    subprocess.run(["hipcc", *B.FLAGS, *B.EXTRA_FLAGS["fast_stat128.hip"], "--cuda-device-only", "-S", os.path.join(B.CSRC, "fast_stat128.hip"), "-o", out],
                   check=True, capture_output=True)
    lines = open(out).read().splitlines()
    assert any("ds_read_b128" in l for l in lines)
    assert pending_read_violations(lines) == []
    assert not any("v_accvgpr" in l or "scratch_" in l for l in lines)
