"""Registers of a kernel that stands at the edge of an occupancy step: at 130 VGPRs instead of 128 it ran
at 0.85 of its speed, with three wavefronts per SIMD instead of four."""
import os
import re
import subprocess

from paper_2605_01774_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_plain_bf16_with_a_velocity_field_keeps_four_wavefronts(tmp_path):
    out = tmp_path / "step_registers.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "-DELBM_Q=27", "-I", build.CSRC, "--offload-device-only", "-S",
                    os.path.join(ROOT, "tests", "native", "step_registers.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    text = out.read_text()
    vgprs = [int(v) for v in re.findall(r"\.amdhsa_next_free_vgpr (\d+)", text)]
    scratch = [int(v) for v in re.findall(r"; ScratchSize: (\d+)", text)]
    assert len(vgprs) == 1 and vgprs[0] <= 128 and scratch == [0]
