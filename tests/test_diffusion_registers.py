"""Registers of the diffusion stage kernel in the gfx950 assembly of the
library build: both forms fit the 96 of five waves per SIMD without a spilled
one (CPU only: cross-compiles, needs hipcc)."""
import os
import re
import shutil
import subprocess

import pytest


def kernel_registers(lines, name_re):
    """{kernel name: (vector registers, spilled ones)} from the metadata."""
    out, cur = {}, {}
    for x in lines:
        m = re.match(r"\s+(?:- )?\.(name|vgpr_count|vgpr_spill_count):\s+(\S+)$", x)
        if not m:
            continue
        cur[m.group(1)] = m.group(2)
        if m.group(1) == "vgpr_spill_count":
            if re.search(name_re, cur["name"]):
                out[cur["name"]] = (int(cur["vgpr_count"]), int(cur["vgpr_spill_count"]))
            cur = {}
    return out


def test_five_waves_per_simd(tmp_path):
    from paper_2604_12672_amd import build
    if shutil.which(build.HIPCC) is None and not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not available")
    src, out = "mhd_diffusion.hip", tmp_path / "diffusion.s"
    flags = [f for f in build.flags_of(src) if f not in ("-shared", "-fPIC")]
    subprocess.run([build.HIPCC] + flags + ["--cuda-device-only", "-S",
                    os.path.join(build.CSRC, src), "-o", str(out)], check=True,
                   capture_output=True)
    regs = kernel_registers(out.read_text().split("\n"), r"^_ZN3mhd17diff_stage_kernelI")
    assert len(regs) == 2, regs
    for name, (count, spilled) in regs.items():
        assert count <= 96 and spilled == 0, (name, count, spilled)
