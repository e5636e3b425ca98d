"""Registers of the multi-RHS hop (gfx950 assembly of csrc/mrhs.hip, built here
from source): in FP64 the links, a half spinor and the next neighbour just fit
the 128 registers a lane has, and a spill would wait for the neighbour as it
arrives."""
import importlib.util
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_fp64_multi_rhs_hop_spills_nothing(tmp_path):
    if not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")):
        pytest.skip("no hipcc")
    spec = importlib.util.spec_from_file_location("_wd_build", os.path.join(ROOT, "paper_0710_2442_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    out = str(tmp_path / "mrhs.s")
    subprocess.run([b._hipcc(), *b.HIP_FLAGS, "--offload-device-only", "-S", os.path.join(b.CSRC, "mrhs.hip"), "-o", out],
                   check=True, capture_output=True)
    text, seen = open(out).read(), 0
    for name, body in re.findall(r"\.amdhsa_kernel (\S*k_dslash_mrhs_splitILi0E\S*)(.*?)\.end_amdhsa_kernel", text, re.S):
        vgpr = int(re.search(r"amdhsa_next_free_vgpr (\d+)", body).group(1))
        scratch = int(re.search(r"amdhsa_private_segment_fixed_size (\d+)", body).group(1))
        assert vgpr <= 128 and scratch == 0, (name, vgpr, scratch)
        seen += 1
    assert seen == 12
