"""Matrix-core sums in the compiled network kernels (gfx950 assembly of
csrc/ptc.hip, built here from source).

Products on the FP64 and 4x4 FP32 matrix instructions take many wait states,
and nothing may rest on how these are counted over branches: the sums of the
weight gradient accumulate in place and are touched by nothing but products
until an explicit wait in the products' own block; the network layers' sums are
read, or waited for, before their block ends.
"""
import importlib.util
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not (shutil.which("hipcc") or os.path.exists("/opt/rocm/bin/hipcc")):
        pytest.skip("no hipcc")
    spec = importlib.util.spec_from_file_location("_wd_build", os.path.join(ROOT, "paper_0710_2442_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    out = str(tmp_path_factory.mktemp("isa") / "ptc.s")
    subprocess.run([b._hipcc(), *b.HIP_FLAGS, "--offload-device-only", "-S", os.path.join(b.CSRC, "ptc.hip"), "-o", out],
                   check=True, capture_output=True)
    found = {}
    for m in re.finditer(r"^(_ZN2wd\w+):[^\n]*\n(.*?)^\.Lfunc_end", open(out).read(), re.S | re.M):
        found[m.group(1)] = m.group(2).splitlines()
    return found


def _registers(text):
    regs = set()
    for a, b, one in re.findall(r"\bv(?:\[(\d+):(\d+)\]|(\d+)\b)", text):
        regs.update(range(int(a), int(b) + 1) if a else [int(one)])
    return regs


def _check(lines, product, strict):
    """Products of one kernel; strict: in place, and touched by products alone
    until the wait (else a read in the same block ends the wait too)."""
    pending, n, in_asm = set(), 0, False
    for line in lines:
        code = line.split(";")[0].strip()
        if "ASMSTART" in line or "ASMEND" in line:
            in_asm = "ASMSTART" in line
        if in_asm and code.startswith("s_nop") and int(code.split()[1]) >= 7:
            pending = set()
        if not code:
            continue
        if code.endswith(":") or code.startswith(("s_cbranch", "s_branch", "s_endpgm")):
            assert not pending, f"products unfinished at the end of a block: {line}"
            continue
        if code.startswith(product):
            ops = [o.strip() for o in code.split(None, 1)[1].split(", ")]
            if strict:
                assert ops[0] == ops[3].split()[0], f"not in place: {code}"
            n += 1
            pending |= _registers(ops[0])
        elif pending & _registers(code):
            assert not strict, f"a sum is touched before the wait: {code}"
            pending -= _registers(code)
    return n


def test_weight_gradient_sums_accumulate_in_place_up_to_the_wait(kernels):
    ks = [k for k in kernels if "k_ptc_wgrad" in k]
    assert len(ks) == 4
    for k in ks:
        assert _check(kernels[k], "v_mfma_f64_16x16x4", True) == 5 * 48, k


def test_network_layer_sums_are_settled_before_their_block_ends(kernels):
    ks = [k for k in kernels if "k_ptc_layer" in k]
    assert len(ks) >= 10
    for k in ks:
        assert _check(kernels[k], "v_mfma_f32_4x4x1", False) > 0, k
