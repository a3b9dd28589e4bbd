"""Finalize writes by block id into arrays sized for the classes that the
refinement counted, before the host has compared that count with the classes
the numbering found (CPU).  The position rule, from the library's own header,
keeps every such write inside the arrays whatever was found; the kernels that
write by block id all go through it."""

import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2111_12493_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_positions_stay_inside():
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    os.makedirs(os.path.join(ROOT, "_build"), exist_ok=True)
    exe = os.path.join(ROOT, "_build", "block_slots_check_%d" % os.getpid())
    subprocess.run([HIPCC, "-O1", "-std=c++17", "-x", "hip", "--offload-arch=gfx950", "-I",
                    os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "native", "block_slots_check.cpp"), "-o", exe],
                   check=True, capture_output=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.startswith("ok "), out.stdout + out.stderr


def test_both_numbering_kernels_use_the_rule():
    with open(os.path.join(CSRC, "bsim_final.hip")) as f:
        src = f.read()
    for kernel in ("k_fin_name", "k_fin_ids"):
        body = re.search(r"__global__[^;{]*\b%s\(.*?\n}" % kernel, src, re.S).group(0)
        assert "block_slot(" in body, kernel
