"""What the device code asks of the compiler, read from the intermediate code that it is given
(before any optimisation): orders and ranges that a run cannot show, since the code that is
generated today may keep them by chance."""
import os
import re
import subprocess

import pytest

from paper_2602_20787_amd import build

CSRC = os.path.join(build.PKG, "csrc")


def device_functions(source, tmp_path):
    """Unoptimised device functions of a HIP source: mangled name -> body."""
    out = tmp_path / "device.ll"
    flags = [f for f in build.FLAGS if f not in ("-O3", "-mllvm") and not f.startswith("-amdgpu")]
    res = subprocess.run([build.HIPCC, *flags, "-O1", "-Xclang", "-disable-llvm-passes", "--offload-device-only", "-S",
                          "-emit-llvm", "-o", str(out), source], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    return dict(re.findall(r"^define [^\n]*?@([\w$.]+)\([^\n]*\{\n(.*?)^\}", out.read_text(), re.S | re.M))


def test_steps_that_hand_lds_slots_on_are_ordered(tmp_path):
    # a lane reads the reaction sums that another lane wrote a step before: without a fence per
    # step the compiler may take the next step's loads before this one's stores
    fns = device_functions(os.path.join(CSRC, "forces_pairwise.hip"), tmp_path)
    fence = [n for n, b in fns.items() if 'fence syncscope("wavefront") acq_rel' in b]
    # near_pass's last template argument but the types: whether the sources react
    passes = [n for n in fns if "8far_pass" in n or ("9near_pass" in n and "ELb1EEE" in n)]
    assert len(passes) >= 30
    for n in passes:
        assert any("@" + f + "(" in fns[n] for f in fence), n


def test_table_positions_take_the_saturating_conversion(tmp_path):
    # a position far outside the table, or NaN, has no conversion in the language: what the
    # compiler makes of it may index anywhere
    fns = device_functions(os.path.join(CSRC, "table.hip"), tmp_path)
    lookups = [n for n in fns if "6lookupILi" in n]
    assert len(lookups) >= 3  # CIC, TSC, TSC from LDS
    for n in lookups:
        assert "fptoui" not in fns[n] and "fptosi" not in fns[n], n
        assert any("@" + f + "(" in fns[n] for f in fns if "v_cvt_u32_f32" in fns[f]), n
