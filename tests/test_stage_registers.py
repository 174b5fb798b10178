"""Registers of the stage kernel, from the compiler's own report for the build's flags:
residuals and stages 1-4 of every mesh, model and schedule keep all their values
in registers; only last stages spill a few (the metric terms of the output plane
carried on general meshes; product meshes with the dynamic model or, in FP32, held
viscosities, which at fewer waves are slower)."""
import concurrent.futures as cf
import os
import re
import subprocess

import pytest

SOURCES = ("residual_fused.hip", "residual_fused_wide.hip", "residual_fused32.hip",
           "residual_fused32_wide.hip")
NAME = re.compile(r"Function Name: \S*k_fusedI([df])Lb(\d)ELi(\d)ELb(\d)ELi(\d)ELb(\d)ELb(\d)E")
SPILL = re.compile(r"\bVGPRs Spill: (\d+)")
EPI_RK_LAST = 2


def _report(src):
    from paper_2301_00817_amd import build as b
    r = subprocess.run([b._hipcc(), *b.CFLAGS, *b.SOURCE_FLAGS.get(src, []), "--cuda-device-only",
                        "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(b.CSRC, src),
                        "-o", os.devnull], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    out, name = {}, None
    for line in r.stderr.splitlines():
        m = NAME.search(line)
        if m:
            name = m.groups()
        m = SPILL.search(line)
        if m and name:
            out[name], name = int(m.group(1)), None
    return out


@pytest.fixture(scope="module")
def spills():
    with cf.ThreadPoolExecutor(len(SOURCES)) as ex:
        return dict(kv for d in ex.map(_report, SOURCES) for kv in d.items())


def test_only_last_stages_spill(spills):
    # T, tile, epilogue, axis, schedule, dynamic, product
    assert len(spills) == 192
    bad = {k: v for k, v in spills.items() if v and int(k[2]) != EPI_RK_LAST}
    assert not bad, bad
    assert max(spills.values()) <= 12


def test_product_fp64_steps_without_spill(spills):
    """The FP64 instances of jets and boxes with a static or no SGS model: none at all."""
    for k, v in spills.items():
        if k[0] == "d" and k[5] == "0" and k[6] == "1":
            assert v == 0, (k, v)


def test_two_pass_faces_without_spill():
    """The face pass of the two-pass residual (256-thread blocks)."""
    from paper_2301_00817_amd import build as b
    r = subprocess.run([b._hipcc(), *b.CFLAGS, "--cuda-device-only",
                        "-Rpass-analysis=kernel-resource-usage", "-c",
                        os.path.join(b.CSRC, "residual_ref.hip"), "-o", os.devnull],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    found = {}
    name = None
    for line in r.stderr.splitlines():
        m = re.search(r"Function Name: \S*k_face_passI([df])E", line)
        if m:
            name = m.group(1)
        m = SPILL.search(line)
        if m and name:
            found[name], name = int(m.group(1)), None
    assert found == {"d": 0, "f": 0}
