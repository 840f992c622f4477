"""The statistics and selection kernels launch with a fixed dynamic LDS size;
with their static LDS it must fit the 160 KiB a gfx950 workgroup can hold,
or every launch fails.  Checked on the CPU from a device-only compile of each
source with the library's own flags (hipcc cross-compiles without a GPU)."""

from __future__ import annotations

import math
import os
import re
import shutil
import subprocess

import pytest

from paper_2606_01790_amd import build as B

LDS_LIMIT = 160 * 1024


def _const(src: str, name: str) -> int:
    m = re.search(r"constexpr int %s = ([0-9* ]+);" % name, src)
    assert m, name
    return math.prod(int(f) for f in m.group(1).split("*"))


def _static_lds(source: str, kernel: str, tmp_path) -> int:
    out = tmp_path / (os.path.basename(source) + ".s")
    flags = [f for f in B.HIP_FLAGS if f != "-fPIC"]
    subprocess.run([B.HIPCC, *flags, "-I", B.INCLUDE, "--cuda-device-only", "-S",
                    "-o", str(out), source], check=True, capture_output=True)
    meta = out.read_text().split("amdhsa.kernels:", 1)[1]
    for blk in meta.split("\n  - ")[1:]:
        name = re.search(r"\.name:\s+(\S+)", blk)
        if name and kernel in name.group(1):
            return int(re.search(r"\.group_segment_fixed_size:\s+(\d+)", blk).group(1))
    raise AssertionError(f"{kernel} not found in {source}")


needs_hipcc = pytest.mark.skipif(not (os.path.exists(B.HIPCC) or shutil.which("hipcc")),
                                 reason="hipcc not available")


def _shape(src: str, nt: int) -> int:
    """Dynamic LDS bytes of the statistics kernel's block shape `nt`, from
    the StatsShape specialisation in the source (constants from the source
    and from stats_shape.h)."""
    consts = {m.group(1): int(m.group(2))
              for m in re.finditer(r"constexpr int (k\w+) = (\d+);",
                                   src + open(os.path.join(B.CSRC, "stats_shape.h")).read())}
    body = src.split("struct StatsShape<%d> {" % nt, 1)[1].split("};", 1)[0]

    def value(name):
        expr = re.search(name + r" = ([^,;]+)", body).group(1)
        for k, v in consts.items():
            expr = re.sub(r"\b%s\b" % k, str(v), expr)
        assert re.fullmatch(r"[0-9*+ ]+", expr), expr
        return eval(expr)

    return 4 * (value("kHistInts") + value("kKeyCache") + value("kCand"))


@needs_hipcc
def test_stats_kernel_lds_fits(tmp_path):
    """The wide shape fits one block per CU; the narrow one, launched when
    the blocks outnumber the CUs, must fit two, and the small one four."""
    path = os.path.join(B.CSRC, "state.hip")
    src = open(path).read()
    for fused in ("0", "1"):
        wide = _shape(src, 1024) + _static_lds(path, "stats_kernelILi1024ELb%sE" % fused,
                                               tmp_path)
        assert wide <= LDS_LIMIT, (fused, wide)
    narrow = _shape(src, 512) + _static_lds(path, "stats_kernelILi512", tmp_path)
    assert 2 * narrow <= LDS_LIMIT, narrow
    small = _shape(src, 256) + _static_lds(path, "stats_kernelILi256", tmp_path)
    assert 4 * small <= LDS_LIMIT, small


@needs_hipcc
def test_stats_kernels_use_no_scratch(tmp_path):
    """Every form of the statistics kernel (three block shapes, with and
    without the selection, visual keys in LDS, few or more, or read from
    memory) keeps its values in registers: scratch memory is set up and touched
    also by calls whose own pass needs none of it.  Each form's LDS fits as above."""
    path = os.path.join(B.CSRC, "state.hip")
    src = open(path).read()
    out = tmp_path / "state.s"
    flags = [f for f in B.HIP_FLAGS if f != "-fPIC"]
    subprocess.run([B.HIPCC, *flags, "-I", B.INCLUDE, "--cuda-device-only", "-S",
                    "-o", str(out), path], check=True, capture_output=True)
    seen = set()
    for blk in out.read_text().split("amdhsa.kernels:", 1)[1].split("\n  - ")[1:]:
        m = re.search(r"\.name:\s+\S*stats_kernelILi(\d+)(\S*)", blk)
        if not m:
            continue
        field = lambda k: int(re.search(r"\.%s:\s+(\d+)" % k, blk).group(1))
        nt = int(m.group(1))
        seen.add((nt, m.group(2)))
        assert field("private_segment_fixed_size") == 0, m.group(0)
        lds = _shape(src, nt) + field("group_segment_fixed_size")
        assert lds * (1024 // nt) <= LDS_LIMIT, (m.group(0), lds)
    assert {nt for nt, _ in seen} == {256, 512, 1024}


@needs_hipcc
def test_select_kernel_lds_fits(tmp_path):
    path = os.path.join(B.CSRC, "select.hip")
    src = open(os.path.join(B.CSRC, "select_body.h")).read()
    dynamic = 4 * _const(src, "kSelLdsKeys")
    static = _static_lds(path, "select_kernel", tmp_path)
    assert static + dynamic <= LDS_LIMIT, (static, dynamic)


@needs_hipcc
def test_float32_unit_holds_float32_kernels_only(tmp_path):
    """The unrolled pass 2 serves bf16 keys with d = 128 alone; the float32
    unit, which can never choose it, does not compile its sixteen kernels."""
    path = os.path.join(B.CSRC, "score_f32.hip")
    out = tmp_path / "score_f32.s"
    flags = [f for f in B.HIP_FLAGS if f != "-fPIC"]
    subprocess.run([B.HIPCC, *flags, "-I", B.INCLUDE, "--cuda-device-only", "-S",
                    "-o", str(out), path], check=True, capture_output=True)
    names = re.findall(r"\.name:\s+(\S*score_pass\S*)", out.read_text())
    assert names and not [n for n in names if "unrolled" in n or "DF16b" in n], names
