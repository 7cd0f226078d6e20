"""Registers of the stage kernels of the detailed model, from the metadata of a compile: the
16 x 16 kernels of every remainder of the component count modulo four keep three wavefronts per
SIMD (512 / 168 registers) and use no scratch memory."""

import concurrent.futures as cf
import os
import re
import subprocess

import pytest

from paper_2504_13750_amd import build

pytestmark = pytest.mark.slow


def _kernels(ns):
    """{stage kernel (width, 1-D tiles, 2-D tiles): (registers, scratch bytes)} of a species count."""
    cmd = [build.HIPCC] + [f for f in build.FLAGS if f != "-fPIC"] + [
        f"-DJANC_NS={ns}", "--cuda-device-only", "-S", os.path.join(build.CSRC, "janc_species.hip"), "-o", "-"]
    asm = subprocess.run(cmd, check=True, capture_output=True, text=True).stdout
    out = {}
    for m in re.finditer(r"\.name: +_ZN4janc12stage_kernelILi2ELi\d+ELi(\d+)ELi\d+ELb(\d)ELb(\d)E"
                         r".*?\.private_segment_fixed_size: (\d+).*?\.vgpr_count: +(\d+)", asm, re.S):
        out[int(m[1]), int(m[2]), int(m[3])] = int(m[5]), int(m[4])
    return out


def test_waves_of_the_default_tiles():
    counts = [2, 3, 4, 9]   # 5, 6, 7 and 12 components
    with cf.ThreadPoolExecutor(4) as ex:
        found = dict(zip(counts, ex.map(_kernels, counts)))
    for ns in counts:
        for kinds in [(0, 1), (1, 0)]:
            regs, scratch = found[ns][(16, *kinds)]
            print(f"{ns} species, kinds {kinds}: {regs} registers, {scratch} bytes of scratch")
            assert regs <= 168 and scratch == 0, (ns, kinds)
