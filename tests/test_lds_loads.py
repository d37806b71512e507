"""Loads straight into LDS (prefill_fa32_kernel) are waited for by the code itself at
every barrier: __syncthreads() does not promise that another wave's loads into LDS have
landed, whatever the compiler of the day puts before it."""
import os
import re
import subprocess

import pytest

from paper_2410_18701_amd import build

SOURCE = """
#include "prefill_attn.hpp"
template __global__ void baton::prefill_fa32_kernel<%d, %d>(const baton::PrefillArgs);
"""


@pytest.mark.parametrize("D,G,own", [(64, 1, 2), (128, 8, 4)])   # own: an iteration's own loads, which may stay in flight
def test_every_barrier_waits(tmp_path, D, G, own):
    src = tmp_path / "k.hip"
    src.write_text(SOURCE % (D, G))
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    out = tmp_path / "k.ll"
    subprocess.run(["hipcc", *flags, "--offload-device-only", "-S", "-emit-llvm", str(src), "-o", str(out)], check=True,
                   stderr=subprocess.DEVNULL)
    body = re.search(r"define [^\n]*prefill_fa32_kernel[^\n]*\n(.*?)\n}", out.read_text(), re.S).group(1)
    lines = [l for l in body.split("\n") if re.search(r"s\.barrier|s\.waitcnt|load\.lds|fence", l)]
    assert sum("load.lds" in l for l in lines) >= 8 and not any(re.match(r"\s*fence", l) for l in lines)
    waits = []
    for before, line in zip(lines, lines[1:]):
        if "s.barrier" in line:
            m = re.search(r"s\.waitcnt\(i32 (?:noundef )?(\d+)\)", before)
            assert m, "a barrier without an explicit wait before it"
            n = int(m.group(1))
            assert n >> 8 & 15 == 0 and n >> 14 == 0, "LDS reads, or vmcnt's high bits"
            waits.append(n & 15)
    assert len(waits) >= 5 and waits[:2] == [0, 0] and set(waits[2:]) == {own}, waits
