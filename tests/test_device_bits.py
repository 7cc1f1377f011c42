"""What can be checked of the device code without a GPU: helpers that are plain
arithmetic, compiled for the host with hipcc and compared with exact integers,
and the compiler's intermediate code of the kernels for gfx950."""
import os
import re
import subprocess

import pytest

from paper_2201_01556_amd import build

MAX = 2**31 - 1

PROGRAM = r"""
#include <cstdio>
#include "hf_device.h"
int main() {
  int v[8];
  while (scanf("%d %d %d %d %d %d %d %d", v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6, v + 7) == 8)
    printf("%u\n", hf::net_residual_bits(v[0], v[1], make_int2(v[2], v[3]), make_int2(v[4], v[5]),
                                         make_int2(v[6], v[7])));
  return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="hipcc not available")
def test_net_residual_bits_at_the_ends_of_int(tmp_path):
    """The bits of a net whose flows sum past INT32_MAX: units that came back
    into e_in over a pin lie on the bridge and in the excess at once."""
    cases = []
    for w in (1, 5, 2**30, 2**30 + 1, MAX):
        for fb in sorted({0, 1, w // 2, w - 1, w}):
            if fb < 0 or fb > w:
                continue
            for x_in in (0, 1, w // 2, w, MAX):
                for part in range(3):  # in the excess, or in one of the pushes not folded yet
                    for x_out in sorted({0, fb // 2, fb}):
                        e = [[0, 0], [0, 0], [0, 0]]
                        e[part][0] = x_in
                        e[(part + 1) % 3][1] = x_out
                        cases.append((fb, w, *e[0], *e[1], *e[2]))
    src = tmp_path / "bits.hip"
    exe = tmp_path / "bits"
    src.write_text(PROGRAM)
    r = subprocess.run([build.HIPCC, *build.FLAGS, str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    out = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases),
                         capture_output=True, text=True, check=True).stdout.split()
    assert len(out) == len(cases)
    for c, got in zip(cases, out):
        fb, w = c[0], c[1]
        x_in, x_out = c[2] + c[4] + c[6], c[3] + c[5] + c[7]
        want = (fb < w) | (fb - x_out > 0) << 1 | (fb > 0) << 2 | (fb + x_in > 0) << 3
        assert int(got) == want, c


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("source,exchanges", [
    ("hf_solve.hip", {"k_bfs_sweep": 4}),
    ("hf_regions.hip", {"k_rg_pins": 2, "k_rg_count_flat": 2, "k_rg_write_flat": 2}),
], ids=lambda x: x if isinstance(x, str) else "")
def test_lds_exchanges_of_a_wave_are_ordered(tmp_path, source, exchanges):
    """Kernels whose lanes hand values to each other through LDS inside a wave
    order the accesses by wavefront fences around a wave barrier: nothing else
    keeps the compiler from using a lane's own last value.  Two exchanges (the
    clearing and the reading) per LDS tally."""
    out = tmp_path / "kernels.ll"
    flags = [f for f in build.FLAGS if f not in ("-O3", "-fPIC")]
    r = subprocess.run([build.HIPCC, *flags, "-O1", "-w", "--cuda-device-only", "-emit-llvm", "-S",
                        os.path.join(build.CSRC, source), "-o", str(out)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    text = out.read_text()
    for kernel, least in exchanges.items():
        body = re.search(r"^define [^\n]*\d" + kernel + r"[A-Z][^\n]*\{\n(.*?)^\}", text, re.S | re.M)
        assert body, kernel
        found = re.findall(r'fence syncscope\("wavefront"\) release\s+'
                           r"(?:tail )?call void @llvm.amdgcn.wave.barrier\(\)[^\n]*\s+"
                           r'fence syncscope\("wavefront"\) acquire', body.group(1))
        assert len(found) >= least, (kernel, len(found))
