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


DEFAULTS = r"""
#include <cstdio>
#include "hf_host.h"
int main() {
  long long V, E, P;
  int arc, flat, pull, bu, gi, tail;
  while (scanf("%lld %lld %lld %d %d %d %d %d %d", &V, &E, &P, &arc, &flat, &pull, &bu, &gi,
               &tail) == 9) {
    fp_options o{};
    o.bfs_flat = flat;
    o.bfs_arc_parallel = arc;
    o.pull_min = pull;
    o.bottom_up_min = bu;
    o.gr_interval = gi;
    o.tail_gr_interval = tail;
    const long long N = ((V + 1) & ~1ll) + 2 * E;
    const bool swept = hf::levels_swept(o, hf::SweepMaps(V, E, P, N));
    const fp_options user = o;
    hf::resolve_by_size(&o, V, E, P, N);
    printf("%d %d %d\n", o.bottom_up_min, o.gr_interval, hf::tail_rounds(o, N, swept));
    fprintf(stderr, "%d\n", hf::forward_min(o, user, N));
  }
  return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="hipcc not available")
def test_defaults_by_size_and_form(tmp_path):
    """Level threshold (0 = never) and relabel intervals that a network's size
    and the form of its levels select.  Large networks whose levels cannot be
    swept (nets with far more pins than nodes, another form of a level chosen)
    and smaller ones with many pins per node expand their levels from N/50 on;
    the former also keep the longer intervals."""
    # V, E, P, bfs_arc_parallel, bfs_flat, pull_min, bottom_up_min, gr_interval, tail -> result
    table = [
        ((2000, 3000, 15_000, 0, 1, 0, 0, 0, 0), (0, 10, 25)),
        ((100_000, 200_000, 740_000, 0, 1, 0, 0, 0, 0), (0, 10, 25)),
        ((1_000_000, 2_000_000, 7_400_000, 0, 1, 0, 0, 0, 0), (312_500, 10, 25)),
        ((1 << 20, 0, 0, 0, 1, 0, 0, 0, 0), (262_144, 10, 25)),
        ((1_000_000, 2_000_000, 7_400_000, 1, 1, 0, 0, 0, 0), (100_000, 16, 64)),
        ((1_000_000, 2_000_000, 7_400_000, 0, -1, 0, 0, 0, 0), (100_000, 16, 64)),
        ((1_000_000, 2_000_000, 7_400_000, 0, 1, 20_000, 0, 0, 0), (100_000, 16, 64)),
        ((100_000, 200_000, 740_000, 1, 1, 0, 0, 0, 0), (0, 10, 25)),
        ((500_000, 300_000, 18_000_000, 0, 1, 0, 0, 0, 0), (22_000, 16, 64)),
        ((100_000, 20_000, 10_000_000, 0, 1, 0, 0, 0, 0), (2800, 10, 25)),
        ((20_000, 10_000, 5_000_000, 0, 1, 0, 0, 0, 0), (1024, 10, 25)),
        ((20_000, 12_000, 720_000, 0, 1, 0, 0, 0, 0), (0, 10, 25)),
        ((100_000, 60_000, 1_800_000, 0, 1, 0, 0, 0, 0), (0, 10, 25)),
        # chosen by the caller
        ((500_000, 300_000, 18_000_000, 0, 1, 0, 77, 8, 30), (77, 8, 30)),
        ((500_000, 300_000, 18_000_000, 0, 1, 0, -1, -1, -1), (0, 0, 0)),
        ((500_000, 300_000, 18_000_000, 0, 1, 0, 0, 8, 0), (22_000, 8, 32)),
        ((100_000, 200_000, 740_000, 0, 1, 0, 0, 8, 0), (0, 8, 20)),
    ]
    src = tmp_path / "defaults.hip"
    exe = tmp_path / "defaults"
    src.write_text(DEFAULTS)
    r = subprocess.run([build.HIPCC, *build.FLAGS, str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    run = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c, _ in table),
                         capture_output=True, text=True, check=True)
    out = run.stdout.splitlines()
    assert [tuple(map(int, line.split())) for line in out] == [want for _, want in table]
    # the forward search: N/50 in large networks by default, else the same
    for (c, want), forward in zip(table, map(int, run.stderr.split())):
        n = ((c[0] + 1) & ~1) + 2 * c[1]
        default = c[6] == 0 and n >= 1 << 20
        assert forward == (n // 50 if default else want[0]), c
