"""Byte offsets of the padded rows at the largest sizes the entry points accept (no GPU): the
kernels' offset functions, compiled for the host, against 64-bit arithmetic. An odd H pads its gate
gradient rows, an H of 1 or 2 its state rows, past the products that the size limits bound."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1904_03409_amd", "csrc")

MAIN = r'''
#include <cstdio>
#include <cstdlib>
#include "levels.h"
#include "contract.h"
int main(int argc, char** argv) {
  for (int i = 1; i + 3 < argc; i += 4) {
    const int np = atoi(argv[i]), nodes = atoi(argv[i + 1]), b = atoi(argv[i + 2]), h = atoi(argv[i + 3]);
    const int h4s = (4 * h + 7) / 8 * 8, hs = (h + 7) / 8 * 8;
    const size_t got = np == 2 ? lev_da_off<2>(nodes - 1, h4s, h - 1) : lev_da_off<1>(nodes - 1, h4s, h - 1);
    printf("%zu %d\n", got, (int)tn_far(nodes + b, hs));
  }
}
'''


def _largest_T(s, B, H, precision):
    lo, hi = 0, 1 << 20
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if s.stacklstm_workspace_bytes(s.make_dims(mid, B, 1, H, precision)):
            lo = mid
        else:
            hi = mid
    return lo


def test_offsets_at_the_largest_sizes(tmp_path):
    hip = "/opt/rocm/include/hip/hip_runtime.h"
    if not os.path.exists(hip):
        pytest.skip("no HIP headers")
    from paper_1904_03409_amd import stacklstm as s
    src, exe = os.path.join(str(tmp_path), "off.cpp"), os.path.join(str(tmp_path), "off")
    open(src, "w").write(MAIN)
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC, src, "-o", exe])
    cases = []
    for precision in (0, 1):
        for H in list(range(1, 34)) + [63, 127, 255, 511]:
            for B in (1, 1000, 8192):
                T = _largest_T(s, B, H, precision)
                assert T > 0
                cases.append((2 if precision == 0 else 1, T * B, B, H))
    args = [str(v) for c in cases for v in c]
    out = subprocess.check_output([exe, *args], text=True).split("\n")
    past = 0
    for (np_, nodes, B, H), line in zip(cases, out):
        got, far = (int(v) for v in line.split())
        want = 2 * ((nodes - 1) * ((4 * H + 7) // 8 * 8) + 4 * (H - 1))
        assert got == want, (np_, nodes, H)
        past += want >= 1 << 32
        assert far == ((nodes + B) * ((H + 7) // 8 * 8) * 2 > 0xffffffff)
        assert not far or H <= 2
    assert past                                            # (H = 3 and on, bf16 mode)
