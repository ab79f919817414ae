"""Which sizes the allocation-free forward serves (no GPU needed: with none, a call that passes the
size checks stops at the missing device before it touches a pointer): the header's rule, and
room in the static array for every size that the rule admits."""
import ctypes
import os
import random
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _up(n):
    return (n + 255) // 256 * 256


def _measure(T, B, I, H, precision):
    return (_up(8448) + _up(4 * B * (T + 1)) + _up(4 * B) + _up(16 * I * H) + 2 * _up(max(16 * T * B * H, 16)) +
            (_up(2 * (T + 1) * B * H) if precision == 1 else 0))


def test_static_forward_serves_what_the_header_says():
    import torch
    if torch.cuda.is_available():
        pytest.skip("the calls pass made-up pointers: only where no device can run them")
    from paper_1904_03409_amd import stacklstm as s
    lib = s.load_library()
    text = open(os.path.join(ROOT, "include", "stacklstm.h")).read()
    size = {k: int(v) << 20 for k, v in re.findall(r"#define (SLSTM_FWD_STATIC\w+) \(\(size_t\)(\d+) << 20\)", text)}
    limit = size["SLSTM_FWD_STATIC_MAX_BYTES"]
    assert limit == s.SLSTM_FWD_STATIC_MAX_BYTES and size["SLSTM_FWD_STATIC_BYTES"] == 256 << 20
    one = ctypes.c_void_p(4096)

    def served(T, B, I, H, precision):
        d = s.make_dims(T, B, I, H, precision)
        rc = lib.stacklstm_fwd_static(ctypes.byref(d), *([one] * 13), ctypes.c_void_p(0))
        assert rc in (4, 6), rc                             # work space too small; no device
        return rc == 6

    rng = random.Random(1)
    checked = 0
    for precision in (0, 1):
        for H in [1, 2, 3, 7, 8, 9, 16, 31, 64, 200, 511, 512] + ([1023, 1024] if precision else []):
            for B in (1, 2, 63, 128, 129, 1000):
                for I in (1, 9, 64, 1000, 1 << 14, 1 << 20):
                    lo, hi = 0, 1 << 23                     # the largest T that the rule admits
                    while hi - lo > 1:
                        mid = (lo + hi) // 2
                        lo, hi = (mid, hi) if _measure(mid, B, I, H, precision) <= limit else (lo, mid)
                    if _measure(lo, B, I, H, precision) > limit or not s.stacklstm_workspace_bytes(
                            s.make_dims(lo, B, I, H, precision)):
                        continue
                    assert served(lo, B, I, H, precision), (lo, B, I, H, precision)
                    assert not served(lo + 1, B, I, H, precision)
                    t = rng.randint(0, lo)
                    assert served(t, B, I, H, precision), (t, B, I, H, precision)
                    checked += 1
    assert checked > 200
