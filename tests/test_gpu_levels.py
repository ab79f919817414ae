"""The level-scheduled kernels at the sizes where they can go wrong: both sides of each compiled
width, nodes with more children than one pass takes, levels of several passes, intervals that
cross the 32-step pieces of the gradient sums and the 64-step pieces of the schedule, sequences
whose walk arrays leave LDS, and an infinite input. Against the oracle, at the tolerances of
the parity tests."""
import numpy as np
import pytest

from paper_1904_03409_amd import workloads as wk
from tests.gpu_helpers import TOL, compare, need_gpu, run_gpu
from tests.torch_ref import normwise

pytestmark = pytest.mark.gpu


def _ops(kind, T, B):
    rng = np.random.default_rng(T + B)
    if kind == "alternate":          # T / 2 children of the initial state, all in one level
        o = np.zeros((T, B), np.int8)
        o[0::2] = 1
        o[1::2] = -1
        return o
    if kind == "held":               # runs of holds from 1 to 100 steps between pushes and pops
        o = np.zeros((T, B), np.int8)
        for b in range(B):
            t, depth = int(rng.integers(0, 70)), 0
            while t < T:
                o[t, b] = -1 if depth and rng.random() < 0.4 else 1
                depth += int(o[t, b])
                t += int(rng.integers(1, 100))
        return o
    if kind == "push":               # no leaves: push nodes in every row of the last tile, or all but a few
        return np.ones((T, B), np.int8)
    if kind == "deep":               # one node per level
        o = np.ones((T, B), np.int8)
        o[(T + 1) // 2:] = -1
        return o
    return wk.ops_random_valid(rng, T, B)


CASES = [
    # (ops, T, B, I, H, precision)
    ("random", 33, 5, 9, 32, 0), ("random", 33, 5, 9, 33, 0), ("random", 40, 9, 40, 65, 0),
    ("random", 40, 9, 40, 129, 0), ("random", 40, 20, 33, 257, 0), ("random", 24, 20, 300, 511, 0),
    ("random", 40, 20, 65, 257, 1), ("random", 24, 20, 129, 385, 1), ("random", 24, 20, 31, 513, 1),
    ("random", 20, 20, 257, 769, 1), ("random", 20, 12, 8, 1023, 1),
    ("alternate", 300, 3, 16, 40, 0), ("alternate", 300, 3, 16, 40, 1), ("alternate", 40, 300, 8, 512, 0),
    ("alternate", 40, 300, 8, 516, 1),
    ("held", 333, 7, 12, 36, 0), ("held", 333, 7, 12, 37, 1), ("held", 64, 7, 12, 36, 0), ("held", 97, 3, 4, 260, 0),
    ("deep", 321, 2, 8, 24, 0), ("random", 20000, 1, 4, 8, 0),
    # one to four quarters of the products' row tile (2, 3 and 4 thousand rows of 16 column tiles)
    ("push", 16, 16, 130, 64, 0), ("push", 13, 20, 33, 64, 1), ("random", 40, 100, 130, 512, 0),
    ("random", 60, 100, 8, 512, 0), ("random", 80, 100, 8, 500, 0), ("random", 40, 100, 72, 1024, 1),
    ("random", 60, 100, 8, 1024, 1),
]


@pytest.mark.parametrize("case", CASES)
def test_levels(oracle_mod, case):
    need_gpu()
    kind, T, B, I, H, precision = case
    print(f"[gpu] {case}", flush=True)
    wl = wk.custom(T=T, B=B, I=I, H=H, seed=T + H, ops=_ops(kind, T, B), wscale=0.3 if H < 300 else 0.1,
                   random_state=True, dc_top=True)
    gpu, _ = run_gpu(wl, precision=precision)
    ref = oracle_mod.run(wl, bf16=precision == 1)
    compare(wl, gpu, ref, precision, alg1=oracle_mod.alg1(wl, bf16=precision == 1))


@pytest.mark.parametrize("precision", [0, 1])
def test_infinite_input(oracle_mod, precision):
    """An infinite input saturates gates; the states stay finite and other rows keep their values."""
    need_gpu()
    from paper_1904_03409_amd.stacklstm import DeviceRun
    print(f"[gpu] infinite input prec={precision}", flush=True)
    wl = wk.custom(T=24, B=4, I=40, H=48, seed=2, wscale=0.3)
    wl.x[0, 0, 3] = np.inf
    wl.x[5, 1, 39] = -np.inf
    r = DeviceRun.from_workload(wl, precision=precision)
    r.forward()
    a1 = oracle_mod.alg1(wl, bf16=precision == 1)
    for k in ("h_cell", "c_cell"):
        got = getattr(r, k).cpu().numpy()
        assert np.all(np.isfinite(a1[k])) and normwise(got, a1[k]) <= TOL[precision], k


@pytest.mark.parametrize("precision", [0, 1])
def test_step_clock(precision):
    """With dims.step_clock the recurrent kernels of every width run as instantiations with stamps: the
    same outputs, and four stamps in order for each level."""
    need_gpu()
    import ctypes
    import torch
    from paper_1904_03409_amd.stacklstm import DeviceRun
    for H in (24, 60, 130, 300, 500) if precision == 0 else (24, 60, 130, 300, 500, 700, 1000):
        print(f"[gpu] step clock H={H} prec={precision}", flush=True)
        wl = wk.custom(T=20, B=5, I=8, H=H, seed=H, ops=_ops("deep", 20, 5), wscale=0.1, random_state=True)
        r = DeviceRun.from_workload(wl, precision=precision)
        r.forward()
        r.backward()
        want = r.results()
        clk = torch.zeros(2, 512, wl.T, 4, dtype=torch.int64, device="cuda")
        r.dims.step_clock = ctypes.c_void_p(clk.data_ptr())
        r.forward()
        r.backward()
        torch.cuda.synchronize()
        got = r.results()
        for k in want:
            assert np.array_equal(got[k], want[k]), (H, k)
        c = clk.cpu().numpy()
        for p, levels in ((0, 11), (1, 10)):              # forward: the initial states' level too
            used = c[p, c[p, :, 0, 0] > 0]
            assert len(used) == 5 * -(-H // 32)
            assert np.all(np.diff(used[:, :levels], axis=2) >= 0) and not used[:, levels:].any()
            step = np.diff(used[:, :levels, 0], axis=1)
            assert np.all(step > 0 if p == 0 else step < 0)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("B,H", [(301, 33), (1000, 8), (130, 200)])
def test_bias_gradient_of_many_groups(precision, B, H):
    """db of equal gate gradients (no weights, one depth) is their number times one of them: the sums over a
    thread's nodes, a workgroup's threads and up to 128 groups lose one rounding, not one per addition."""
    need_gpu()
    from paper_1904_03409_amd.stacklstm import DeviceRun
    T = 58
    print(f"[gpu] db of equal gradients B={B} H={H} prec={precision}", flush=True)
    wl = wk.custom(T=T, B=B, I=4, H=H, seed=1, ops=_ops("alternate", T, B))
    for a in (wl.x, wl.W, wl.U, wl.b, wl.h0, wl.c0):
        a[...] = 0
    v = np.linspace(0.1, 0.7, H).astype(np.float32)
    wl.dh_top[...] = v
    r = DeviceRun.from_workload(wl, precision=precision)
    r.forward()
    r.backward()
    db = r.db.cpu().numpy().astype(np.float64)
    want = 0.25 * v.astype(np.float64) * (B * T // 2)      # o i of a gate at 0, g alone: 0.5 0.5
    assert np.all(np.abs(db[2 * H:3 * H] / want - 1) <= 2.0 ** -23)
    assert not db[:2 * H].any() and not db[3 * H:].any()
