"""Infinities and NaN in fp32 mode: the same outputs are NaN, +inf and -inf as in the fp64 oracle and
the others keep their values, at widths whose state rows are no whole number of 128-byte lines, in
levels of several passes."""
import numpy as np
import pytest

from paper_1904_03409_amd import workloads as wk
from tests.gpu_helpers import TOL, need_gpu
from tests.torch_ref import normwise

pytestmark = pytest.mark.gpu


def _same(got, ref, what):
    for f, name in ((np.isnan, "NaN"), (np.isposinf, "+inf"), (np.isneginf, "-inf")):
        assert np.array_equal(f(got), f(ref)), (what, name, int(f(got).sum()), int(f(ref).sum()))
    ok = np.isfinite(ref)
    if ok.any():
        assert normwise(got[ok], ref[ok]) <= TOL[0], what


def _forward(wl):
    import torch
    from paper_1904_03409_amd.stacklstm import DeviceRun
    r = DeviceRun.from_workload(wl, precision=0)
    r.forward()
    torch.cuda.synchronize()
    return r


def _ops(T, B):
    """Pushes on the initial state and one deeper push after every eighth: levels of many states."""
    o = np.zeros((T, B), np.int8)
    for t in range(T):
        k = t % 8
        o[t] = (1, -1, 1, -1, 1, 1, -1, -1)[k]
    return o


@pytest.mark.parametrize("H", [36, 100, 130, 500])
def test_infinite_weight_and_late_nan(oracle_mod, H):
    """A weight of U is infinite (every product with it has to be made infinite, not NaN), and a
    NaN enters with an input late in the sequence: in a level's second pass or later."""
    need_gpu()
    T, B = 400, 2
    print(f"[gpu] infinite U, NaN in x, H={H}", flush=True)
    wl = wk.custom(T=T, B=B, I=12, H=H, seed=H, ops=_ops(T, B), wscale=0.3 if H < 300 else 0.1, random_state=True)
    wl.U[5, 3] = np.inf
    wl.U[H - 1, 2 * H + 7] = -np.inf
    wl.x[332, 0, 1] = np.nan                              # (t % 8 == 4: a state with a child)
    r = _forward(wl)
    a1 = oracle_mod.alg1(wl)
    assert np.isnan(a1["h_cell"][332, 0]).all() and np.isnan(a1["h_cell"][333, 0]).all()
    assert np.isfinite(a1["h_cell"][:, 1]).all()
    for k in ("h_cell", "c_cell"):
        _same(getattr(r, k).cpu().numpy(), a1[k], k)


@pytest.mark.parametrize("H", [36, 130])
def test_infinite_initial_state(oracle_mod, H):
    need_gpu()
    T, B = 40, 3
    print(f"[gpu] infinite h0, H={H}", flush=True)
    wl = wk.custom(T=T, B=B, I=12, H=H, seed=H + 1, ops=_ops(T, B), wscale=0.3, random_state=True)
    wl.h0[1, 4] = np.inf
    wl.h0[2, H - 1] = -np.inf
    r = _forward(wl)
    a1 = oracle_mod.alg1(wl)
    for k in ("h_cell", "c_cell"):
        _same(getattr(r, k).cpu().numpy(), a1[k], k)


def _backward(oracle_mod, wl, keys=("dx", "dh0", "dc0", "dW", "dU", "db")):
    import torch
    r = _forward(wl)
    r.backward()
    torch.cuda.synchronize()
    got, ref = r.results(), oracle_mod.run(wl)
    for k in keys:
        _same(got[k], ref[k], k)
    return ref


@pytest.mark.parametrize("H", [36, 100, 130, 500])
def test_infinite_upstream_gradient(oracle_mod, H):
    """Infinite gradients of two steps late in the sequence: their nodes' ancestors get infinities
    and NaN, the others' gradients stay."""
    need_gpu()
    T, B = 400, 2
    print(f"[gpu] infinite dh_top, H={H}", flush=True)
    wl = wk.custom(T=T, B=B, I=12, H=H, seed=H, ops=_ops(T, B), wscale=0.3 if H < 300 else 0.1, random_state=True)
    wl.dh_top[333, 0, 4] = np.inf                        # (t % 8 == 5: the child of a state)
    wl.dh_top[213, 0, H - 1] = -np.inf
    ref = _backward(oracle_mod, wl)
    assert not np.isfinite(ref["dx"][333, 0]).any() and np.isfinite(ref["dx"][:, 1]).all()


@pytest.mark.parametrize("H", [36, 130])
def test_infinite_weight_backward(oracle_mod, H):
    need_gpu()
    T, B = 200, 2
    print(f"[gpu] infinite U, backward, H={H}", flush=True)
    wl = wk.custom(T=T, B=B, I=12, H=H, seed=H, ops=_ops(T, B), wscale=0.3, random_state=True)
    wl.U[5, 3 * H + 7] = np.inf
    _backward(oracle_mod, wl, keys=("dx", "dh0", "dc0"))


@pytest.mark.parametrize("I,H", [(13, 36), (130, 130)])
@pytest.mark.parametrize("where", ["x", "W"])
def test_infinite_inputs_of_the_products(oracle_mod, where, I, H):
    """Infinities in x or W, forward and backward: x W, dW and dx over them (the gates saturate, so
    the gate gradients they meet are exactly 0 in places: NaN there too)."""
    need_gpu()
    T, B = 45, 3
    print(f"[gpu] infinite {where}, I={I} H={H}", flush=True)
    wl = wk.custom(T=T, B=B, I=I, H=H, seed=I + H, wscale=0.3 if H < 100 else 0.1, random_state=True)
    if where == "x":
        wl.x[2, 0, 3] = np.inf
        wl.x[30, 1, I - 1] = -np.inf
    else:
        wl.W[2, 2 * H + 5] = np.inf
        wl.W[I - 1, 3 * H + 7] = -np.inf
    a1 = oracle_mod.alg1(wl)
    r = _forward(wl)
    for k in ("h_cell", "c_cell"):
        _same(getattr(r, k).cpu().numpy(), a1[k], k)
    _backward(oracle_mod, wl)


def test_diverged_step_takes_about_as_long(oracle_mod):
    """A training step whose gradients are all NaN: every NaN result is repeated on the matrix units
    (1.1 times the ordinary step; one lane for each result took 40 times)."""
    need_gpu()
    import torch
    from paper_1904_03409_amd.stacklstm import DeviceRun
    r = DeviceRun.from_workload(wk.make("parser"), precision=0)

    def step():
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        r.forward()
        r.backward()
        b.record()
        b.synchronize()
        return a.elapsed_time(b)

    plain = min(step() for _ in range(5))
    r.dh_top.fill_(float("nan"))
    nan = min(step() for _ in range(5))
    print(f"[gpu] step {plain:.3f} ms, all NaN {nan:.3f} ms", flush=True)
    assert np.isnan(r.results()["dW"]).all()
    assert nan < 5 * plain
