"""fp32 mode holds its gradients and states over fp32's exponent range: gradients that shrink by
tens of orders of magnitude on their way down a deep stack, gradients scaled up or down, weights
and initial states far from one. Judged step by step against the fp64 oracle, each step's gradient
on its own norm, at the parity tolerance (plain fp32 arithmetic stays within 2e-6)."""
import numpy as np
import pytest

from paper_1904_03409_amd import workloads as wk
from tests.gpu_helpers import TOL, need_gpu, run_gpu
from tests.torch_ref import normwise

pytestmark = pytest.mark.gpu


def _errors(wl, gpu, ref):
    errs = {k: normwise(gpu[k], ref[k]) for k in ("h_top", "c_top", "dh0", "dc0", "dW", "dU", "db")}
    errs["dx"] = max(normwise(gpu["dx"][t], ref["dx"][t]) for t in range(wl.T) if np.any(ref["dx"][t]))
    return errs


def _check(oracle_mod, wl):
    need_gpu()
    print(f"[gpu] {wl.name} T={wl.T} B={wl.B} I={wl.I} H={wl.H}", flush=True)
    gpu, _ = run_gpu(wl, precision=0)
    errs = _errors(wl, gpu, oracle_mod.run(wl))
    print(f"[gpu] errors {errs}", flush=True)
    bad = {k: v for k, v in errs.items() if not v <= TOL[0]}
    assert not bad, (bad, errs)


# (T, H): the last is where dh0 is near the smallest normal fp32 number
LAST = [(60, 64), (100, 64), (150, 64), (110, 200), (100, 512)]


@pytest.mark.parametrize("T,H", LAST)
def test_loss_on_the_last_step_of_a_deep_stack(oracle_mod, T, H):
    wl = wk.custom(T=T, B=3, I=16, H=H, seed=T + H, ops=np.ones((T, 3), np.int8), wscale=0.08, random_state=True,
                   name="last step")
    wl.dh_top[:-1] = 0
    _check(oracle_mod, wl)


@pytest.mark.parametrize("H", [64, 130])
@pytest.mark.parametrize("scale", [1e-34, 1e-26, 1e24, 1e32])
def test_scaled_gradients(oracle_mod, scale, H):
    wl = wk.custom(T=24, B=5, I=20, H=H, seed=3, wscale=0.3, random_state=True, dc_top=True, name=f"gradients x {scale}")
    wl.dh_top *= np.float32(scale)
    wl.dc_top *= np.float32(scale)
    _check(oracle_mod, wl)


@pytest.mark.parametrize("scale", [1e-30, 1e-20])
def test_small_recurrent_weights(oracle_mod, scale):
    """All that dh0 holds came through U (a stack of pushes alone)."""
    wl = wk.custom(T=6, B=5, I=20, H=64, seed=4, ops=np.ones((6, 5), np.int8), wscale=0.3, random_state=True,
                   name=f"U x {scale}")
    wl.U[:] *= np.float32(scale)
    wl.dh_top[:-1] = 0
    _check(oracle_mod, wl)


@pytest.mark.parametrize("scale", [1e-30, 1e-12, 1e12, 1e30])
def test_initial_state_far_from_one(oracle_mod, scale):
    """Depth one only (pushes on the initial state), h0 U of ordinary size."""
    ops = np.zeros((12, 4), np.int8)
    ops[0::2] = 1
    ops[1::2] = -1
    wl = wk.custom(T=12, B=4, I=20, H=64, seed=5, ops=ops, wscale=0.3, random_state=True, name=f"h0 x {scale}")
    wl.h0[:] *= np.float32(scale)
    wl.U[:] /= np.float32(scale)
    _check(oracle_mod, wl)
