"""Error paths of the C-ABI: every bad input returns its status code, nothing faults."""
import numpy as np
import pytest
import torch

from paper_1904_03409_amd import workloads as wk
from tests.gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu


def _run(wl, **kw):
    from paper_1904_03409_amd.stacklstm import DeviceRun
    r = DeviceRun.from_workload(wl, **kw)
    return r, r.forward(check=False)


def test_bad_op_and_underflow():
    need_gpu()
    ops = np.ones((10, 4), np.int8)
    ops[3, 2] = 5
    r, rc = _run(wk.custom(T=10, B=4, I=3, H=8, seed=0, ops=ops))
    assert rc == 2
    ops = np.ones((10, 4), np.int8)
    ops[0, 1] = -1
    r, rc = _run(wk.custom(T=10, B=4, I=3, H=8, seed=0, ops=ops))
    assert rc == 3
    ops = np.zeros((10, 4), np.int8)
    ops[2, 3] = 1
    ops[3, 3] = -1
    ops[4, 3] = -1                # second pop of element 3 underflows at step 4
    ops[6, 3] = 7                 # a later bad op does not change the code of element 3
    r, rc = _run(wk.custom(T=10, B=4, I=3, H=8, seed=0, ops=ops))
    assert rc == 3


def test_workspace_dims_and_null():
    need_gpu()
    from paper_1904_03409_amd import stacklstm as s
    wl = wk.custom(T=8, B=4, I=3, H=8, seed=0)
    r, rc = _run(wl)
    assert rc == 0
    small = torch.empty(r.workspace.numel() - 256, dtype=torch.uint8, device="cuda")
    rc = s.stacklstm_fwd(r.dims, r.x, r.ops, r.W, r.U, r.b, r.h0, r.c0, r.h_cell, r.c_cell, None, None, r.ptr,
                         r.top, small, check=False)
    assert rc == 4
    bad = s.make_dims(8, 4, 3, 2000)
    assert s.stacklstm_workspace_bytes(bad) == 0
    rc = s.stacklstm_fwd(bad, r.x, r.ops, r.W, r.U, r.b, r.h0, r.c0, r.h_cell, r.c_cell, None, None, r.ptr, r.top,
                         r.workspace, check=False)
    assert rc == 1
    rc = s.stacklstm_fwd(r.dims, None, r.ops, r.W, r.U, r.b, r.h0, r.c0, r.h_cell, r.c_cell, None, None, r.ptr,
                         r.top, r.workspace, check=False)
    assert rc == 1


def test_spin_limit_timeout_reported():
    """A one-poll barrier limit forced from the host: the kernels give up, every
    workgroup leaves its loop, and the call reports SLSTM_ETIMEOUT (also through
    stacklstm_sync_status)."""
    need_gpu()
    from paper_1904_03409_amd import stacklstm as s
    wl = wk.make("parser")
    r, rc = _run(wl, spin_limit=1)
    assert rc == 7
    assert s.stacklstm_sync_status(r.workspace) == 7
    torch.cuda.synchronize()
    # the same buffers run normally afterwards
    r2, rc2 = _run(wl)
    assert rc2 == 0
    assert s.stacklstm_sync_status(r2.workspace) == 0


def test_spin_limit_timeout_reported_polling():
    """The bf16 forward on the deep-stack streams (hundreds of levels, a wait at each): with a
    one-poll limit some wait finds another workgroup not yet there and gives up, the kernels leave
    their loops and the call reports SLSTM_ETIMEOUT; the same buffers then run normally."""
    need_gpu()
    from paper_1904_03409_amd import stacklstm as s
    deep = wk.make("deep")
    wl = wk.custom(T=deep.T, B=deep.B, I=544, H=deep.H, seed=104, ops=deep.ops, wscale=0.08)
    r, rc = _run(wl, precision=1, spin_limit=1)
    assert rc == 7
    torch.cuda.synchronize()
    r2, rc2 = _run(wl, precision=1)
    assert rc2 == 0
    assert s.stacklstm_sync_status(r2.workspace) == 0
    r2.backward()
    torch.cuda.synchronize()
    assert s.stacklstm_sync_status(r2.workspace) == 0


def test_empty_T():
    need_gpu()
    wl = wk.custom(T=0, B=3, I=2, H=4, seed=0, ops=np.zeros((0, 3), np.int8))
    from paper_1904_03409_amd.stacklstm import DeviceRun
    r = DeviceRun.from_workload(wl)
    r.forward()
    r.backward()
    torch.cuda.synchronize()
    out = r.results()
    assert np.all(out["ptr"] == 0)
    for k in ("dW", "dU", "db", "dh0", "dc0"):
        assert np.all(out[k] == 0)


@pytest.mark.parametrize("precision", [0, 1])
def test_corrupted_top_reported(precision):
    """A producer table that is not the forward's (indices past their step, below -1) passed
    to stacklstm_bwd: every kernel still finishes (each bad index is replaced by -1 before any
    access), and the call returns SLSTM_EINDEX instead of OK. The same work space then runs a
    normal backward with status OK."""
    need_gpu()
    from paper_1904_03409_amd import stacklstm as s
    wl = wk.make("tiny")
    r, rc = _run(wl, precision=precision)
    assert rc == 0
    torch.cuda.synchronize()
    good = r.top.clone()
    bad = good.clone()
    bad[5:, 1] = 1000                 # past every step
    bad[9, 3] = -7                    # below the initial state's -1
    print(f"[gpu] corrupted top, tiny, precision={precision}", flush=True)
    rc = s.stacklstm_bwd(r.dims, r.x, r.ops, r.W, r.U, r.h0, r.c0, r.h_cell, r.c_cell, bad, r.workspace, r.dh_top,
                         r.dc_top, r.dx, r.dW, r.dU, r.db, r.dh0, r.dc0, check=False)
    assert rc == 8
    assert s.stacklstm_sync_status(r.workspace) == 8
    rc = s.stacklstm_bwd(r.dims, r.x, r.ops, r.W, r.U, r.h0, r.c0, r.h_cell, r.c_cell, good, r.workspace, r.dh_top,
                         r.dc_top, r.dx, r.dW, r.dU, r.db, r.dh0, r.dc0, check=False)
    assert rc == 0
    assert s.stacklstm_sync_status(r.workspace) == 0


def test_deferred_status():
    """Deferred calls return OK without a read-back; they give the same results as ordinary
    calls, keep the first error of any of them for stacklstm_sync_status, and an ordinary call
    resets it."""
    need_gpu()
    from paper_1904_03409_amd.stacklstm import DeviceRun, stacklstm_sync_status
    wl = wk.custom(T=12, B=40, I=8, H=32, seed=3)
    ref = DeviceRun.from_workload(wl)
    assert ref.forward(check=False) == 0 and ref.backward(check=False) == 0
    want = ref.results()
    r = DeviceRun.from_workload(wl)
    assert r.forward(check=False) == 0 and r.backward(check=False) == 0   # resets the error words
    r.dims.defer_status = 1
    for _ in range(2):
        assert r.forward(check=False) == 0 and r.backward(check=False) == 0
    torch.cuda.synchronize()
    assert stacklstm_sync_status(r.workspace) == 0
    got = r.results()
    for k in want:
        assert np.array_equal(want[k], got[k]), k
    # an invalid op in a deferred call, then valid deferred calls: still reported
    bad_ops = wl.ops.copy()
    bad_ops[4, 7] = 5
    rb = DeviceRun.from_workload(wk.custom(T=12, B=40, I=8, H=32, seed=3, ops=bad_ops))
    assert rb.forward(check=False) == 2                                      # ordinary call: its own status
    rb.dims.defer_status = 1
    assert rb.forward(check=False) == 0 and rb.backward(check=False) == 0
    rb.ops.copy_(torch.from_numpy(wl.ops).to(rb.ops.device))
    assert rb.forward(check=False) == 0 and rb.backward(check=False) == 0
    torch.cuda.synchronize()
    assert stacklstm_sync_status(rb.workspace) == 2
    rb.dims.defer_status = 0
    assert rb.forward(check=False) == 0                                      # resets: valid ops now
    assert stacklstm_sync_status(rb.workspace) == 0


def _bwd_code(r, ws):
    from paper_1904_03409_amd import stacklstm as s
    return s.stacklstm_bwd(r.dims, r.x, r.ops, r.W, r.U, r.h0, r.c0, r.h_cell, r.c_cell, r.top, ws, r.dh_top, r.dc_top,
                           r.dx, r.dW, r.dU, r.db, r.dh0, r.dc0, check=False)


@pytest.mark.parametrize("precision", [0, 1])
def test_backward_without_its_forward(precision):
    """A work space that holds no forward of the backward's sizes (never written, or by a forward of
    other sizes) gives SLSTM_EINDEX, also deferred; the kernels follow none of its indices. The forward
    and backward then run as usual."""
    need_gpu()
    from paper_1904_03409_amd import stacklstm as s
    from paper_1904_03409_amd.stacklstm import DeviceRun
    wl = wk.custom(T=33, B=7, I=12, H=40, seed=1, dc_top=True)
    r = DeviceRun.from_workload(wl, precision=precision)
    assert r.forward(check=False) == 0 and r.backward(check=False) == 0
    torch.cuda.synchronize()
    want = r.results()
    for fill in (0, 255):
        ws = torch.full_like(r.workspace, fill)
        print(f"[gpu] backward on a work space of {fill}, precision={precision}", flush=True)
        assert _bwd_code(r, ws) == 8
        assert s.stacklstm_sync_status(ws) == 8
    other = DeviceRun.from_workload(wk.custom(T=30, B=8, I=12, H=40, seed=2), precision=precision)
    ws = torch.zeros(max(r.workspace.numel(), other.workspace.numel()), dtype=torch.uint8, device="cuda")
    other.workspace = ws
    assert other.forward(check=False) == 0
    print(f"[gpu] backward after another forward, precision={precision}", flush=True)
    assert _bwd_code(r, ws) == 8
    r.workspace = ws
    assert r.forward(check=False) == 0
    other.dims.defer_status = 1
    assert _bwd_code(other, ws) == 0
    torch.cuda.synchronize()
    assert s.stacklstm_sync_status(ws) == 8
    assert r.forward(check=False) == 0 and r.backward(check=False) == 0
    torch.cuda.synchronize()
    got = r.results()
    for k in want:
        assert np.array_equal(got[k], want[k]), k
