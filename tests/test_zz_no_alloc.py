"""The allocation-free forward (stacklstm_fwd_static: static per-GPU work space) against the
forward on a caller work space (stacklstm_fwd): two calls in a row, the second on a smaller
problem, in both precisions. The outputs must be identical bit for bit (same kernels, same
arithmetic), which is within the parity bar of the forward itself; dims whose forward work
space exceeds the static array are rejected with SLSTM_EWORKSPACE."""
import numpy as np
import pytest
import torch

from paper_1904_03409_amd import workloads as wk
from tests.gpu_helpers import need_gpu

pytestmark = pytest.mark.gpu

OUTS = ("h_cell", "c_cell", "h_top", "c_top", "ptr", "top")


def _static_forward(run):
    from paper_1904_03409_amd.stacklstm import stacklstm_fwd_static
    out = {k: torch.full_like(getattr(run, k), -7 if k in ("ptr", "top") else float("nan")) for k in OUTS}
    rc = stacklstm_fwd_static(run.dims, run.x, run.ops, run.W, run.U, run.b, run.h0, run.c0, out["h_cell"],
                              out["c_cell"], out["h_top"], out["c_top"], out["ptr"], out["top"], check=False)
    torch.cuda.synchronize()
    return rc, {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("precision", [0, 1])
def test_static_forward_matches_forward(precision):
    need_gpu()
    from paper_1904_03409_amd.stacklstm import DeviceRun
    for wl in (wk.make("parser", precision=precision), wk.make("tiny", precision=precision)):
        print(f"[gpu] static forward {wl.name} T={wl.T} B={wl.B} I={wl.I} H={wl.H} prec={precision}", flush=True)
        run = DeviceRun.from_workload(wl, precision=precision, want_top=True)
        run.forward()
        torch.cuda.synchronize()
        ref = {k: getattr(run, k).cpu().numpy() for k in OUTS}
        rc, got = _static_forward(run)
        assert rc == 0
        for k in OUTS:
            assert np.array_equal(got[k], ref[k], equal_nan=True), (wl.name, k)


def test_static_forward_rejects_large_dims():
    need_gpu()
    from paper_1904_03409_amd import stacklstm as s
    # the large workload's forward work space (about 0.5 GB) exceeds the static array
    wl = wk.make("large")
    run = s.DeviceRun.from_workload(wl, want_top=True)
    rc, _ = _static_forward(run)
    assert rc == 4


PIECES = [
    # (T, B, I, H, precision): planes of x that take several ranges of columns (the last one short; rows of x
    # without 16-byte alignment), and of which not even 64 columns of all rows fit
    (100, 300, 2048, 16, 0), (100, 300, 2046, 16, 0), (100, 800, 2048, 16, 1), (100, 800, 2046, 16, 1),
    (700, 1000, 72, 4, 0),
]


@pytest.mark.parametrize("shape", PIECES)
def test_static_forward_in_pieces(shape):
    """Inputs whose operand planes have no room in the static array beside the rest: the projection goes on
    over ranges of their columns (and rows): the same outputs."""
    need_gpu()
    from paper_1904_03409_amd import stacklstm as s
    T, B, I, H, precision = shape
    print(f"[gpu] static forward in pieces {shape}", flush=True)
    wl = wk.custom(T=T, B=B, I=4, H=H, seed=I)
    g = torch.Generator(device="cuda")
    g.manual_seed(I)
    x = torch.randn(T, B, I, generator=g, device="cuda")
    W = torch.randn(I, 4 * H, generator=g, device="cuda") * 0.02
    x[3, 5, 10], x[3, 5, I - 1] = float("inf"), -float("inf")   # infinities of one step in two pieces: NaN or not
    x[9, 6, 7] = x[9, 6, I - 2] = float("inf")
    x[20, 7, I - 1] = float("inf")
    up = lambda a: torch.from_numpy(a).to("cuda")
    args = (x, up(wl.ops), W, up(wl.U), up(wl.b), up(wl.h0), up(wl.c0))
    dims = s.make_dims(T, B, I, H, precision)
    ws = torch.empty(s.stacklstm_workspace_bytes(dims), dtype=torch.uint8, device="cuda")
    outs = []
    for static in (False, True):
        out = [torch.full((T, B, H), float("nan"), device="cuda") for _ in range(4)]
        out += [torch.full((n, B), -7, dtype=torch.int32, device="cuda") for n in (T + 1, T)]
        rc = s.stacklstm_fwd_static(dims, *args, *out, check=False) if static else \
            s.stacklstm_fwd(dims, *args, *out, ws, check=False)
        assert rc == 0
        torch.cuda.synchronize()
        outs.append(out)
    planes = (3 if precision == 0 else 1) * T * B * I * 2
    assert planes > (256 << 20)
    for k, a, b in zip(OUTS, *outs):
        assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.nan_to_num(a), torch.nan_to_num(b)), k
