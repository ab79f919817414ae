"""Every variant of the recurrent kernels, and every kind of group, runs against the oracle.

The compiled width (K chunks) and the rows per pass follow from H and the precision; the number of
groups, the elements of a group and whether the groups are even follow from B as well. The test
sweeps a grid of (precision, H, B), asks the planner for each, and keeps the first grid point of each
class: (precision, width compiled and in use, how state rows lie in cache lines; groups of one element,
of one pass, of several passes at the first level; even or uneven groups). Each runs once (short T)
against the oracle: traces of every column, floats of sampled columns, and the weight gradients of
a second backward whose upstream gradient is zero outside the sampled columns."""
import numpy as np
import pytest

from paper_1904_03409_amd import workloads as wk
from tests.gpu_helpers import TOL, need_gpu
from tests.torch_ref import normwise

pytestmark = pytest.mark.gpu

GRID_H = {0: [1, 40, 64, 100, 128, 200, 252, 256, 300, 508, 512],
          1: [1, 64, 100, 128, 200, 256, 300, 384, 504, 512, 520, 768, 1020, 1024]}
GRID_B = [1, 17, 64, 100, 128, 129, 200, 256, 257, 300, 384, 400, 512, 513, 600, 700, 768, 769, 900, 1000, 1024, 1500, 3000, 5000, 5120]
KEYS = ("fwd_tiles", "k_chunk_cap")


def reachable_variants():
    """{variant: (precision, H, B) of the first grid point that reaches it}."""
    from paper_1904_03409_amd.stacklstm import StackLSTMError, make_dims, stacklstm_plan
    out = {}
    for prec, hs in GRID_H.items():
        for H in hs:
            for B in GRID_B:
                try:
                    plan = stacklstm_plan(make_dims(8, B, 8, H, prec, 0))
                except StackLSTMError:
                    continue
                key = (prec,) + tuple(plan[k] for k in KEYS) + row_class(prec, H, plan) + group_class(B, plan)
                out.setdefault(key, (prec, H, B))
    return out


def row_class(prec, H, plan):
    """How the kernels copy state rows for this H: every K chunk in use, rows of whole 1 KB
    segments, rows of whole 128-byte lines (no line shared by two rows). (A plane has 2 bytes a unit.)"""
    nbytes = H * 2
    return (int(plan["k_chunks"] == plan["k_chunk_cap"]), int(nbytes % 1024 == 0), int(nbytes % 128 == 0))


def group_class(B, plan):
    """Groups of one element, of one pass of states, of more; whether some group has an element less."""
    rows = plan["rows_per_group"]
    assert rows == -(-B // plan["groups"]) and plan["groups"] <= B
    return (1 if rows == 1 else 2 if rows <= 16 * plan["fwd_tiles"] else 3, int(B % plan["groups"] != 0))


# shapes run whatever variant they map to: the largest batches at the largest hidden sizes
EXTRA = [(0, 512, 1024), (1, 512, 1024), (1, 1020, 1024), (1, 1024, 1024)]


def _sampled_parity(oracle_mod, wl, precision, ncols=3):
    import torch
    from paper_1904_03409_amd.stacklstm import DeviceRun
    sel = np.unique(np.linspace(0, wl.B - 1, ncols).astype(np.int32))
    run = DeviceRun.from_workload(wl, precision=precision)
    run.forward()
    run.backward()
    torch.cuda.synchronize()
    got = run.results()
    ref = oracle_mod.run(wl, sel=sel, bf16=precision == 1)
    ptr = np.vstack([np.zeros((1, wl.B), np.int64), np.cumsum(wl.ops.astype(np.int64), axis=0)])
    assert np.array_equal(got["ptr"], ptr)
    assert np.array_equal(got["top"][:, sel], ref["top"])
    errs = {k: normwise(got[k][:, sel], ref[k]) for k in ("h_top", "c_top", "dx")}
    errs.update({k: normwise(got[k][sel], ref[k]) for k in ("dh0", "dc0")})
    push = wl.ops[:, sel] == 1
    errs["h_cell_push"] = normwise(got["h_cell"][:, sel][push], ref["h_cell"][push])
    assert np.all(got["dx"][:, sel][~push] == 0)
    mask = np.zeros(wl.B, np.float32)
    mask[sel] = 1.0
    run.dh_top.copy_(torch.from_numpy(wl.dh_top * mask[None, :, None]).to(run.dh_top.device))
    run.dc_top.copy_(torch.from_numpy(wl.dc_top * mask[None, :, None]).to(run.dc_top.device))
    run.backward()
    torch.cuda.synchronize()
    gw = run.results()
    errs.update({k: normwise(gw[k], ref[k]) for k in ("dW", "dU", "db")})
    return errs


def test_every_planner_variant(oracle_mod):
    need_gpu()
    variants = reachable_variants()
    print(f"[gpu] {len(variants)} variants: precision, fwd tiles, K-chunk cap, all chunks used, 1 KB rows, "
          f"128-byte rows, group size class, uneven groups -> first (precision, H, B)", flush=True)
    for prec, caps in ((0, {2, 4, 8, 16}), (1, {2, 4, 8, 12, 16, 24, 32})):
        assert {k[2] for k in variants if k[0] == prec} == caps
        for cap in caps:                                   # every width: one element, one pass and several
            assert {k[6] for k in variants if k[0] == prec and k[2] == cap} == {1, 2, 3}, (prec, cap)
    failures = {}
    cases = sorted(variants.items()) + [(("extra",), s) for s in EXTRA]
    for key, (prec, H, B) in cases:
        T = 10
        wl = wk.custom(T=T, B=B, I=24, H=H, seed=1000 + H + B, wscale=0.3, random_state=True, dc_top=True)
        print(f"[gpu] variant {key} at H={H} B={B} T={T}", flush=True)
        errs = _sampled_parity(oracle_mod, wl, prec)
        bad = {k: v for k, v in errs.items() if not v <= TOL[prec]}
        print(f"[gpu]   max err {max(errs.values()):.2e}" + (f" FAILED {bad}" if bad else ""), flush=True)
        if bad:
            failures[key] = bad
    assert not failures, failures
