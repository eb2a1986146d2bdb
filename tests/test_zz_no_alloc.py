"""hpsgd_local_step_all_static: the entry point that allocates nothing, through the C ABI,
against hpsgd_local_step_all on the same inputs."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2009_02701_amd import binding as hb
from paper_2009_02701_amd import harness
from paper_2009_02701_amd import workloads as wl

from parity import TOL_BF16, TOL_FP32, workload

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

BIG = wl.scaled(wl.CONFIGS["gru_lm"], vocab=264, embed=72, hidden=160, seq_len=19, batch=16, K=2)   # 17 MiB, bf16
SMALL = wl.CONFIGS["tiny_gru"]                                                                     # 0.24 MiB, fp32


def _both_entry_points(cfg, steps=2, fits=True):
    """`steps` local steps through each entry point, raw C-ABI calls; returns (replicas, losses) of both."""
    init, shards, orders, _ = workload(cfg)
    tr = harness.Trainer(cfg, init, shards, orders, device=DEV)
    lib, ctx = hb.load_library(), tr.ctx
    assert (ctx.workspace_bytes <= (32 << 20)) == fits
    tr.sync_all(0)
    tr.sync_all(1)
    torch.cuda.synchronize()
    st = torch.cuda.current_stream()
    out = []
    for gen, static in ((0, False), (1, True)):
        R = tr.R[gen]
        loss = torch.zeros(steps, cfg["K"], device=DEV)
        for i in range(steps):
            tr.gather(i)
            args = [ctx._h, C.c_void_p(R.data_ptr()), C.c_void_p(R.data_ptr()), C.c_size_t(R.stride(0)),
                    C.c_void_p(tr.xb.data_ptr()), C.c_void_p(tr.yb.data_ptr()), C.c_float(cfg["lr"]),
                    C.c_void_p(loss[i].data_ptr())]
            if static:
                rc = lib.hpsgd_local_step_all_static(*args, C.c_void_p(st.cuda_stream))
            else:
                rc = lib.hpsgd_local_step_all(*args, ctx._ws_ptr(tr.ws[0]), C.c_void_p(st.cuda_stream))
            assert rc == 0, rc
        torch.cuda.synchronize()
        out.append((R[:, :tr.P].clone(), loss.clone()))
    return out


def test_static_workspace_entry_point_twice_in_a_row_second_call_smaller():
    """Two uses in a row, the second with a smaller model (the array then still holds the first
    one's contents): each gives the bits of hpsgd_local_step_all, losses included."""
    for cfg in (BIG, SMALL, BIG):
        (r0, l0), (r1, l1) = _both_entry_points(cfg)
        assert torch.isfinite(r0).all() and torch.isfinite(l0).all()
        assert torch.equal(r0, r1), cfg
        assert torch.equal(l0, l1), cfg


@pytest.mark.parametrize("base,sizes,tol", [
    ("gru_lm", dict(prec="bf16", layers=1, vocab=408, embed=2, hidden=196, seq_len=27, batch=2, K=7), TOL_BF16),
    ("gru_cls", dict(prec="fp32", layers=2, input=3, hidden=139, seq_len=13, batch=124, classes=14, K=2), TOL_FP32),
])
def test_static_workspace_entry_point_in_the_smaller_layout(base, sizes, tol):
    """Models that fit the array only without padding and partial sums: the change of every parameter against the
    usual layout's, at the tolerance of one step (the two differ in the order of their sums)."""
    cfg = wl.scaled(wl.CONFIGS[base], lr=8.0, **sizes)
    (r0, l0), (r1, l1) = _both_entry_points(cfg, steps=1, fits=False)
    start = torch.from_numpy(hb.Context(cfg).flatten(wl.init_params(cfg))).to(DEV)
    assert float((r0 - r1).abs().max()) <= tol * float((r0 - start).abs().max())
    assert torch.allclose(l0, l1, rtol=tol, atol=0)


def test_static_workspace_entry_point_rejects_models_beyond_its_array():
    cfg = wl.CONFIGS["gru_cls"]   # 276 MiB of workspace
    ctx = hb.Context(cfg)
    lib = hb.load_library()
    R = torch.zeros(cfg["K"], ctx.stride, device=DEV)
    x = torch.zeros(cfg["K"], cfg["seq_len"], cfg["batch"], cfg["input"], device=DEV)
    y = torch.zeros(cfg["K"], cfg["batch"], dtype=torch.int32, device=DEV)
    rc = lib.hpsgd_local_step_all_static(ctx._h, C.c_void_p(R.data_ptr()), C.c_void_p(R.data_ptr()),
                                         C.c_size_t(R.stride(0)), C.c_void_p(x.data_ptr()), C.c_void_p(y.data_ptr()),
                                         C.c_float(0.1), None, None)
    assert rc == 5  # HPSGD_EWORKSPACE
    assert float(R.abs().sum()) == 0.0


@pytest.mark.parametrize("base,sizes,tol", [
    ("gru_cls", dict(layers=2, input=40, hidden=100, batch=20, seq_len=44, classes=7, K=4), TOL_FP32),
    ("gru_lm", dict(prec="fp32", layers=2, vocab=150, embed=40, hidden=100, batch=20, seq_len=35, K=4), TOL_FP32),
    ("gru_lm", dict(prec="bf16", layers=2, vocab=203, embed=24, hidden=128, batch=16, seq_len=22, K=4), TOL_BF16),
])
def test_static_workspace_entry_point_with_the_layers_one_after_the_other(base, sizes, tol):
    """Two narrow layers that fit the array only without the second buffers of their joint launches keep all else of the
    usual layout: a recurrence launch per layer where that has one for both."""
    cfg = wl.scaled(wl.CONFIGS[base], lr=8.0, **sizes)
    (r0, l0), (r1, l1) = _both_entry_points(cfg, steps=1, fits=False)
    start = torch.from_numpy(hb.Context(cfg).flatten(wl.init_params(cfg))).to(DEV)
    assert float((r0 - r1).abs().max()) <= tol * float((r0 - start).abs().max())
    assert torch.allclose(l0, l1, rtol=tol, atol=0)
    init, shards, orders, _ = workload(cfg)
    tr = harness.Trainer(cfg, init, shards, orders, device=DEV)
    tr.gather(0)
    tr.sync_all(0)
    fwd = tr.ctx.role_names().index("gemm_recurrent_fwd")
    tr.ctx.timer_enable([fwd])
    for joint in (True, False):
        if joint:
            tr.local_step(0, cfg["lr"])
        else:
            tr.ctx.local_step_all_static(tr.R[0], tr.R[0], tr.xb, tr.yb, cfg["lr"], tr.loss)
        torch.cuda.synchronize()
        assert tr.ctx.timer_read(fwd)[0] == (1 if joint else 2)
        assert tr.ctx.recurrence_info()[0] == 2
    tr.ctx.timer_enable([])
