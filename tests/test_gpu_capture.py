"""Graph capture of the fused GEMV whose plan has one column slab.

  forced    WH_GEMV_SLABS=1 keeps the call from the context's workspace: it is
            captured, and every replay equals the eager call
  by cost   256 x 1024 has one slab by the planner's cost but several by the
            rule that decides about capture: wh_gemv refuses, wh_gemv_noalloc
            is captured

A context can be made while a capture is under way, on this thread or another.
"""
import threading

import numpy as np
import pytest
import torch

import oracle
from paper_1902_08018_amd import synth, wh

pytestmark = pytest.mark.gpu


def replays_equal_eager(ctx, call, rows, cols):
    u, y = torch.empty(cols, device="cuda"), torch.empty(rows, device="cuda")
    us = [torch.from_numpy(synth.uniform(cols, seed=s)).cuda() for s in (1, 2, 3)]
    u.copy_(us[0])
    call(u, y)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call(u, y)
    for rep in range(6):
        u.copy_(us[rep % 3])
        g.replay()
        torch.cuda.synchronize()
        got = y.cpu().numpy().copy()
        eager = torch.empty_like(y)
        call(u, eager)
        torch.cuda.synchronize()
        assert np.array_equal(got.view(np.uint32), eager.cpu().numpy().view(np.uint32)), rep


@pytest.mark.parametrize("rows,cols,rate", [(512, 8192, 8), (256, 1024, 16)])
def test_one_forced_slab_is_captured(monkeypatch, rows, cols, rate):
    monkeypatch.setenv("WH_GEMV_SLABS", "1")
    ctx = wh.wh_create(0, 0)
    try:
        s = oracle.encode(synth.matrix(synth.MatrixSpec(rows, cols, 32, 8.0, seed=81)), rate)
        mat = wh.wh_load_compressed(ctx, rows, cols, wh.WH_FMT_ZFP_FIXED_RATE, rate, s)
        h = torch.empty(s.size, dtype=torch.uint8, pin_memory=True)
        h.copy_(torch.from_numpy(s))
        replays_equal_eager(ctx, lambda u, y: wh.wh_gemv(ctx, mat, u, y, 0, rows), rows, cols)
        replays_equal_eager(ctx, lambda u, y: wh.wh_gemv_host(ctx, h, rows, cols, rate, u, y,
                                                              flags=wh.WH_HOST_DIRECT), rows, cols)
    finally:
        wh.wh_destroy(ctx)


def test_one_slab_by_cost(gpu_ctx):
    rows, cols, rate = 256, 1024, 16
    assert wh.wh_gemv_plan_info(rows, cols, 0, rows, rate=rate)["nslab"] == 1
    s = oracle.encode(synth.matrix(synth.MatrixSpec(rows, cols, 32, 8.0, seed=82)), rate)
    mat = wh.wh_load_compressed(gpu_ctx, rows, cols, wh.WH_FMT_ZFP_FIXED_RATE, rate, s)
    replays_equal_eager(gpu_ctx, lambda u, y: wh.wh_gemv_noalloc(gpu_ctx, mat, u, y, 0, rows), rows, cols)
    u, y = torch.ones(cols, device="cuda"), torch.empty(rows, device="cuda")
    refused = None
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        try:
            wh.wh_gemv(gpu_ctx, mat, u, y, 0, rows)
        except wh.WhError as e:
            refused = e.status
        y.zero_()
    assert refused == wh.WH_ERR_INVALID
    wh.wh_unload(gpu_ctx, mat)


@pytest.mark.parametrize("other_thread", [False, True])
def test_create_during_a_capture(gpu_ctx, other_thread):
    x = torch.zeros(1000, device="cuda")
    made = []

    def create():
        made.append(wh.wh_create(0, 0))

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        x.add_(1.0)
        if other_thread:
            t = threading.Thread(target=create)
            t.start()
            t.join()
        else:
            create()
        x.add_(1.0)
    for rep in range(4):
        g.replay()
        torch.cuda.synchronize()
        assert torch.all(x == 2.0 * (rep + 1))
    # the context's workspace is usable: a product that splits its columns
    rows, cols, rate = 512, 8192, 8
    s = oracle.encode(synth.matrix(synth.MatrixSpec(rows, cols, 32, 8.0, seed=83)), rate)
    mat = wh.wh_load_compressed(made[0], rows, cols, wh.WH_FMT_ZFP_FIXED_RATE, rate, s)
    u = synth.uniform(cols, seed=84)
    y = torch.empty(rows, device="cuda")
    wh.wh_gemv(made[0], mat, torch.from_numpy(u).cuda(), y, 0, rows)
    torch.cuda.synchronize()
    ref = oracle.gemv_fp64(s, rows, cols, rate, u)
    assert np.linalg.norm(y.cpu().numpy() - ref) <= 1e-6 * np.linalg.norm(ref)
    wh.wh_destroy(made[0])
