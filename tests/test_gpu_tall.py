"""GPU tests of tall, narrow matrices: many tiles of block rows and few steps
of block columns, where the multi-RHS planner's slab count changes most with
the number of right-hand sides (40000 x 256 at rate 8: two slabs for 8, one
for 16).

  serving   requests of every bucket of right-hand sides against the FP64
            product with the decoded matrix, within 1e-6 relative L2 (the
            stated tolerance of FP32 right-hand sides)
  batched   the same counts through wh_gemv_batched, FP32 1e-6 and BF16 2e-3
"""
import time

import numpy as np
import pytest
import torch

import oracle
from paper_1902_08018_amd import synth, wh

pytestmark = pytest.mark.gpu

SHAPES = [(40000, 256, 8), (28085, 106, 20)]


def case(rows, cols, rate):
    s = oracle.encode(synth.matrix(synth.MatrixSpec(rows, cols, 32, 8.0, seed=71)), rate)
    return s, oracle.decode(s, rows, cols, rate).astype(np.float64)


def worst(Y, U, ref_M):
    ref = U.astype(np.float64) @ ref_M.T
    return float((np.linalg.norm(Y - ref, axis=1) / np.linalg.norm(ref, axis=1)).max())


@pytest.mark.parametrize("rows,cols,rate", SHAPES)
def test_serving(rows, cols, rate):
    s, ref_M = case(rows, cols, rate)
    ctx = wh.wh_create(0, 256 << 20)
    try:
        mat = wh.wh_load_compressed(ctx, rows, cols, wh.WH_FMT_ZFP_FIXED_RATE, rate, s)
        for k in (8, 2, 4, 1, 16, 32, 48, 64):
            U = synth.uniform(k * cols, seed=k).reshape(k, cols)
            Ud, Y = torch.from_numpy(U).cuda(), torch.full((k, rows), float("nan"), device="cuda")
            torch.cuda.synchronize()
            t = wh.wh_submit(ctx, wh.wh_request(mat=mat, U=Ud.data_ptr(), u_on_device=1, k=k, Y=Y.data_ptr(),
                                                y_on_device=1, deadline_ns=10 ** 9, arrival_ns=0))
            end = time.monotonic() + 30.0
            while True:
                st, r = wh.wh_poll(ctx, t)
                if st == wh.WH_OK:
                    break
                assert time.monotonic() < end, "the request did not complete"
                time.sleep(0.0002)
            torch.cuda.synchronize()
            assert r.status == wh.WH_OK
            assert worst(Y.cpu().numpy(), U, ref_M) <= 1e-6, k
    finally:
        wh.wh_destroy(ctx)


@pytest.mark.parametrize("rows,cols,rate", SHAPES)
@pytest.mark.parametrize("dtype,tol", [(torch.float32, 1e-6), (torch.bfloat16, 2e-3)])
def test_batched(gpu_ctx, rows, cols, rate, dtype, tol):
    s, ref_M = case(rows, cols, rate)
    mat = wh.wh_load_compressed(gpu_ctx, rows, cols, wh.WH_FMT_ZFP_FIXED_RATE, rate, s)
    for k in (2, 8, 16, 20, 64):
        U = torch.from_numpy(synth.uniform(k * cols, seed=100 + k).reshape(k, cols)).to(dtype)
        Y = torch.full((k, rows), float("nan"), device="cuda")
        wh.wh_gemv_batched(gpu_ctx, mat, U.cuda(), Y)
        torch.cuda.synchronize()
        assert worst(Y.cpu().numpy(), U.float().numpy(), ref_M) <= tol, k
    wh.wh_unload(gpu_ctx, mat)
