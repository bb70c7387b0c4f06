"""WH_GEMV_ROWS at the rates whose kernels differ in workgroup and LDS layout
(1024 lanes, 768, and 1024 with one workgroup a CU): the call gives the
oracle's y (1e-6 relative L2, the stated tolerance) whether the kernel takes
several block rows a group or keeps to one, and the context stays usable."""
import numpy as np
import pytest
import torch

import oracle
from paper_1902_08018_amd import synth, wh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rpg", [2, 4])
@pytest.mark.parametrize("rate", [8, 14, 16, 20, 24, 32])
def test_rows_per_group(monkeypatch, rate, rpg):
    monkeypatch.setenv("WH_GEMV_LANES", "64")
    monkeypatch.setenv("WH_GEMV_ROWS", str(rpg))
    rows, cols = 378, 1030  # 95 block rows: tiles of 16 or 12 groups, the last one partial
    s = oracle.encode(synth.matrix(synth.MatrixSpec(rows, cols, 32, 8.0, seed=91)), rate)
    u = synth.uniform(cols, seed=92)
    ref = oracle.gemv_fp64(s, rows, cols, rate, u)
    ud = torch.from_numpy(u).cuda()
    ctx = wh.wh_create(0, 0)
    try:
        mat = wh.wh_load_compressed(ctx, rows, cols, wh.WH_FMT_ZFP_FIXED_RATE, rate, s)
        for rb, re in [(0, rows), (3, rows - 2)]:
            for flags in (wh.WH_ACC_DEFAULT, wh.WH_ACC_TWOSUM, wh.WH_PAPER_MP):
                y = torch.full((re - rb + 2,), -7.0, device="cuda")
                wh.wh_gemv(ctx, mat, ud, y, rb, re, flags)
                torch.cuda.synchronize()
                got = y.cpu().numpy()
                assert np.linalg.norm(got[:re - rb] - ref[rb:re]) <= 1e-6 * np.linalg.norm(ref[rb:re]), (rb, re, flags)
                assert np.all(got[re - rb:] == -7.0)
    finally:
        wh.wh_destroy(ctx)
