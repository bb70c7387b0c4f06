"""The thermal step on both sides of the size at which its workgroups widen
from 64 to 512 lanes (a workgroup of 512 for every CU), rows of 0 to 11
entries: every product is exact in FP64 and a row's sum has the kernel's order,
so the results are equal."""
import numpy as np
import pytest
import torch

from paper_1902_08018_amd import wh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("off", [-1, 0, 65])
def test_around_the_wider_workgroups(gpu_ctx, off):
    n = 512 * torch.cuda.get_device_properties(0).multi_processor_count + off
    rng = np.random.default_rng(n)
    counts = np.arange(n) % 12
    row_ptr = np.concatenate([[0], np.cumsum(counts)])
    rows = np.repeat(np.arange(n), counts)
    col = np.clip(rows + rng.integers(-700, 701, rows.size), 0, n - 1)
    val = rng.uniform(-1, 1, rows.size).astype(np.float32)
    b = rng.uniform(0, 1, n).astype(np.float32)
    T = rng.uniform(19, 21, n).astype(np.float32)
    U = rng.uniform(0, 1, (3, n)).astype(np.float32)
    want = T
    for k in range(3):
        s = np.zeros(n)
        for e in range(11):  # entry e of every row that has one
            has = counts > e
            p = row_ptr[:-1][has] + e
            s[has] += val[p].astype(np.float64) * want[col[p]].astype(np.float64)
        want = (s + b.astype(np.float64) * U[k].astype(np.float64)).astype(np.float32)
    sysm = wh.ThermalSystem(row_ptr.astype(np.uint32), col.astype(np.uint32), val, b)
    Td, Ud = torch.from_numpy(T).cuda(), torch.from_numpy(U).cuda()
    step = torch.empty_like(Td)
    wh.wh_thermal_step(gpu_ctx, sysm, Td, Ud[0], step)
    wh.wh_thermal_run(gpu_ctx, sysm, Td, Ud, torch.empty_like(Td))
    torch.cuda.synchronize()
    assert np.array_equal(Td.cpu().numpy(), want)
    s0 = np.zeros(n)
    np.add.at(s0, rows, val.astype(np.float64) * T[col].astype(np.float64))
    assert np.allclose(step.cpu().numpy(), s0 + b.astype(np.float64) * U[0], rtol=2.0 ** -23, atol=2.0 ** -20)
