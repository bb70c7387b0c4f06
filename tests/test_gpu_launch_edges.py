"""GPU parity at the edges of the kernels' own limits.

  slab vectors   the fused GEMV holds B^T u of a slab in LDS up to a limit
                 that depends on the rate, and makes it per block above:
                 slabs on both sides of it, within 1e-6 relative L2 of the
                 FP64 oracle (the stated tolerance of every mode)
  batched tiles  the multi-RHS kernels' tiles lie in the staged blocks' place
                 as far as a block's words reach: every count of words, more
                 than one step of block columns, the last one partial, on
                 every math (1e-6 FP32, 2e-3 BF16: the stated tolerances)
  thermal rows   rows of 0 to 11 entries (the kernel takes five at a time),
                 columns out of range and infinities where nothing reads
  decode         workgroups of 16, 12 and 8 waves (by rate), the last one's
                 waves partly without a patch of blocks: exact
  encode         a stream that starts on 4 bytes but not on 16; more blocks
                 than one sweep of the grid
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1902_08018_amd import synth, wh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [wh.WH_ACC_DEFAULT, wh.WH_ACC_TWOSUM, wh.WH_PAPER_MP])
@pytest.mark.parametrize("rate", [2, 4, 8, 12, 16, 20, 24, 32])
def test_slab_vector_limits(monkeypatch, rate, flags):
    rows, cols = 61, 4 * 400 + 2  # 401 block columns, the last one partial
    spec = synth.MatrixSpec(rows, cols, 48, 8.0, seed=61)
    s = oracle.encode(synth.matrix(spec), rate)
    u = synth.u_vector(spec)
    ref = oracle.gemv_fp64(s, rows, cols, rate, u)
    ud = torch.from_numpy(u).cuda()
    monkeypatch.setenv("WH_GEMV_LANES", "8")
    for slabs in (1, 2, 4, 7):  # 408, 208, 104 and 64 block columns
        monkeypatch.setenv("WH_GEMV_SLABS", str(slabs))
        ctx = wh.wh_create(0, 0)
        try:
            mat = wh.wh_load_compressed(ctx, rows, cols, wh.WH_FMT_ZFP_FIXED_RATE, rate, s)
            y = torch.full((rows,), float("nan"), device="cuda")
            wh.wh_gemv(ctx, mat, ud, y, 0, rows, flags)
            torch.cuda.synchronize()
            err = np.linalg.norm(y.cpu().numpy() - ref) / np.linalg.norm(ref)
            assert err <= 1e-6, (slabs, err)
        finally:
            wh.wh_destroy(ctx)


@pytest.mark.parametrize("k,dtype", [(3, "f32"), (16, "f32"), (20, "f32"), (64, "f32"), (16, "bf16"), (40, "bf16")])
@pytest.mark.parametrize("rate", [2, 4, 6, 8, 10, 12, 14, 16, 20, 24, 32])
def test_batched_tile_places(gpu_ctx, rate, k, dtype):
    rows, cols = 131, 4 * 37 + 2  # 33 block rows; 38 block columns, 3 steps
    spec = synth.MatrixSpec(rows, cols, 40, 8.0, seed=64)
    s = oracle.encode(synth.matrix(spec), rate)
    Mhat = oracle.decode(s, rows, cols, rate).astype(np.float64)
    U = torch.from_numpy(synth.u_batch(spec, k)).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    ref = U.double().numpy() @ Mhat.T
    mat = wh.wh_load_compressed(gpu_ctx, rows, cols, wh.WH_FMT_ZFP_FIXED_RATE, rate, s)
    Y = torch.full((k, rows), float("nan"), device="cuda")
    wh.wh_gemv_batched(gpu_ctx, mat, U.cuda(), Y)
    torch.cuda.synchronize()
    err = np.linalg.norm(Y.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() <= (2e-3 if dtype == "bf16" else 1e-6), err.max()
    wh.wh_unload(gpu_ctx, mat)


@pytest.mark.parametrize("rate", [16, 20, 24, 32])
def test_decode_workgroups(gpu_ctx, rate):
    rows, cols = 4 * 8 * 5 - 2, 4 * 8 * 5 - 4  # 5 x 5 patches of 8 x 8 blocks
    s = oracle.encode(synth.matrix(synth.MatrixSpec(rows, cols, 16, 4.0, seed=65)), rate)
    mat = wh.wh_load_compressed(gpu_ctx, rows, cols, wh.WH_FMT_ZFP_FIXED_RATE, rate, s)
    out = torch.full((rows, cols), float("nan"), device="cuda")
    wh.wh_decode(gpu_ctx, mat, out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), oracle.decode(s, rows, cols, rate))
    wh.wh_unload(gpu_ctx, mat)


@pytest.mark.parametrize("rate", [8, 16, 6])
def test_encode_into_word_aligned_stream(gpu_ctx, rate):
    rows, cols = 37, 150
    M = synth.matrix(synth.MatrixSpec(rows, cols, 16, 4.0, seed=62))
    want = oracle.encode(M, rate)
    buf = torch.zeros(want.size + 8, dtype=torch.uint8, device="cuda")
    wh.wh_encode(gpu_ctx, torch.from_numpy(M).cuda(), rate, buf[4:4 + want.size])
    torch.cuda.synchronize()
    got = buf.cpu().numpy()
    assert np.array_equal(got[4:4 + want.size], want)
    assert not got[:4].any() and not got[4 + want.size:].any()


def test_encode_more_blocks_than_one_sweep(gpu_ctx):
    # 65536 workgroups of 256 lanes are one sweep: 16,777,216 blocks.  The
    # parts are encoded by launches below that, so a block's code must not
    # depend on the sweep it is in
    rows, cols, rate, cut = 4 * 1025, 4 * 16385, 2, 4 * 512
    M = torch.rand(rows, cols, device="cuda", generator=torch.Generator("cuda").manual_seed(5))
    whole = torch.empty(wh.stream_bytes(rows, cols, rate), dtype=torch.uint8, device="cuda")
    wh.wh_encode(gpu_ctx, M, rate, whole)
    at = wh.stream_bytes(cut, cols, rate)
    parts = torch.empty_like(whole)
    wh.wh_encode(gpu_ctx, M[:cut], rate, parts[:at])
    wh.wh_encode(gpu_ctx, M[cut:], rate, parts[at:])
    torch.cuda.synchronize()
    assert torch.equal(whole, parts)


@pytest.mark.parametrize("n", [1, 511, 512, 513, 1500])
def test_thermal_row_lengths(gpu_ctx, n):
    rng = np.random.default_rng(n)
    counts = np.arange(n) % 12
    row_ptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.uint32)
    nnz = int(row_ptr[-1])
    col = rng.integers(0, n, nnz).astype(np.uint32)
    val = rng.uniform(-1, 1, nnz).astype(np.float32)
    bad = rng.random(nnz) < 0.05
    col[bad] = n + rng.integers(0, 5, int(bad.sum()))  # skipped
    if nnz:
        col[(col == 0)] = min(1, n - 1)
    b = rng.uniform(0, 1, n).astype(np.float32)
    T = rng.uniform(19, 21, n).astype(np.float32)
    u = rng.uniform(0, 1, n).astype(np.float32)
    if n > 1:
        T[0] = np.inf  # no entry reads cell 0
    want = np.empty(n, np.float32)
    for i in range(n):
        s = 0.0  # every product is exact in FP64, the sum rounds as the kernel's
        for p in range(int(row_ptr[i]), int(row_ptr[i + 1])):
            if col[p] < n:
                s += float(val[p]) * float(T[col[p]])
        want[i] = np.float32(s + float(b[i]) * float(u[i]))
    sysm = wh.ThermalSystem(row_ptr, col, val, b)
    out = torch.empty(n, device="cuda")
    wh.wh_thermal_step(gpu_ctx, sysm, torch.from_numpy(T).cuda(), torch.from_numpy(u).cuda(), out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), want)
