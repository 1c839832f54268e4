"""Calls of one kernel with half a column tile to a workgroup (up to 16 tokens) against the separate calls, bit for bit:
sums of one pair of k-tiles and of several (waves without one, batches that are full, cut and empty), numbers of columns on
both sides of half and whole tiles, every number of chunks of X per thread, W with and without 16-bit rows, and outlier
buffers on both sides of the slots that are fetched ahead."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_out_close, bits, through
from paper_2208_07339_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s,h,o,n", [
    (1, 8, 1, 1), (1, 64, 16, 1), (2, 130, 17, 2), (16, 128, 31, 2), (3, 1000, 32, 3), (16, 512, 2033, 5), (13, 1024, 48, 20),
    (1, 8192, 1030, 7), (1, 5120, 20480, 7), (1, 8320, 8192, 9), (2, 8192, 12288, 7), (1, 32768, 100, 4), (8, 4096, 4090, 6),
    (5, 6000, 513, 40), (9, 1801, 4100, 35)])
@pytest.mark.parametrize("rows16", [True, False])
def test_half_tiles_against_the_separate_calls(s, h, o, n, rows16):
    import torch

    import paper_2208_07339_amd as L
    cap = 64 if n > 32 else 32
    d = wl.make_custom(s, h, o, min(n, h // 4), seed=s + 3 * h + o)
    X, W = d["X"], d["W"]
    Xd, Wd = (torch.from_numpy(a.view(np.int16)).cuda().view(torch.float16) for a in (X, W))
    ws = L.Workspace.allocate(s, h, o, cap)
    qw = L.quantize_weight(Wd, ws)
    if not rows16:
        qw.W = None
    outl = L.Outliers(*(torch.full((k,), -7, dtype=torch.int32, device="cuda") for k in (cap, 1, 1)), cap)
    rows = L.QuantizedRows(torch.full((L.xq_bytes(s, h),), 99, dtype=torch.int8, device="cuda"),
                           torch.full((s,), 7.0, dtype=torch.float16, device="cuda"),
                           torch.full((s, L.opad(cap)), 7.0, dtype=torch.float16, device="cuda"), s, h)
    out = torch.full((s, o), 3.0, dtype=torch.float16, device="cuda")
    L.linear(Xd, qw, 6.0, outl, rows, ws, out)
    outl2 = L.find_outliers(Xd, 6.0, cap, ws)
    rows2 = L.quantize_rows(Xd, outl2)
    out2 = L.matmul(rows2, outl2, qw, ws)
    k = int(outl2.count.item())
    assert int(outl.count.item()) == k and int(outl.status.item()) == int(outl2.status.item())
    assert outl.idx[:k].cpu().tolist() == outl2.idx[:k].cpu().tolist() == oracle.find_outliers(X, 6.0)[:cap].tolist()
    for a, b in ((rows.Xq, rows2.Xq), (rows.cx, rows2.cx), (rows.Xo, rows2.Xo), (out, out2)):
        assert np.array_equal(bits(a.cpu().numpy().ravel()) if a.dtype == torch.float16 else a.cpu().numpy(),
                              bits(b.cpu().numpy().ravel()) if b.dtype == torch.float16 else b.cpu().numpy())
    if rows16:
        assert_out_close(out.cpu().numpy(), oracle.linear(X, W, 6.0)["Out"])


@pytest.mark.parametrize("zeropoint", [False, True])
@pytest.mark.parametrize("cap,n", [(64, 33), (64, 64), (256, 97), (250, 250)])
@pytest.mark.parametrize("s,h,o", [(1, 5000, 513), (9, 2000, 2049), (16, 4096, 1000), (17, 2048, 1030), (32, 700, 2016)])
def test_columns_past_the_32nd_with_k_split_over_the_waves(s, h, o, cap, n, zeropoint):
    """Up to 32 tokens, against the weight-streaming kernel, which adds up in the same order: the same bits."""
    import torch

    import paper_2208_07339_amd as L
    d = wl.make_custom(s, h, o, n, seed=s + h + n)
    Xd, Wd = (torch.from_numpy(a.view(np.int16)).cuda().view(torch.float16) for a in (d["X"], d["W"]))
    ws = L.Workspace.allocate(s, h, o, cap)
    outl = L.find_outliers(Xd, 6.0, cap, ws)
    assert int(outl.count.item()) > 32
    qw, rows = (L.zp_quantize_weight(Wd, ws), L.zp_quantize_rows(Xd, outl)) if zeropoint else (L.quantize_weight(Wd, ws), L.quantize_rows(Xd, outl))
    product = L.zp_matmul if zeropoint else L.matmul
    assert L.debug_kernel_for(s, h, o, zeropoint) >= 2
    out = product(rows, outl, qw, ws)
    with through("streaming"):
        want = product(rows, outl, qw, ws)
    assert np.array_equal(bits(out.cpu().numpy()), bits(want.cpu().numpy()))
    if not zeropoint:
        qw.W = None
        out = L.matmul(rows, outl, qw, ws)
        with through("streaming"):
            want = L.matmul(rows, outl, qw, ws)
        assert np.array_equal(bits(out.cpu().numpy()), bits(want.cpu().numpy()))
