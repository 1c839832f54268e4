"""The pre-pass that reads X once (rows held in registers, the outlier set settled afterwards) and the stand-alone calls
that share its kernels, against the oracle, bit for bit.

Sizes: one on each side of every rule that picks rows per workgroup, threads and groups per thread, feature counts that are
multiples of 128, of 8 and of nothing.  Data: outlier columns that one row alone reaches (the other rows' entries there
went into their constants and codes and have to go), with the largest entry of some rows in such a column (the row is made
anew), and more columns than the buffer takes."""
import numpy as np
import pytest

import oracle
from gpu_util import bits

pytestmark = pytest.mark.gpu

SIZES = [(2, 16392), (9, 12288), (16, 40001), (32, 4100),                                     # up to 32 tokens
         (33, 8), (40, 264), (64, 4104), (100, 16384), (45, 20479), (200, 40000),        # one row, and more where rows are short
         (512, 136), (520, 1000), (600, 12288), (513, 16400), (514, 20481), (515, 50176),  # two rows
         (2048, 264), (2049, 2048), (2050, 2056), (2048, 5120), (2051, 8200), (2048, 10248)]  # eight rows, or what fits


def hidden_states(s, h, n, one_sided, seed):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((s, h), dtype=np.float32)
    if one_sided:
        X = np.maximum(X, -0.25)
    cols = np.sort(rng.choice(h, size=min(n, h // 2), replace=False))
    for q, j in enumerate(cols):
        X[rng.integers(0, s), j] = 9.0 + q         # one row alone
        X[rng.integers(0, s, 3), j] = 5.75         # the largest ordinary entry of its row, in an outlier column
        X[rng.integers(0, s, 3), j] = -0.25 if one_sided else -5.75
    if s > 3:
        X[1] = 0.0
        X[2, :] = 0.5
    return X.astype(np.float16)


def device(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda().view(torch.float16)


def buffers(s, h, cap, zp):
    import torch

    import paper_2208_07339_amd as L
    outl = L.Outliers(*(torch.full((n,), -7, dtype=torch.int32, device="cuda") for n in (cap, 1, 1)), cap)
    Xq = torch.full((L.xq_bytes(s, h),), 99, dtype=torch.int8, device="cuda")
    Xo = torch.full((s, L.opad(cap)), 7.0, dtype=torch.float16, device="cuda")
    if zp:
        return outl, L.ZpRows(Xq, torch.full((s, 4), 77, dtype=torch.int32, device="cuda"), Xo, s, h)
    return outl, L.QuantizedRows(Xq, torch.full((s,), 7.0, dtype=torch.float16, device="cuda"), Xo, s, h)


def check(X, outl, rows, alpha, cap, zp):
    import torch

    import paper_2208_07339_amd as L
    torch.cuda.synchronize()
    s, h = X.shape
    full = oracle.find_outliers(X, alpha)
    idx = full[:cap]
    assert int(outl.status.item()) == (1 if len(full) > cap else 0)
    n = int(outl.count.item())
    assert outl.idx[:n].cpu().numpy().tolist() == idx.tolist()
    Xo = rows.Xo.cpu().numpy()
    assert np.array_equal(bits(Xo[:, :n]), bits(X[:, idx])) and not bits(Xo[:, n:]).any()
    if zp:
        x = oracle.zp_quantize_rows(X, idx)
        zc = rows.zc.cpu().numpy()
        assert np.array_equal(zc[:, 0] & 0xffff, bits(x["lo"]).ravel()) and np.array_equal((zc[:, 0] >> 16) & 0xffff, bits(x["hi"]).ravel())
        assert np.array_equal(zc[:, 1], x["zp"]) and np.array_equal(zc[:, 2], x["rowsum"]) and not zc[:, 3].any()
        want = x["Xq"]
    else:
        want, cx = oracle.quantize_rows(X, idx)
        assert np.array_equal(bits(rows.cx.cpu().numpy()), bits(cx))
    assert np.array_equal(L.export_rows(L.QuantizedRows(rows.Xq, None, None, s, h)).cpu().numpy(), want)


@pytest.mark.parametrize("zp", [False, True])
@pytest.mark.parametrize("cap", [32, 6])
@pytest.mark.parametrize("s,h", SIZES)
def test_rows_against_the_oracle(s, h, cap, zp):
    import paper_2208_07339_amd as L
    n, alpha, o = 9 if cap == 6 else 17, 6.0, 40
    X = hidden_states(s, h, n, zp, seed=s * 31 + h)
    Xd, Wd = device(X), device(np.random.default_rng(5).standard_normal((h, o)).astype(np.float16))
    ws = L.Workspace.allocate(s, h, o, cap)
    qw = L.zp_quantize_weight(Wd, ws) if zp else L.quantize_weight(Wd, ws)
    outl, rows = buffers(s, h, cap, zp)
    for _ in range(2):  # twice: what the first call left in the workspace must not matter
        out = (L.zp_linear if zp else L.linear)(Xd, qw, alpha, outl, rows, ws)
    check(X, outl, rows, alpha, cap, zp)
    # the stand-alone calls: the same bits, and the same product from them
    outl2, rows2 = buffers(s, h, cap, zp)
    L.find_outliers(Xd, alpha, cap, ws, outl2)
    (L.zp_quantize_rows if zp else L.quantize_rows)(Xd, outl2, rows2)
    check(X, outl2, rows2, alpha, cap, zp)
    out2 = (L.zp_matmul if zp else L.matmul)(rows2, outl2, qw, ws)
    assert np.array_equal(bits(out.cpu().numpy()), bits(out2.cpu().numpy()))


@pytest.mark.parametrize("zp", [False, True])
@pytest.mark.parametrize("alpha,cap", [(0.0, 256), (0.0, 8), (1e9, 8), (3.0, 256)])
def test_thresholds_that_every_or_no_entry_reaches(alpha, cap, zp):
    """Every column an outlier (and the columns past the buffer's end ordinary again), none, and about as many as fit."""
    import paper_2208_07339_amd as L
    s, h, o = 70, 250, 40
    X = hidden_states(s, h, 3, zp, seed=11)
    Xd, Wd = device(X), device(np.random.default_rng(6).standard_normal((h, o)).astype(np.float16))
    ws = L.Workspace.allocate(s, h, 4096, cap)
    qw = L.zp_quantize_weight(Wd, ws) if zp else L.quantize_weight(Wd, ws)
    outl, rows = buffers(s, h, cap, zp)
    (L.zp_linear if zp else L.linear)(Xd, qw, alpha, outl, rows, ws)
    check(X, outl, rows, alpha, cap, zp)
    outl, rows = buffers(s, h, cap, zp)
    L.find_outliers(Xd, alpha, cap, ws, outl)
    (L.zp_quantize_rows if zp else L.quantize_rows)(Xd, outl, rows)
    check(X, outl, rows, alpha, cap, zp)


@pytest.mark.parametrize("offset", [1, 3, 8])
def test_hidden_states_that_start_anywhere(offset):
    """X at any element of an allocation, an h that would otherwise take whole chunks."""
    import torch

    import paper_2208_07339_amd as L
    s, h, o, cap = 90, 1024, 40, 32
    X = hidden_states(s, h, 5, False, seed=offset)
    room = torch.empty(s * h + 16, dtype=torch.float16, device="cuda")
    Xd = room[offset:offset + s * h].view(s, h)
    Xd.copy_(device(X))
    ws = L.Workspace.allocate(s, h, o, cap)
    qw = L.quantize_weight(device(np.random.default_rng(7).standard_normal((h, o)).astype(np.float16)), ws)
    outl, rows = buffers(s, h, cap, False)
    L.linear(Xd, qw, 6.0, outl, rows, ws)
    check(X, outl, rows, 6.0, cap, False)


# One size per work split (rows of a workgroup, groups and threads) in which threads whose last group lies past the row hold the
# row's last group once more, with 96 to 128 features in the last 128.
REPEATED_END = [(40, 113), (40, 640), (33, 1272), (48, 4220), (96, 5120), (64, 12288), (40, 20480), (100, 28672), (33, 33020),
                (34, 43008), (33, 56064), (40, 64512), (600, 2300), (514, 4220), (600, 5120), (513, 6656), (520, 9216), (530, 11264),
                (514, 14336), (520, 18432), (514, 21118), (516, 28672), (513, 33020), (514, 43008), (516, 56064), (515, 64512),
                (2048, 640), (2050, 1272), (2049, 1790), (2051, 2300), (2048, 3200), (2050, 4220), (2049, 5374), (2048, 6656),
                (2050, 9216), (2048, 7168)]


@pytest.mark.parametrize("zp", [False, True])
@pytest.mark.parametrize("s,h", REPEATED_END)
def test_a_row_whose_extreme_goes_with_a_column_at_either_end(s, h, zp):
    """Outlier columns among the last and the first 16 features that row 0 alone reaches, in which rows of other workgroups
    have their only smallest or largest entry below the threshold: these rows are made anew."""
    import paper_2208_07339_amd as L
    o, cap, alpha = 40, 32, 6.0
    X = np.clip(np.random.default_rng(s + h).standard_normal((s, h), dtype=np.float32), -0.25 if zp else -4.0, 4.0)
    for t, j in enumerate((h - 1, h - 3, h - 16, 0, 2, 15)):
        X[0, j] = 9.0
        X[s - 1 - 2 * t, j] = 5.5      # the largest of its row, by magnitude too
        X[s - 2 - 2 * t, j] = -5.5     # the smallest
        X[s - 13 - t, j], X[s - 13 - t, 7] = 5.5, -5.25
    X = X.astype(np.float16)
    Xd, Wd = device(X), device(np.random.default_rng(8).standard_normal((h, o)).astype(np.float16))
    ws = L.Workspace.allocate(s, h, o, cap)
    qw = L.zp_quantize_weight(Wd, ws) if zp else L.quantize_weight(Wd, ws)
    outl, rows = buffers(s, h, cap, zp)
    (L.zp_linear if zp else L.linear)(Xd, qw, alpha, outl, rows, ws)
    check(X, outl, rows, alpha, cap, zp)


@pytest.mark.parametrize("zp", [False, True])
@pytest.mark.parametrize("s,h", [(40, 8), (41, 27), (600, 30)])
def test_constant_rows_where_every_column_is_an_outlier(s, h, zp):
    """One row reaches the threshold everywhere; rows of other workgroups, constant ones among them, have no ordinary
    column left: their constants are zero."""
    import paper_2208_07339_amd as L
    o, cap, alpha = 4096, 32, 6.0  # (a W wide enough for the scratch to hold the records)
    X = np.random.default_rng(h).uniform(-0.25 if zp else -4.0, 4.0, (s, h))
    X[0] = 9.0
    X[20], X[25], X[30] = 0.5, -0.25, 0.0
    X = X.astype(np.float16)
    Xd, Wd = device(X), device(np.random.default_rng(8).standard_normal((h, o)).astype(np.float16))
    ws = L.Workspace.allocate(s, h, o, cap)
    qw = L.zp_quantize_weight(Wd, ws) if zp else L.quantize_weight(Wd, ws)
    outl, rows = buffers(s, h, cap, zp)
    (L.zp_linear if zp else L.linear)(Xd, qw, alpha, outl, rows, ws)
    check(X, outl, rows, alpha, cap, zp)


def scratch_for_records(s, h, o, cap):
    """Bytes that the workspace of a call has for the records."""
    import paper_2208_07339_amd as L

    def up(n):
        return (n + 255) // 256 * 256
    scan = L.workspace_bytes(s, h, o, cap) - 256 - up(L.opad(cap) * o * 2) - 24 * (up(o) + 256)
    return scan - up(4096 + (h + 255) // 256 * min(cap, 256) * 4 + (h + 511) // 512 * 128)


@pytest.mark.parametrize("zp", [False, True])
@pytest.mark.parametrize("cap,n", [(256, 45), (256, 200), (256, 300), (60, 50), (32, 33), (32, 32)])
@pytest.mark.parametrize("s,h,records", [(40, 5120, 64), (256, 4096, 256), (258, 4100, 288), (600, 8200, 304), (1024, 8192, 512), (1030, 4096, 528),
                                         (2050, 1000, 260), (2048, 12288, 1024)])
def test_many_columns_in_the_records(s, h, records, cap, n, zp):
    """Records of up to more columns than a thread looks at, as many as the buffer takes and more; joined by each workgroup
    for itself or by a kernel of their own (more than 256 records, or 512 of a buffer of up to 32)."""
    import paper_2208_07339_amd as L
    o, alpha = 4096, 6.0
    assert scratch_for_records(s, h, o, cap) >= records * (cap + 17) // 16 * 32 + (h + 255) // 256 * 32
    rng = np.random.default_rng(s + h + n)
    X = np.clip(rng.standard_normal((s, h), dtype=np.float32), -0.25 if zp else -4.0, 4.0)
    for t, j in enumerate(rng.choice(h, size=n, replace=False)):  # from one row alone to nearly all
        X[:, j] = np.where(rng.random(s) < t / n, 9.0, X[:, j])
        X[rng.integers(0, s), j] = 9.0
        X[rng.integers(0, s), j] = 5.5
    X = X.astype(np.float16)
    Xd, Wd = device(X), device(rng.standard_normal((h, o), dtype=np.float32).astype(np.float16))
    ws = L.Workspace.allocate(s, h, o, cap)
    qw = L.zp_quantize_weight(Wd, ws) if zp else L.quantize_weight(Wd, ws)
    outl, rows = buffers(s, h, cap, zp)
    for _ in range(2):  # twice: what the first call left in the workspace must not matter
        (L.zp_linear if zp else L.linear)(Xd, qw, alpha, outl, rows, ws)
    check(X, outl, rows, alpha, cap, zp)
