"""The unguarded kernels that use 16 x 16 x 64 MFMAs: tiles of 256 tokens on grids that cover three quarters of the
compute units (192 of 256).  Every one of their outputs against the kernel of 128 x 128 tiles, which keeps 32 x 32 x 32
MFMAs and is held against the oracle elsewhere: any tile gives the same bits."""
import pytest

from gpu_util import have_gpu

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="needs a GPU")]

COLS = {0: 256, 1: 192, 2: 128}  # forced tile: its columns


@pytest.fixture
def forced_tile():
    import paper_2208_07339_amd as L
    yield L.debug_prefill_tile
    L.debug_prefill_tile(-1)


@pytest.mark.parametrize("zeropoint", [False, True])
@pytest.mark.parametrize("tile", [0, 1, 2])
@pytest.mark.parametrize("s,col_blocks,h,outliers,cap", [
    (1021, 48, 64, 3, 16),     # 192 tiles, two K stages, 16 outlier slots, a last token block of 253
    (1024, 48, 136, 0, 32),    # no outlier column
    (769, 64, 640, 20, 32),    # 256 tiles, the last token block of one token
    (1000, 96, 320, 32, 48),   # 384 tiles: workgroups with a second tile; a buffer of more than 32 columns, 32 found
    (1021, 48, 200, 40, 48),   # more than 32 found: these kernels leave the call to the guarded ones
    (1017, 47, 256, 7, 32),    # 188 tiles: just below the line
])
def test_the_same_bits_as_the_other_mfma(tile, s, col_blocks, h, outliers, cap, zeropoint, forced_tile):
    import torch

    import paper_2208_07339_amd as L
    o = COLS[tile] * col_blocks - 8
    g = torch.Generator(device="cuda").manual_seed(s + h + outliers)
    X = torch.empty((s, h), dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    cols = torch.randperm(h, device="cuda", generator=g)[:outliers]
    X[:, cols] = X[:, cols] * 4 + 20
    W = torch.empty((h, o), dtype=torch.float16, device="cuda").normal_(0.0, 0.02, generator=g)
    ws = L.Workspace.allocate(s, h, o, cap)
    outl = L.find_outliers(X, 6.0, cap, ws)
    if zeropoint:
        qw, rows = L.zp_quantize_weight(W, ws), L.zp_quantize_rows(X, outl)
        product = L.zp_matmul
    else:
        qw, rows = L.quantize_weight(W, ws), L.quantize_rows(X, outl)
        product = L.matmul
    out = []
    for t in (tile, 3):
        forced_tile(t)
        out.append(product(rows, outl, qw, ws).view(torch.int16).cpu())
    assert int(outl.count.item()) == outliers
    assert torch.equal(out[0], out[1])
