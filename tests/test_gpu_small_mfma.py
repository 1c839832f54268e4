"""The unguarded kernels with tiles of 256 tokens, 16 x 16 x 64 MFMAs and 32 x 32 x 32 (llmint8_debug_mfma_for says which a
product takes).  Every one of their outputs against the kernel of 128 x 128 tiles, which keeps 32 x 32 x 32
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


def compare_with_the_small_tile(s, h, o, outliers, cap, tile, zeropoint, force, fp16_rows=True):
    import torch

    import paper_2208_07339_amd as L
    g = torch.Generator(device="cuda").manual_seed(s + h + outliers)
    X = torch.empty((s, h), dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=g)
    X.clamp_(-5.0, 5.0)  # of 20 million samples one may reach the threshold of 6 (2e-9 each): a column more
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
    if not fp16_rows:
        qw.W = None
    out = []
    for t in (tile, 3):
        force(t)
        out.append(product(rows, outl, qw, ws).view(torch.int16).cpu())
    assert int(outl.count.item()) == outliers
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("zeropoint", [False, True])
@pytest.mark.parametrize("tile", [0, 1, 2])
@pytest.mark.parametrize("s,quarters,outliers,cap,fp16_rows", [
    (1021, 3, 3, 16, True),      # three quarters of the compute units, 16 outlier slots, a last token block of 253
    (1024, 4, 0, 32, True),      # a full round, no outlier column
    (769, 4, 20, 32, True),      # the last token block of one token
    (1000, 8, 32, 48, True),     # workgroups with a second tile; a buffer of more than 32 columns, 32 found
    (1021, 4, 40, 48, True),     # more than 32 found: these kernels leave the call to the guarded ones
    (1021, 4, 9, 32, False),     # rows of W rebuilt from the codes
])
def test_sixteen_wide_mfma_from_the_shortest_sum_on(tile, s, quarters, outliers, cap, fp16_rows, zeropoint, forced_tile):
    """The smallest K that the rule gives to 16 x 16 x 64, for a grid of that many quarters of the compute units."""
    import torch

    import paper_2208_07339_amd as L
    if zeropoint and not fp16_rows:
        pytest.skip("the zeropoint calls need W in fp16")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    o = COLS[tile] * (cus // 4 * quarters // 4) - 8
    forced_tile(tile)
    lo, hi = 1, 65536
    assert L.debug_mfma_for(s, lo, o, zeropoint) == 32 and L.debug_mfma_for(s, hi, o, zeropoint) == 16
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if L.debug_mfma_for(s, mid, o, zeropoint) == 16 else (mid, hi)
    compare_with_the_small_tile(s, hi, o, outliers, cap, tile, zeropoint, forced_tile, fp16_rows)


@pytest.mark.parametrize("zeropoint", [False, True])
@pytest.mark.parametrize("tile", [0, 1, 2])
@pytest.mark.parametrize("s,col_blocks,h,outliers,cap", [
    (1021, 48, 64, 3, 16),     # 192 tiles, two K stages, 16 outlier slots, a last token block of 253
    (1024, 48, 136, 0, 32),    # no outlier column
    (769, 64, 640, 20, 32),    # 256 tiles, the last token block of one token
    (1000, 96, 320, 32, 48),   # 384 tiles: workgroups with a second tile; a buffer of more than 32 columns, 32 found
    (1021, 48, 200, 40, 48),   # more than 32 found: these kernels leave the call to the guarded ones
    (1017, 47, 256, 7, 32),    # 188 tiles
])
def test_the_same_bits_as_the_other_mfma(tile, s, col_blocks, h, outliers, cap, zeropoint, forced_tile):
    """Short sums, for which all these shapes use 32 x 32 x 32 (but absmax at 640 features in 128 and 256 columns)."""
    compare_with_the_small_tile(s, h, COLS[tile] * col_blocks - 8, outliers, cap, tile, zeropoint, forced_tile)
