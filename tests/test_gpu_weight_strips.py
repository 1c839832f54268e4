"""The weight conversion that reads W once (32 columns to a workgroup, held in registers) and the one that reads it twice at the
edges of their units and of the rule between them, against the oracle: codes, constants and padding, bit for bit."""
import numpy as np
import pytest

import oracle
from gpu_util import have_gpu

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not have_gpu(), reason="needs a GPU")]

# features: one lane group, one unit and one more, the last with one unit per wave and the first with two (absmax), more of
# them with few columns, which are read twice; columns: the fewest, one past a tile, a ragged last tile, nothing aligned
SIZES = [(16, 8), (1, 33), (255, 40), (257, 100), (2048, 72), (2049, 65), (4096, 33), (4097, 31), (5000, 77), (6144, 64),
         (6145, 64), (300, 7)]

# read once: the last with one unit per wave and the first with three (zeropoint), one unit more than whole waves, an odd number of
# units, the largest, and the largest less one row
TALL = [(2305, 33), (4096, 1003), (4097, 999), (4353, 1000), (5000, 997), (6144, 1000), (6143, 1023)]
# more tiles than the eight XCDs deal out evenly, than compute units and than twice as many (two workgroups to a unit)
MANY_TILES = [(70, 773), (300, 4104), (2047, 1029), (129, 8300), (64, 16424)]
# what the kernels that read W twice keep: more features than fit, badly filled rounds, few columns; rows that do not start on 16 bytes,
# one and several blocks of 512 columns with a remainder, last rows that a 16-byte load would reach past, several steps
# to a workgroup (zeropoint)
TWO_READS = [(6145, 9), (6200, 511), (6159, 1031), (8200, 77), (9000, 1541), (2100, 257 * 32 + 5), (5120, 7), (6144, 512)]


def convert_and_compare(h, o, zeropoint, offset=0):
    import torch

    import paper_2208_07339_amd as L
    rng = np.random.default_rng([h, o])
    W = rng.normal(0.0, 0.02, (h, o)).astype(np.float16)
    W[:, 0] = 0                                # constant 0
    W[h // 2, o - 1] = np.float16(3.0)         # the extremes in the last column and the last row
    W[h - 1, o // 2] = np.float16(-5.0)
    if zeropoint:
        W[:, 1] = np.abs(W[:, 1]) + np.float16(1.0)   # a zeropoint far from 0
    # what lies before and behind the matrix is not a weight
    around = torch.full((h * o + 64,), 777.0, dtype=torch.float16, device="cuda")
    Wd = around[offset:offset + h * o].view(h, o)
    Wd.copy_(torch.from_numpy(W.view(np.int16)).cuda().view(torch.float16))
    ws = L.Workspace.allocate(1, h, o, 1)
    qw = L.zp_quantize_weight(Wd, ws) if zeropoint else L.quantize_weight(Wd, ws)
    codes = L.export_weight(L.QuantizedWeight(qw.Wq, None, None, h, o)).cpu().numpy()
    if zeropoint:
        want = oracle.zp_quantize_weight(W)
        zc = qw.zc.cpu().numpy()
        assert np.array_equal(codes, want["Wq"])
        assert np.array_equal(zc[:, 0] & 0xffff, want["lo"].view(np.uint16) & 0xffff)
        assert np.array_equal((zc[:, 0] >> 16) & 0xffff, want["hi"].view(np.uint16) & 0xffff)
        assert np.array_equal(zc[:, 1], want["zp"]) and np.array_equal(zc[:, 2], want["colsum"])
    else:
        Wq, cw = oracle.quantize_weight(W)
        assert np.array_equal(codes, Wq) and np.array_equal(qw.cw.cpu().numpy(), cw)
    # the padding (columns up to a multiple of 32, features up to a multiple of 128) is zero: the buffer sums to the codes
    assert int(qw.Wq.cpu().to(torch.int64).abs().sum()) == int(np.abs(codes.astype(np.int64)).sum())


@pytest.mark.parametrize("h,o", SIZES)
@pytest.mark.parametrize("zeropoint", [False, True])
def test_codes_and_constants(h, o, zeropoint):
    convert_and_compare(h, o, zeropoint)


@pytest.mark.parametrize("h,o", TALL + MANY_TILES)
@pytest.mark.parametrize("zeropoint", [False, True])
def test_conversions_that_read_w_once(h, o, zeropoint):
    import paper_2208_07339_amd as L
    assert L.debug_weight_reads_for(h, o, zeropoint) == 1
    convert_and_compare(h, o, zeropoint, offset=1)


@pytest.mark.parametrize("h,o", TWO_READS)
@pytest.mark.parametrize("zeropoint", [False, True])
def test_conversions_that_read_w_twice(h, o, zeropoint):
    import paper_2208_07339_amd as L
    assert L.debug_weight_reads_for(h, o, zeropoint) == 2
    convert_and_compare(h, o, zeropoint, offset=1)


def test_the_first_conversion_of_a_process_sets_up_the_conversions_only():
    """In a fresh process the first conversion takes a small part of what llmint8_init still has to do after it: 0.09.  With
    the set-up of every kernel in the first conversion, 0.37."""
    import os
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    code = r'''
import sys, time
sys.path.insert(0, %r)
import torch
import paper_2208_07339_amd as L
W = torch.zeros((512, 1024), dtype=torch.float16, device="cuda")
ws = L.Workspace.allocate(1, 512, 1024, 1)
torch.cuda.synchronize()
t = [time.perf_counter()]
for f in (lambda: L.zp_quantize_weight(W, ws), L.init):
    f()
    t.append(time.perf_counter())
print("ratio", (t[1] - t[0]) / (t[2] - t[1]))
''' % root
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    assert float(r.stdout.split()[1]) < 0.22


# two reads with the next step requested ahead (zeropoint): workgroups of one step and of several with a short last one, rows past
# the last feature within a step, a last block of 512 columns that is nearly empty, and the sizes on both sides of its rule
@pytest.mark.parametrize("h,o", [(6500, 3001), (10240, 1541), (10241, 1541), (20481, 1027), (9001, 2056), (3000, 9001)])
def test_two_reads_with_the_next_step_requested_ahead(h, o):
    convert_and_compare(h, o, True, offset=1)
