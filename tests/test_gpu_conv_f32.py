"""The fp32 channels-first convolution at the edges of its tiling: blocks of one pixel to
2048 (in parts of 256), output-channel groups of four, few and many groups per workgroup,
chunked input channels, kernels with and without a compile-time size, from one tap to the
largest, stride 2, batches, ragged everything, with an index and without. Integer operands
make every fp32 sum exact, so the comparison is byte for byte."""
import numpy as np
import pytest

import oracle
import synth
from _util import block_select, from_dev, to_dev, weights_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2108_09376_amd import bc
    return bc


# n, cin, cout, gh, gw, bh, bw, k, stride, residual, active fraction; k: an edge or (kh, kw)
CASES = [
    (1, 16, 16, 4, 4, 8, 8, 3, 1, False, 0.4),       # a channel group per wave
    (1, 1, 1, 1, 1, 1, 1, 1, 1, False, 1.0),          # one output
    (2, 3, 5, 2, 3, 5, 5, 3, 2, True, 0.5),           # 25 pixels, 5 channels, stride 2
    (1, 7, 17, 2, 2, 5, 13, 3, 1, False, 0.7),        # 65 pixels: a second, nearly empty group
    (1, 40, 9, 2, 2, 12, 12, 3, 1, True, 0.7),        # 144 pixels, chunked channels
    (1, 64, 6, 1, 2, 32, 32, 3, 1, False, 0.6),       # 1024 pixels: four parts of 8 rows
    (1, 5, 3, 1, 2, 32, 64, 1, 1, True, 1.0),         # 2048 pixels: eight parts
    (1, 12, 20, 2, 2, 8, 8, 5, 1, False, 0.6),
    (1, 4, 4, 2, 2, 6, 6, 7, 2, False, 0.6),
    (1, 5, 9, 2, 1, 20, 30, 3, 2, True, 0.6),         # parts that begin and end inside rows
    (2, 2, 4, 1, 2, 7, 257, 3, 1, False, 0.6),        # rows longer than a part
    (1, 3, 5, 2, 2, 1, 600, 5, 1, False, 0.6),        # one row in three parts
    (1, 9, 130, 24, 24, 1, 1, 3, 1, True, 0.5),       # one pixel: 33 channel groups, two idle lanes
    (1, 64, 70, 8, 8, 4, 4, 3, 1, False, 0.4),        # few blocks: 16 channels per workgroup
    (1, 64, 24, 48, 48, 2, 2, 3, 1, False, 0.3),      # many small blocks, rounds of weights only
    (1, 20, 40, 24, 32, 3, 5, 1, 1, False, 0.4),      # 1x1: channels read in eights, a ragged last
    (1, 11, 6, 2, 3, 8, 8, (3, 5), 1, True, 0.6),     # not square: no compile-time size
    (1, 2, 3, 2, 2, 8, 8, 51, 1, False, 0.8),         # the halo tile and four channels of 2601 taps
    (1, 2, 1, 2, 2, 8, 8, 73, 1, False, 0.8),         # the largest kernel of an 8x8 block
]


@pytest.mark.parametrize("case", CASES, ids=[f"n{c[0]}_c{c[1]}-{c[2]}_{c[5]}x{c[6]}_k{c[7]}s{c[8]}".replace(" ", "") for c in CASES])
def test_conv_f32_integer_exact(B, case):
    n, cin, cout, gh, gw, bh, bw, k, s, res, frac = case
    kh, kw = k if isinstance(k, tuple) else (k, k)
    r = synth.rng(7300 + cin + cout + bh * bw)
    h, w = gh * bh, gw * bw
    p = kw // 2                                       # (3, 5): the output is two rows taller
    x = synth.to_storage_bits(synth.small_ints(r, (n, cin, h * s - 2 * p + kh - 1 if kh != kw else h * s, w * s)), "f32")
    wt = synth.to_storage_bits(synth.small_ints(r, (cout, cin, kh, kw)), "f32")
    bias = synth.small_ints(r, (cout,))
    prev = synth.nan_canaries(r, (n, cout, h, w), "f32")
    rb = synth.to_storage_bits(synth.small_ints(r, (n, cout, h, w)), "f32") if res else None
    mask = (r.random((n, gh, gw)) < frac).astype(np.uint8)
    mask.reshape(-1)[-1] = 1
    m = torch.from_numpy(mask).cuda()
    idx = torch.empty(n * gh * gw, dtype=torch.int32, device="cuda")
    cnt = torch.empty(1, dtype=torch.int32, device="cuda")
    B.bc_build_block_index(m, n, (gh, gw), idx, cnt)
    out, dense = to_dev(prev, "f32", nhwc=False), to_dev(prev, "f32", nhwc=False)
    args = ((kh, kw, s, p, 1), to_dev(x, "f32", nhwc=False), B.BC_NCHW, weights_dev(wt, "f32", nhwc=False),
            torch.from_numpy(bias).cuda(), to_dev(rb, "f32", nhwc=False) if res else None)
    print("conv f32", case, flush=True)
    B.bc_sparse_conv2d(*args, out, (gh, gw), idx, cnt)
    B.bc_sparse_conv2d(*args, dense, (gh, gw), None, None)      # every block, no index
    torch.cuda.synchronize()
    got = from_dev(out, nhwc=False)
    want = oracle.sparse_conv2d(x, wt, np.ones_like(mask), prev, "f32", s, p, bias, rb, True)
    sel = block_select(mask, got.shape)
    assert np.array_equal(got[~sel], prev[~sel])
    assert np.array_equal(got[sel], want[sel])
    assert np.array_equal(from_dev(dense, nhwc=False), want)


def test_conv_f32_many_channels_on_many_blocks(B):
    """1200 blocks of one pixel with 240000 output channels: 16 channels per workgroup would
    be 2^32 threads and more."""
    cout = 240000
    x = (torch.arange(1200, device="cuda") % 7 - 3).float().reshape(1, 1, 30, 40)
    w = (torch.arange(cout, device="cuda") % 5 - 2).float().reshape(cout, 1, 1, 1)
    out = torch.full((1, cout, 30, 40), float("nan"), device="cuda")
    B.bc_sparse_conv2d((1, 1, 1, 0, 0), x, B.BC_NCHW, w, None, None, out, (30, 40), None, None)
    assert torch.equal(out, x * w.reshape(1, cout, 1, 1))


def test_conv_f32_most_blocks(B):
    """2^20 blocks of one pixel with more output channels than 16 workgroups of 256 threads
    per block could cover within the runtime's 2^32 threads per launch."""
    cout = 272
    x = (torch.arange(1 << 20, device="cuda") % 7 - 3).float().reshape(1, 1, 1024, 1024)
    w = (torch.arange(cout, device="cuda") % 5 - 2).float().reshape(cout, 1, 1, 1)
    out = torch.full((1, cout, 1024, 1024), float("nan"), device="cuda")
    B.bc_sparse_conv2d((1, 1, 1, 0, 0), x, B.BC_NCHW, w, None, None, out, (1024, 1024), None, None)
    assert torch.equal(out, x * w.reshape(1, cout, 1, 1))
