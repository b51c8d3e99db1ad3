"""The fp32 channels-first convolution at the edges of its tiling: pixel groups of 64 (one
to 32 per block), output-channel groups of four, chunked input channels, kernels with and
without a compile-time size, stride 2, batches, ragged everything. Integer operands make
every fp32 sum exact, so the comparison is byte for byte."""
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


# n, cin, cout, gh, gw, bh, bw, k, stride, residual, active fraction
CASES = [
    (1, 16, 16, 4, 4, 8, 8, 3, 1, False, 0.4),       # one item per wave
    (1, 1, 1, 1, 1, 1, 1, 1, 1, False, 1.0),          # one output
    (2, 3, 5, 2, 3, 5, 5, 3, 2, True, 0.5),           # 25 pixels, 5 channels, stride 2
    (1, 7, 17, 2, 2, 5, 13, 3, 1, False, 0.7),        # 65 pixels: a second, nearly empty group
    (1, 40, 9, 2, 2, 12, 12, 3, 1, True, 0.7),        # 144 pixels, chunked channels
    (1, 64, 6, 1, 2, 32, 32, 3, 1, False, 0.6),       # 1024 pixels: four items per wave
    (1, 5, 3, 1, 2, 32, 64, 1, 1, True, 1.0),         # 2048 pixels: eight items per wave
    (1, 12, 20, 2, 2, 8, 8, 5, 1, False, 0.6),        # a kernel without a compile-time size
    (1, 4, 4, 2, 2, 6, 6, 7, 2, False, 0.6),
]


@pytest.mark.parametrize("case", CASES, ids=[f"n{c[0]}_c{c[1]}-{c[2]}_{c[5]}x{c[6]}_k{c[7]}s{c[8]}" for c in CASES])
def test_conv_f32_integer_exact(B, case):
    n, cin, cout, gh, gw, bh, bw, k, s, res, frac = case
    r = synth.rng(7300 + cin + cout + bh * bw)
    h, w = gh * bh, gw * bw
    x = synth.to_storage_bits(synth.small_ints(r, (n, cin, h * s, w * s)), "f32")
    wt = synth.to_storage_bits(synth.small_ints(r, (cout, cin, k, k)), "f32")
    bias = synth.small_ints(r, (cout,))
    prev = synth.nan_canaries(r, (n, cout, h, w), "f32")
    rb = synth.to_storage_bits(synth.small_ints(r, (n, cout, h, w)), "f32") if res else None
    mask = (r.random((n, gh, gw)) < frac).astype(np.uint8)
    mask.reshape(-1)[-1] = 1
    m = torch.from_numpy(mask).cuda()
    idx = torch.empty(n * gh * gw, dtype=torch.int32, device="cuda")
    cnt = torch.empty(1, dtype=torch.int32, device="cuda")
    B.bc_build_block_index(m, n, (gh, gw), idx, cnt)
    out = to_dev(prev, "f32", nhwc=False)
    print("conv f32", case, flush=True)
    B.bc_sparse_conv2d((k, k, s, k // 2, 1), to_dev(x, "f32", nhwc=False), B.BC_NCHW,
                       weights_dev(wt, "f32", nhwc=False), torch.from_numpy(bias).cuda(),
                       to_dev(rb, "f32", nhwc=False) if res else None, out, (gh, gw), idx, cnt)
    torch.cuda.synchronize()
    got = from_dev(out, nhwc=False)
    want = oracle.sparse_conv2d(x, wt, mask, prev, "f32", s, k // 2, bias, rb, True)
    sel = block_select(mask, got.shape)
    assert np.array_equal(got[~sel], prev[~sel])
    assert np.array_equal(got[sel], want[sel])
