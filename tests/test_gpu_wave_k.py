"""The wave-K convolution form (3x3, stride 1, four waves splitting K) at the sizes where
it can go wrong: ragged channel counts, waves with unequal or no work, one and several
patches per tile, every LDS halo size, batches, single blocks, K slices by several
workgroups and by one in turn, K whole on few and many tiles; and some shapes just outside,
which other forms compute. Operands are small integers, so every sum is exact in fp32
and the comparison is byte for byte whatever the order of the sums."""
import numpy as np
import pytest

import oracle
import synth
from _util import block_select, from_dev, shifted, to_dev, weights_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2108_09376_amd import bc
    return bc


# n, cin, cout, gh, gw, bh, bw, dtype, residual, active fraction
CASES = [
    (1, 512, 64, 2, 3, 8, 8, "bf16", False, 0.5),     # four K slices, one chunk per wave
    (1, 488, 64, 3, 2, 8, 8, "f16", True, 0.5),       # the last chunk ragged
    (2, 520, 128, 2, 2, 8, 8, "bf16", True, 0.6),     # 17 chunks: the last slice shorter
    (1, 616, 64, 4, 5, 4, 4, "bf16", False, 0.4),     # four 4x4 patches per tile, ragged last patch
    (1, 256, 320, 6, 9, 8, 8, "bf16", True, 0.3),     # 270 tiles, K whole, two chunks per wave
    (1, 232, 320, 6, 9, 8, 8, "f16", False, 0.3),     # eight chunks, the last of 8 channels
    (1, 512, 64, 2, 2, 16, 16, "bf16", False, 0.5),   # bands of a 16-wide block
    (1, 512, 64, 1, 2, 32, 32, "f16", False, 1.0),    # a 32-wide block cut into 8x8 tiles
    (1, 512, 64, 2, 2, 12, 32, "bf16", True, 0.6),    # cut into 4x16 tiles
    (1, 512, 64, 2, 2, 2, 32, "f16", False, 0.6),     # two rows: not cut, a 136-slot halo
    (1, 512, 64, 1, 1, 4, 64, "bf16", True, 1.0),     # 64 wide: the halo is too large, another form
    (1, 512, 64, 4, 4, 2, 4, "bf16", False, 0.4),     # eight 2x4 patches: the largest halo
    (1, 512, 64, 3, 5, 8, 8, "bf16", False, 0.07),    # one active block
    (1, 232, 64, 3, 5, 8, 8, "bf16", False, 0.3),     # few tiles, eight chunks: another form
    (1, 520, 192, 6, 8, 8, 8, "f16", True, 0.3),      # 144 tiles: 288 slices by workgroups of their
                                                      # own, in turn without an index, the last shorter
    (1, 520, 640, 6, 9, 8, 8, "bf16", True, 0.3),     # 540 tiles, K whole
]


@pytest.mark.parametrize("case", CASES, ids=[f"n{c[0]}_c{c[1]}-{c[2]}_{c[5]}x{c[6]}_{c[7]}" for c in CASES])
def test_wave_k_integer_exact(B, case):
    n, cin, cout, gh, gw, bh, bw, dt, res, frac = case
    r = synth.rng(7000 + cin + cout + bh)
    h, w = gh * bh, gw * bw
    x = synth.to_storage_bits(synth.small_ints(r, (n, cin, h, w), -2, 2), dt)
    wt = synth.to_storage_bits(synth.small_ints(r, (cout, cin, 3, 3), -1, 1), dt)
    bias = synth.small_ints(r, (cout,), -3, 3)
    prev = synth.nan_canaries(r, (n, cout, h, w), dt)
    rb = synth.to_storage_bits(synth.small_ints(r, (n, cout, h, w), -3, 3), dt) if res else None
    mask = (r.random((n, gh, gw)) < frac).astype(np.uint8)
    mask.reshape(-1)[0] = 1
    m = torch.from_numpy(mask).cuda()
    idx = torch.empty(n * gh * gw, dtype=torch.int32, device="cuda")
    cnt = torch.empty(1, dtype=torch.int32, device="cuda")
    B.bc_build_block_index(m, n, (gh, gw), idx, cnt)
    args = ((3, 3, 1, 1, 1), to_dev(x, dt), B.BC_NHWC, weights_dev(wt, dt), torch.from_numpy(bias).cuda(),
            to_dev(rb, dt) if res else None)
    print("wave-K", case, flush=True)
    out, dense = to_dev(prev, dt), to_dev(prev, dt)
    B.bc_sparse_conv2d(*args, out, (gh, gw), idx, cnt)
    B.bc_sparse_conv2d(*args, dense, (gh, gw), None, None)      # every block, no index
    torch.cuda.synchronize()
    got, full = from_dev(out), from_dev(dense)
    want = oracle.sparse_conv2d(x, wt, np.ones_like(mask), prev, dt, 1, 1, bias, rb, True)
    sel = block_select(mask, got.shape)
    assert np.array_equal(full, want)
    assert np.array_equal(got[sel], want[sel])
    assert np.array_equal(got[~sel], prev[~sel])                # copied blocks: previous bits


@pytest.mark.parametrize("shape", [(512, 128, 16, 16, 8, 8), (512, 512, 8, 16, 4, 4), (256, 256, 8, 16, 8, 8)])
def test_wave_k_bits_do_not_depend_on_the_call(B, shape):
    """An active block has the same bits alone, with others, and in a call without an index
    (where K slices may run in turn instead of in workgroups of their own)."""
    cin, cout, gh, gw, bh, bw = shape
    r = synth.rng(7100 + bh)
    h, w = gh * bh, gw * bw
    x = to_dev(synth.to_storage_bits(synth.normal(r, (1, cin, h, w)), "bf16"), "bf16")
    wt = weights_dev(synth.to_storage_bits(synth.he_normal(r, cout, cin, 3, 3), "bf16"), "bf16")
    conv = (3, 3, 1, 1, 1)
    dense = torch.zeros((1, h, w, cout), dtype=torch.bfloat16, device="cuda")
    B.bc_sparse_conv2d(conv, x, B.BC_NHWC, wt, None, None, dense, (gh, gw), None, None)
    full = from_dev(dense)
    for frac in (0.0, 0.2, 0.9):
        mask = (r.random((1, gh, gw)) < frac).astype(np.uint8)
        mask[0, gh - 1, gw - 1] = 1
        m = torch.from_numpy(mask).cuda()
        idx = torch.empty(gh * gw, dtype=torch.int32, device="cuda")
        cnt = torch.empty(1, dtype=torch.int32, device="cuda")
        B.bc_build_block_index(m, 1, (gh, gw), idx, cnt)
        out = torch.zeros_like(dense)
        B.bc_sparse_conv2d(conv, x, B.BC_NHWC, wt, None, None, out, (gh, gw), idx, cnt)
        torch.cuda.synchronize()
        got = from_dev(out)
        sel = block_select(mask, got.shape)
        assert np.array_equal(got[sel], full[sel]), frac
        assert not got[~sel].any()


@pytest.mark.parametrize("which", ["x", "w"])
def test_wave_k_shapes_take_any_alignment(B, which):
    """A map or weights that start 8 bytes off a 16-byte boundary (a view into a buffer) give
    the exact result too: the form whose loads need the alignment is not taken."""
    r = synth.rng(7150)
    x = to_dev(synth.to_storage_bits(synth.small_ints(r, (1, 512, 24, 32), -2, 2), "bf16"), "bf16")
    wt = weights_dev(synth.to_storage_bits(synth.small_ints(r, (128, 512, 3, 3), -1, 1), "bf16"), "bf16")
    outs = []
    for off in (0, 4):
        out = torch.zeros((1, 24, 32, 128), dtype=torch.bfloat16, device="cuda")
        xs, ws = (shifted(x, off), wt) if which == "x" else (x, shifted(wt, off))
        B.bc_sparse_conv2d((3, 3, 1, 1, 0), xs, B.BC_NHWC, ws, None, None, out, (3, 4), None, None)
        outs.append(out)
    assert outs[0].float().abs().sum() > 0 and torch.equal(outs[0], outs[1])
