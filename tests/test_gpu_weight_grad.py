"""Weight and bias gradients at the edges of the kernel-row form (output maps that divide
into 8 x 8 tiles): one and many tiles per run, ragged input channels, both strides and
kernel sizes, batches, both formats, and the sizes just below its range. Small integers
make every product and sum exact in fp32, so the comparison is exact and the order of the
atomic additions does not matter."""
import numpy as np
import pytest

import synth
from _util import shifted, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# n, cin, cout, k, stride, hout, wout, dtype, bias
CASES = [
    (1, 64, 64, 3, 1, 32, 32, "bf16", True),      # 16 tiles: the smallest 3x3 map
    (1, 64, 64, 3, 1, 24, 40, "bf16", True),      # 960 pixels: the general form
    (2, 72, 128, 3, 1, 24, 24, "f16", True),      # ragged second ci tile, two images
    (1, 8, 64, 3, 2, 32, 40, "bf16", False),      # eight input channels, stride 2
    (3, 136, 64, 3, 2, 16, 24, "bf16", True),     # a run that crosses images
    (1, 64, 64, 1, 1, 8, 8, "bf16", True),        # one tile
    (1, 200, 192, 1, 2, 16, 8, "f16", True),
    (1, 64, 64, 3, 1, 128, 64, "bf16", True),     # several tiles per run, a shorter last run
    (1, 256, 256, 3, 1, 32, 32, "bf16", True),    # as many tiles of (co, ci) as workgroups
    (1, 512, 256, 3, 1, 48, 56, "f16", True),     # runs of 21 tiles: one batch joined, a shorter one
    (1, 512, 512, 3, 1, 48, 48, "bf16", True),    # one run of 36 tiles: two batches joined
]


@pytest.mark.parametrize("case", CASES, ids=["_".join(map(str, c)) for c in CASES])
def test_weight_grad_integer_exact(case):
    from paper_2108_09376_amd import bc
    n, cin, cout, k, s, h, w, dt, bias = case
    r = synth.rng(7500 + cin + cout + h)
    x = synth.small_ints(r, (n, cin, h * s, w * s), -2, 2)
    g = synth.small_ints(r, (n, cout, h, w), -2, 2)
    xp = np.pad(x, ((0, 0), (0, 0), (k // 2, k // 2), (k // 2, k // 2))).astype(np.float64)
    gf = g.astype(np.float64).transpose(1, 0, 2, 3).reshape(cout, -1)
    want = np.empty((cout, k, k, cin))
    for i in range(k):
        for j in range(k):
            t = xp[:, :, i:i + s * (h - 1) + 1:s, j:j + s * (w - 1) + 1:s]
            want[:, i, j] = gf @ t.transpose(1, 0, 2, 3).reshape(cin, -1).T
    dw0 = synth.small_ints(r, (cout, k, k, cin))
    dw = torch.from_numpy(dw0.copy()).cuda()
    db = torch.full((cout,), 3.0, device="cuda") if bias else None
    print("weight gradient", case, flush=True)
    bc.bc_conv2d_weight_grad((k, k, s, k // 2, 0), to_dev(synth.to_storage_bits(x, dt), dt),
                             to_dev(synth.to_storage_bits(g, dt), dt), dw, db)
    torch.cuda.synchronize()
    assert np.array_equal(dw.cpu().numpy(), (want + dw0).astype(np.float32))
    if bias:
        assert np.array_equal(db.cpu().numpy(), (gf.sum(1) + 3.0).astype(np.float32))


def test_weight_grad_outside_values_stay_out():
    """Padding is zero and pixels that a tap does not reach do not enter its sum: an
    infinity in the last input column reaches only the taps that read that column."""
    from paper_2108_09376_amd import bc
    x = torch.ones((1, 32, 32, 64), dtype=torch.bfloat16, device="cuda")
    x[0, :, 31, 5] = float("inf")
    g = torch.ones((1, 32, 32, 64), dtype=torch.bfloat16, device="cuda")
    dw = torch.zeros((64, 3, 3, 64), device="cuda")
    bc.bc_conv2d_weight_grad((3, 3, 1, 1, 0), x, g, dw, None)
    bad = ~torch.isfinite(dw)
    assert bool(bad[:, :, 1:, 5].all()) and int(bad.sum()) == 64 * 3 * 2


@pytest.mark.parametrize("which", ["x", "g"])
def test_weight_grad_takes_any_alignment(which):
    """Maps that start 8 bytes off a 16-byte boundary give the exact result too (small
    integers): the form whose loads need the alignment is not taken."""
    from paper_2108_09376_amd import bc
    r = synth.rng(7650)
    x = to_dev(synth.to_storage_bits(synth.small_ints(r, (1, 64, 32, 40), -2, 2), "bf16"), "bf16")
    g = to_dev(synth.to_storage_bits(synth.small_ints(r, (1, 64, 32, 40), -2, 2), "bf16"), "bf16")
    res = []
    for off in (0, 4):
        dw, db = torch.zeros((64, 3, 3, 64), device="cuda"), torch.zeros(64, device="cuda")
        xs, gs = (shifted(x, off), g) if which == "x" else (x, shifted(g, off))
        bc.bc_conv2d_weight_grad((3, 3, 1, 1, 0), xs, gs, dw, db)
        res.append((dw, db))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])


@pytest.mark.parametrize("cin,cout,k", [(256, 256, 3), (64, 64, 1)])
def test_weight_grad_no_less_accurate_than_the_general_form(cin, cout, k):
    """Long sums of values of one sign, where every rounding counts: the gradients of a map
    of whole 8 x 8 tiles (64 x 128) are at most as far from 64 bits as those of a map of
    about as many pixels that the general form takes (64 x 124; 3 % fewer terms, 5 % for
    the spread between inputs)."""
    from paper_2108_09376_amd import bc
    g = torch.Generator(device="cuda").manual_seed(11)
    err = {}
    for w in (128, 124):
        x = torch.randn((1, 64, w, cin), generator=g, device="cuda").relu().bfloat16()
        go = (torch.randn((1, 64, w, cout), generator=g, device="cuda").abs() * 0.1).bfloat16()
        dw = torch.zeros((cout, k, k, cin), device="cuda")
        db = torch.zeros(cout, device="cuda")
        bc.bc_conv2d_weight_grad((k, k, 1, k // 2, 0), x, go, dw, db)
        xp = torch.nn.functional.pad(x.double(), (0, 0, k // 2, k // 2, k // 2, k // 2))
        gd = go.double().reshape(-1, cout).t().contiguous()
        want = torch.stack([gd @ xp[:, i:i + 64, j:j + w].reshape(-1, cin) for i in range(k) for j in range(k)], 1)
        rel = lambda a, b: float((a.double() - b).norm() / b.norm())
        err[w] = rel(dw.reshape(want.shape), want), rel(db, gd.sum(1))
    print(err)
    assert err[128][0] <= 1.08 * err[124][0]
    # 64 or 256 sums only: their spread between inputs is about 1 / sqrt(2 * 64) each side
    assert err[128][1] <= 1.3 * err[124][1]


@pytest.mark.parametrize("counts", [(1, 255, 1024, 1025), (4096, 2049, 3), (262145,), (300000, 5),
                                    (1, 262144, 1023, 1024, 1025, 2049, 255, 256, 257)])
def test_rmsprop_many_elements_per_workgroup(counts):
    """Tensors that end inside, at and just past a workgroup's 256 or 1024 elements (few or
    many workgroups) take the same step as one by one, byte for byte, with and without a
    16-bit copy."""
    from paper_2108_09376_amd import bc
    r = synth.rng(7700 + len(counts))
    make = lambda: [tuple(torch.from_numpy(a).cuda() for a in t) for t in data]
    data = [(synth.normal(r, n), np.abs(synth.normal(r, n)), synth.normal(r, n)) for n in counts]
    many, single = make(), make()
    c16 = [torch.zeros(n, dtype=torch.bfloat16, device="cuda") if i % 2 else None for i, n in enumerate(counts)]
    s16 = [None if c is None else c.clone() for c in c16]
    bc.bc_rmsprop_step_many([(w, v, g, c) for (w, v, g), c in zip(many, c16)], 1e-2, 0.9, 1e-8, 1e-3)
    for (w, v, g), c in zip(single, s16):
        bc.bc_rmsprop_step(w, v, g, 1e-2, 0.9, 1e-8, 1e-3, c)
    torch.cuda.synchronize()
    for a, b in zip(many, single):
        assert all(torch.equal(x, y) for x, y in zip(a, b))
    for a, b in zip(c16, s16):
        assert a is None or torch.equal(a, b)
