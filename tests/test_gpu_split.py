"""Kernels that multiply operands cut into terms on a faster matrix unit, at the edges of their tiles, against the plain sums in
float64."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _sites(call):
    from paper_2505_05086_amd import binding as B
    B.asi_profile_enable(True)
    try:
        call()
        torch.cuda.synchronize()
        return list(B.asi_profile_report())
    finally:
        B.asi_profile_enable(False)


def _factors(rng, dims, ranks):
    return [torch.from_numpy(np.linalg.qr(rng.standard_normal((n, r)))[0].astype(np.float32)).cuda() for n, r in zip(dims, ranks)]


def _dense_dw(S, U, gy, stride, pad, dil):
    x = S.double()
    for u in U:
        x = torch.tensordot(x, u.double().t().contiguous(), dims=([0], [0]))
    x = torch.nn.functional.pad(x, (pad[1], pad[1], pad[0], pad[0]))
    ho, wo = gy.shape[2:]                                # (dilation along H only)
    g2 = gy.double().transpose(0, 1).reshape(gy.shape[1], -1).contiguous()
    out = torch.empty(gy.shape[1], x.shape[1], 3, 3, dtype=torch.float64, device="cuda")
    for a in range(3):
        for b in range(3):
            xs = x[:, :, a * dil[0]:a * dil[0] + (ho - 1) * stride[0] + 1:stride[0], b:b + (wo - 1) * stride[1] + 1:stride[1]]
            out[:, :, a, b] = g2 @ xs.transpose(0, 1).reshape(x.shape[1], -1).t().contiguous()
    return out


# Output rows of one position, one short of / just past a group of eight and of the widest map; maps with fewer core channels
# than a chunk takes and with a ragged last chunk of rows; channels past a tile of 64, core channels past one of 16; strides and
# dilations along H, paddings other than 1 (0: windows that end at the map's edge; 2: more positions than the map is wide); the same
# with a stride of two along W over maps of odd and even width.
@pytest.mark.parametrize("dims,ranks,cout,stride,pad,dil", [
    ((5, 20, 3, 3), (3, 17, 2, 2), 65, 1, 0, 1),
    ((5, 20, 3, 4), (3, 17, 2, 2), 65, (1, 2), 0, 1),
    ((6, 18, 17, 15), (6, 18, 5, 5), 66, (2, 2), 1, 1),
    ((3, 12, 30, 34), (3, 12, 6, 6), 20, (2, 2), 1, 1),
    ((2, 10, 21, 127), (2, 9, 6, 9), 18, (1, 2), 1, 1),
    ((2, 10, 20, 61), (2, 9, 6, 9), 18, (2, 2), 2, 2),
    ((6, 33, 7, 7), (5, 16, 4, 4), 64, 1, 1, 1),
    ((9, 18, 8, 9), (9, 18, 5, 5), 63, 1, 1, 1),
    ((4, 24, 17, 18), (3, 9, 6, 6), 130, 1, 0, 1),
    ((3, 20, 66, 63), (2, 5, 9, 9), 40, 1, 1, 1),
    ((3, 12, 45, 62), (3, 12, 7, 8), 17, 1, 2, 1),
    ((4, 16, 41, 24), (4, 16, 6, 6), 32, 2, 1, 1),
    ((4, 16, 23, 31), (3, 16, 6, 6), 32, 1, 1, 3),
])
def test_split_correlation_at_the_edges_of_its_tiles(dims, ranks, cout, stride, pad, dil):
    """Bound: fp32 sums of K products, K up to 4000, are off by about sqrt(K) 2^-25 of a typical entry; 1e-5 of the largest."""
    from paper_2505_05086_amd import binding as B
    rng = np.random.default_rng(sum(dims) + cout)
    stride = stride if isinstance(stride, tuple) else (stride, 1)
    ho = (dims[2] + 2 * pad - 2 * dil - 1) // stride[0] + 1
    wo = (dims[3] + 2 * pad - 3) // stride[1] + 1
    desc, conv = B.make_desc(dims, ranks, "f32"), B.make_conv(cout, 3, 3, stride, (pad, pad), (dil, 1), 1)
    U = _factors(rng, dims, ranks)
    S = torch.from_numpy(rng.standard_normal(ranks).astype(np.float32)).cuda()
    gy = torch.from_numpy(rng.standard_normal((dims[0], cout, ho, wo)).astype(np.float32)).cuda()
    dW = torch.empty(cout, dims[1], 3, 3, device="cuda")
    ws = B.alloc_workspace(desc, conv, 0)
    ws.fill_(255)                                        # NaN wherever nothing was written
    sites = _sites(lambda: B.asi_weight_grad_conv2d(desc, S, U, gy, conv, dW, False, ws))
    assert any("k_corr_mfma_split<9, %s, %d>" % ("true" if wo % 8 else "false", stride[1]) in s for s in sites), sites
    want = _dense_dw(S, U, gy, stride, (pad, pad), (dil, 1))
    assert float((dW - want).abs().max() / want.abs().max()) <= 1e-5


@pytest.mark.parametrize("value", [float("inf"), 3.4e38])
def test_split_correlation_of_an_entry_without_finite_terms(value):
    """An infinite grad_out entry makes its output channel's gradient Inf or NaN where the plain sums have it, and nowhere else; an
    entry that rounds to an infinite bf16 value is computed like any other."""
    from paper_2505_05086_amd import binding as B
    rng = np.random.default_rng(3)
    dims, ranks, cout = (4, 16, 10, 12), (4, 8, 5, 5), 70
    desc, conv = B.make_desc(dims, ranks, "f32"), B.make_conv(cout, 3, 3, (1, 1), (1, 1), (1, 1), 1)
    U = _factors(rng, dims, ranks)
    U[0] = torch.eye(4, device="cuda")                   # the batch entries stay apart
    S = torch.from_numpy((1e-3 * rng.standard_normal(ranks)).astype(np.float32)).cuda()
    gy = torch.from_numpy(rng.standard_normal((4, cout, 10, 12)).astype(np.float32)).cuda()
    gy[2, 66, 4, 5] = value
    dW = torch.empty(cout, 16, 3, 3, device="cuda")
    B.asi_weight_grad_conv2d(desc, S, U, gy, conv, dW, False, B.alloc_workspace(desc, conv, 0))
    rest = torch.arange(cout, device="cuda") != 66
    want = _dense_dw(S, U, gy, (1, 1), (1, 1), (1, 1))
    assert bool(torch.isfinite(dW[rest]).all())
    assert float((dW[rest] - want[rest]).abs().max() / want[rest].abs().max()) <= 1e-5
    if np.isfinite(value):
        assert float((dW[66] - want[66]).abs().max() / want[66].abs().max()) <= 1e-5
    else:
        assert not bool(torch.isfinite(dW[66]).any())


# A single batch entry and core channel, so that a gradient entry meets one value of Z: infinite, NaN or too large for a bf16 term,
# inside the map and where windows hang over its edge (zeros times Inf); several that cancel; finite sums that overflow; maps that are no
# multiple of eight positions, strides of one and two.
@pytest.mark.parametrize("hw,stride", [((10, 12), 1), ((9, 16), 1), ((11, 14), 2)])
@pytest.mark.parametrize("entries", [{(4, 5): "inf"}, {(4, 5): "-inf"}, {(0, 0): "inf", (3, 2): "nan"}, {(0, 0): "inf"}, {(1, 2): "inf", (3, 4): "-inf"},
                                     {(2, 3): "3.4e38"}, {(2, 3): "3.4e38", (0, 0): "inf"}, {}, "all nan", "all inf", "overflow"])
def test_split_correlation_of_special_values(hw, stride, entries):
    from paper_2505_05086_amd import binding as B
    rng = np.random.default_rng(7)
    dims, ranks, cout = (1, 16, *hw), (1, 1, 5, 5), 70
    ho, wo = ((x - 1) // stride + 1 for x in hw)
    desc, conv = B.make_desc(dims, ranks, "f32"), B.make_conv(cout, 3, 3, (stride, stride), (1, 1), (1, 1), 1)
    U = _factors(rng, dims, ranks)
    U[0] = torch.ones(1, 1, device="cuda")
    S = torch.from_numpy((1e-3 * rng.standard_normal(ranks)).astype(np.float32)).cuda()
    gy = torch.from_numpy(rng.standard_normal((1, cout, ho, wo)).astype(np.float32)).cuda()
    if isinstance(entries, dict):
        for (y, x), v in entries.items():
            gy[0, 66, y, x] = float(v)
    elif entries == "overflow":
        gy[0, 66] = 1e38
        S = S.abs() * 1e6
    else:
        gy.fill_(float(entries.split()[1]))
    dW = torch.empty(cout, 16, 3, 3, device="cuda")
    sites = _sites(lambda: B.asi_weight_grad_conv2d(desc, S, U, gy, conv, dW, False, B.alloc_workspace(desc, conv, 0)))
    assert any("k_corr_mfma_split" in s for s in sites), sites
    want = _dense_dw(S, U, gy, (stride, stride), (1, 1), (1, 1))
    if entries == "overflow":                            # (infinite or NaN, by the order of the sums, where fp32 has no number)
        over = want.abs() > 3.5e38
        assert bool(over.any()) and not bool(torch.isfinite(dW[over]).any())
    else:
        assert torch.equal(torch.isnan(dW), torch.isnan(want))
        assert torch.equal(torch.isposinf(dW), torch.isposinf(want)) and torch.equal(torch.isneginf(dW), torch.isneginf(want))
    rest, row = torch.isfinite(want), torch.arange(cout, device="cuda") == 66
    for rows in (~row, row)[:1 if entries == "overflow" else 2]:
        part = rest & rows[:, None, None, None]
        if bool(part.any()):
            assert float((dW - want)[part].abs().max() / want[part].abs().max()) <= 1e-5


def test_split_correlation_of_a_nan_gradient_is_not_summed_entry_by_entry():
    """Twice the finite time, with room for the noise of a measurement (entry by entry it took 65 times as long)."""
    from paper_2505_05086_amd import binding as B
    rng = np.random.default_rng(8)
    dims, ranks, cout = (8, 256, 64, 64), (8, 48, 32, 32), 256
    desc, conv = B.make_desc(dims, ranks, "f32"), B.make_conv(cout, 3, 3, (1, 1), (1, 1), (1, 1), 1)
    U = _factors(rng, dims, ranks)
    S = torch.from_numpy(rng.standard_normal(ranks).astype(np.float32)).cuda()
    gy = torch.randn(dims[0], cout, 64, 64, device="cuda")
    dW, ws = torch.empty(cout, dims[1], 3, 3, device="cuda"), B.alloc_workspace(desc, conv, 0)

    def time(g):
        best = float("inf")
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                B.asi_weight_grad_conv2d(desc, S, U, g, conv, dW, False, ws)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    finite = time(gy)
    for value in ("nan", "inf"):
        assert time(torch.full_like(gy, float(value))) <= 4 * finite


def _exact_factor(A, u, mode):
    """Q of P = A_m (A_m^T u) in float64, positive diagonal of R."""
    m = A.double().movedim(mode, 0).reshape(A.shape[mode], -1)
    P = torch.zeros(u.shape, dtype=torch.float64, device="cuda")
    for c in range(0, m.shape[1], 1 << 18):
        a = m[:, c:c + (1 << 18)].contiguous()
        P += a @ (a.t().contiguous() @ u.double())
    Q, R = torch.linalg.qr(P.cpu())
    return (Q * torch.sign(torch.diagonal(R))).cuda()


def _low_rank(rng, dims, ranks):
    x = torch.from_numpy(rng.standard_normal(ranks).astype(np.float32)).cuda()
    U = _factors(rng, dims, ranks)
    for u in U:
        x = torch.tensordot(x, u.t().contiguous(), dims=([0], [0]))
    return x / x.square().mean().sqrt(), U


# 40 batch entries (three row blocks, the last ragged) and 130 tokens (nine, 45 blocks in one part) or 240 (fifteen, 120 blocks in
# three parts), inner extents that end inside a tile; hidden modes and columns that are no multiple of 64, ranks that fill one, two and
# three blocks per wave and not.
_DIGITS = [
    ((40, 130, 3400), (20, 64, 70), ("gram_digits<4>", "gram_digits<1>", "pair_digits<2>")),
    ((38, 240, 2504), (12, 60, 60), ("gram_digits<4>", "pair_digits<1>")),
    ((24, 240, 5000), (12, 64, 34), ("gram_digits<1>", "pair_digits<1>")),
    ((17, 251, 1000), (9, 20, 150), ("pair_digits<3>",)),
]


_LARGEST = 1e4                      # the one entry that sets the scale of the digits: the last one is worth 2^-30 to 2^-29 of it


def _two_blocks(rng, dims, ranks, small, scale, g):
    """A tensor that is zero but for a block of small values in a corner and one of ordinary values behind it, one of which is large, and
    factors whose last two columns see the small block alone: what these columns become depends on the small values only."""
    A = torch.zeros(dims, device="cuda")
    big = tuple(n - k for n, k in zip(dims, small))
    x, U = _low_rank(rng, big, tuple(r - 2 for r in ranks))
    x += 1e-3 * torch.randn(big, device="cuda", generator=g)
    x[3, 20, 30] = _LARGEST
    A[small[0]:, small[1]:, small[2]:] = x
    A[:small[0], :small[1], :small[2]] = scale * torch.randn(small, device="cuda", generator=g)
    full = []
    for n, r, k, u in zip(dims, ranks, small, U):
        f = torch.zeros(n, r, device="cuda")
        f[k:, :r - 2] = u
        f[:k, r - 2:] = torch.linalg.qr(torch.randn(k, 2, device="cuda", generator=g).cpu())[0].cuda()
        full.append(f)
    return A, full


def _step(A, dims, ranks, prev, kernels):
    from paper_2505_05086_amd import binding as B
    desc = B.make_desc(dims, ranks, "bf16")
    info, ws = torch.zeros(1, dtype=torch.int32, device="cuda"), B.alloc_workspace(desc, None, 0)
    out = [torch.empty_like(u) for u in prev]
    ws.fill_(255)                                        # NaN wherever nothing was written
    sites = _sites(lambda: B.asi_compress(desc, A, prev, out, ws, info))
    if kernels is None:
        assert not any("digits" in s for s in sites), sites
    else:
        assert all(any(k in s for s in sites) for k in kernels), sites
    assert int(info.item()) == 0
    return out


def _off(out, want, rows):
    """Relative error of the first `rows` rows and of the others, the larger."""
    return max(float((o - w).norm() / w.norm()) for o, w in ((out[:rows], want[:rows]), (out[rows:], want[rows:])) if o.numel())


# Ordinary values (now and then one has bits below the last digit, a rest); a few small values, three to a column, some with a rest (the
# list); more than the list holds (the fp64 MFMA from their tile on), with digits left and mostly below the last digit; one entry that dwarfs
# all others; every tile full of rests; token norms that spread over five decades; magnitudes where the scale ends.
@pytest.mark.parametrize("dims,ranks,kernels", _DIGITS)
@pytest.mark.parametrize("data", ["ordinary", "few", "block", "below", "dwarfed", "gelu", "tokens", "tiny"])
def test_steps_on_digits_against_float64(dims, ranks, kernels, data):
    """Factors of one step from a nearby basis, by rows of the small values and the others.  fp32 rounding of the result is 3e-8; the hidden
    mode's V has its factor in two bf16 terms (2^-18), which ordinary values hardly amplify: 1e-5.  And no further off than the same step on
    the fp64 MFMA (an activation that is not 16-byte aligned takes that), but for the rounding of the result."""
    rng = np.random.default_rng(sum(dims))
    g = torch.Generator("cuda").manual_seed(1)
    rows = (0, 0, 0)
    if data in ("few", "block", "below"):
        rows = (3, 3, 3) if data == "few" else (4, 60, 300)
        x, prev = _two_blocks(rng, dims, ranks, rows, _LARGEST * {"few": 1e-6, "block": 6e-7, "below": 2e-7}[data], g)
    else:
        x, U = _low_rank(rng, dims, ranks)
        x += 1e-3 * torch.randn(dims, device="cuda", generator=g)
        if data == "dwarfed":
            x[5, 7, 11] = 3e6
        elif data == "gelu":
            x = torch.nn.functional.gelu(2 * x)
        elif data == "tokens":
            x *= torch.exp(2 * torch.randn(dims[0], dims[1], 1, device="cuda", generator=g))
        elif data == "tiny":
            x *= 2.0 ** -112
        prev = [torch.linalg.qr((u + 0.02 / u.shape[0] ** 0.5 * torch.randn(u.shape, device="cuda", generator=g)).cpu())[0].cuda().contiguous() for u in U]
    A = x.to(torch.bfloat16).contiguous()
    apart = torch.empty(A.numel() + 1, dtype=A.dtype, device="cuda")[1:].view(dims).copy_(A)
    outs = [_step(A, dims, ranks, prev, kernels) for _ in range(2)]
    wide = _step(apart, dims, ranks, prev, None)
    for m in range(3):
        assert torch.equal(outs[0][m], outs[1][m]), m      # the same sums in every run
        want = _exact_factor(A, prev[m], m)
        got, ref = _off(outs[0][m], want, rows[m]), _off(wide[m], want, rows[m])
        print(f"{data} {dims} mode {m}: {got:.2e}, on fp64 {ref:.2e}")
        assert got <= max(1.2 * ref, 1e-7), (m, got, ref)
        if m < 2 or data == "ordinary":
            assert got <= (1e-5 if m == 2 else 1e-6), (m, got)


def test_steps_on_digits_report_a_tensor_that_is_not_finite():
    from paper_2505_05086_amd import binding as B
    dims, ranks = (40, 130, 3400), (20, 64, 70)
    rng = np.random.default_rng(5)
    x, U = _low_rank(rng, dims, ranks)
    A = x.to(torch.bfloat16).contiguous()
    A[3, 7, 11] = float("inf")
    desc = B.make_desc(dims, ranks, "bf16")
    out, info = [torch.empty_like(u) for u in U], torch.zeros(1, dtype=torch.int32, device="cuda")
    sites = _sites(lambda: B.asi_compress(desc, A, U, out, B.alloc_workspace(desc, None, 0), info))
    assert any("digits" in s for s in sites), sites
    assert int(info.item()) != 0
    assert all(not bool(torch.isfinite(u).any()) for u in out)
