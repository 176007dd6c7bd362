"""Mode products and pair products at the edges of their tiles, against the plain sums in float64."""
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
        return {site: v["workgroups"] for site, v in B.asi_profile_report().items()}
    finally:
        B.asi_profile_enable(False)


def _dev(x, dtype="f32"):
    return torch.from_numpy(x.astype(np.float32)).cuda().to(torch.float32 if dtype == "f32" else torch.bfloat16)


def _modes(x, mats):
    """x multiplied along every mode by mats[m] (n_m x r_m), in float64."""
    x = x.double()
    for m in mats:
        x = torch.tensordot(x, m.double(), dims=([0], [0]))
    return x


# The channel mode (not a multiple of the four entries of a step; fewer steps than waves times the steps in flight, and more), 15 to 65
# outputs (one to four blocks, two tiles), columns short of and past one, two and many blocks, an inner extent of 1 x 2 to 9 x 11.
@pytest.mark.parametrize("dims,ranks", [
    ((3, 65, 1, 2), (3, 6, 1, 2)), ((2, 97, 5, 7), (2, 16, 2, 7)), ((70, 100, 7, 7), (40, 17, 3, 5)), ((5, 131, 9, 11), (5, 47, 4, 3)),
    ((300, 66, 3, 5), (60, 33, 2, 5)), ((9, 515, 7, 7), (9, 63, 5, 5)), ((4, 1029, 5, 7), (4, 65, 5, 7)), ((170, 258, 7, 7), (10, 20, 2, 2)),
    ((170, 97, 7, 7), (160, 4, 7, 7)), ((9, 160, 5, 7), (9, 40, 5, 7)), ((9, 161, 5, 7), (9, 40, 5, 7)), ((190, 68, 9, 5), (180, 50, 9, 5))])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_product_along_a_long_mode_with_few_columns(dims, ranks, dtype):
    """Bound: fp32 sums of at most 1029 products, off by about sqrt(K) 2^-25 of a typical entry; 2e-6 of the largest."""
    from paper_2505_05086_amd import binding as B
    rng = np.random.default_rng(sum(dims) + sum(ranks))
    x = _dev(rng.standard_normal(dims), dtype)
    U = [_dev(np.linalg.qr(rng.standard_normal((n, r)))[0]) for n, r in zip(dims, ranks)]
    desc = B.make_desc(dims, ranks, dtype)
    S = torch.empty(ranks, device="cuda")
    ws = B.alloc_workspace(desc, None, 0)
    ws.fill_(255)                                        # NaN wherever nothing was written
    sites = _sites(lambda: B.asi_core_project(desc, x, U, S, ws))
    waves = 4 if dims[1] <= 160 else 8
    assert any("k_ttm_ksplit" in s and ", true, %d>" % waves in s for s in sites), sites
    want = _modes(x, U)
    assert float((S - want).abs().max() / want.abs().max()) <= 2e-6


@pytest.mark.parametrize("r2,cout,cb", [(65, 30, 1), (130, 7, 1), (97, 31, 1), (149, 911, 2), (66, 920, 2)])
def test_product_with_a_transposed_matrix_along_a_long_mode(r2, cout, cb):
    """The last step of a 3 x 3 weight gradient with more than 64 core channels (17 to 38 steps of four entries, the last one whole or not;
    one and two blocks of columns a workgroup); bound as above, over two chained sums."""
    from paper_2505_05086_amd import binding as B
    rng = np.random.default_rng(r2)
    dims, ranks = (4, 150, 9, 9), (4, r2, 9, 9)
    x = _dev(rng.standard_normal(dims))
    U = [_dev(np.linalg.qr(rng.standard_normal((n, r)))[0]) for n, r in zip(dims, ranks)]
    S = _modes(x, U).float()
    gy = _dev(rng.standard_normal((4, cout, 9, 9)))
    desc, conv = B.make_desc(dims, ranks, "f32"), B.make_conv(cout, 3, 3, (1, 1), (1, 1), (1, 1), 1)
    dW = torch.empty(cout, 150, 3, 3, device="cuda")
    ws = B.alloc_workspace(desc, conv, 0)
    ws.fill_(255)
    sites = _sites(lambda: B.asi_weight_grad_conv2d(desc, S, U, gy, conv, dW, False, ws))
    assert any("k_ttm_ksplit<float, 4, %d, false, 4>" % cb in s for s in sites), sites
    xr = _modes(S, [u.t().contiguous() for u in U])
    want = torch.nn.grad.conv2d_weight(xr.cpu(), dW.shape, gy.double().cpu(), padding=1).cuda()
    assert float((dW - want).abs().max() / want.abs().max()) <= 5e-6


# (mode): rows short of and past a tile of 64, ranks of one to four blocks of 16 and of two tiles, columns short of a block of 16, of a
# chunk of 64 and past several, inner extents of 1, odd, a multiple of four above and below a chunk; the activation one element off.
@pytest.mark.parametrize("dims,ranks,mode", [
    ((3, 65, 1, 7), (3, 15, 1, 7), 1), ((9, 127, 3, 5), (9, 16, 3, 5), 1), ((40, 130, 7, 7), (20, 33, 5, 5), 1), ((5, 513, 9, 11), (5, 48, 5, 5), 1),
    ((6, 515, 2, 2), (6, 24, 2, 2), 1), ((4, 640, 4, 8), (4, 49, 4, 4), 1), ((3, 600, 6, 12), (3, 70, 6, 12), 1), ((2, 100, 9, 80), (2, 17, 5, 9), 1),
    ((3, 35, 514), (3, 20, 50), 2), ((2, 33, 577), (2, 33, 17), 2), ((4, 1100, 66), (4, 64, 31), 1),
    ((3, 70, 335), (3, 20, 40), 2), ((2, 130, 402), (2, 50, 70), 2)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shift", [0, 1])
def test_pair_product_at_the_edges_of_its_tiles(dims, ranks, mode, dtype, shift):
    """The factor of a mode that goes through V and P, against float64.  P's condition is that of random data, 5 to 340; V is fp32,
    2^-24 of its entries, which the condition (below 500) takes to 3e-5 of the factor's largest entry.  bf16 last modes cut U_prev in two bf16 terms: 2^-17 of its
    entries, 2e-4."""
    from paper_2505_05086_amd import binding as B
    rng = np.random.default_rng(sum(dims) + sum(ranks) + shift)
    numel = int(np.prod(dims))
    flat = _dev(rng.standard_normal(numel + 1), dtype)
    x = flat[shift:shift + numel].view(dims)
    U = [_dev(np.linalg.qr(rng.standard_normal((n, r)))[0]) for n, r in zip(dims, ranks)]
    out = [torch.full_like(u, float("nan")) for u in U]
    desc = B.make_desc(dims, ranks, dtype)
    info = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    ws = B.alloc_workspace(desc, None, 0)
    ws.fill_(255)
    sites = _sites(lambda: B.asi_compress(desc, x, U, out, ws, info))
    assert any("k_pair" in s for s in sites), sites
    assert int(info) == 0
    a = x.double().movedim(mode, 0).reshape(dims[mode], -1)
    p = a @ (a.t().contiguous() @ U[mode].double())
    q, r = torch.linalg.qr(p)
    want = q * torch.sign(torch.diagonal(r))
    assert float(torch.linalg.cond(p)) < 500
    err = float((out[mode] - want).abs().max() / want.abs().max())
    assert err <= (2e-4 if dtype == "bf16" and mode == len(dims) - 1 else 3e-5), err


# Planes of one to four blocks of 16 rows and columns (one, two and four waves a plane; the last workgroup of planes not full), ranks of
# one and two blocks that are no multiple of four; G1 streamed (a million entries of grad_out), tiled, and grad_out itself (r1 = B).
@pytest.mark.parametrize("dims,ranks,cout", [
    ((40, 9, 7, 7), (8, 5, 5, 5), 520), ((20, 6, 13, 17), (12, 5, 9, 17), 240), ((18, 7, 31, 18), (8, 5, 13, 6), 112), ((6, 8, 33, 50), (5, 7, 19, 31), 30),
    ((64, 11, 14, 14), (16, 7, 7, 7), 100), ((5, 9, 64, 63), (5, 5, 29, 32), 11), ((9, 10, 2, 16), (5, 9, 2, 9), 33), ((33, 6, 49, 8), (4, 6, 6, 5), 90)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_plane_products_of_any_size(dims, ranks, cout, dtype):
    """Core and 1 x 1 weight gradient against float64: chains of fp32 sums of at most 500 terms, 2e-6 of the largest entry per product."""
    from paper_2505_05086_amd import binding as B
    rng = np.random.default_rng(sum(dims) + sum(ranks))
    x = _dev(rng.standard_normal(dims), dtype)
    U = [_dev(np.linalg.qr(rng.standard_normal((n, r)))[0]) for n, r in zip(dims, ranks)]
    desc, conv = B.make_desc(dims, ranks, dtype), B.make_conv(cout, 1, 1, (1, 1), (0, 0), (1, 1), 1)
    S = torch.empty(ranks, device="cuda")
    ws = B.alloc_workspace(desc, conv, 0)
    ws.fill_(255)                                        # NaN wherever nothing was written
    sites = _sites(lambda: B.asi_core_project(desc, x, U, S, ws))
    want = _modes(x, U)
    assert float((S - want).abs().max() / want.abs().max()) <= 5e-6
    gy = _dev(rng.standard_normal((dims[0], cout) + dims[2:]), dtype)
    dW = torch.empty(cout, dims[1], 1, 1, device="cuda")
    ws.fill_(255)
    sites = _sites(lambda: B.asi_weight_grad_conv2d(desc, S, U, gy, conv, dW, False, ws))
    assert any("k_z_planes" in s or "+Z" in s for s in sites), sites
    assert not any(s.endswith(":Z1") for s in sites), sites
    xr = _modes(S, [u.t().contiguous() for u in U])
    ref = gy.double().transpose(0, 1).reshape(cout, -1).contiguous() @ xr.transpose(0, 1).reshape(dims[1], -1).t().contiguous()
    assert float((dW.view(cout, -1) - ref).abs().max() / ref.abs().max()) <= 1e-5


# The H and W products of the core on an intermediate in fp32, rows in 16-byte pieces and element by element: one, two and four waves a
# plane (up to 16, 32 and 64 rows), one to four blocks of columns, planes that take one product with the factors' Kronecker product where they
# come first (7 x 7, 8 x 8) and here do not, the last workgroup of planes not full.
@pytest.mark.parametrize("dims,ranks,form", [
    ((40, 90, 7, 7), (7, 9, 5, 5), "1, false"), ((6, 90, 8, 8), (3, 9, 8, 5), "1"), ((9, 60, 2, 16), (3, 5, 2, 9), "1"), ((33, 60, 49, 8), (4, 6, 6, 5), "1"),
    ((20, 60, 13, 17), (5, 6, 9, 11), "2, false"), ((18, 40, 31, 20), (4, 5, 13, 6), "2"), ((6, 80, 20, 45), (3, 7, 17, 31), "3, false"),
    ((8, 90, 29, 48), (3, 5, 9, 13), "3"), ((6, 80, 33, 50), (3, 7, 19, 31), "4, false"), ((5, 90, 64, 63), (2, 5, 29, 32), "4, false"), ((6, 80, 40, 52), (3, 7, 19, 31), "4")])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_core_by_planes_of_any_size(dims, ranks, form, dtype):
    """Against float64: chains of fp32 sums of at most 90 terms a mode, 2e-6 of the largest entry per product."""
    from paper_2505_05086_amd import binding as B
    rng = np.random.default_rng(sum(dims) + sum(ranks))
    x = _dev(rng.standard_normal(dims), dtype)
    U = [_dev(np.linalg.qr(rng.standard_normal((n, r)))[0]) for n, r in zip(dims, ranks)]
    desc, S = B.make_desc(dims, ranks, dtype), torch.empty(ranks, device="cuda")
    ws = B.alloc_workspace(desc, None, 0)
    ws.fill_(255)                                        # NaN wherever nothing was written
    sites = _sites(lambda: B.asi_core_project(desc, x, U, S, ws))
    assert any("k_core_planes<%s>" % form in s for s in sites), sites
    want = _modes(x, U)
    assert float((S - want).abs().max() / want.abs().max()) <= 5e-6


# The same on planes of up to 64 entries whose waves (the layers' together) fill the chip once and no longer, and one more plane than that: one
# product with the factors' Kronecker product.
@pytest.mark.parametrize("dims,ranks,layers,planes", [
    ((150, 256, 7, 7), (16, 40, 3, 3), 1, True), ((150, 257, 7, 7), (16, 40, 3, 3), 1, False), ((90, 128, 8, 8), (8, 80, 4, 5), 4, True),
    ((90, 129, 8, 8), (8, 80, 4, 5), 4, False), ((60, 128, 60, 1), (8, 24, 9, 1), 1, True), ((60, 129, 60, 1), (8, 24, 9, 1), 1, False),
    ((90, 256, 4, 4), (8, 60, 2, 2), 1, True), ((90, 257, 4, 4), (8, 60, 2, 2), 1, False)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_core_by_planes_or_by_the_kronecker_product(dims, ranks, layers, planes, dtype):
    """Against float64: chains of fp32 sums of at most 257 terms a mode, 2e-6 of the largest entry per product."""
    from paper_2505_05086_amd import binding as B
    rng = np.random.default_rng(sum(dims) + layers)
    xs = [_dev(rng.standard_normal(dims), dtype) for _ in range(layers)]
    U = [_dev(np.linalg.qr(rng.standard_normal((n, r)))[0]) for n, r in zip(dims, ranks)]
    desc, S = B.make_desc(dims, ranks, dtype), [torch.empty(ranks, device="cuda") for _ in xs]
    ws = [B.alloc_workspace(desc, None, 0) for _ in xs]
    for w in ws:
        w.fill_(255)                                     # NaN wherever nothing was written
    sites = _sites(lambda: B.asi_core_project_batch([desc] * layers, xs, [U] * layers, S, ws))
    assert any("k_core_planes" in s for s in sites) == planes, sites
    for s, x in zip(S, xs):
        want = _modes(x, U)
        assert float((s - want).abs().max() / want.abs().max()) <= 5e-6


# Cores of one to fifteen planes with ranks that are no multiple of four, and the first of sixteen: Z rides in the launch of G1, tiled or
# (the two after: a million entries of grad_out) streaming, where planes have up to 256 entries; last, planes that the plane kernels do not
# take (a row or a column longer than 64, a rank above 32), beside a G1 of few and of a million entries.
@pytest.mark.parametrize("dims,ranks,cout,k", [
    ((8, 6, 5, 5), (1, 1, 3, 3), 9, 3), ((64, 32, 7, 7), (2, 5, 5, 5), 32, 3), ((9, 6, 13, 9), (3, 5, 5, 6), 20, 1), ((5, 7, 16, 15), (3, 5, 1, 2), 3, 1),
    ((11, 9, 6, 7), (2, 8, 5, 3), 17, 3), ((64, 8, 14, 14), (4, 3, 7, 7), 100, 1), ((64, 5, 7, 8), (16, 1, 5, 7), 520, 1),
    ((16, 20, 1, 100), (4, 8, 1, 20), 30, 1), ((64, 9, 1, 200), (8, 5, 1, 40), 128, 1), ((32, 7, 128, 1), (4, 3, 30, 1), 64, 3), ((7, 9, 3, 80), (3, 4, 2, 29), 11, 3)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_small_cores_keep_g1_and_z_in_one_launch(dims, ranks, cout, k, dtype):
    """The weight gradient against float64: chains of fp32 sums of at most 1100 terms, 2e-6 of the largest entry per product."""
    from paper_2505_05086_amd import binding as B
    rng = np.random.default_rng(sum(dims) + sum(ranks))
    U = [_dev(np.linalg.qr(rng.standard_normal((n, r)))[0]) for n, r in zip(dims, ranks)]
    S = _dev(rng.standard_normal(ranks))
    gy = _dev(rng.standard_normal((dims[0], cout) + dims[2:]), dtype)
    desc, conv = B.make_desc(dims, ranks, dtype), B.make_conv(cout, k, k, (1, 1), (k // 2, k // 2), (1, 1), 1)
    dW = torch.empty(cout, dims[1], k, k, device="cuda")
    ws = B.alloc_workspace(desc, conv, 0)
    ws.fill_(255)                                        # NaN wherever nothing was written
    sites = _sites(lambda: B.asi_weight_grad_conv2d(desc, S, U, gy, conv, dW, False, ws))
    assert any(s.endswith(":G1+Z") for s in sites), sites
    xr = _modes(S, [u.t().contiguous() for u in U])
    want = torch.nn.grad.conv2d_weight(xr.cpu(), dW.shape, gy.double().cpu(), padding=k // 2).cuda()
    assert float((dW - want).abs().max() / want.abs().max()) <= 1e-5


# Planes whose waves fill the chip once (4096) and no longer, of few entries (one product with the factors' Kronecker product beyond the line) and
# of 160 entries a wave and more; the layers of a batch together.
@pytest.mark.parametrize("dims,ranks,layers,planes", [
    ((64, 64, 4, 5), (64, 64, 1, 2), 1, True), ((65, 64, 4, 5), (65, 64, 1, 2), 1, False), ((64, 70, 7, 7), (16, 64, 2, 3), 4, True), ((64, 70, 7, 7), (16, 64, 2, 3), 5, False),
    ((64, 64, 41, 6), (16, 64, 5, 1), 1, True), ((64, 66, 41, 6), (16, 65, 5, 1), 1, False), ((70, 64, 16, 10), (65, 64, 3, 2), 1, True)])
def test_z_by_planes_or_by_the_kronecker_product(dims, ranks, layers, planes):
    """A 1 x 1 gradient against float64: chains of fp32 sums of at most 500 terms, 2e-6 of the largest entry per product."""
    from paper_2505_05086_amd import binding as B
    rng = np.random.default_rng(sum(dims) + layers)
    cout = 3
    U = [_dev(np.linalg.qr(rng.standard_normal((n, r)))[0]) for n, r in zip(dims, ranks)]
    S, gy = _dev(rng.standard_normal(ranks)), _dev(rng.standard_normal((dims[0], cout) + dims[2:]))
    desc, conv = B.make_desc(dims, ranks, "f32"), B.make_conv(cout, 1, 1, (1, 1), (0, 0), (1, 1), 1)
    ws = [B.alloc_workspace(desc, conv, 0) for _ in range(layers)]
    for w in ws:
        w.fill_(255)
    dW = [torch.empty(cout, dims[1], 1, 1, device="cuda") for _ in range(layers)]
    sites = _sites(lambda: B.asi_weight_grad_conv2d_batch([desc] * layers, [S] * layers, [U] * layers, [gy] * layers, [conv] * layers, dW, [False] * layers, ws))
    z = [s.split("|")[1] for s in sites if s.endswith("Z")]
    assert len(z) == 1 and (", true>" not in z[0] and "k_ttm_mfma" not in z[0]) == planes, sites
    xr = _modes(S, [u.t().contiguous() for u in U])
    want = gy.double().transpose(0, 1).reshape(cout, -1).contiguous() @ xr.transpose(0, 1).reshape(dims[1], -1).t().contiguous()
    for d in dW:
        assert float((d.view(cout, -1) - want).abs().max() / want.abs().max()) <= 1e-5


def _check_factors(dims, ranks, modes, dtype, shift, label, tol, ws_bytes=None):
    from paper_2505_05086_amd import binding as B
    rng = np.random.default_rng(sum(dims) + sum(ranks) + shift)
    numel = int(np.prod(dims))
    flat = _dev(rng.standard_normal(numel + 1), dtype)
    x = flat[shift:shift + numel].view(dims)
    U = [_dev(np.linalg.qr(rng.standard_normal((n, r)))[0]) for n, r in zip(dims, ranks)]
    out = [torch.full_like(u, float("nan")) for u in U]
    desc = B.make_desc(dims, ranks, dtype)
    info = torch.full((1,), 7, dtype=torch.int32, device="cuda")
    ws = B.alloc_workspace(desc, None, 0)
    ws.fill_(255)
    assert ws_bytes is None or ws_bytes < ws.numel()
    ws, past = ws[:ws_bytes], ws[ws_bytes:] if ws_bytes else None
    sites = _sites(lambda: B.asi_compress(desc, x, U, out, ws, info))
    assert any(label in s for s in sites), sites
    assert int(info) == 0
    assert past is None or bool((past == 255).all())     # (nothing is written behind the scratch)
    for m in modes:
        a = x.double().movedim(m, 0).reshape(dims[m], -1)
        p = a @ (a.t().contiguous() @ U[m].double())
        q, r = torch.linalg.qr(p)
        want = q * torch.sign(torch.diagonal(r))
        assert float(torch.linalg.cond(p)) < 500
        err = float((out[m] - want).abs().max() / want.abs().max())
        assert err <= tol, (m, err)
    return sites


# Odd numbers of planes (two share an operand), a last tile that is not full, tiles whose bytes are no multiple of a copy's 16, one
# plane, one row, one column, planes of 64 and of one element, the last rows of an operand past the planes; one element off.  Tiles of 128 planes, whole and one over, of 256
# from 65536 planes on and of 512 (elements of up to 2 x 2 and 3 x 2 in bf16) from 131072 on.
@pytest.mark.parametrize("dims,ranks", [
    ((9, 9, 7, 7), (4, 5, 5, 5)), ((1, 163, 5, 5), (1, 9, 5, 3)), ((1, 1, 8, 8), (1, 1, 1, 1)), ((3, 701, 1, 8), (3, 7, 1, 8)), ((5, 103, 8, 3), (3, 4, 8, 3)),
    ((67, 65, 6, 7), (9, 8, 1, 7)), ((1, 4099, 1, 1), (1, 1, 1, 1)), ((700, 31, 8, 8), (6, 5, 8, 8)), ((257, 129, 4, 2), (5, 6, 3, 2)),
    ((16, 8, 3, 5), (5, 4, 2, 3)), ((43, 3, 2, 4), (5, 2, 2, 3)), ((257, 255, 3, 2), (7, 6, 2, 1)), ((256, 256, 2, 3), (7, 6, 2, 2)), ((512, 256, 2, 2), (6, 5, 1, 2)),
    ((521, 257, 3, 2), (6, 5, 2, 1))])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shift", [0, 1])
def test_tiny_planes_at_the_edges_of_their_tiles(dims, ranks, dtype, shift):
    """Sums in fp64 from the activation on: the factor is rounded to fp32 once, 1e-6 of its largest entry with a condition below 500
    (2^-53 of P's entries times the condition's square, as the factorisation is of P's Gram matrix, is below 1e-10)."""
    want = "k_subspace_tiny<%s, %s>" % ("float" if dtype == "f32" else "asi::bf16_t", "false" if shift else "true")
    _check_factors(dims, ranks, (2, 3), dtype, shift, want, 1e-6)


# Modes of 49 to 64 entries over a long inner extent: columns that are no multiple of four, of a block of 16, exactly whole blocks; one
# block and more blocks than waves, several outer slices; ranks of one to a whole block; one element off.
@pytest.mark.parametrize("dims,ranks,mode", [
    ((49, 1, 1, 128), (1, 1, 1, 16), 0), ((64, 5, 3, 11), (16, 3, 3, 7), 0), ((50, 33, 7, 7), (9, 7, 5, 5), 0), ((64, 65, 14, 14), (16, 7, 5, 5), 0),
    ((57, 700, 7, 7), (12, 6, 5, 5), 0), ((3, 63, 9, 17), (3, 13, 9, 7), 1), ((70, 53, 16, 16), (8, 16, 7, 7), 1), ((51, 1031, 129), (7, 9, 11), 0)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shift", [0, 1])
def test_subspace_step_of_49_to_64_entries(dims, ranks, mode, dtype, shift):
    """V is fp32: 2^-24 of its entries, which the condition (below 500) takes to 3e-5 of the factor's largest entry."""
    inner = int(np.prod(dims[mode + 1:]))
    want = "k_subspace_cols<%s, %s>" % ("float" if dtype == "f32" else "asi::bf16_t", "false" if shift or inner % 4 else "true")
    _check_factors(dims, ranks, (mode,), dtype, shift, want, 3e-5)


# Two and three modes' steps in one launch: both Gram forms and planes of one block; columns beside tiny planes (another mode's step, on its
# own, between them), beside a Gram form and planes of two blocks.
@pytest.mark.parametrize("dims,ranks,modes,names", [
    ((8, 32, 16, 16), (4, 8, 6, 6), (0, 1, 2, 3), ("gram", "gram", "planes")), ((64, 40, 7, 8), (16, 9, 5, 5), (0, 2, 3), ("cols", "tiny")),
    ((50, 5, 20, 28), (7, 5, 6, 9), (0, 1, 2, 3), ("cols", "gram", "planes")), ((4, 3, 12, 12), (2, 3, 4, 5), (0, 1, 2, 3), ("gram", "gram", "planes")),
    ((130, 9, 6, 8), (8, 5, 3, 5), (2, 3), ("tiny",)), ((7, 19, 9, 16), (3, 8, 4, 5), (0, 1, 2, 3), ("gram", "gram", "planes"))])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_subspace_steps_of_several_modes(dims, ranks, modes, names, dtype):
    """As for the steps alone: V in fp32 (columns), 3e-5; sums in fp64, 1e-6."""
    tn = "float" if dtype == "f32" else "asi::bf16_t"
    label = "k_subspace_%s<%s" % (("steps" if len(names) > 1 else names[0]), tn)
    sites = [s.split("|")[1] for s in _check_factors(dims, ranks, modes, dtype, 0, label, 3e-5 if "cols" in names else 1e-6)]
    steps = [s.split(" = ")[1].split(" + ") for s in sites if s.startswith("k_subspace_steps")]
    if len(names) > 1:                                   # the parts in their order, and none of them on its own
        assert [tuple(p[len("k_subspace_"):p.index("<")] for p in parts) for parts in steps] == [names], sites
        assert not any(s in parts for parts in steps for s in sites), sites
    else:
        assert steps == [], sites


# Scratch that holds a partial sum for every 256 columns of a pair product and for every 128 planes (or 16 KB of them) of up to 8 x 8, but not the more and
# smaller splits that the library asks room for: the same calls, with fewer splits.
@pytest.mark.parametrize("dims,ranks,ws_bytes", [
    ((84, 172, 7, 7), (84, 37, 7, 6), 5658112), ((6, 1182, 8, 8), (6, 124, 8, 8), 6432768), ((10, 156, 8, 8), (10, 98, 8, 8), 1130496),
    ((3, 70, 335), (3, 20, 40), 467968), ((2, 130, 402), (2, 50, 70), 1530624), ((172, 360, 5, 5), (2, 128, 5, 5), 9788160)])
def test_compress_with_scratch_for_fewer_partial_sums(dims, ranks, ws_bytes):
    """V is fp32 (pair products): 3e-5 of the factor's largest entry, as above."""
    _check_factors(dims, ranks, range(len(dims)), "f32", 0, "k_orth", 3e-5, ws_bytes)


# Tiles of 32 for ranks of four blocks over inner extents that are no multiple of four while 32 splits of them have a CU each (four tiles of 64
# rows); one row more, a multiple of four, a rank of three blocks: as wide as the rank.
@pytest.mark.parametrize("dims,ranks,mode,form", [
    ((3, 256, 333), (2, 64, 9), 1, "k_pair<%s, false, false, 32>"), ((3, 257, 333), (2, 64, 9), 1, "k_pair<%s, false, false, 64>"),
    ((3, 100, 332), (2, 49, 9), 1, "k_pair_vec<%s, 64>"), ((5, 100, 331), (2, 49, 9), 1, "k_pair<%s, false, false, 32>"),
    ((5, 100, 331), (2, 48, 9), 1, "k_pair<%s, false, false, 48>"), ((9, 130, 5, 7), (5, 50, 5, 5), 1, "k_pair<%s, false, false, 32>")])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_pair_tiles_over_inner_extents_that_are_no_multiple_of_four(dims, ranks, mode, form, dtype):
    """V is fp32: 3e-5 of the factor's largest entry, as above."""
    _check_factors(dims, ranks, (mode,), dtype, 0, form % ("float" if dtype == "f32" else "asi::bf16_t"), 3e-5)


# The splits of a pair product along the last mode at a rank of three blocks where one round trip of partial sums and two tie: 26 of them
# over 3232 columns of 376 rows (six tiles) and over 3328 of 77 (two).
@pytest.mark.parametrize("dims,ranks,least", [((16, 202, 376), (4, 16, 38), 26 * 6), ((64, 52, 77), (4, 16, 37), 26 * 2)])
def test_splits_of_pair_products_at_ranks_of_three_blocks(dims, ranks, least):
    """V is fp32: 3e-5 of the factor's largest entry, as above."""
    from paper_2505_05086_amd import binding as B
    _check_factors(dims, ranks, (2,), "f32", 0, "k_pair<float, true, false, 48>", 3e-5)
    rng = np.random.default_rng(3)
    x, U = _dev(rng.standard_normal(dims)), [_dev(np.linalg.qr(rng.standard_normal((n, r)))[0]) for n, r in zip(dims, ranks)]
    desc, info = B.make_desc(dims, ranks, "f32"), torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = B.alloc_workspace(desc, None, 0)
    B.asi_profile_enable(True)
    try:
        B.asi_compress(desc, x, U, [torch.empty_like(u) for u in U], ws, info)
        wgs = [v["workgroups"] for s, v in B.asi_profile_report().items() if "k_pair<float, true, false, 48>" in s]
    finally:
        B.asi_profile_enable(False)
    assert len(wgs) == 1 and wgs[0] >= least, wgs        # (and those of the partial sums that ride along)


@pytest.mark.parametrize("dims,ranks,dout,ws_bytes", [((11, 297, 200), (6, 34, 60), 904, 7832576), ((5, 352, 66), (3, 44, 55), 1623, 8784128)])
def test_linear_gradient_with_scratch_for_fewer_partial_sums(dims, ranks, dout, ws_bytes):
    """Against float64: four chained fp32 sums of at most 352 terms, 2e-6 of the largest entry each."""
    from paper_2505_05086_amd import binding as B
    rng = np.random.default_rng(dout)
    U = [_dev(np.linalg.qr(rng.standard_normal((n, r)))[0]) for n, r in zip(dims, ranks)]
    S, gy = _dev(rng.standard_normal(ranks)), _dev(rng.standard_normal(dims[:2] + (dout,)))
    desc = B.make_desc(dims, ranks, "f32")
    ws = B.alloc_workspace(desc, None, dout)
    assert ws_bytes < ws.numel()
    ws.fill_(255)
    dW = torch.empty(dout, dims[2], device="cuda")
    B.asi_weight_grad_linear(desc, S, U, gy, dout, dW, False, ws[:ws_bytes])
    assert bool((ws[ws_bytes:] == 255).all())            # (nothing is written behind the scratch)
    xr = _modes(S, [u.t().contiguous() for u in U])
    want = gy.double().reshape(-1, dout).t().contiguous() @ xr.reshape(-1, dims[2])
    assert float((dW - want).abs().max() / want.abs().max()) <= 1e-5


# The pair product of a linear gradient (dout rows of the core's r1 x r2 columns, r3 outputs): tiles of 32 up to 128 columns while every tile
# has a CU (128 rows of tiles of a rank of four blocks), the widest that the rank fills otherwise; the last
# block and the last row of tiles not full.
@pytest.mark.parametrize("dims,ranks,dout,tile", [
    ((20, 30, 70), (8, 16, 50), 131, 32), ((20, 30, 70), (6, 22, 50), 131, 64), ((20, 50, 90), (3, 42, 33), 64, 32), ((20, 50, 90), (6, 9, 40), 4100, 32),
    ((9, 30, 150), (2, 9, 100), 70, 32), ((9, 30, 90), (5, 7, 64), 8192, 32), ((9, 30, 90), (5, 7, 64), 8193, 64), ((20, 30, 70), (8, 16, 32), 70, 32),
    ((20, 30, 70), (8, 16, 15), 70, 16)])
def test_pair_product_of_few_columns(dims, ranks, dout, tile):
    """Against float64: four chained fp32 sums of at most 270 terms, 2e-6 of the largest entry each."""
    from paper_2505_05086_amd import binding as B
    rng = np.random.default_rng(sum(ranks) + dout)
    U = [_dev(np.linalg.qr(rng.standard_normal((n, r)))[0]) for n, r in zip(dims, ranks)]
    S, gy = _dev(rng.standard_normal(ranks)), _dev(rng.standard_normal(dims[:2] + (dout,)))
    desc, dW = B.make_desc(dims, ranks, "f32"), torch.empty(dout, dims[2], device="cuda")
    ws = B.alloc_workspace(desc, None, dout)
    ws.fill_(255)
    sites = _sites(lambda: B.asi_weight_grad_linear(desc, S, U, gy, dout, dW, False, ws))
    assert any("k_pair<float, true, false, %d>" % tile in s for s in sites), sites
    xr = _modes(S, [u.t().contiguous() for u in U])
    want = gy.double().reshape(-1, dout).t().contiguous() @ xr.reshape(-1, dims[2])
    assert float((dW - want).abs().max() / want.abs().max()) <= 1e-5


# Planes in 33 to 64 tiles: half as many workgroups where their partial sums alone would need a launch of the summing tree (up to 32 x 32),
# not where another mode's do (a Gram form of 36 splits) or a pair product carries it (70 entries over 3 x 256 columns).
# wgs: of the launch that the planes share with the Gram forms before them.
@pytest.mark.parametrize("dims,ranks,wgs,tree", [
    ((8, 32, 16, 16), (4, 4, 5, 5), 16 + 16 + 32, False), ((4, 38, 20, 23), (2, 4, 6, 7), 18 + 19, False), ((1, 133, 16, 3), (1, 9, 5, 2), 7 + 34, False),
    ((6, 32, 28, 28), (3, 4, 9, 9), 49 + 42 + 48, True), ((3, 70, 16, 16), (2, 4, 5, 5), 18 + 53, False), ((4, 40, 33, 20), (2, 4, 9, 6), 40, True)])
def test_workgroups_of_planes_in_33_to_64_tiles(dims, ranks, wgs, tree):
    """Sums in fp64 from the activation on: 1e-6, as above."""
    sites = _check_factors(dims, ranks, (2, 3), "f32", 0, "k_subspace_planes", 1e-6)
    assert [w for s, w in sites.items() if "k_subspace_planes" in s] == [wgs], sites
    assert any("presum" in s for s in sites) == tree, sites
