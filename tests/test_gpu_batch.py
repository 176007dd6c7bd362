"""Batched entry points: every launch serves several layers.  The factors must be bit-identical to
the single-layer calls (which the parity tests check against the float64 oracle); core and weight
gradient may differ at fp32 rounding level, because a batch takes the m-mode products of the
core projection in one common order."""
import numpy as np
import pytest
import torch

from asi_inputs import CONFIGS, Layer, LayerStream
from paper_2505_05086_amd.runner import BatchRunner, LayerRunner

pytestmark = pytest.mark.gpu


def _run_pair(cfg_index, layer_ids, steps=2):
    cfg = CONFIGS[cfg_index]
    _run_layers(cfg_index, layer_ids, [cfg.layers[i] for i in layer_ids],
                [LayerStream(cfg.index, i, cfg.layers[i], cfg.theta) for i in layer_ids], steps)


def _run_layers(cfg_index, layer_ids, layers, streams, steps):
    singles = [LayerRunner(lay) for lay in layers]
    batch = BatchRunner(layers)
    for r, b, st in zip(singles, batch.runs, streams):
        r.set_factors(st.u_prev0())
        b.set_factors(st.u_prev0())
    for t in range(steps):
        A = [r.upload(st.activation(t)) for r, st in zip(singles, streams)]
        dY = [r.upload(st.grad_out(t)) for r, st in zip(singles, streams)]
        for r, a, g in zip(singles, A, dY):
            r.step(a, g)
        batch.step(A, dY)
        torch.cuda.synchronize()
        for li, (r, b) in enumerate(zip(singles, batch.runs)):
            assert int(r.info.item()) == 0 and int(b.info.item()) == 0
            for m, (u1, u2) in enumerate(zip(r.factors(), b.factors())):
                assert torch.equal(u1, u2), f"cfg{cfg_index} layer {layer_ids[li]} step {t} factor {m}"
            for name, x, y in (("core", r.S, b.S), ("dW", r.dW, b.dW)):
                err = float((x - y).abs().max() / x.abs().max())
                assert err <= 2e-6, f"cfg{cfg_index} layer {layer_ids[li]} step {t} {name}: {err:.2e}"


def test_batch_equals_single_config2_all_layers():
    _run_pair(2, [0, 1, 2, 3])


def test_batch_equals_single_config3_mixed_shapes_and_groups():
    _run_pair(3, list(range(len(CONFIGS[3].layers))))


def test_batch_equals_single_config5_linear_bf16():
    _run_pair(5, list(range(len(CONFIGS[5].layers))), steps=1)


@pytest.mark.parametrize("hw,k,r1,cout", [((7, 8), 3, 5, 130), ((8, 8), 3, 7, 130), ((7, 7), 5, 3, 64), ((14, 13), 3, 5, 70), ((7, 7), 1, 4, 33)])
def test_batch_of_equal_layers_shares_the_correlation(hw, k, r1, cout):
    """Three equal layers: the correlation's K is split into fewer parts than for one (the single layer's is the reference that
    the parity tests hold against the oracle); slabs of Z one step below and above the short form's, a partial last split."""
    lay = Layer("share", (9, 40, *hw), (r1, 18, 5, 5), "f32", "conv2d", cout, k=k, pad=(k - 1) // 2, alpha=0.7, noise=1e-2)
    _run_layers(9, [21, 22, 23], [lay] * 3, [LayerStream(9, 21 + i, lay) for i in range(3)], 1)


def test_batch_of_one_and_repeated_layer():
    _run_pair(1, [0])
    _run_pair(2, [1, 1, 2])


def test_batch_of_eight_layers():
    """The largest batch the ABI takes: every launch serves eight argument blocks."""
    _run_pair(2, [0, 1, 2, 3, 3, 2, 1, 0], steps=1)
    _run_pair(3, [0, 3, 0, 3, 1, 2, 0, 3], steps=1)


def test_correlations_that_share_no_launch_are_split_like_layers_alone():
    """3x3, 1x1 and 5x5 kernels over the same map: the correlations of such a batch run one after the other, and each must fill
    the chip by itself.  A second 3x3 layer shares its launch, and the two take fewer splits together than two alone."""
    from paper_2505_05086_amd import binding as B

    def corr_workgroups(step):
        torch.cuda.synchronize()
        B.asi_profile_enable(True)
        try:
            step()
            torch.cuda.synchronize()
            return {s: v["workgroups"] for s, v in B.asi_profile_report().items() if "k_corr" in s}
        finally:
            B.asi_profile_enable(False)

    layers = [Layer("mix", (16, 128, 7, 7), (12, 48, 5, 5), "f32", "conv2d", 512, k=k, pad=(k - 1) // 2, alpha=0.7, noise=1e-2)
              for k in (3, 1, 5)]
    streams = [LayerStream(9, 31 + i, lay) for i, lay in enumerate(layers)]
    _run_layers(9, [31, 32, 33], layers, streams, 1)
    alone = {}
    for lay, st in zip(layers, streams):
        r = LayerRunner(lay)
        r.set_factors(st.u_prev0())
        a, g = r.upload(st.activation(0)), r.upload(st.grad_out(0))
        alone.update(corr_workgroups(lambda: r.step(a, g)))
    assert len(alone) == 3

    def together(idx):
        batch = BatchRunner([layers[i] for i in idx])
        for r, i in zip(batch.runs, idx):
            r.set_factors(streams[i].u_prev0())
        A = [r.upload(streams[i].activation(0)) for r, i in zip(batch.runs, idx)]
        dY = [r.upload(streams[i].grad_out(0)) for r, i in zip(batch.runs, idx)]
        return corr_workgroups(lambda: batch.step(A, dY))

    assert together([0, 1, 2]) == alone
    four = together([0, 1, 2, 0])
    pair = [s for s in alone if "<9, " in s][0]
    assert {s: w for s, w in four.items() if s != pair} == {s: w for s, w in alone.items() if s != pair}
    assert alone[pair] <= four[pair] <= 2 * alone[pair]


@pytest.mark.parametrize("count,parts", [(1, 3), (2, 3), (4, 2), (8, 2)])
def test_steps_of_a_batch_share_a_launch_while_it_fills_the_chip_no_more_often(count, parts):
    """16 x 32 x 20 x 20: 50 and 64 workgroups of two Gram forms, one resident per CU as in a joined launch, and 128 of the planes, of which
    two are.  Two layers fill 256 CUs twice joined (484) and three times apart; four layers' Gram forms join (456: twice either way) and their
    planes do not (968: four times instead of three); eight layers' Gram forms would be 912 workgroups, four fillings like apart: joined."""
    from paper_2505_05086_amd import binding as B
    lay = Layer("steps", (16, 32, 20, 20), (4, 8, 6, 6), "f32", "conv2d", 9, k=1, alpha=0.7, noise=1e-2)
    streams = [LayerStream(9, 61 + i, lay) for i in range(count)]
    _run_layers(9, [61 + i for i in range(count)], [lay] * count, streams, 1)
    batch = BatchRunner([lay] * count)
    for r, st in zip(batch.runs, streams):
        r.set_factors(st.u_prev0())
    A = [r.upload(st.activation(0)) for r, st in zip(batch.runs, streams)]
    torch.cuda.synchronize()
    B.asi_profile_enable(True)
    try:
        batch.compress(A)
        torch.cuda.synchronize()
        sites = [s.split("|")[1] for s in B.asi_profile_report()]
    finally:
        B.asi_profile_enable(False)
    steps = [s for s in sites if s.startswith("k_subspace_steps")]
    assert [s.count("k_subspace_") - 1 for s in steps] == [parts], sites
    assert any(s.startswith("k_subspace_planes") for s in sites) == (parts < 3), sites


@pytest.mark.parametrize("ratio", [0.9, 0.02])
def test_batch_with_more_runs_of_slices_than_workgroups_of_the_orthogonalisation(ratio):
    """Eight layers of 3, 700 and 620 rows: 344 runs of 32 rows, two a workgroup where the chip holds 256; the first pass certified (0.9) and, in the
    two long modes, measured and repeated (0.02).  Bit for bit the factors of single layers, whose workgroups take a run each."""
    from paper_2505_05086_amd import binding as B
    dims, ranks = (3, 700, 620), (3, 20, 18)
    desc = B.make_desc(dims, ranks, "f32")
    A, U, one, many, ws, info = [], [], [], [], [], []
    for i in range(8):
        rng = np.random.default_rng(900 + i)
        x = rng.standard_normal(ranks)
        for m, (n, r) in enumerate(zip(dims, ranks)):
            q = np.linalg.qr(rng.standard_normal((n, r)))[0] * (ratio ** (np.arange(r) / (r - 1)))
            x = np.moveaxis(np.tensordot(q, x, axes=(1, m)), 0, m)
        A.append(torch.from_numpy(np.ascontiguousarray(x / np.abs(x).max(), dtype=np.float32)).cuda())
        U.append([torch.from_numpy(np.ascontiguousarray(np.linalg.qr(rng.standard_normal((n, r)))[0], dtype=np.float32)).cuda() for n, r in zip(dims, ranks)])
        one.append([torch.full_like(u, float("nan")) for u in U[-1]])
        many.append([torch.full_like(u, float("nan")) for u in U[-1]])
        ws.append(B.alloc_workspace(desc, None, 0))
        info.append(torch.full((1,), 7, dtype=torch.int32, device="cuda"))
    for i in range(8):
        B.asi_compress(desc, A[i], U[i], one[i], ws[i], info[i])
        assert int(info[i]) == 0
    for w in ws:
        w.fill_(255)
    B.asi_compress_batch([desc] * 8, A, U, many, ws, info)
    for i in range(8):
        assert int(info[i]) == 0
        for a, b in zip(one[i], many[i]):
            assert torch.equal(a, b), i
            assert float((b.double().t() @ b.double() - torch.eye(b.shape[1], device="cuda", dtype=torch.float64)).abs().max()) < 1e-5
