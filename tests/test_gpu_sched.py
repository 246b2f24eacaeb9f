"""Two-stream scheduling (Algorithm 2, §IV-E) and the interaction head on the
GPU: the enqueue order of each mode, and the cross network + MLP forward
against the fp64 oracle in every mode."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2606_21101_amd import dpi

pytestmark = pytest.mark.gpu


def recording_ops(n, module, log):
    ops, keep = [], []
    for i in range(n):
        def fn(ctx, stream, i=i):
            log.append((module, i, stream))
            return dpi.DPI_OK
        cb = dpi.DPI_OP_FN(fn)
        keep.append(cb)
        ops.append(dpi.dpi_op(cb, None))
    return ops, keep


@pytest.mark.parametrize("ne,ni", [(3, 5), (4, 4), (6, 1), (0, 3)])
def test_enqueue_order_and_streams(ne, ni):
    se, si = torch.cuda.Stream(), torch.cuda.Stream()
    after = torch.cuda.current_stream()
    for mode in (dpi.DPI_SCHED_BREADTH_FIRST, dpi.DPI_SCHED_DEPTH_FIRST, dpi.DPI_SCHED_ONE_STREAM):
        log = []
        eo, k1 = recording_ops(ne, "E", log)
        io, k2 = recording_ops(ni, "I", log)
        dpi.dpi_launch_two_streams(eo, io, mode, se, si, after)
        torch.cuda.synchronize()
        order = [(m, i) for m, i, _ in log]
        if mode == dpi.DPI_SCHED_BREADTH_FIRST:
            assert order == oracle.breadth_first_order(ne, ni)
        else:
            assert order == [("E", i) for i in range(ne)] + [("I", j) for j in range(ni)]
        streams = {m: {s for mm, _, s in log if mm == m} for m in ("E", "I")}
        if ne:
            assert streams["E"] == {se.cuda_stream}
        if ni:
            assert streams["I"] == ({se.cuda_stream} if mode == dpi.DPI_SCHED_ONE_STREAM else {si.cuda_stream})


def make_head(rng, B, d, n_cross, mlp_dims):
    cw = [torch.from_numpy((rng.standard_normal((d, d)) / np.sqrt(d)).astype(np.float32)).cuda() for _ in range(n_cross)]
    cb = [torch.from_numpy((rng.standard_normal(d) * 0.1).astype(np.float32)).cuda() for _ in range(n_cross)]
    mw, mb, prev = [], [], d
    for h in mlp_dims:
        mw.append(torch.from_numpy((rng.standard_normal((h, prev)) / np.sqrt(prev)).astype(np.float32)).cuda())
        mb.append(torch.from_numpy((rng.standard_normal(h) * 0.1).astype(np.float32)).cuda())
        prev = h
    return dpi.DcnHead(B, d, cw, cb, mw, mb), cw, cb, mw, mb


@pytest.mark.parametrize("B,d,n_cross,mlp_dims", [(300, 64, 2, [128, 32]), (1000, 416, 3, [512, 256, 130]),
                                                  (7, 13, 1, [5])])
def test_dcn_forward_all_modes(B, d, n_cross, mlp_dims):
    rng = np.random.default_rng(B + d)
    head, cw, cb, mw, mb = make_head(rng, B, d, n_cross, mlp_dims)
    x0_np = (rng.standard_normal((B, d)) * 0.5).astype(np.float32)
    x0 = torch.from_numpy(x0_np).cuda()
    ref_x, ref_h, mag_x, mag_h = oracle.dcn_forward(x0_np, [w.cpu().numpy() for w in cw], [b.cpu().numpy() for b in cb],
                                                    [w.cpu().numpy() for w in mw], [b.cpu().numpy() for b in mb])
    tol_x = n_cross * (d + 8) * 2.0 ** -24
    dims = [d] + mlp_dims
    tol_h = sum(k + 8 for k in dims[:-1]) * 2.0 ** -24
    se, si = torch.cuda.Stream(), torch.cuda.Stream()
    after = torch.cuda.current_stream()
    outs = []
    for mode in (dpi.DPI_SCHED_BREADTH_FIRST, dpi.DPI_SCHED_DEPTH_FIRST, dpi.DPI_SCHED_ONE_STREAM):
        oc = torch.full((B, d), float("nan"), device="cuda")
        om = torch.full((B, mlp_dims[-1]), float("nan"), device="cuda")
        marks = torch.zeros(2, dtype=torch.int64, device="cuda")
        head.forward(x0, oc, om, mode, se, si, after, marks)
        torch.cuda.synchronize()
        yx, yh = oc.double().cpu().numpy(), om.double().cpu().numpy()
        assert np.all(np.abs(yx - ref_x) <= tol_x * mag_x + 1e-30), f"cross, mode {mode}"
        assert np.all(np.abs(yh - ref_h) <= tol_h * mag_h + 1e-30), f"mlp, mode {mode}"
        assert torch.all(marks > 0)
        outs.append((oc, om))
    for oc, om in outs[1:]:       # the order of enqueueing changes nothing computed
        assert torch.equal(oc, outs[0][0]) and torch.equal(om, outs[0][1])


def test_dcn_forward_waits_for_after_stream():
    rng = np.random.default_rng(3)
    B, d = 2048, 64
    head, *_ = make_head(rng, B, d, 2, [64])
    x0 = torch.zeros((B, d), device="cuda")
    after = torch.cuda.Stream()
    se, si = torch.cuda.Stream(), torch.cuda.Stream()
    src = torch.from_numpy((rng.standard_normal((B, d))).astype(np.float32)).cuda()
    torch.cuda.synchronize()
    with torch.cuda.stream(after):
        for _ in range(20):                       # queue some work that writes x0 last
            x0.copy_(src)
    oc1 = torch.empty((B, d), device="cuda")
    om1 = torch.empty((B, 64), device="cuda")
    head.forward(x0, oc1, om1, dpi.DPI_SCHED_BREADTH_FIRST, se, si, after)
    after.synchronize()
    oc2 = torch.empty_like(oc1)
    om2 = torch.empty_like(om1)
    head.forward(x0, oc2, om2, dpi.DPI_SCHED_BREADTH_FIRST, se, si, after)
    after.synchronize()
    assert torch.equal(oc1, oc2) and torch.equal(om1, om2)


@pytest.mark.parametrize("B,d,mlp_dims", [
    (1, 1, [1]),                # one K block of one column
    (33, 31, [33]),             # odd depths: dword reads; a row and a column past the tile
    (31, 34, [32, 66]),         # depths 2 mod 4: pairs of dwords; two K blocks
    (64, 96, [36, 100]),        # whole rounds of three K blocks, none left over
    (65, 128, [68, 7]),         # ... with one left over
    (40, 164, [4]),             # ... with two and a part
    (24577, 4, [256]),          # 64-column tiles (more than 1536 of them), a row past the last
    (24577, 6, [250]),          # ... read as pairs, columns that are no multiple of 4
    (24577, 7, [253]),          # ... read as quads shifted back into the row
    (8200, 3, [32, 35]), (40, 3, [1, 9]),   # depths of 1 and 3: single columns
    (40, 5, [6, 1000, 34]),     # two groups share K: one K block for both, 32 of them
])
def test_layer_tiles(B, d, mlp_dims):
    """The layer kernel at the edges of its tiles, K blocks and read widths; the
    cross network also where out_cross is x0."""
    rng = np.random.default_rng(B + d)
    head, cw, cb, mw, mb = make_head(rng, B, d, 1, mlp_dims)
    x0_np = (rng.standard_normal((B, d)) * 0.5).astype(np.float32)
    x0 = torch.from_numpy(x0_np).cuda()
    ref_x, ref_h, mag_x, mag_h = oracle.dcn_forward(x0_np, [w.cpu().numpy() for w in cw], [b.cpu().numpy() for b in cb],
                                                    [w.cpu().numpy() for w in mw], [b.cpu().numpy() for b in mb])
    tol_x = (d + 8) * 2.0 ** -24
    tol_h = sum(k + 8 for k in ([d] + mlp_dims)[:-1]) * 2.0 ** -24
    s = torch.cuda.Stream()
    oc = torch.full((B, d), float("nan"), device="cuda")
    om = torch.full((B, mlp_dims[-1]), float("nan"), device="cuda")
    head.forward(x0, oc, om, dpi.DPI_SCHED_BREADTH_FIRST, s, torch.cuda.Stream())
    torch.cuda.synchronize()
    assert np.all(np.abs(oc.double().cpu().numpy() - ref_x) <= tol_x * mag_x + 1e-30)
    assert np.all(np.abs(om.double().cpu().numpy() - ref_h) <= tol_h * mag_h + 1e-30)
    om2 = torch.empty_like(om)
    head.forward(x0, x0, om2, dpi.DPI_SCHED_ONE_STREAM, s, s)
    torch.cuda.synchronize()
    assert torch.equal(x0, oc)


def test_layer_special_values():
    """Infinities and NaN stay in their own rows and columns (depths with a part of a K block)."""
    B, d = 40, 37
    rng = np.random.default_rng(11)
    head, cw, cb, mw, mb = make_head(rng, B, d, 1, [35])
    x0 = torch.from_numpy(rng.standard_normal((B, d)).astype(np.float32)).cuda()
    x0[3, 36], x0[20, 0] = float("inf"), float("nan")
    s = torch.cuda.Stream()
    oc, om = torch.empty((B, d), device="cuda"), torch.empty((B, 35), device="cuda")
    head.forward(x0, oc, om, dpi.DPI_SCHED_BREADTH_FIRST, s, torch.cuda.Stream())
    torch.cuda.synchronize()
    rows = [b for b in range(B) if b not in (3, 20)]
    assert torch.isfinite(oc[rows]).all() and torch.isfinite(om[rows]).all()
    assert torch.isnan(oc[20]).all() and not torch.isfinite(oc[3]).any()


@pytest.mark.parametrize("B,d,mlp_dims", [
    # tiles of 64 by 64 in both epilogues: 12, 13 and 14 K blocks (three in flight), each read width
    (16400, 384, [1024]), (16400, 416, [1024]), (16400, 448, []), (16400, 390, []), (16400, 391, [1021]),
    (2000, 1568, []), (2000, 1566, []), (2000, 1567, []), (2000, 1600, []),     # ... at depth
    # ... with two groups: 25 K blocks each, 51 in all, and the other read widths
    (1000, 1600, []), (1000, 1632, []), (1000, 1634, []), (1000, 1655, [1601]),
    # tiles of 32 by 32: two groups (16 K blocks each); at depth four (12 and 13 each), and two sums
    (33, 1024, []), (33, 1536, []), (33, 1539, [35]), (40, 1538, []), (40, 1568, []),
    (300, 1600, []), (300, 1601, []), (300, 1602, []),
])
def test_layer_variants(B, d, mlp_dims):
    """Each form of the layer kernel over several rounds of K blocks, in both epilogues; with no MLP listed, one of d."""
    rng = np.random.default_rng(B + d)
    mlp_dims = mlp_dims or [d]
    head, cw, cb, mw, mb = make_head(rng, B, d, 1, mlp_dims)
    x0_np = (rng.standard_normal((B, d)) * 0.5).astype(np.float32)
    ref_x, ref_h, mag_x, mag_h = oracle.dcn_forward(x0_np, [w.cpu().numpy() for w in cw], [b.cpu().numpy() for b in cb],
                                                    [w.cpu().numpy() for w in mw], [b.cpu().numpy() for b in mb])
    oc = torch.full((B, d), float("nan"), device="cuda")
    om = torch.full((B, mlp_dims[-1]), float("nan"), device="cuda")
    head.forward(torch.from_numpy(x0_np).cuda(), oc, om, dpi.DPI_SCHED_BREADTH_FIRST, torch.cuda.Stream(),
                 torch.cuda.Stream())
    torch.cuda.synchronize()
    tol = (d + 8) * 2.0 ** -24
    assert np.all(np.abs(oc.double().cpu().numpy() - ref_x) <= tol * mag_x + 1e-30)
    assert np.all(np.abs(om.double().cpu().numpy() - ref_h) <= tol * mag_h + 1e-30)


@pytest.mark.parametrize("n_cross,mlp_dims", [(1, [48]), (2, [30, 48]), (3, [50, 20, 48])])
@pytest.mark.parametrize("over", ["cross", "mlp", "shifted"])
def test_outputs_over_x0(n_cross, mlp_dims, over):
    """An output that is x0, or overlaps it, takes nothing from the other module's input, in every mode."""
    B, d = 700, 48
    rng = np.random.default_rng(n_cross)
    head, cw, cb, mw, mb = make_head(rng, B, d, n_cross, mlp_dims)
    x0_np = (rng.standard_normal((B, d)) * 0.5).astype(np.float32)
    ref_x, ref_h, mag_x, mag_h = oracle.dcn_forward(x0_np, [w.cpu().numpy() for w in cw], [b.cpu().numpy() for b in cb],
                                                    [w.cpu().numpy() for w in mw], [b.cpu().numpy() for b in mb])
    tol_x = n_cross * (d + 8) * 2.0 ** -24
    tol_h = sum(k + 8 for k in ([d] + mlp_dims)[:-1]) * 2.0 ** -24
    se, si = torch.cuda.Stream(), torch.cuda.Stream()
    for mode in (dpi.DPI_SCHED_BREADTH_FIRST, dpi.DPI_SCHED_DEPTH_FIRST, dpi.DPI_SCHED_ONE_STREAM):
        store = torch.zeros(2 * B * d, device="cuda")
        x0 = store[: B * d].view(B, d)
        x0.copy_(torch.from_numpy(x0_np))
        oc, om = (torch.full((B, d), float("nan"), device="cuda") for _ in range(2))
        if over == "mlp":
            om = x0
        else:
            oc = x0 if over == "cross" else store[64: 64 + B * d].view(B, d)
        head.forward(x0, oc, om, mode, se, si)
        torch.cuda.synchronize()
        assert np.all(np.abs(oc.double().cpu().numpy() - ref_x) <= tol_x * mag_x + 1e-30), f"cross, mode {mode}"
        assert np.all(np.abs(om.double().cpu().numpy() - ref_h) <= tol_h * mag_h + 1e-30), f"mlp, mode {mode}"
