"""Rows of every byte length the lookups take, through each kernel that reads
them, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_21101_amd import dpi
from paper_2606_21101_amd.lookup import FusedLookup
from parity import check_outputs
from test_gpu_edges import check, random_problem, run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,dtype", [(12, 0), (60, 0), (100, 0), (192, 0), (24, 1), (120, 1)])
def test_one_class_rows_shorter_than_their_lanes(dim, dtype):
    """Fields of one dim whose rows do not fill their power of two of lanes,
    pooled through the plan's partition (the single-row-class kernel)."""
    rng = np.random.default_rng(500 + dim)
    dims, dtypes = [dim] * 3, [dtype] * 3
    tables, ids, offs, pool = random_problem(rng, dims, dtypes, 61, 40, rows=70)
    for od in (torch.float32, torch.float16):
        for W in (1, 29):
            out, st, _, _ = run_case(tables, ids, offs, pool, 61, od, num_waves=W)
            assert st == dpi.DPI_OK
            check(tables, ids, offs, pool, 61, out)


ODD_ROWS = {
    "f32": ([1, 2, 3, 5, 7, 10, 18, 50, 255], [0] * 9),     # 4 .. 1020 bytes
    "f16": ([2, 4, 6, 10, 18, 50, 254, 510], [1] * 8),      # 4 .. 1020 bytes
    "both": ([1, 6, 4, 8, 13, 34, 300], [0, 1, 0, 1, 0, 1, 0]),   # with a row above 1024 bytes
}


@pytest.mark.parametrize("name", sorted(ODD_ROWS))
@pytest.mark.parametrize("B,max_len", [(37, 30), (5, 300), (1100, 9)])   # one launch; long bags; planned first
def test_rows_of_any_length(name, B, max_len):
    dims, dtypes = ODD_ROWS[name]
    rng = np.random.default_rng(B + len(dims))
    tables, ids, offs, pool = random_problem(rng, dims, dtypes, B, max_len, rows=40)
    for W, flags in ((0, 0), (41, 0), (0, dpi.DPI_FLAG_INPUT_FIRST)):
        for od in (torch.float32, torch.float16):
            out, st, _, _ = run_case(tables, ids, offs, pool, B, od, num_waves=W, flags=flags)
            assert st == dpi.DPI_OK
            check(tables, ids, offs, pool, B, out)


@pytest.mark.parametrize("dims,dtype", [([1, 1], 0), ([3, 3], 0), ([7, 7, 7], 0), ([10, 11], 0), ([6, 6], 1), ([50], 1),
                                        ([3, 4, 1, 2], 0), ([8, 2, 6], 1)])   # rows below 16 bytes beside one of 16
@pytest.mark.parametrize("B", [1, 129, 1500])
def test_onehot_rows_of_any_length(dims, dtype, B):
    rng = np.random.default_rng(B + sum(dims))
    tables, _, _, pool = random_problem(rng, dims, [dtype] * len(dims), B, 1, rows=33)
    ids = rng.integers(0, 33, B * len(dims)).astype(np.int32)
    ids[-1] = 32                                         # the last row: a piece ends where the table does
    for od in (torch.float32, torch.float16):
        out, st, _, _ = run_case(tables, ids, None, pool, B, od)
        assert st == dpi.DPI_OK
        check(tables, ids, None, pool, B, out, exact=od == torch.float32)


def test_row_before_a_neighbour_stays_in_its_columns():
    """A field's last piece is shifted back into its row: the next field's
    columns are untouched by it, and so is what follows the block."""
    rng = np.random.default_rng(77)
    dims, B = [5, 3, 9], 64
    tables, ids, offs, pool = random_problem(rng, dims, [0, 0, 0], B, 6)
    tables[1][:] = np.inf
    out, st, fl, plan = run_case(tables, ids, offs, pool, B)
    assert st == dpi.DPI_OK
    store = torch.full((B * fl.total_dim + 64,), 7.0, device="cuda")
    fl.lookup(plan, torch.from_numpy(ids).cuda(), torch.from_numpy(offs).cuda(), out=store[: B * fl.total_dim])
    torch.cuda.synchronize()
    assert torch.equal(store[: B * fl.total_dim].view(B, -1), out) and bool((store[B * fl.total_dim:] == 7.0).all())
    assert bool(torch.isfinite(out[:, :5]).all()) and bool(torch.isfinite(out[:, 8:]).all())


@pytest.mark.parametrize("T,dim,dtype", [(3, 15, 0), (70, 9, 0), (5, 30, 1), (70, 60, 1), (2, 255, 0), (4, 32, 0)])
@pytest.mark.parametrize("B", [1, 7, 8, 9, 777])
def test_onehot_pieces(T, dim, dtype, B):
    """One-hot fields of one dim (one launch, and more fields than that takes):
    the rows are copied bit for bit, an id outside its table gives zeros and is
    reported, -0 becomes +0, and nothing past the block is written."""
    rng = np.random.default_rng(T + dim + B)
    tables = [rng.standard_normal((19, dim)).astype(np.float16 if dtype else np.float32) for _ in range(T)]
    tables[0][3] = -0.0
    tables[0][4, :2] = [np.inf, -np.inf]
    ids = rng.integers(0, 19, T * B).astype(np.int32)
    ids[0], ids[-1] = 3, 18
    for od in (torch.float32, torch.float16):
        out, st, fl, plan = run_case(tables, ids, None, [0] * T, B, od)
        assert st == dpi.DPI_OK
        want = torch.cat([torch.from_numpy(tables[t][ids[t * B:(t + 1) * B]]) for t in range(T)], 1).to(od) + 0.0
        got = out.cpu()
        as_int = torch.int32 if od == torch.float32 else torch.int16
        assert torch.equal(got.view(as_int), want.view(as_int))
        broken = ids.copy()
        broken[B * T // 2], broken[0] = 19, -1
        store = torch.full((B * fl.total_dim + 64,), 7.0, dtype=od, device="cuda")
        block = store[: B * fl.total_dim].view(B, -1)
        plan = fl.plan(None, B, T * B)
        fl.lookup(plan, torch.from_numpy(broken).cuda(), None, out=block)
        assert dpi.dpi_plan_sync_status(plan) == dpi.DPI_ERR_BAD_ID
        for i in (B * T // 2, 0):
            t, b = divmod(i, B)
            want[b, t * dim:(t + 1) * dim] = 0
        assert torch.equal(block.cpu().view(as_int), want.view(as_int)) and bool((store[B * fl.total_dim:] == 7.0).all())


@pytest.mark.parametrize("T,dims,dtype", [(3, [64], 1), (70, [32], 0), (3, [16], 0), (3, [15], 0), (4, [12, 16], 0),
                                          (70, [40, 64], 1), (3, [4], 0), (4, [3, 4], 0), (70, [2, 4], 1)])
@pytest.mark.parametrize("B", [1, 129, 1000])
def test_onehot_ids_outside_their_tables(T, dims, dtype, B):
    """One-hot rows by fields and by pieces: an id outside its table gives zeros
    whatever row 0 holds, and the others are copied."""
    rng = np.random.default_rng(T + B + sum(dims))
    ds = [dims[t % len(dims)] for t in range(T)]
    tables = [rng.standard_normal((19, d)).astype(np.float16 if dtype else np.float32) for d in ds]
    for t in tables:
        t[0] = np.nan
    ids = rng.integers(1, 19, T * B).astype(np.int32)
    out_of = rng.random(T * B) < 0.2
    out_of[-1] = True
    ids[out_of] = rng.choice([-1, 19, 2 ** 31 - 1, -2 ** 31], out_of.sum())
    want = np.concatenate([np.where(out_of[t * B:(t + 1) * B, None], 0, tables[t][ids[t * B:(t + 1) * B] % 19])
                           for t in range(T)], 1).astype(np.float32)
    for od in (torch.float32, torch.float16):
        out, st, _, _ = run_case(tables, ids, None, [0] * T, B, od)
        assert st == dpi.DPI_ERR_BAD_ID
        assert torch.equal(out.cpu(), torch.from_numpy(want).to(od))


@pytest.mark.parametrize("dim,B", [(16, 3999), (16, 4000), (48, 3999), (48, 4000), (32, 4000)])
def test_onehot_large_batches_of_half_lines(dim, B):
    """200 fields: below and from 800,000 bags on (pieces of the output row), and
    rows that fill whole lines."""
    T, rows = 200, 50
    gen = torch.Generator(device="cuda")
    gen.manual_seed(dim + B)
    tables = [torch.randn((rows, dim), generator=gen, device="cuda") for _ in range(T)]
    ids = torch.randint(0, rows, (T, B), generator=gen, device="cuda", dtype=torch.int32)
    out = FusedLookup(tables, [0] * T, torch.float32)(ids.reshape(-1), None, B)
    for t in range(T):
        assert torch.equal(out[:, t * dim:(t + 1) * dim], tables[t][ids[t].long()])


@pytest.mark.parametrize("dim,limit", [(60, 2 ** 32 - 256), (3, 2 ** 32 - 16)])   # 240- and 12-byte rows
@pytest.mark.parametrize("past", [0, 1, 2])
@pytest.mark.parametrize("beside", [False, True])
def test_masked_rows_at_the_buffer_limit(dim, limit, past, beside):
    """Ragged fp32 rows in a table of the largest size read by masked buffer loads
    (the byte past the last masked lane is 2^32), one row larger (64-bit
    addresses where masking is needed) and two (above 4 GiB), alone and beside a
    field of another row class.  Bags of 3 ids leave most row slots masked; the
    row after the table holds a marker that a load past it would add."""
    rows = limit // (4 * dim) + past
    assert limit % (4 * dim) == 0
    rng = np.random.default_rng(dim + past)
    n_set, B, L = 3000, 1500, 3
    store = torch.empty((rows + 1, dim), device="cuda")
    ends = (rng.integers(-64, 64, size=(2 * n_set, dim)) / 64.0).astype(np.float32)
    store[:n_set] = torch.from_numpy(ends[:n_set]).cuda()
    store[rows - n_set:rows] = torch.from_numpy(ends[n_set:]).cuda()
    store[rows] = 1000.0
    small_ids = rng.integers(0, 2 * n_set, L * B)
    big_ids = np.where(small_ids < n_set, small_ids, small_ids + rows - 2 * n_set).astype(np.int32)
    offs = np.arange(0, L * B + 1, L, dtype=np.int32)[None]
    tables, host, ids, ref_ids = [store[:rows]], [ends], big_ids, small_ids.astype(np.int32)
    if beside:
        other = rng.standard_normal((40, 8)).astype(np.float32)
        other_ids = rng.integers(0, 40, L * B).astype(np.int32)
        tables, host, offs = tables + [torch.from_numpy(other).cuda()], host + [other], np.concatenate([offs, offs])
        ids, ref_ids = np.concatenate([ids, other_ids]), np.concatenate([ref_ids, other_ids])
    T = len(tables)
    ref, mag = oracle.lookup([t.shape[1] for t in host], host, ref_ids, offs, [0] * T, B)
    fl = FusedLookup(tables, [0] * T, torch.float32)
    d_ids, d_offs = torch.from_numpy(ids).cuda(), torch.from_numpy(offs).cuda()
    for waves in (64, 0):                     # the plan's partition; bag by bag
        plan = fl.plan(d_offs, B, len(ids), num_waves=waves)
        out = fl.lookup(plan, d_ids, d_offs)
        assert dpi.dpi_plan_sync_status(plan) == dpi.DPI_OK
        check_outputs(out.double().cpu().numpy(), ref, mag, False, False)
    del store, tables, fl
    torch.cuda.empty_cache()
