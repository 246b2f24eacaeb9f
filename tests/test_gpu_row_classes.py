"""Rows of every byte length the lookups take, through each kernel that reads
them, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2606_21101_amd import dpi
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
