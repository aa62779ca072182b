"""The schedule of a call without an explicit plan (CPU): the estimate picks a
tile of the table for every shape, kind and output, never needs more than the
planner's plan, and reaches each tile that only such calls run on."""
import ctypes

import numpy as np
import pytest

from paper_2607_12505_amd import nmspmm
from paper_2607_12505_amd.nmprobe import stream_out
from schedule_cases import CASES, PATTERN, schedule_tile


@pytest.mark.parametrize("kind", nmspmm.ALL_KINDS)
def test_every_shape_gets_a_tile_of_the_table(kind):
    rng = np.random.default_rng(kind)
    for _ in range(400):
        m, n, k = int(np.exp(rng.uniform(0, 12))), 4 * int(np.exp(rng.uniform(0, 8))), 16 * int(np.exp(rng.uniform(0, 6)))
        mode = int(rng.integers(1, 8))
        planned = int(rng.integers(0, nmspmm.num_tiles()))
        tile = schedule_tile(kind, m, n, k, mode, planned)
        assert 0 <= tile < 16
        assert tile != 13 or kind in (nmspmm.NM_KIND_SP42, nmspmm.NM_KIND_DENSE)
        assert tile != 14 or kind not in (nmspmm.NM_KIND_MK3, nmspmm.NM_KIND_MK4, nmspmm.NM_KIND_MK5)
        assert tile == schedule_tile(kind, m, n, k, mode, planned)


@pytest.mark.parametrize("case", CASES, ids=str)
def test_cases_reach_the_unplanned_tiles(case):
    m, n, k, kind, mode, want = case
    d = nmspmm.compress_size(n, k, *PATTERN[kind])
    p = nmspmm.spmm_plan(d, m, mode)
    assert p.expand == 0 and p.tile < nmspmm.num_tiles() and p.split_k == 1
    assert schedule_tile(kind, m, n, k, mode, p.tile) == want


def test_internal_tiles_are_no_plans():
    d = nmspmm.compress_size(256, 256, 2, 4)
    for tile in (12, 15, 16):
        with pytest.raises(nmspmm.NmError):
            nmspmm.spmm_plan_complete(d, 100, nmspmm.make_plan(nmspmm.NM_KIND_SP42, tile, 1))
        with pytest.raises(nmspmm.NmError):
            nmspmm.tile_info(tile)


# reductions longer than any the estimate was fitted to, whose switch away from
# the planner's tile cost 13-25 % (the kind is the one that runs)
@pytest.mark.parametrize("m,n,k,kind,mode,planned", [
    (2458, 1508, 15120, nmspmm.NM_KIND_SP42, nmspmm.NM_OUT_I32, 1),
    (7550, 484, 6576, nmspmm.NM_KIND_SP42, nmspmm.NM_OUT_I32, 1),
    (2604, 1416, 6240, nmspmm.NM_KIND_SP42, nmspmm.NM_OUT_I32, 1),
    (5273, 548, 5072, nmspmm.NM_KIND_SP42, nmspmm.NM_OUT_I8, 1),
    (1462, 788, 8848, nmspmm.NM_KIND_MK5, nmspmm.NM_OUT_I32, 3),
    (12178, 424, 12096, nmspmm.NM_KIND_DENSE, nmspmm.NM_OUT_F16, 0),
    (1116, 4180, 5616, nmspmm.NM_KIND_C14, nmspmm.NM_OUT_I8, 1),
    (253, 1804, 5680, nmspmm.NM_KIND_C28, nmspmm.NM_OUT_I32, 10),
])
def test_small_promises_past_the_fitted_reductions_are_not_taken(m, n, k, kind, mode, planned):
    assert schedule_tile(kind, m, n, k, mode, planned) == planned


def test_large_promises_past_the_fitted_reductions_are_taken():
    assert schedule_tile(nmspmm.NM_KIND_SP42, 18464, 1024, 8192, nmspmm.NM_OUT_I32, 0) == 15


def test_store_policy_of_rows_on_and_off_the_lines():
    # rows on 128-byte lines: non-temporal whatever the reduction
    assert stream_out(100352, 512, 128) == stream_out(1000, 512, 4096) == 7
    assert stream_out(1000, 64, 128) == 6 and stream_out(1000, 32, 128) == 4
    # off the lines: through L2, but int32 of a long reduction as before the rows went through L2 at all
    assert stream_out(30000, 500, 256) == 0
    assert stream_out(44423, 2152, 2048) == 4
    assert [stream_out(30000, 500, k) for k in (768, 1408, 1424)] == [0, 0, 4]
    # ... from 7 k-steps where the output passes 256 MB
    assert [stream_out(140000, 500, k) for k in (768, 784)] == [0, 4]
    assert [stream_out(m, 500, 1024) for m in (134217, 134218)] == [0, 4]
