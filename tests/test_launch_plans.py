"""How calls are cut into launches, asked of the library on the host: no GPU needed."""
import numpy as np
import pytest

import paper_2407_20761_amd as ob
import synth_inputs as si
from oracle import block as orc


def _segments(lens):
    seg = ob.Segments(si.lengths_to_cu(lens), device=None)
    seg.c.cu_dev = 0x1000      # never read: the plan is host work
    return seg


def _lengths(total, median, longest, seed):
    rng, out, left = np.random.default_rng(seed), [], total
    while left:
        n = int(min(max(1, np.exp(np.log(median) + 1.1 * rng.standard_normal())), longest, left))
        out.append(n)
        left -= n
    return out


# 57344 tokens fill the table with tiles of 64 key rows, 172032 with the 192 rows of the six-pair shape
@pytest.mark.parametrize("d,nq,nkv,mask", [(64, 16, 4, orc.MASK_CAUSAL), (64, 16, 16, orc.MASK_BIDIR), (64, 2, 1, orc.MASK_CAUSAL),
                                           (128, 32, 8, orc.MASK_CAUSAL), (128, 2, 1, orc.MASK_CAUSAL)])
@pytest.mark.parametrize("total", [64, 700, 16327, 57344, 57409, 90000, 114000, 160000])
def test_dkv_order_covers_every_tile_heaviest_first(d, nq, nkv, mask, total):
    lens = _lengths(total, 2000, 8000, total + d)
    cu = si.lengths_to_cu(lens)
    plan, rows = ob.ob_varlen_attn_bwd_plan(_segments(lens), nq, nkv, d, mask)
    tiles = np.concatenate([np.arange(a, b, plan.key_rows) for a, b in zip(cu[:-1], cu[1:])])
    assert np.array_equal(np.sort(rows[rows >= 0]), tiles)
    if plan.key_rows == 64 or total < 114000:
        assert plan.order_rows > 0, "a batch that had an order of work in 192-row tiles has one in 64-row tiles"
    if plan.order_rows:
        seg = np.searchsorted(cu, np.maximum(rows, 0), side="right") - 1
        work = cu[seg + 1] - rows if mask == orc.MASK_CAUSAL else cu[seg + 1] - cu[seg]
        per = plan.order_rows // plan.key_rows
        first = -(-work[::per] // 64)                       # of the heaviest tile of each unit
        assert (rows[::per] >= 0).all() and (np.diff(first) <= 0).all()
        assert len(rows) % per == 0 and (rows < 0).sum() < per * len(lens)
