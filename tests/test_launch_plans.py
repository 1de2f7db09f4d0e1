"""How calls are cut into launches, asked of the library on the host: no GPU needed."""
import numpy as np
import pytest

import gemm_launches
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


def test_gpu_cases_reach_the_kernels_they_name():
    for layout, M, N, K, want in gemm_launches.FORMS:
        assert gemm_launches.named(gemm_launches.forms(layout, M, N, K)) == want, (layout, M, N, K)
    for Ht, grid, tiles, want in gemm_launches.ROW_LIST:
        assert gemm_launches.named(gemm_launches.forms(0, tiles * (grid // 2) ** 2, Ht, Ht)) == want, (Ht, grid, tiles)
    left = {"whole": set(), "split": set()}      # K steps modulo the trip's four that a deep tile walks
    for M, N, K in gemm_launches.DEEP:
        (launch,) = ob.ob_gemm_plan(0, M, N, K)
        kind, how = gemm_launches.form(launch)
        assert kind == "deep"
        left[how].add(gemm_launches.steps(launch, K)[-1] % 4)
    assert left == {"whole": {0, 1, 2, 3}, "split": {0, 1, 2, 3}}


def test_every_gemm_form_has_a_gpu_case():
    """Whatever the plan takes over sizes of every magnitude, the GPU tests run: each kind of tile, whole, split and mixed, per
    layout, and each pair of launches a GEMM is cut into, by the kind of the first and of the second and whether that is split."""
    def seen(layout, forms):
        out = {(layout, *f) for f in forms}
        if len(forms) == 2:
            out |= {(layout, "head", forms[0][0]), (layout, "rest", forms[1][0], forms[1][1] != "whole")}
        return out

    covered = set().union(*(seen(layout, gemm_launches.forms(layout, M, N, K)) for layout, M, N, K, _ in gemm_launches.FORMS))
    rng = np.random.default_rng(5)
    dims = [256, 512, 640, 768, 1024, 1088, 2048, 2112, 2560, 3072, 3200, 4096, 5120, 6144, 9600, 12288, 12800, 14336, 16384, 28672]
    for i in range(30000):
        a, b = (int(rng.choice(dims)) if rng.random() < 0.8 else 64 * int(rng.integers(1, 400)) for _ in range(2))
        T, layout = int(2 ** rng.uniform(0, 15)), i % 3
        M, N, K = (a, b, T) if layout == 2 else (T, a, b)
        missing = seen(layout, gemm_launches.forms(layout, M, N, K, i % 5 != 0)) - covered
        assert not missing, (layout, M, N, K, missing)


def test_every_activation_launch_has_a_gpu_case():
    covered = {(mlp, i, tile) for mlp, _, _, _, _, _, tiles in gemm_launches.ACTIVATIONS for i, tile in enumerate(tiles)}
    rng = np.random.default_rng(7)
    for i in range(20000):
        mlp, backward = (si.MLP_GELU, si.MLP_SWIGLU)[i & 1], i >> 1 & 1
        T, hidden, F = int(2 ** rng.uniform(0, 15)), 64 * int(2 ** rng.uniform(0, 7)), 64 * int(2 ** rng.uniform(0, 9))
        plan = ob.ob_gemm_act_plan(mlp, backward, T, F, hidden, i % 3 != 0)
        if plan is not None:
            assert (mlp, backward, (plan.tile_rows, plan.ring_slots, plan.slices)) in covered and (plan.row0, plan.rows) == (0, T), (mlp, backward, T, F, hidden)


def test_every_dkv_kernel_has_a_gpu_case():
    """Whichever kernel a batch of any layout takes, the walks of the GPU tests are walked in it, under the same mask."""
    covered = set()
    for d, nq, nkv, lens, *want in gemm_launches.DKV_WALKS:
        for mask, kernel in zip((orc.MASK_BIDIR, orc.MASK_CAUSAL), want):
            assert gemm_launches.dkv_kernel(lens, nq, nkv, d, mask) == kernel, (d, nq, nkv, lens, mask)
            covered.add((d, mask, kernel))
    rng = np.random.default_rng(6)
    for i in range(4000):
        d, mask, nkv = (64, 128)[i & 1], (orc.MASK_BIDIR, orc.MASK_CAUSAL)[i >> 1 & 1], int(rng.integers(1, 49))
        total = int(2 ** rng.uniform(0, 14))
        lens = [total] if i % 3 == 0 else [1025] * (1 + total // 1025) if i % 3 == 1 else _lengths(total, 300, 4096, i)
        assert (d, mask, gemm_launches.dkv_kernel(lens, nkv * int(rng.integers(1, 7)), nkv, d, mask)) in covered, (d, mask, nkv, lens)


# bidirectional, heads of 64: six pairs where two need a second round of two workgroups to a CU and they do not (256 CUs)
@pytest.mark.parametrize("nkv,lens,six", [(10, [1025] * 3, False), (8, [1025] * 4, True), (8, [4097], True), (8, [1025] * 6, False), (16, [2000], False),
                                          (4, [1025] * 7, False), (4, [1025] * 8, True)])
def test_dkv_six_pairs_save_a_round(nkv, lens, six):
    plan, _ = ob.ob_varlen_attn_bwd_plan(_segments(lens), nkv, nkv, 64, orc.MASK_BIDIR)
    assert (plan.key_rows == 192) == six
