"""Kernels that come in several launch shapes, at the sizes where the choice between them changes and at
the edges of their tiles: against the CPU oracle, and against each other where they promise the same bits."""
import math

import numpy as np
import pytest
import torch

import paper_2407_20761_amd as ob
import synth_inputs as si
from gpu_util import bytes_buf, run_block, saved_view, to_dev, to_np
from oracle import block as orc
from oracle import connector as orc_conn

pytestmark = pytest.mark.gpu

TOL = 2e-2      # bf16 storage of every result and of the probabilities on the way (up to 2^-8 each), as in the parity tests


def _attention(qkv, d_o, lens, nq, nkv, d, mask):
    """(o, dq, dk, dv) of one packed batch; qkv [T, (nq + 2 nkv) d], d_o [T, nq d] on the device"""
    T, ld = qkv.shape
    seg = ob.Segments(si.lengths_to_cu(lens))
    o, lse = torch.empty_like(d_o), torch.empty((nq, T), dtype=torch.float32, device="cuda")
    dqkv = torch.full_like(qkv, float("nan"))
    cols = (slice(0, nq * d), slice(nq * d, (nq + nkv) * d), slice((nq + nkv) * d, ld))
    q, k, v = (qkv[:, c] for c in cols)
    dq, dk, dv = (dqkv[:, c] for c in cols)
    ob.ob_varlen_attn_fwd(q, k, v, o, lse, ld, ld, nq * d, seg, nq, nkv, d, d ** -0.5, mask)
    ws = bytes_buf(ob.ob_varlen_attn_bwd_workspace_bytes(T, nq, nkv, d))
    ob.ob_varlen_attn_bwd(d_o, q, k, v, o, lse, dq, dk, dv, ld, ld, nq * d, seg, nq, nkv, d, d ** -0.5, mask, ws)
    return o, dq, dk, dv


@pytest.mark.parametrize("mask", [orc.MASK_BIDIR, orc.MASK_CAUSAL])
@pytest.mark.parametrize("d,nq,nkv", [(64, 16, 16), (64, 16, 8), (64, 10, 10), (128, 8, 8), (128, 16, 8)])
def test_dkv_shapes_give_the_same_bits(d, nq, nkv, mask):
    """Many short segments fill the chip (the shape for throughput), each alone leaves it idle (the shape for the
    shorter trip): lengths on and beside the 32-, 64- and 128-row borders, oracle on two of them.
    (64, 10, 10): the bidirectional batch is about one round of the six-pair shape."""
    lens = [1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 191, 193, 257] * (1 if nkv == 10 else 8) + [385]
    print(f"dkv shapes d={d} nq={nq} nkv={nkv} mask={mask}", flush=True)
    cu = si.lengths_to_cu(lens)
    T = int(cu[-1])
    q, k, v, d_o_np = si.qkv_tensors(T, nq, nkv, d, seed=d + nq)
    qkv = to_dev(np.concatenate([q.reshape(T, -1), k.reshape(T, -1), v.reshape(T, -1)], axis=1))
    d_o = to_dev(d_o_np.reshape(T, -1))
    packed = _attention(qkv, d_o, lens, nq, nkv, d, mask)
    for j in list(range(17)) + [len(lens) - 1]:
        a, b = int(cu[j]), int(cu[j + 1])
        alone = _attention(qkv[a:b].contiguous(), d_o[a:b].contiguous(), [b - a], nq, nkv, d, mask)
        for name, x, y in zip(("o", "dq", "dk", "dv"), packed, alone):
            assert torch.equal(x[a:b].view(torch.int16), y.view(torch.int16)), (name, j, b - a)
        if j in (9, len(lens) - 1):
            ref = orc.attention_bwd_masked(*(t[a:b].astype(np.float64) for t in (d_o_np, q, k, v)), [0, b - a], mask, d ** -0.5)
            for name, x, r in zip(("dq", "dk", "dv"), packed[1:], ref):
                got = to_np(x[a:b]).reshape(r.shape)
                assert np.abs(got - r).max() <= TOL * np.abs(r).max(), (name, j)


@pytest.mark.parametrize("mask", [orc.MASK_BIDIR, orc.MASK_CAUSAL])
@pytest.mark.parametrize("d,unit", [(64, 128), (64, 256), (128, 128)])
def test_dkv_order_in_units_of_tiles(d, unit, mask):
    """Batches with more 64-row key tiles than the order table holds: the table's entries are two or four tiles, the last of a
    segment's places have none.  Segments on and beside the borders of tiles and units give the bits they give alone."""
    edges = [1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 700, 1987]
    total = 59000 if unit == 128 else 117000
    rest = [12000] + [300] * 150 if d == 128 else [3000] * ((total - sum(edges)) // 3000)      # (d = 128: one long walk)
    lens = edges + rest
    print(f"dkv order in units d={d} unit={unit} mask={mask}", flush=True)
    nq, nkv = 2, 1
    cu = si.lengths_to_cu(lens)
    plan, _ = ob.ob_varlen_attn_bwd_plan(ob.Segments(cu), nq, nkv, d, mask)
    assert plan.key_rows == 64 and plan.order_rows == unit
    gen = torch.Generator(device="cuda").manual_seed(d + unit)
    T = int(cu[-1])
    qkv = torch.randn((T, (nq + 2 * nkv) * d), generator=gen, device="cuda", dtype=torch.bfloat16)
    d_o = torch.randn((T, nq * d), generator=gen, device="cuda", dtype=torch.bfloat16)
    packed = _attention(qkv, d_o, lens, nq, nkv, d, mask)
    assert all(torch.isfinite(t.float()).all() for t in packed)
    for j in list(range(len(edges) + 1)) + [len(lens) - 1]:
        a, b = int(cu[j]), int(cu[j + 1])
        alone = _attention(qkv[a:b].contiguous(), d_o[a:b].contiguous(), [b - a], nq, nkv, d, mask)
        for name, x, y in zip(("o", "dq", "dk", "dv"), packed, alone):
            assert torch.equal(x[a:b].view(torch.int16), y.view(torch.int16)), (name, j, b - a)


@pytest.mark.parametrize("M,N,K", [(1, 64, 640), (127, 192, 704), (129, 320, 768), (300, 4160, 832), (557, 1088, 1088),
                                   (257, 256, 4096), (300, 4096, 4096), (200, 768, 4224)])
def test_gemm_deep_ring(M, N, K):
    """"NT" launches of few tiles walk K over a ring of eight slots and may leave it in the middle (K of 10 - 66 steps of
    64, every remainder modulo the four steps of a trip), whole or in slices, on ragged edges; with bias and residual."""
    print(f"deep ring {M} {N} {K}", flush=True)
    rng = np.random.default_rng(M + N + K)
    A = si.round_to_bf16(rng.standard_normal((M, K), dtype=np.float32))
    B = si.round_to_bf16(rng.standard_normal((N, K), dtype=np.float32))
    bias = si.round_to_bf16(rng.standard_normal((N,), dtype=np.float32))
    R = si.round_to_bf16(rng.standard_normal((M, N), dtype=np.float32) * 4)
    prod = A.astype(np.float64) @ B.astype(np.float64).T
    for ws in (None, bytes_buf(ob.ob_gemm_workspace_bytes(0, M, N, K))):
        for b, r in ((None, None), (bias, R)):
            C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
            ob.ob_gemm_bf16(0, M, N, K, to_dev(A), to_dev(B), C, None if b is None else to_dev(b), None if r is None else to_dev(r), ws)
            ref = prod if b is None else prod + b + r
            # one rounding to bf16 (8 significant bits: 2^-8 of the value at most) behind fp32 sums
            assert np.abs(to_np(C) - ref).max() <= 2.0 ** -8 * np.abs(ref).max(), (ws is not None, b is not None)


@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(64, 64, 64), (1, 64, 128), (65, 128, 192), (130, 192, 640), (200, 768, 768), (63, 448, 1088),
                                   (1025, 768, 832), (64, 4096, 4224)])
def test_gemm_fine_tiles(layout, M, N, K):
    """Launches that 64 x 64 tiles are chosen for (and their neighbours), all layouts: ragged rows and columns, every
    remainder of the eight-slot ring, token counts that are no multiple of 32."""
    if layout == 2:
        M, K = (M + 63) // 64 * 64, K + 37
    print(f"fine tiles layout={layout} {M} {N} {K}", flush=True)
    rng = np.random.default_rng(M + N + K + layout)
    A = si.round_to_bf16(rng.standard_normal((M, K), dtype=np.float32))
    B = si.round_to_bf16(rng.standard_normal((N, K), dtype=np.float32))
    R = si.round_to_bf16(rng.standard_normal((M, N), dtype=np.float32) * 4)
    ref = A.astype(np.float64) @ B.astype(np.float64).T + R
    a_dev = to_dev(A if layout != 2 else np.ascontiguousarray(A.T))
    b_dev = to_dev(B if layout == 0 else np.ascontiguousarray(B.T))
    for ws in (None, bytes_buf(ob.ob_gemm_workspace_bytes(layout, M, N, K))):
        C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        ob.ob_gemm_bf16(layout, M, N, K, a_dev, b_dev, C, None, to_dev(R), ws)
        assert np.abs(to_np(C) - ref).max() <= 2.0 ** -8 * np.abs(ref).max(), ws is not None


@pytest.mark.parametrize("Hv,Ht,grid,tiles", [(64, 128, 2, 3), (1024, 64, 32, 1), (1088, 128, 16, 5), (2048, 64, 16, 4), (2112, 64, 32, 2),
                                              (4096, 64, 18, 3)])
def test_connector_widths(Hv, Ht, grid, tiles):
    """The hand-over's row kernels at the widths where their launch shape changes, with token counts that leave groups and
    workgroups without a token, and few enough (81 and less) or enough for the one launch of all column sums."""
    print(f"connector widths {Hv} {Ht} {grid} {tiles}", flush=True)
    rng = np.random.default_rng(Hv + grid)
    n_tok, rows_v = tiles * (grid // 2) ** 2, tiles * (grid * grid + 1)
    w = si.connector_weights(Hv, Ht, seed=1)
    v = si.round_to_bf16(rng.standard_normal((rows_v, Hv), dtype=np.float32))
    llm = n_tok + 7
    dst = rng.permutation(llm)[:n_tok].astype(np.int32)
    dx = si.round_to_bf16(rng.standard_normal((llm, Ht), dtype=np.float32))
    desc = ob.make_connector_desc(Hv, Ht, grid, 1e-5)
    wd = {n: to_dev(t) for n, t in w.items()}
    gd = {n: torch.full_like(t, float("nan")) for n, t in wd.items()}
    vd, dv, x = to_dev(v), torch.full((rows_v, Hv), float("nan"), dtype=torch.bfloat16, device="cuda"), torch.zeros((llm, Ht), dtype=torch.bfloat16, device="cuda")
    rows = ob.RowIndex(dst)
    saved, ws = bytes_buf(ob.ob_connector_saved_bytes(desc, tiles)), bytes_buf(ob.ob_connector_workspace_bytes(desc, tiles))
    ob.ob_connector_fwd(desc, wd, vd, tiles, rows, x, llm, saved, ws)
    ob.ob_connector_bwd(desc, wd, gd, 0, vd, to_dev(dx), dv, tiles, rows, llm, saved, ws)
    x_ref, cache = orc_conn.connector_fwd(w, v, tiles, grid, 1e-5, np.zeros((llm, Ht)), dst)
    dv_ref, g_ref = orc_conn.connector_bwd(w, cache, dx, tiles, grid, 1e-5, dst)
    got = {"x": to_np(x), "dv": to_np(dv), **{n: to_np(t) for n, t in gd.items()}}
    ref = {"x": x_ref, "dv": dv_ref, **g_ref}
    for n in ref:
        assert np.abs(got[n] - ref[n]).max() <= TOL * np.abs(ref[n]).max(), n


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("M,N,K", [(2050, 4032, 896), (2050, 4096, 960), (2112, 4096, 1024), (1921, 4096, 1088), (3072, 4096, 2048)])
def test_gemm_rectangular_tiles(layout, M, N, K):
    """Launches that 192 x 256 tiles are chosen for: ragged and whole rows and columns, every remainder of the trip's two
    K steps, sampled rows against fp64."""
    print(f"rectangular tiles layout={layout} {M} {N} {K}", flush=True)
    rng = np.random.default_rng(M + N + K + layout)
    A = si.round_to_bf16(rng.standard_normal((M, K), dtype=np.float32))
    B = si.round_to_bf16(rng.standard_normal((N, K), dtype=np.float32))
    bias = si.round_to_bf16(rng.standard_normal((N,), dtype=np.float32))
    R = si.round_to_bf16(rng.standard_normal((M, N), dtype=np.float32) * 4)
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    ob.ob_gemm_bf16(layout, M, N, K, to_dev(A), to_dev(B if layout == 0 else np.ascontiguousarray(B.T)), C, to_dev(bias), to_dev(R), None)
    rows = np.unique(np.concatenate([np.arange(0, M, 37), [95, 96, 191, 192, 287, 288, M - 2, M - 1]]))
    ref = A[rows].astype(np.float64) @ B.astype(np.float64).T + bias + R[rows]
    got = to_np(C)
    assert np.isfinite(got).all()
    assert np.abs(got[rows] - ref).max() <= 2.0 ** -8 * np.abs(ref).max()


@pytest.mark.parametrize("hidden,T", [(64, 1), (64, 2051), (1024, 2047), (1088, 3), (2112, 700), (4096, 513), (4160, 257), (6144, 40),
                                      (8192, 300)])
@pytest.mark.parametrize("norm", [si.NORM_LAYERNORM, si.NORM_RMSNORM])
def test_norm_bwd_widths(hidden, T, norm):
    """The norm's backward at the widths and row counts where its launch shape changes (folded waves; one to eight waves to a
    row; fewer rows than workgroups, one more), through a block whose other sizes are the smallest: input and gain / beta /
    bias gradients against the oracle."""
    print(f"norm bwd hidden={hidden} T={T} norm={norm}", flush=True)
    ln = norm == si.NORM_LAYERNORM
    shape = si.small_shape(hidden=hidden, n_q_heads=1, n_kv_heads=1, head_dim=64, mlp_dim=64, norm=norm, mlp=si.MLP_GELU,
                           mask=si.MASK_BIDIR, has_bias=ln, norm_eps=1e-5)
    lens = [T] if T < 64 else [T - 33, 33]
    cu = si.lengths_to_cu(lens)
    w = si.block_weights(shape, seed=2)
    x, dy = si.activations(T, hidden, seed=3, std=1.0)
    _, y, dx, g = run_block(shape, w, x, dy, cu)
    y_ref, cache = orc.block_fwd(shape, w, x, cu)
    dx_ref, g_ref, _ = orc.block_bwd(shape, w, cache, dy, cu)
    for n, got, ref in [("y", y, y_ref), ("dx", dx, dx_ref)] + [(n, g[n], g_ref[n]) for n in g]:
        assert np.abs(got - ref).max() <= TOL * np.abs(ref).max(), n


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("M,N,K", [(2049, 8192, 1024), (1030, 16384, 768), (4444, 4096, 2048), (2500, 14336, 1024)])
def test_gemm_row_cut(layout, M, N, K):
    """Launches whose last rows go out on their own, behind whole rounds of tiles: one row, a few, more than a tile; with
    bias, residual and slice sums allowed.  Rows on both sides of every possible cut against fp64; a row's values do not
    depend on what is launched with it, up to the rounding of sums in another order where a contraction is split."""
    print(f"row cut layout={layout} {M} {N} {K}", flush=True)
    rng = np.random.default_rng(M + N + K + layout)
    A = si.round_to_bf16(rng.standard_normal((M, K), dtype=np.float32))
    B = si.round_to_bf16(rng.standard_normal((N, K), dtype=np.float32))
    bias = si.round_to_bf16(rng.standard_normal((N,), dtype=np.float32))
    R = si.round_to_bf16(rng.standard_normal((M, N), dtype=np.float32) * 4)
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = bytes_buf(max(ob.ob_gemm_workspace_bytes(layout, M, N, K), 16))
    ob.ob_gemm_bf16(layout, M, N, K, to_dev(A), to_dev(B if layout == 0 else np.ascontiguousarray(B.T)), C, to_dev(bias), to_dev(R), ws)
    edges = np.concatenate([np.arange(t, M, t) for t in (192, 256)])
    rows = np.unique(np.concatenate([edges - 1, edges, [0, M - 2, M - 1]]))
    ref = A[rows].astype(np.float64) @ B.astype(np.float64).T + bias + R[rows]
    got = to_np(C)
    assert np.isfinite(got).all()
    assert np.abs(got[rows] - ref).max() <= 2.0 ** -8 * np.abs(ref).max()


def test_connector_row_cut():
    """The hand-over's GEMMs cut by rows (4352 tokens, 4096 wide): both launches of the last store through the row list.  The first
    and the last tile of the batch against the oracle on those tiles alone; rows that no token has stay as they were."""
    Hv, Ht, grid, tiles = 64, 4096, 32, 17
    print(f"connector row cut {Hv} {Ht} {grid} {tiles}", flush=True)
    rng = np.random.default_rng(11)
    per, n_tok, rows_v = 256, tiles * 256, grid * grid + 1
    w = si.connector_weights(Hv, Ht, seed=1)
    v = si.round_to_bf16(rng.standard_normal((tiles * rows_v, Hv), dtype=np.float32))
    llm = n_tok + 5
    dst = rng.permutation(llm)[:n_tok].astype(np.int32)
    desc = ob.make_connector_desc(Hv, Ht, grid, 1e-5)
    x = torch.full((llm, Ht), 3.0, dtype=torch.bfloat16, device="cuda")
    saved, ws = bytes_buf(ob.ob_connector_saved_bytes(desc, tiles)), bytes_buf(ob.ob_connector_workspace_bytes(desc, tiles))
    ob.ob_connector_fwd(desc, {n: to_dev(t) for n, t in w.items()}, to_dev(v), tiles, ob.RowIndex(dst), x, llm, saved, ws)
    got = to_np(x)
    assert (np.delete(got, dst, axis=0) == 3.0).all()
    for t in (0, tiles - 1):
        ref, _ = orc_conn.connector_fwd(w, v[t * rows_v:(t + 1) * rows_v], 1, grid, 1e-5, np.zeros((per, Ht)), np.arange(per))
        assert np.abs(got[dst[t * per:(t + 1) * per]] - ref).max() <= TOL * np.abs(ref).max()


def test_gelu_and_derivative_element_by_element():
    """GELU and its derivative at every bf16 argument of 2^-12 .. 13.1 in size, each against its own value and not the tensor's
    maximum: one rounding to bf16 (8 significant bits: 2^-8 of the value at most) and the functions' own error (1.2e-5 of the value in the tails, 7e-8
    around the derivative's zero).  One token through a block whose up projection gives its bias, whose down projection and
    dy give the derivative a factor of one, so that the bias gradient is the derivative as stored."""
    print("gelu element by element", flush=True)
    z = (np.arange(65536, dtype=np.uint32) << 16).view(np.float32)
    with np.errstate(invalid="ignore"):
        z = z[(np.abs(z) >= 2.0 ** -12) & (np.abs(z) <= 13.1)]
    F = (len(z) + 63) // 64 * 64
    z = np.concatenate([z, np.zeros(F - len(z), np.float32)])
    shape = si.small_shape(hidden=64, n_q_heads=1, n_kv_heads=1, head_dim=64, mlp_dim=F, norm=si.NORM_LAYERNORM, mlp=si.MLP_GELU,
                           mask=si.MASK_BIDIR, has_bias=True, norm_eps=1e-5)
    w = si.block_weights(shape, seed=2)
    w["w_up"], w["b_up"], w["w_down"] = np.zeros_like(w["w_up"]), z, np.zeros_like(w["w_down"])
    w["w_down"][0] = 1.0
    x, dy = si.activations(1, 64, seed=3, std=1.0)
    dy[:] = 0.0
    dy[0, 0] = 1.0
    run, _, _, g = run_block(shape, w, x, dy, si.lengths_to_cu([1]))
    act = to_np(saved_view(run.desc, 1, run.saved, "act", (1, F)))[0]
    z = z.astype(np.float64)
    cdf = np.array([0.5 * math.erfc(-t / math.sqrt(2.0)) for t in z])
    density = np.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi)
    for name, got, ref, around in (("gelu", act, z * cdf, 0.0), ("derivative", g["b_up"], cdf + z * density, 7e-8)):
        # (values below 2^-126 may be flushed)
        bound = (2.0 ** -8 + 2e-5) * np.abs(ref) + np.where(np.abs(z) < 2.0, around, 2.0 ** -126)
        bad = np.abs(got - ref) > bound
        assert not bad.any(), (name, z[bad][:4], got[bad][:4], ref[bad][:4])
