"""Kernels that come in several launch shapes, at the sizes where the choice between them changes and at
the edges of their tiles: against the CPU oracle, and against each other where they promise the same bits."""
import math

import numpy as np
import pytest
import torch

import gemm_launches
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
@pytest.mark.parametrize("d,nq,nkv", [(64, 16, 16), (64, 16, 8), (64, 10, 10), (128, 8, 8), (128, 16, 8), (128, 16, 16)])
def test_dkv_shapes_give_the_same_bits(d, nq, nkv, mask):
    """Many short segments fill the chip (the shape for throughput), each alone leaves it idle (a shape for the
    shorter trip): lengths on and beside the 32-, 64- and 128-row borders, oracle on two of them.
    (64, 10, 10): two pairs would need a second round for the bidirectional batch, six do not.  (128, 16, 16): two pairs of heads of
    128 walk seven tiles, three to a trip."""
    lens = [1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 191, 193, 257] * 8 + [385]
    if nkv == 10:
        lens = [1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 257, 513, 1025, 385]
    if (d, nkv) == (128, 16):
        lens = [448, 385, 320, 191, 129, 65] * 3 + [385]
    want = gemm_launches.FOUR if d == 128 else gemm_launches.SR32 if nkv != 10 else gemm_launches.SR64 if mask else gemm_launches.SIX
    assert gemm_launches.dkv_kernel(lens, nq, nkv, d, mask) == want
    seen = set()
    print(f"dkv shapes d={d} nq={nq} nkv={nkv} mask={mask}", flush=True)
    cu = si.lengths_to_cu(lens)
    T = int(cu[-1])
    q, k, v, d_o_np = si.qkv_tensors(T, nq, nkv, d, seed=d + nq)
    qkv = to_dev(np.concatenate([q.reshape(T, -1), k.reshape(T, -1), v.reshape(T, -1)], axis=1))
    d_o = to_dev(d_o_np.reshape(T, -1))
    packed = _attention(qkv, d_o, lens, nq, nkv, d, mask)
    for j in list(range(min(17, len(lens) - 1))) + [len(lens) - 1]:
        a, b = int(cu[j]), int(cu[j + 1])
        seen.add(gemm_launches.dkv_kernel([b - a], nq, nkv, d, mask))
        alone = _attention(qkv[a:b].contiguous(), d_o[a:b].contiguous(), [b - a], nq, nkv, d, mask)
        for name, x, y in zip(("o", "dq", "dk", "dv"), packed, alone):
            assert torch.equal(x[a:b].view(torch.int16), y.view(torch.int16)), (name, j, b - a)
        if j in (9, len(lens) - 1):
            ref = orc.attention_bwd_masked(*(t[a:b].astype(np.float64) for t in (d_o_np, q, k, v)), [0, b - a], mask, d ** -0.5)
            for name, x, r in zip(("dq", "dk", "dv"), packed[1:], ref):
                got = to_np(x[a:b]).reshape(r.shape)
                assert np.abs(got - r).max() <= TOL * np.abs(r).max(), (name, j)
    short = gemm_launches.TWO if mask == orc.MASK_BIDIR else gemm_launches.FOUR      # (causal: segments of up to 64)
    assert seen == ({gemm_launches.SR64} if d == 64 else {gemm_launches.BLOCKS} if mask and min(lens) > 64 else {gemm_launches.BLOCKS, short})


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


@pytest.mark.parametrize("mask", [orc.MASK_BIDIR, orc.MASK_CAUSAL])
@pytest.mark.parametrize("d,nq,nkv,lens,bidir,causal", gemm_launches.DKV_WALKS)
def test_dkv_walks(d, nq, nkv, lens, bidir, causal, mask):
    """Walks of more query tiles than one descriptor of the requests serves (64), of a tile or two, and of odd and even numbers of them:
    dK, dV of the first and the last segment against float32 products on the device (their own error is below 1e-5)."""
    print(f"dkv walks d={d} nq={nq} nkv={nkv} mask={mask} {lens}", flush=True)
    assert gemm_launches.dkv_kernel(lens, nq, nkv, d, mask) == (causal if mask == orc.MASK_CAUSAL else bidir)
    gen = torch.Generator(device="cuda").manual_seed(d + nq + len(lens))
    cu = si.lengths_to_cu(lens)
    T, group = int(cu[-1]), nq // nkv
    qkv = torch.randn((T, (nq + 2 * nkv) * d), generator=gen, device="cuda", dtype=torch.bfloat16)
    d_o = torch.randn((T, nq * d), generator=gen, device="cuda", dtype=torch.bfloat16)
    _, _, dk, dv = _attention(qkv, d_o, lens, nq, nkv, d, mask)
    for a, b in ((int(cu[0]), int(cu[1])), (int(cu[-2]), int(cu[-1]))):
        q, k, v = (x.float() for x in qkv[a:b].split([nq * d, nkv * d, nkv * d], 1))
        hidden = torch.ones((b - a, b - a), dtype=torch.bool, device="cuda").triu_(1) if mask == orc.MASK_CAUSAL else None
        for h in (0, nkv - 1):
            c = slice(h * d, (h + 1) * d)
            want_k, want_v = torch.zeros_like(k[:, c]), torch.zeros_like(v[:, c])
            for g in range(h * group, (h + 1) * group):
                qh, go = q[:, g * d:(g + 1) * d], d_o[a:b, g * d:(g + 1) * d].float()
                S = (qh @ k[:, c].t()) * d ** -0.5
                P = (S if hidden is None else S.masked_fill_(hidden, -math.inf)).softmax(1)
                dP = go @ v[:, c].t()
                want_v += P.t() @ go
                want_k += (P * (dP - (P * dP).sum(1, keepdim=True))).t() @ qh * d ** -0.5
            for name, got, want in (("dk", dk[a:b, c], want_k), ("dv", dv[a:b, c], want_v)):
                assert (got.float() - want).abs().max() <= TOL * want.abs().max(), (name, a, h)


@pytest.mark.parametrize("d,nq,nkv,T,ld,mask,kernel", [(64, 2, 1, 4160, 530000, orc.MASK_CAUSAL, gemm_launches.SR64), (64, 24, 24, 2176, 1060000, orc.MASK_BIDIR, gemm_launches.SR32),
                                                       (64, 8, 8, 4160, 530000, orc.MASK_BIDIR, gemm_launches.SIX), (128, 8, 8, 4160, 530000, orc.MASK_BIDIR, gemm_launches.FOUR),
                                                       (128, 2, 1, 4160, 530000, orc.MASK_CAUSAL, gemm_launches.BLOCKS),
                                                       (64, 2, 1, 385, 34200000, orc.MASK_CAUSAL, gemm_launches.SR64), (64, 320, 320, 130, 68000000, orc.MASK_BIDIR, gemm_launches.SR32),
                                                       (128, 3, 1, 193, 34200000, orc.MASK_CAUSAL, gemm_launches.BLOCKS), (128, 1, 1, 257, 34200000, orc.MASK_BIDIR, gemm_launches.BLOCKS)])
def test_attention_in_rows_far_apart(d, nq, nkv, T, ld, mask, kernel):
    """Heads in columns of a wide buffer, rows so far apart that the 64 query tiles that a descriptor of dK / dV serves elsewhere span
    more than 2^32 bytes, or a single tile of the kernel they would have does (then keys and values, of which 64 rows have to fit, lie side by side; for
    T = 385 queries alone are apart): the bits of the same heads side by side."""
    print(f"rows far apart d={d} nq={nq} nkv={nkv} T={T} ld={ld} mask={mask}", flush=True)
    one_tile = kernel[1] * ld * 2 > 2 ** 32
    assert gemm_launches.dkv_kernel([T], nq, nkv, d, mask) == kernel and 64 * kernel[1] * ld * 2 > 2 ** 32 and one_tile == (ld > 1060000)
    gen = torch.Generator(device="cuda").manual_seed(d + nq)
    qkv = torch.randn((T, (nq + 2 * nkv) * d), generator=gen, device="cuda", dtype=torch.bfloat16)
    d_o = torch.randn((T, nq * d), generator=gen, device="cuda", dtype=torch.bfloat16)
    want = _attention(qkv, d_o, [T], nq, nkv, d, mask)
    buf, at, views = torch.empty((T, ld), device="cuda", dtype=torch.bfloat16), 8, []
    ldkv, ldo = nkv * d if one_tile else ld, nq * d if T == 385 else ld
    for i, n in enumerate((nq, nkv, nkv, nq, nq, nq, nkv, nkv)):          # q k v d_o o dq dk dv, from the row's second vector on
        apart = (ldkv if i in (1, 2, 6, 7) else ldo if i in (3, 4) else ld) == ld
        views.append(buf[:, at:at + n * d] if apart else torch.empty((T, n * d), device="cuda", dtype=torch.bfloat16))
        at += n * d
    q, k, v, go, o, dq, dk, dv = views
    for to, x in zip((q, k, v), qkv.split([nq * d, nkv * d, nkv * d], 1)):
        to.copy_(x)
    go.copy_(d_o)
    seg, lse = ob.Segments(si.lengths_to_cu([T])), torch.empty((nq, T), dtype=torch.float32, device="cuda")
    ob.ob_varlen_attn_fwd(q, k, v, o, lse, ld, ldkv, ldo, seg, nq, nkv, d, d ** -0.5, mask)
    ws = bytes_buf(ob.ob_varlen_attn_bwd_workspace_bytes(T, nq, nkv, d))
    ob.ob_varlen_attn_bwd(go, q, k, v, o, lse, dq, dk, dv, ld, ldkv, ldo, seg, nq, nkv, d, d ** -0.5, mask, ws)
    for name, got, ref in zip(("o", "dq", "dk", "dv"), (o, dq, dk, dv), want):
        assert torch.equal(got.contiguous().view(torch.int16), ref.contiguous().view(torch.int16)), name


def _normal_gemm(layout, M, N, K, seed):
    """operands of N(0, 1) as the library takes them, bias, residual, and A, B as [M, K], [N, K] views"""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    new = lambda *size: torch.randn(size, generator=gen, device="cuda", dtype=torch.bfloat16)
    A, B = new(K, M) if layout == 2 else new(M, K), new(N, K) if layout == 0 else new(K, N)
    return A, B, new(N), new(M, N) * 4, A.T if layout == 2 else A, B if layout == 0 else B.T


@pytest.mark.parametrize("layout,M,N,K,want", gemm_launches.FORMS + [(0, *c, None) for c in gemm_launches.DEEP])
def test_gemm_forms(layout, M, N, K, want):
    """Every kind of tile in every layout that has it, whole, in slices and whole beside sliced, and launches cut by rows in two:
    the rows on and beside every border of a tile, whole, against fp64; plain, and with bias and residual in place of the result.
    Scratch and result hold garbage before."""
    print(f"gemm forms layout={layout} {M} {N} {K} {want}", flush=True)
    assert want is None or gemm_launches.named(gemm_launches.forms(layout, M, N, K)) == want
    A, B, bias, R, a, b = _normal_gemm(layout, M, N, K, seed=M + N + K + layout)
    edges = np.concatenate([np.arange(t, M, t) for t in (64, 192)] + [[0, M - 1]])
    rows = torch.from_numpy(np.unique(np.concatenate([edges - 1, edges, [min(M - 1, 33)]]).clip(0))).cuda()
    ref = a[rows].double() @ b.double().T
    ws = bytes_buf(ob.ob_gemm_workspace_bytes(layout, M, N, K))
    for plain in (True, False):
        ws.fill_(0x7F)
        C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda") if plain else R.clone()
        ob.ob_gemm_bf16(layout, M, N, K, A, B, C, None if plain else bias, None if plain else C, ws)
        want_rows = ref if plain else ref + bias.double() + R[rows].double()
        assert torch.isfinite(C).all()
        # one rounding to bf16 (8 significant bits: 2^-8 of the value at most) behind fp32 sums
        assert (C[rows].double() - want_rows).abs().max() <= 2.0 ** -8 * want_rows.abs().max(), plain


@pytest.mark.parametrize("M,N,K", [(1, 64, 640), (127, 192, 704), (129, 320, 768), (300, 4160, 832), (557, 1088, 1088),
                                   (257, 256, 4096), (300, 4096, 4096), (200, 768, 4224)] + gemm_launches.DEEP[:5])
def test_gemm_deep_ring(M, N, K):
    """"NT" launches of few rows walk K over a ring of eight slots and may leave it in the middle, in 64 x 64 tiles (the first
    eight but one) and 128 x 128 ones (K steps of every remainder modulo the four of a trip), whole or in slices, on ragged edges;
    with bias and residual."""
    for scratch in (False, True):
        plan = ob.ob_gemm_plan(0, M, N, K, scratch)
        assert all(p.ring_slots == 8 for p in plan)
        assert (M, N, K) not in gemm_launches.DEEP or plan[0].tile_rows == 128
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
    """Launches that 64 x 64 tiles are chosen for, all layouts: ragged rows and columns, every remainder of the eight-slot
    ring, token counts that are no multiple of 32."""
    if layout == 2:
        M, K = (M + 63) // 64 * 64, K + 37
    assert all(k == "fine" for scratch in (False, True) for k, _ in gemm_launches.forms(layout, M, N, K, scratch))
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
                                              (4096, 64, 18, 3), (64, 64, 2, 1536), (64, 64, 2, 1537), (1088, 64, 2, 768),
                                              (1088, 64, 2, 769), (2112, 64, 2, 256), (2112, 64, 2, 257), (2112, 64, 16, 48), (2112, 64, 16, 49)])
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
@pytest.mark.parametrize("M,N,K", [(2050, 4032, 896), (2050, 4096, 960), (2112, 4096, 1024), (2881, 4096, 1088), (3072, 4096, 2048)])
def test_gemm_rectangular_tiles(layout, M, N, K):
    """Launches that 192 x 256 tiles are chosen for: ragged and whole rows and columns, every remainder of the trip's two
    K steps, sampled rows against fp64."""
    print(f"rectangular tiles layout={layout} {M} {N} {K}", flush=True)
    assert gemm_launches.forms(layout, M, N, K, False) == [("mid", "whole")]
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


@pytest.mark.parametrize("hidden,T", [(64, 1), (64, 2051), (1024, 2047), (1088, 3), (1088, 4095), (1088, 4096), (2048, 4097), (2112, 4097), (2112, 700), (4096, 513), (4160, 257), (6144, 40),
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


@pytest.mark.parametrize("layout,M,N,K", [(0, 2049, 8192, 1024), (0, 1030, 16384, 768), (0, 4444, 4096, 2048), (0, 2500, 14336, 1024),
                                          (0, 6012, 3072, 2560), (1, 2049, 8192, 1024), (1, 2500, 14336, 1024), (1, 4494, 4096, 2496)])
def test_gemm_row_cut(layout, M, N, K):
    """Launches whose last rows go out on their own, behind whole rounds of tiles: one row, a few, more than a tile, some
    of them in slices; with bias and residual.  Rows on both sides of every possible cut against fp64; a row's values do not
    depend on what is launched with it, up to the rounding of sums in another order where a contraction is split."""
    print(f"row cut layout={layout} {M} {N} {K}", flush=True)
    head, rest = ob.ob_gemm_plan(layout, M, N, K)
    assert head.rows + rest.rows == M and rest.row0 == head.rows
    assert (rest.slices > 1) == (K > 2400)
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


@pytest.mark.parametrize("Ht,grid,tiles,want", gemm_launches.ROW_LIST)
def test_connector_row_list(Ht, grid, tiles, want):
    """The hand-over's last GEMM stores through the row list from every kind of tile, whole and in slices, and from both launches
    of one cut by rows.  The first, the middle and the last tile of the batch against the oracle on those tiles alone; rows that no token
    has stay as they were."""
    Hv = 64
    print(f"connector row list {Ht} {grid} {tiles} {want}", flush=True)
    rng = np.random.default_rng(11)
    per, rows_v = (grid // 2) ** 2, grid * grid + 1
    n_tok = tiles * per
    assert gemm_launches.named(gemm_launches.forms(0, n_tok, Ht, Ht)) == want
    w = si.connector_weights(Hv, Ht, seed=1)
    v = si.round_to_bf16(rng.standard_normal((tiles * rows_v, Hv), dtype=np.float32))
    llm = n_tok + 5
    dst = rng.permutation(llm)[:n_tok].astype(np.int32)
    desc = ob.make_connector_desc(Hv, Ht, grid, 1e-5)
    x = torch.full((llm, Ht), 3.0, dtype=torch.bfloat16, device="cuda")
    saved, ws = bytes_buf(ob.ob_connector_saved_bytes(desc, tiles)), bytes_buf(ob.ob_connector_workspace_bytes(desc, tiles))
    ws.fill_(0x7F)
    ob.ob_connector_fwd(desc, {n: to_dev(t) for n, t in w.items()}, to_dev(v), tiles, ob.RowIndex(dst), x, llm, saved, ws)
    got = to_np(x)
    assert np.isfinite(got).all() and (np.delete(got, dst, axis=0) == 3.0).all()
    for t in (0, tiles // 2, tiles - 1):
        ref, _ = orc_conn.connector_fwd(w, v[t * rows_v:(t + 1) * rows_v], 1, grid, 1e-5, np.zeros((per, Ht)), np.arange(per))
        assert np.abs(got[dst[t * per:(t + 1) * per]] - ref).max() <= TOL * np.abs(ref).max()


@pytest.mark.parametrize("hidden,mlp,T,want", [(256, 1024, 200, ("fine", "whole")), (640, 2560, 300, ("small", "whole")),
                                               (1024, 4096, 557, ("big", "whole")), (256, 1024, 12300, ("big", "split"))])
def test_grouped_weight_gradients_by_tile(hidden, mlp, T, want):
    """A block's four weight gradients in one launch, in each kind of tile that the group takes, whole and in slices: against the
    oracle, and accumulated onto themselves."""
    print(f"grouped weight gradients {hidden} {mlp} T={T}", flush=True)
    shape = si.small_shape(hidden=hidden, n_q_heads=hidden // 64, n_kv_heads=hidden // 64, head_dim=64, mlp_dim=mlp,
                           norm=si.NORM_LAYERNORM, mlp=si.MLP_GELU, mask=si.MASK_BIDIR, has_bias=True, norm_eps=1e-5)
    lens = [100] * (T // 100) + ([T % 100] if T % 100 else [])
    cu = si.lengths_to_cu(lens)
    w = si.block_weights(shape, seed=2)
    x, dy = si.activations(T, hidden, seed=3, std=1.0)
    run, y, dx, g = run_block(shape, w, x, dy, cu)
    sizes = [(3 * hidden, hidden), (hidden, hidden), (mlp, hidden), (hidden, mlp)]
    launch = ob.ob_gemm_group_plan(sizes, T, ob.ob_block_workspace_bytes(run.desc, T))
    assert launch and gemm_launches.form(launch) == want
    y_ref, cache = orc.block_fwd(shape, w, x, cu)
    dx_ref, g_ref, _ = orc.block_bwd(shape, w, cache, dy, cu)
    for n, got, ref in [("y", y, y_ref), ("dx", dx, dx_ref)] + [(n, g[n], g_ref[n]) for n in g]:
        assert np.abs(got - ref).max() <= TOL * np.abs(ref).max(), n
    once = {n: t.clone() for n, t in run.g.items()}
    run.bwd(to_dev(x), to_dev(dy), ob.Segments(cu), accumulate=True)
    for n in once:
        assert torch.equal((2 * once[n].float()).to(torch.bfloat16).view(torch.int16), run.g[n].view(torch.int16)), n


def _act_launches(shape, T):
    """the launches that apply the block's activation to a GEMM's result, forward and backward: (tile, ring slots, slices), None: a pass of its own"""
    H, F, up = shape.hidden, shape.mlp_dim, shape.mlp_dim * (2 if shape.mlp == si.MLP_SWIGLU else 1)
    scratch = any(ob.ob_gemm_workspace_bytes(0, T, n, k) for n, k in (((shape.n_q_heads + 2 * shape.n_kv_heads) * shape.head_dim, H), (H, H), (up, H), (H, F)))
    plans = (ob.ob_gemm_act_plan(shape.mlp, 0, T, F, H, scratch), ob.ob_gemm_act_plan(shape.mlp, 1, T, F, H))
    return tuple(p and (p.tile_rows, p.ring_slots, p.slices) for p in plans)


@pytest.mark.parametrize("mlp,bias,T,hidden,F,more,tiles", gemm_launches.ACTIVATIONS)
def test_epilogue_and_pass_give_the_same_bits(mlp, bias, T, hidden, F, more, tiles):
    """A batch whose GEMMs apply the activation and the same segments in front of a batch for which it is a pass of its own: up -> act over
    every row, and d act -> d up in single rows (the only ones with a gradient, so that the weight gradient is that row's d up times h2, and the bias
    gradient is the row), bit for bit."""
    print(f"epilogue and pass mlp={mlp} bias={bias} T={T} {hidden} {F}", flush=True)
    shape = si.small_shape(hidden=hidden, n_q_heads=hidden // 64, n_kv_heads=hidden // 64, head_dim=64, mlp_dim=F,
                           norm=si.NORM_LAYERNORM if bias else si.NORM_RMSNORM, mlp=mlp, mask=si.MASK_BIDIR, has_bias=bias, norm_eps=1e-5)
    assert _act_launches(shape, T) == tiles and _act_launches(shape, T + more) == (None, None)
    lens = [100] * (T // 100) + ([T % 100] if T % 100 else [])
    w = si.block_weights(shape, seed=2)
    x, dy = si.activations(T + more, hidden, seed=3, std=1.0)
    for row in (0, T // 2, T - 1):
        only = np.zeros_like(dy)
        only[row] = dy[row]
        short, _, _, _ = run_block(shape, w, x[:T], only[:T], si.lengths_to_cu(lens))
        long, _, _, _ = run_block(shape, w, x, only, si.lengths_to_cu(lens + [100] * (more // 100)))
        for name, n in (("up", F * (2 if mlp == si.MLP_SWIGLU else 1)), ("act", F)):
            a, b = (saved_view(r.desc, t, r.saved, name, (t, n))[:T] for r, t in ((short, T), (long, T + more)))
            assert torch.equal(a.view(torch.int16), b.view(torch.int16)), name
        for name in ("w_up",) + (("b_up",) if bias else ()):
            assert torch.equal(short.g[name], long.g[name]) and short.g[name].any(), (name, row)      # (a zero's sign depends on the sums' order)


@pytest.mark.parametrize("mlp,T,hidden,F,tile", [(si.MLP_GELU, 1, 128, 192, (64, 8)), (si.MLP_GELU, 65, 256, 512, (64, 8)),
                                                 (si.MLP_GELU, 1025, 640, 2560, (128, 4)), (si.MLP_GELU, 1500, 768, 2112, (128, 8)),
                                                 (si.MLP_SWIGLU, 129, 256, 1088, (64, 8)), (si.MLP_SWIGLU, 1700, 640, 2560, (128, 4))])
def test_activations_in_the_epilogue(mlp, T, hidden, F, tile):
    """Activations applied to a GEMM's result on its way out, forward (GELU) and backward, with the column sums that come with the backward:
    each kind of tile that takes them, rows and columns on and beside the tiles' borders, against the oracle."""
    print(f"activation in the epilogue mlp={mlp} T={T} {hidden} {F}", flush=True)
    shape = si.small_shape(hidden=hidden, n_q_heads=hidden // 64, n_kv_heads=hidden // 64, head_dim=64, mlp_dim=F,
                           norm=si.NORM_LAYERNORM, mlp=mlp, mask=si.MASK_BIDIR, has_bias=True, norm_eps=1e-5)
    assert _act_launches(shape, T) == ((tile[0], tile[1], 1) if mlp == si.MLP_GELU else None, (tile[0], 8 if tile[0] == 64 else 4, 1))
    lens = [100] * (T // 100) + ([T % 100] if T % 100 else [])
    cu = si.lengths_to_cu(lens)
    w = si.block_weights(shape, seed=2)
    x, dy = si.activations(T, hidden, seed=3, std=1.0)
    run, y, dx, g = run_block(shape, w, x, dy, cu)
    y_ref, cache = orc.block_fwd(shape, w, x, cu)
    dx_ref, g_ref, _ = orc.block_bwd(shape, w, cache, dy, cu)
    for n, got, ref in [("y", y, y_ref), ("dx", dx, dx_ref)] + [(n, g[n], g_ref[n]) for n in g]:
        if n != "b_qkv" or T > 1:      # (one token: no gradient through its softmax, and the oracle's rounding as the scale)
            assert np.abs(got - ref).max() <= TOL * np.abs(ref).max(), n


@pytest.mark.parametrize("T,F", [(2051, 4160), (4102, 2112)])
def test_column_sums_beside_the_passes(T, F):
    """Where the GEMM in front has large tiles, GELU's backward is a pass of its own that leaves the column sums of its result, and so is the
    hand-over's gather: columns that do not fill the last workgroup, rows that do not fill the last walk.  Against the oracle."""
    print(f"column sums beside the passes T={T} F={F}", flush=True)
    assert ob.ob_gemm_act_plan(si.MLP_GELU, 1, T, F, 256) is None
    shape = si.small_shape(hidden=256, n_q_heads=4, n_kv_heads=4, head_dim=64, mlp_dim=F, norm=si.NORM_LAYERNORM, mlp=si.MLP_GELU,
                           mask=si.MASK_BIDIR, has_bias=True, norm_eps=1e-5)
    cu = si.lengths_to_cu([100] * (T // 100) + [T % 100])
    w = si.block_weights(shape, seed=2)
    x, dy = si.activations(T, 256, seed=3, std=1.0)
    _, _, dx, g = run_block(shape, w, x, dy, cu)
    _, cache = orc.block_fwd(shape, w, x, cu)
    dx_ref, g_ref, _ = orc.block_bwd(shape, w, cache, dy, cu)
    for n, got, ref in [("dx", dx, dx_ref)] + [(n, g[n], g_ref[n]) for n in g]:
        assert np.abs(got - ref).max() <= TOL * np.abs(ref).max(), n
    if F == 2112:      # the hand-over over as many tokens, a square GEMM in front
        assert ob.ob_gemm_act_plan(si.MLP_GELU, 1, T, F, F) is None
        test_connector_widths(64, F, 2, T)


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
