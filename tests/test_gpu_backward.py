"""Backward pass on the GPU against the CPU oracle, through the C ABI (needs an MI355X).

The kernels are fed the ORACLE's forward results (weights rounded to bfloat16, metadata converted
to the library's order), so that both sides differentiate through exactly the same selection; the
composition with the GPU forward pass is checked on integer-valued Q, K, where the selection is exact.
Tolerances: operands are bfloat16 (8 significant bits) and sums run in fp32, so results agree to
about 2^-8 of the magnitudes involved; each bound below is stated next to its check.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2203_00091_amd as dfss
from paper_2203_00091_amd import Shape, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _dev(t):
    return t.to(DEV).contiguous()


def _np(t):
    return t.detach().to("cpu", torch.float32).numpy()


def _bf16(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).to(torch.bfloat16)


def _oracle_forward(Qn, Kn, N, M, scale):
    """Per head: kept indices, bf16-rounded weights, canonical metadata."""
    kidx, P, meta = [], [], []
    for h in range(Qn.shape[0]):
        S = oracle.scores(Qn[h], Kn[h], scale)
        _, vals, ki = oracle.prune(S, N, M)
        P.append(oracle.round_bf16(oracle.softmax_kept(oracle.round_bf16(vals))))
        kidx.append(ki)
        meta.append(oracle.encode_meta(ki, Kn.shape[1]))
    return np.stack(kidx), np.stack(P), np.stack(meta)


@pytest.mark.parametrize("BH,Lq,Lk,d,N,M", [
    (2, 128, 256, 64, 2, 4),
    (3, 192, 128, 64, 1, 2),      # more queries than keys, three query steps
    (2, 64, 384, 128, 2, 4),      # d = 128, one query step
])
def test_transposed_spmm(BH, Lq, Lk, d, N, M):
    Q, K, _ = synth.gaussian_qkv(BH, Lq, Lk, d, 1.0, seed=9300 + Lq + Lk)
    g = torch.Generator().manual_seed(9301 + d)
    X = torch.randn(BH, Lq, d, generator=g).to(torch.bfloat16)
    s = Shape(1, BH, Lq, Lk, d, N, M)
    Qn, Kn, Xn = (synth.to_numpy_f32(t) for t in (Q, K, X))
    kidx, P, meta_c = _oracle_forward(Qn, Kn, N, M, 1.0 / math.sqrt(d))
    meta = dfss.dfss_meta_from_canonical(_dev(torch.from_numpy(meta_c.view(np.int16))), s)
    out = dfss.dfss_spmm_t(_dev(_bf16(P)), meta, _dev(X), s)
    torch.cuda.synchronize()
    out = _np(out)
    for h in range(BH):
        Pd = np.zeros((Lq, Lk))
        np.put_along_axis(Pd, kidx[h].astype(np.int64), P[h].astype(np.float64), axis=1)
        ref = Pd.T @ Xn[h].astype(np.float64)
        # bf16 output rounding (2^-9 relative) + fp32 accumulation of <= Lq terms
        assert np.max(np.abs(out[h] - ref)) <= 2.0 ** -8 * np.max(np.abs(ref)) + 1e-4


def _oracle_backward_case(BH, Lq, Lk, d, N, M, seed, scale):
    Q, K, V = synth.gaussian_qkv(BH, Lq, Lk, d, 1.0, seed=seed)
    g = torch.Generator().manual_seed(seed + 1)
    dO = torch.randn(BH, Lq, d, generator=g).to(torch.bfloat16)
    Qn, Kn, Vn, dOn = (synth.to_numpy_f32(t) for t in (Q, K, V, dO))
    kidx, P, meta_c = _oracle_forward(Qn, Kn, N, M, scale)
    O = np.stack([oracle.round_bf16(oracle.spmm(P[h], kidx[h], Vn[h])) for h in range(BH)])
    return (Q, K, V, dO), (Qn, Kn, Vn, dOn), kidx, P, meta_c, O


@pytest.mark.parametrize("BH,Lq,Lk,d,N,M", [
    (2, 128, 256, 64, 2, 4),
    (2, 192, 384, 64, 1, 2),       # three tiles of 64 queries, three pairs of key blocks
    (2, 128, 128, 128, 2, 4),      # d = 128
])
def test_backward_against_oracle_through_the_same_selection(BH, Lq, Lk, d, N, M):
    scale = 1.0 / math.sqrt(d)
    (Q, K, V, dO), (Qn, Kn, Vn, dOn), kidx, P, meta_c, O = _oracle_backward_case(BH, Lq, Lk, d, N, M, 9400 + Lq + d, scale)
    s = Shape(1, BH, Lq, Lk, d, N, M)
    meta = dfss.dfss_meta_from_canonical(_dev(torch.from_numpy(meta_c.view(np.int16))), s)
    dQ, dK, dV = dfss.dfss_attention_backward(_dev(dO), _dev(Q), _dev(K), _dev(V), _dev(_bf16(O)), _dev(_bf16(P)),
                                              meta, s, scale)
    torch.cuda.synchronize()
    dQ, dK, dV = _np(dQ), _np(dK), _np(dV)
    for h in range(BH):
        rQ, rK, rV = oracle.attention_backward(Qn[h], Kn[h], Vn[h], dOn[h], P[h], kidx[h], scale)
        for name, got, ref in (("dQ", dQ[h], rQ), ("dK", dK[h], rK), ("dV", dV[h], rV)):
            # operands (P, dS, O) and results are bfloat16 (2^-9 relative each); observed <= 0.0053 of the largest entry
            tol = 2.0 ** -7 * np.max(np.abs(ref)) + 1e-4
            err = np.max(np.abs(got - ref))
            assert err <= tol, (name, h, err, tol)


def test_forward_stages_then_backward_on_exact_scores():
    """GPU forward (three stage calls, integer Q and K: the selection equals the oracle's exactly)
    followed by the GPU backward, against the oracle end to end."""
    BH, L, d = 2, 256, 64
    Q, K, V = synth.integer_qkv(BH, L, L, d, seed=9500)
    Q, K = (Q.float() * 0.25).to(torch.bfloat16), (K.float() * 0.25).to(torch.bfloat16)   # keeps the softmax soft
    g = torch.Generator().manual_seed(9501)
    dO = torch.randn(BH, L, d, generator=g).to(torch.bfloat16)
    s = Shape(1, BH, L, L, d, 2, 4)
    Qd, Kd, Vd, dOd = _dev(Q), _dev(K), _dev(V), _dev(dO)
    vals, meta = dfss.dfss_sddmm_prune(Qd, Kd, s, 0.125)
    dfss.dfss_sparse_softmax(vals, s)
    O = dfss.dfss_spmm(vals, meta, Vd, s)
    dQ, dK, dV = dfss.dfss_attention_backward(dOd, Qd, Kd, Vd, O, vals, meta, s, 0.125)
    torch.cuda.synchronize()
    Qn, Kn, Vn, dOn = (synth.to_numpy_f32(t) for t in (Q, K, V, dO))
    kidx, P, meta_c = _oracle_forward(Qn, Kn, 2, 4, 0.125)
    canon = dfss.dfss_meta_to_canonical(meta, s)
    torch.cuda.synchronize()
    assert np.array_equal(canon.cpu().numpy().view(np.uint16), meta_c)       # same selection on both sides
    for h in range(BH):
        rQ, rK, rV = oracle.attention_backward(Qn[h], Kn[h], Vn[h], dOn[h], P[h], kidx[h], 0.125)
        for name, got, ref in (("dQ", _np(dQ[h]), rQ), ("dK", _np(dK[h]), rK), ("dV", _np(dV[h]), rV)):
            tol = 2.0 ** -7 * np.max(np.abs(ref)) + 1e-4
            assert np.max(np.abs(got - ref)) <= tol, (name, h)


@pytest.mark.parametrize("BH,Lq,Lk,d,N,M", [
    (192, 320, 384, 64, 1, 2),     # 128-query workgroups, the last one of a head half empty
    (96, 704, 704, 64, 2, 4),      # 11 blocks of 64 keys: a single one in the last pair
    (140, 512, 256, 128, 2, 4),    # d = 128, 128-query workgroups
    (192, 300, 388, 64, 2, 4),     # no tile multiples: the last workgroup of a head half empty, and absent rows and keys
    (180, 330, 260, 128, 1, 2),
    (512, 256, 128, 64, 2, 4),     # (dQ and dK, dV each on both sides of the rule that keeps workgroups level: a part-filled last round
    (512, 200, 132, 64, 1, 2),     # does not, all at once do)
    (128, 512, 256, 128, 2, 4),
    (256, 200, 260, 128, 1, 2),
    (90, 192, 384, 64, 2, 4),      # 64-query workgroups
    (90, 150, 332, 64, 1, 2),
    (70, 256, 512, 128, 1, 2),
    (70, 230, 400, 128, 2, 4),
])
def test_backward_on_grids_that_fill_the_chip(BH, Lq, Lk, d, N, M):
    """Waves that compete for the matrix unit see its results later than a lone wave does; sampled heads against the
    oracle, differentiating through the GPU's own forward results.  What the rows of the weights past Lq hold must not
    matter (NaN here); nothing is written behind a gradient."""
    scale = 1.0 / math.sqrt(d)
    Q, K, V = synth.gaussian_qkv(BH, Lq, Lk, d, 1.0, seed=9800 + Lq + d)
    g = torch.Generator().manual_seed(9801 + d)
    dO = torch.randn(BH, Lq, d, generator=g).to(torch.bfloat16)
    s = Shape(1, BH, Lq, Lk, d, N, M)
    Qd, Kd, Vd, dOd = _dev(Q), _dev(K), _dev(V), _dev(dO)
    P, meta = dfss.dfss_sddmm_prune(Qd, Kd, s, scale)
    dfss.dfss_sparse_softmax(P, s)
    O = dfss.dfss_spmm(P, meta, Vd, s)
    P[:, Lq:] = math.nan
    bufs = [torch.full((BH * L * d + 4096,), 777.0, dtype=torch.bfloat16, device=DEV) for L in (Lq, Lk, Lk)]
    dQ, dK, dV = (x[:BH * L * d].view(BH, L, d) for x, L in zip(bufs, (Lq, Lk, Lk)))
    dfss.dfss_attention_backward(dOd, Qd, Kd, Vd, O, P, meta, s, scale, dQ=dQ, dK=dK, dV=dV)
    canon = dfss.dfss_meta_to_canonical(meta, s)
    torch.cuda.synchronize()
    for x in bufs:
        assert bool((x[-4096:] == 777.0).all()), "wrote behind a gradient"
    for h in (0, BH // 3, BH // 2 + 1, BH - 1):
        kidx = oracle.decode_meta(canon[h].cpu().numpy().view(np.uint16), s.LkP)[:Lq]
        Ph = _np(P[h])[:Lq]
        real = kidx < Lk
        assert np.all(Ph[~real] == 0.0)
        ki, Pr = np.where(real, kidx, 0).astype(np.int32), np.where(real, Ph, 0.0).astype(np.float32)
        Qn, Kn, Vn, dOn = (synth.to_numpy_f32(t[h]) for t in (Q, K, V, dO))
        rQ, rK, rV = oracle.attention_backward(Qn, Kn, Vn, dOn, Pr, ki, scale)
        for name, got, ref in (("dQ", _np(dQ[h]), rQ), ("dK", _np(dK[h]), rK), ("dV", _np(dV[h]), rV)):
            tol = 2.0 ** -7 * np.max(np.abs(ref)) + 1e-4      # as above
            assert np.max(np.abs(got - ref)) <= tol, (name, h)


def _sharing_bytes(s, keys, queries):
    """The workspace of a backward pass whose dQ tiles are shared by `keys` workgroups, whose dV, dK tiles by `queries` (1: none):
    the row terms, then the fp32 sums."""
    up = lambda n: (n + 255) // 256 * 256
    return (up(4 * s.BH * s.LqP) + (up(4 * keys * s.BH * s.Lq * s.d) if keys > 1 else 0)
            + (up(8 * queries * s.BH * s.Lk * s.d) if queries > 1 else 0))


@pytest.mark.parametrize("BH,Lq,Lk,d,N,M,keys,queries", [
    (1, 64, 512, 128, 2, 4, 2, 1),      # dQ: two workgroups share the keys of a query tile
    (2, 128, 640, 128, 1, 2, 2, 1),     # ... five pairs of key blocks for two
    (1, 1, 8192, 128, 2, 4, 32, 1),     # ... 32 workgroups; one query
    (2, 70, 580, 128, 2, 4, 2, 1),      # ... no tile multiples; four keys in the last block
    (2, 70, 572, 128, 2, 4, 2, 1),      # ... a single block in the last pair
    (2, 70, 2092, 128, 1, 2, 8, 1),     # ... 17 pairs for eight workgroups
    (1, 64, 4096, 64, 1, 2, 16, 1),     # ... d = 64
    (3, 100, 4100, 64, 2, 4, 16, 1),
    (9, 60, 4096, 64, 2, 4, 16, 1),
    (1, 100, 1400, 64, 1, 2, 5, 1),     # ... five: two pairs each, the last one three
    (2, 128, 256, 64, 2, 4, 1, 1),      # (nobody shares)
    (1, 1100, 256, 64, 2, 4, 1, 4),     # dV, dK: workgroups share the queries of a key tile; a partial last block of queries
    (2, 640, 128, 128, 1, 2, 1, 2),     # ... d = 128
    (3, 1000, 1500, 64, 2, 4, 6, 4),    # ... and the keys in dQ, no tile multiples
    (1, 2048, 1024, 128, 2, 4, 4, 8),
    (1, 1990, 1020, 128, 1, 2, 4, 8),
    (1, 700, 260, 128, 2, 4, 1, 2),
])
def test_backward_with_a_workspace_of_exactly_the_size_it_asks_for(BH, Lq, Lk, d, N, M, keys, queries):
    """Few queries against many keys and the other way round, against the oracle; poisoned scratch of exactly
    dfss_backward_workspace_bytes, which tells how many workgroups share, and guards behind it and behind every gradient."""
    assert dfss.dfss_backward_workspace_bytes(Shape(1, BH, Lq, Lk, d, N, M)) == _sharing_bytes(Shape(1, BH, Lq, Lk, d, N, M), keys, queries)
    scale = 1.0 / math.sqrt(d)
    Q, K, V = synth.gaussian_qkv(BH, Lq, Lk, d, 1.0, seed=9900 + Lq + Lk + d)
    dO = torch.randn(BH, Lq, d, generator=torch.Generator().manual_seed(9901 + Lk)).to(torch.bfloat16)
    Qn, Kn, Vn, dOn = (synth.to_numpy_f32(t) for t in (Q, K, V, dO))
    s = Shape(1, BH, Lq, Lk, d, N, M)
    kidx, P, Pp, mp = _padded_forward(Qn, Kn, N, M, scale, s)
    O = []
    for h in range(BH):
        Pd = np.zeros((Lq, s.LkP))
        np.put_along_axis(Pd, kidx[h].astype(np.int64), P[h].astype(np.float64), axis=1)
        O.append((Pd[:, :Lk] @ Vn[h].astype(np.float64)).astype(np.float32))
    meta = dfss.dfss_meta_from_canonical(_dev(torch.from_numpy(mp.view(np.int16))), s)
    guard, need = 4096, dfss.dfss_backward_workspace_bytes(s)
    ws = torch.full((need + guard,), 0xFF, dtype=torch.uint8, device=DEV)
    bufs = [torch.full((BH * L * d + guard,), 777.0, dtype=torch.bfloat16, device=DEV) for L in (Lq, Lk, Lk)]
    dQ, dK, dV = (b[:b.numel() - guard].view(BH, L, d) for b, L in zip(bufs, (Lq, Lk, Lk)))
    dfss.dfss_attention_backward(_dev(dO), _dev(Q), _dev(K), _dev(V), _dev(_bf16(np.stack(O))), _dev(_bf16(Pp)), meta, s,
                                 scale, dQ=dQ, dK=dK, dV=dV, ws=ws[:need])
    torch.cuda.synchronize()
    assert bool((ws[need:] == 0xFF).all()), "wrote behind the workspace"
    for b in bufs:
        assert bool((b[b.numel() - guard:] == 777.0).all()), "wrote behind a gradient"
    dQ, dK, dV = _np(dQ), _np(dK), _np(dV)
    for h in range(BH):
        real = kidx[h] < Lk
        ki, Pr = np.where(real, kidx[h], 0).astype(np.int32), np.where(real, P[h], 0.0).astype(np.float32)
        rQ, rK, rV = oracle.attention_backward(Qn[h], Kn[h], Vn[h], dOn[h], Pr, ki, scale)
        for name, got, ref in (("dQ", dQ[h], rQ), ("dK", dK[h], rK), ("dV", dV[h], rV)):
            tol = 2.0 ** -7 * np.max(np.abs(ref)) + 1e-4      # as above
            assert np.max(np.abs(got - ref)) <= tol, (name, h)


def test_backward_with_a_workspace_that_holds_the_row_terms_only():
    """A workspace of a larger shape's size serves a smaller shape whose workgroups would share keys: the same gradients
    but for the order of the sums in dQ; one that does not hold the row terms is refused."""
    large, s = Shape(1, 64, 512, 512, 128), Shape(1, 2, 64, 2048, 128)
    least, need = 4 * s.BH * s.LqP, dfss.dfss_backward_workspace_bytes(s)
    assert least <= dfss.dfss_backward_workspace_bytes(large) < need
    g = torch.Generator().manual_seed(9950)
    Q, K, V, dO = (torch.randn(s.BH, L, s.d, generator=g).to(DEV, torch.bfloat16) for L in (s.Lq, s.Lk, s.Lk, s.Lq))
    scale = 1.0 / math.sqrt(s.d)
    P, meta = dfss.dfss_sddmm_prune(Q, K, s, scale)
    dfss.dfss_sparse_softmax(P, s)
    O = dfss.dfss_spmm(P, meta, V, s)

    def run(n):
        ws = torch.full((n + 4096,), 0xFF, dtype=torch.uint8, device=DEV)
        out = dfss.dfss_attention_backward(dO, Q, K, V, O, P, meta, s, scale, ws=ws[:n])
        torch.cuda.synchronize()
        assert bool((ws[n:] == 0xFF).all())
        return out

    shared, alone, alone2 = run(need), run(dfss.dfss_backward_workspace_bytes(large)), run(least)
    for a, b, c in zip(shared, alone, alone2):
        assert torch.equal(b, c)
        # fp32 sums in another order, rounded to bfloat16: half a unit in the last place apart at most, and rarely
        assert (a.float() - b.float()).abs().max() <= 2.0 ** -8 * b.float().abs().max()
    assert torch.equal(shared[1], alone[1]) and torch.equal(shared[2], alone[2])      # dK, dV
    with pytest.raises(dfss.DfssError):
        run(least - 256)


@pytest.mark.parametrize("Lq,Lk", [(2048, 1152), (1990, 1020)])
def test_backward_shares_as_far_as_the_workspace_reaches(Lq, Lk):
    """Shared keys and shared queries need two parts of a workspace.  One that holds fewer sums, or those of one part only, is used for
    these; all of them give the oracle's gradients, and what is shared shows in the order of the sums."""
    s, scale = Shape(1, 1, Lq, Lk, 128), 1.0 / math.sqrt(128)
    g = torch.Generator().manual_seed(9960)
    Q, K, V, dO = (torch.randn(1, L, 128, generator=g).to(DEV, torch.bfloat16) for L in (Lq, Lk, Lk, Lq))
    P, meta = dfss.dfss_sddmm_prune(Q, K, s, scale)
    dfss.dfss_sparse_softmax(P, s)
    O = dfss.dfss_spmm(P, meta, V, s)
    kidx = oracle.decode_meta(dfss.dfss_meta_to_canonical(meta, s)[0].cpu().numpy().view(np.uint16), s.LkP)[:Lq]
    real, Ph = kidx < Lk, _np(P[0])[:Lq]
    refs = oracle.attention_backward(*(_np(t[0]) for t in (Q, K, V, dO)), np.where(real, Ph, 0.0).astype(np.float32),
                                     np.where(real, kidx, 0).astype(np.int32), scale)

    def run(n):
        ws = torch.full((n + 4096,), 0xFF, dtype=torch.uint8, device=DEV)
        out = dfss.dfss_attention_backward(dO, Q, K, V, O, P, meta, s, scale, ws=ws[:n])
        torch.cuda.synchronize()
        assert bool((ws[n:] == 0xFF).all()), "wrote behind the workspace"
        for got, ref in zip(out, refs):
            assert np.max(np.abs(_np(got[0]) - ref)) <= 2.0 ** -7 * np.max(np.abs(ref)) + 1e-4      # as above
        return out

    assert dfss.dfss_backward_workspace_bytes(s) == _sharing_bytes(s, 4, 8)
    both, queries, fewer, keys, alone = (run(n) for n in (_sharing_bytes(s, 4, 8), _sharing_bytes(s, 1, 8), _sharing_bytes(s, 1, 2),
                                                          _sharing_bytes(s, 2, 1), _sharing_bytes(s, 1, 1)))
    same = [[torch.equal(a, b) for a, b in zip(x, alone)] for x in (both, queries, fewer, keys)]
    assert same == [[False, False, False], [True, False, False], [True, False, False], [False, True, True]]
    assert torch.equal(queries[1], both[1]) and not torch.equal(fewer[1], both[1])      # eight, and two


@pytest.mark.parametrize("BH,Lq,Lk,d,N,M", [
    (2, 128, 256, 64, 2, 4), (2, 192, 128, 64, 1, 2), (2, 64, 384, 128, 2, 4),
    (2, 100, 132, 64, 2, 4), (2, 70, 260, 128, 1, 2),       # no tile multiples
    (1, 1088, 128, 64, 2, 4), (1, 700, 260, 128, 1, 2),     # queries shared: one of the workgroups starts again
])
@pytest.mark.parametrize("what", ["V", "dO", "P", "one weight"])
def test_what_is_not_finite_reaches_the_kept_places_only(what, BH, Lq, Lk, d, N, M):
    """Infinities and NaN in a row of V that no query kept, in a row of dO, in a row of weights, in a single weight: every
    gradient that they do not enter through a kept place is, bit for bit, what it is with zeros instead."""
    scale = 1.0 / math.sqrt(d)
    Q, K, V = synth.gaussian_qkv(BH, Lq, Lk, d, 1.0, seed=9600 + Lq + d)
    dO = torch.randn(BH, Lq, d, generator=torch.Generator().manual_seed(9601 + Lq)).to(torch.bfloat16)
    Qn, Kn, Vn = (synth.to_numpy_f32(t) for t in (Q, K, V))
    s = Shape(1, BH, Lq, Lk, d, N, M)
    never = [5, 70, 99, Lk - 2]            # one key of a run each: masked, so that no query keeps it
    kidx, O = [], []
    P = np.full((BH, s.LqP, s.Lc), 0.25, dtype=np.float32)
    meta_c = np.full((BH, s.LqP, s.meta_words), 0x4444, dtype=np.uint16)
    for h in range(BH):
        S = np.full((Lq, s.LkP), -np.inf, dtype=np.float32)
        S[:, :Lk] = oracle.scores(Qn[h], Kn[h], scale)
        S[:, never] = -np.inf
        _, vals, ki = oracle.prune(S, N, M)
        assert not np.isin(never, ki).any()
        kidx.append(ki)
        P[h, :Lq] = oracle.round_bf16(oracle.softmax_kept(oracle.round_bf16(vals)))
        meta_c[h, :Lq] = oracle.encode_meta(ki, s.LkP)
        Pd = np.zeros((Lq, s.LkP))
        np.put_along_axis(Pd, ki.astype(np.int64), P[h, :Lq].astype(np.float64), axis=1)
        O.append((Pd[:, :Lk] @ Vn[h].astype(np.float64)).astype(np.float32))
    meta = dfss.dfss_meta_from_canonical(_dev(torch.from_numpy(meta_c.view(np.int16))), s)
    Qd, Kd, Od = _dev(Q), _dev(K), _dev(_bf16(np.stack(O)))
    q0, e0 = 37, 21                        # the row; the kept entry of the single weight
    for bad in (math.nan, math.inf, -math.inf):
        got = []
        for x in (0.0, bad):
            V_, dO_, P_ = V.clone(), dO.clone(), _bf16(P)
            if what == "V":
                V_[0, never] = x
            elif what == "dO":
                dO_[0, q0] = x
            elif what == "P":
                P_[0, q0] = x
            else:
                P_[0, q0, e0] = x
            grads = dfss.dfss_attention_backward(_dev(dO_), Qd, Kd, _dev(V_), Od, _dev(P_), meta, s, scale)
            torch.cuda.synchronize()
            got.append([_np(t) for t in grads])
        rows = np.ones((BH, Lq), bool)     # rows of dQ, and of dK and dV, that have to agree
        keys = {"dK": np.ones((BH, Lk), bool), "dV": np.ones((BH, Lk), bool)}
        if what != "V":
            rows[0, q0] = False
            hit = kidx[0][q0] if what != "one weight" else kidx[0][q0, e0:e0 + 1]
            for k in keys.values():
                k[0, hit[hit < Lk]] = False
            if what == "dO":               # dO itself is a factor of dV: every key of the head
                keys["dV"][0] = False
        (zQ, zK, zV), (bQ, bK, bV) = got
        for name, z, b, sel in (("dQ", zQ, bQ, rows), ("dK", zK, bK, keys["dK"]), ("dV", zV, bV, keys["dV"])):
            assert np.isfinite(z).all() and np.array_equal(z[sel], b[sel]), (name, bad)
            if name != "dQ" and what != "V":
                assert not np.isfinite(b[~sel]).any(), (name, bad)


# ----------------------------------------------------------------------------------
# lengths that are not tile multiples: P and meta keep the layout of the padded lengths
# ----------------------------------------------------------------------------------
def _padded_forward(Qn, Kn, N, M, scale, s):
    """The oracle's forward results in the padded layout: absent keys count as -inf; the rows past Lq hold finite
    junk (weights 0.25, codes 0x4) that no gradient may depend on."""
    BH, Lq, Lk = Qn.shape[0], Qn.shape[1], Kn.shape[1]
    kidx, P = [], []
    Pp = np.full((BH, s.LqP, s.Lc), 0.25, dtype=np.float32)
    mp = np.full((BH, s.LqP, s.meta_words), 0x4444, dtype=np.uint16)
    for h in range(BH):
        Sp = np.full((Lq, s.LkP), -np.inf, dtype=np.float32)
        Sp[:, :Lk] = oracle.scores(Qn[h], Kn[h], scale)
        _, vals, ki = oracle.prune(Sp, N, M)
        Ph = oracle.round_bf16(oracle.softmax_kept(oracle.round_bf16(vals)))
        Pp[h, :Lq] = Ph
        mp[h, :Lq] = oracle.encode_meta(ki, s.LkP)
        # for the oracle's backward pass: the kept entries that are real keys (the absent ones have weight 0)
        kidx.append(ki)
        P.append(Ph)
    return kidx, P, Pp, mp


@pytest.mark.parametrize("BH,Lq,Lk,d,N,M", [
    (2, 100, 132, 64, 2, 4),       # one partial query tile, a partial second key block
    (2, 250, 516, 64, 1, 2),       # 4 real keys in the last block
    (2, 70, 260, 128, 2, 4),       # d = 128
])
def test_backward_on_unpadded_lengths(BH, Lq, Lk, d, N, M):
    scale = 1.0 / math.sqrt(d)
    Q, K, V = synth.gaussian_qkv(BH, Lq, Lk, d, 1.0, seed=9700 + Lq + d)
    g = torch.Generator().manual_seed(9701 + Lq)
    dO = torch.randn(BH, Lq, d, generator=g).to(torch.bfloat16)
    Qn, Kn, Vn, dOn = (synth.to_numpy_f32(t) for t in (Q, K, V, dO))
    s = Shape(1, BH, Lq, Lk, d, N, M)
    assert (s.LqP, s.LkP) != (Lq, Lk)
    kidx, P, Pp, mp = _padded_forward(Qn, Kn, N, M, scale, s)
    # O of the forward pass from the real keys only (weights of absent keys are 0; their indices point past Lk)
    O = []
    for h in range(BH):
        Pd = np.zeros((Lq, s.LkP))
        np.put_along_axis(Pd, kidx[h].astype(np.int64), P[h].astype(np.float64), axis=1)
        O.append(oracle.round_bf16((Pd[:, :Lk] @ Vn[h].astype(np.float64)).astype(np.float32)))
    O = np.stack(O)
    meta = dfss.dfss_meta_from_canonical(_dev(torch.from_numpy(mp.view(np.int16))), s)
    guard = 4096
    bufs = [torch.full((n + guard,), 777.0, dtype=torch.bfloat16, device=DEV) for n in (BH * Lq * d, BH * Lk * d, BH * Lk * d)]
    dQ, dK, dV = (b[:b.numel() - guard].view(BH, L, d) for b, L in zip(bufs, (Lq, Lk, Lk)))
    dfss.dfss_attention_backward(_dev(dO), _dev(Q), _dev(K), _dev(V), _dev(_bf16(O)), _dev(_bf16(Pp)), meta, s, scale,
                                 dQ=dQ, dK=dK, dV=dV)
    X = torch.randn(BH, Lq, d, generator=g).to(torch.bfloat16)
    T = dfss.dfss_spmm_t(_dev(_bf16(Pp)), meta, _dev(X), s)
    torch.cuda.synchronize()
    for b in bufs:
        assert bool((b[b.numel() - guard:] == 777.0).all()), "wrote behind a gradient"
    assert tuple(T.shape) == (BH, Lk, d)
    dQ, dK, dV, T, Xn = _np(dQ), _np(dK), _np(dV), _np(T), synth.to_numpy_f32(X)
    for h in range(BH):
        real = kidx[h] < Lk                          # kept entries that are real keys
        ki = np.where(real, kidx[h], 0)
        Pr = np.where(real, P[h], 0.0).astype(np.float32)
        assert np.all(P[h][~real] == 0.0)
        rQ, rK, rV = oracle.attention_backward(Qn[h], Kn[h], Vn[h], dOn[h], Pr, ki.astype(np.int32), scale)
        for name, got, ref in (("dQ", dQ[h], rQ), ("dK", dK[h], rK), ("dV", dV[h], rV)):
            assert np.isfinite(got).all(), name
            tol = 2.0 ** -7 * np.max(np.abs(ref)) + 1e-4
            err = np.max(np.abs(got - ref))
            assert err <= tol, (name, h, err, tol)
        Pd = np.zeros((Lq, s.LkP))
        np.put_along_axis(Pd, kidx[h].astype(np.int64), P[h].astype(np.float64), axis=1)
        refT = Pd[:, :Lk].T @ Xn[h].astype(np.float64)
        assert np.max(np.abs(T[h] - refT)) <= 2.0 ** -8 * np.max(np.abs(refT)) + 1e-4
