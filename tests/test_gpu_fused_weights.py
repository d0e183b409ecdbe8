"""Element-wise check of the one-kernel paths (needs an MI355X).

The one-kernel forward pass writes neither kept scores nor metadata, so its selection cannot be read
back directly.  It can be made visible: with V = the identity on d consecutive keys j0 .. j0+d-1 and zero
elsewhere, O[i, c] IS the softmax weight of key j0 + c in row i.  Sweeping j0 over the key axis shows the
whole weight matrix, which is compared with the oracle entry by entry:

  * a key the oracle drops must have weight exactly 0 (a wrong pick, or two swapped position codes inside a
    run of four, puts a weight on a dropped key);
  * a kept key must carry the oracle's weight up to the bfloat16 roundings of weight, row sum and output.

Q and K hold small integers, so every score is exact in fp32 on both sides and equal scores (ties) abound:
the selection must then agree with the oracle's rank rule exactly, ties included.
"""
import ctypes
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2203_00091_amd as dfss
from paper_2203_00091_amd import DFSS_BF16, DFSS_F32_BF16X3, Shape, binding, synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# Three bfloat16 roundings stack up in a weight: the weight itself, the dominant weight of its row (through the
# row sum) and the output.  Each is at most 2^-8 relative (half the spacing at the bottom of a binade):
# 3 * 2^-8 in the worst case, so 2^-6.  A wrong pick is off by 100 %.
REL, ABS = 2.0 ** -6, 1e-6


def _dense_weights(Qn, Kn, N, M, scale, key_bias=None, block_mask=None, mask=None):
    """The oracle's weight matrix of one head, dense [Lq, Lk] (0 at dropped keys), and the kept mask."""
    S = oracle.scores(Qn, Kn, scale)
    if key_bias is not None:
        S = oracle.add_key_bias(S, key_bias)
    if mask is not None:
        S = oracle.add_mask(S, mask)
    if block_mask is not None:
        S = oracle.apply_block_mask(S, block_mask, 64)
    mask, vals, kidx = oracle.prune(S, N, M)
    P = oracle.softmax_kept(vals)
    W = np.zeros(S.shape, np.float64)
    np.put_along_axis(W, kidx.astype(np.int64), P.astype(np.float64), axis=1)
    kept = np.zeros(S.shape, bool)
    np.put_along_axis(kept, kidx.astype(np.int64), True, axis=1)
    assert kept.sum() == kidx.size and np.array_equal(kept, mask.astype(bool))
    return W, kept, S


def _weights_through_identity_v(run, BH, Lq, Lk, d, tdtype):
    """Run `run(V)` once per block of d keys with V = identity on that block; returns [BH, Lq, Lk] weights."""
    out = np.empty((BH, Lq, Lk), np.float32)
    eye = torch.eye(d, dtype=tdtype, device=DEV)
    for j0 in range(0, Lk, d):
        V = torch.zeros((BH, Lk, d), dtype=tdtype, device=DEV)
        n = min(d, Lk - j0)
        V[:, j0:j0 + n, :] = eye[:n]
        O = run(V)
        torch.cuda.synchronize()
        out[:, :, j0:j0 + n] = O.float().cpu().numpy()[:, :, :n]
    return out


def _compare(Wgpu, Qn, Kn, N, M, scale, key_bias=None, H=1, block_mask=None, rel=REL, mask=None):
    ties = 0
    for h in range(Qn.shape[0]):
        kb = None if key_bias is None else key_bias[h // H]
        W, kept, S = _dense_weights(Qn[h], Kn[h], N, M, scale, kb, block_mask, mask)
        got = Wgpu[h].astype(np.float64)
        dropped_weight = np.abs(got[~kept])
        assert dropped_weight.max(initial=0.0) == 0.0, \
            f"head {h}: {int((dropped_weight > 0).sum())} dropped keys carry weight (largest {dropped_weight.max():.3e})"
        err = np.abs(got - W)
        assert (err <= rel * W + ABS).all(), f"head {h}: weight off by {err.max():.3e}"
        G = S.reshape(S.shape[0], -1, M)
        srt = np.sort(G, axis=-1)
        ties += int((srt[..., M - N] == srt[..., M - N - 1]).sum())   # N-th and (N+1)-th largest equal
    return ties


def _int_qk(BH, Lq, Lk, d, seed, tdtype=torch.bfloat16):
    Q, K, _ = synth.integer_qkv(BH, Lq, Lk, d, seed=seed, dtype=tdtype)
    return Q, K, synth.to_numpy_f32(Q), synth.to_numpy_f32(K)


VARIANTS = [binding.VARIANT_Q16, binding.VARIANT_Q16X2, binding.VARIANT_Q32W2, binding.VARIANT_Q32W4,
            binding.VARIANT_Q32K2, binding.VARIANT_FEW]


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("BH,Lq,Lk,d,N,M,scale", [
    (2, 128, 512, 64, 2, 4, 0.125),
    (2, 128, 384, 64, 1, 2, 0.125),
    (1, 128, 512, 128, 2, 4, 0.125),
    (1, 256, 256, 128, 1, 2, float(np.float32(1.0 / math.sqrt(128.0)))),   # scale that is not a power of two
    (2, 256, 384, 64, 2, 4, float(np.float32(1.0 / 3.0))),
])
def test_every_tiling_selects_and_weighs_like_the_oracle(variant, BH, Lq, Lk, d, N, M, scale):
    Q, K, Qn, Kn = _int_qk(BH, Lq, Lk, d, seed=8100 + Lk + d + N)
    s = Shape(1, BH, Lq, Lk, d, N, M)
    Qd, Kd = Q.to(DEV), K.to(DEV)
    W = _weights_through_identity_v(
        lambda V: binding.internal_attention_variant(Qd, Kd, V, None, s, scale, variant), BH, Lq, Lk, d, torch.bfloat16)
    ties = _compare(W, Qn, Kn, N, M, scale)
    assert ties > 100          # the tie rule was exercised


def _ragged_without_workspace(Q, K, V, key_bias, s, scale):
    """The C entry dfss_attention_ragged itself, at shapes whose Python call goes through a workspace."""
    assert key_bias is None
    O = torch.empty_like(Q)
    st = dfss.load_library().dfss_attention_ragged(Q.data_ptr(), K.data_ptr(), V.data_ptr(), None, ctypes.byref(s.c()), scale,
                                                   O.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert st == 0
    return O


@pytest.mark.parametrize("BH,Lq,Lk,d,N,M,scale,bias", [
    (3, 1, 132, 64, 2, 4, 0.125, False),       # (fewer than 256 keys: the kernel of the masked calls)
    (3, 1, 260, 64, 2, 4, 0.125, False),       # one query; one run of keys in the last block, most waves without a block
    (2, 16, 576, 64, 1, 2, 1.0 / 3.0, False),  # a whole query tile; nine blocks: one wave takes two
    (2, 17, 1092, 64, 2, 4, 0.125, True),      # a tile with one query; 18 blocks, list of live blocks
    (2, 33, 324, 128, 2, 4, 1.0 / 3.0, True),
    (1, 5, 260, 128, 1, 2, 0.125, False),
    (260, 1, 324, 64, 2, 4, 0.125, True),      # more tiles than compute units: two waves per workgroup
    (257, 2, 196, 128, 1, 2, 0.125, False),    # (fewer than 256 keys)
    (257, 1, 260, 128, 1, 2, 0.125, False),    # more tiles than compute units, d = 128
    (768, 1, 260, 128, 2, 4, 0.125, True),     # ... with a key bias (d = 128: from 768 heads on again)
    (320, 1, 260, 128, 2, 4, 0.125, True),     # (... the kernel below)
    (3, 3, 3076, 64, 2, 4, 0.125, False),      # 49 blocks shared between workgroups (d = 64: from 48 on)
    (2, 16, 1540, 128, 1, 2, 1.0 / 3.0, False),   # ... d = 128: from 24 on
    (70, 1, 1536, 128, 2, 4, 0.125, False),    # ... three workgroups per tile
])
def test_few_queries(BH, Lq, Lk, d, N, M, scale, bias):
    """The kernel whose waves share the keys: the weights of every key, through the public calls that take it (where
    several workgroups share keys, the call with a workspace and the one without)."""
    scale = float(np.float32(scale))
    Q, K, Qn, Kn = _int_qk(BH, Lq, Lk, d, seed=8700 + Lk + d + N)
    kb = None
    if bias:   # finite integers, and padding that ends in a block and leaves whole blocks masked
        kb = torch.randint(-2, 3, (BH, Lk), generator=torch.Generator().manual_seed(8701)).float()
        kb[0, Lk // 3 + 2:] = -math.inf
        kb[1, 64:128] = -math.inf
    s = Shape(BH, 1, Lq, Lk, d, N, M)
    Qd, Kd, kbd = Q.to(DEV), K.to(DEV), None if kb is None else kb.to(DEV)
    calls = [dfss.dfss_attention_ragged]
    if dfss.dfss_ragged_split_workspace_bytes(s) and not bias:
        calls.append(_ragged_without_workspace)
    for call in calls:
        W = _weights_through_identity_v(lambda V: call(Qd, Kd, V, kbd, s, scale), BH, Lq, Lk, d, torch.bfloat16)
        _compare(W, Qn, Kn, N, M, scale, key_bias=None if kb is None else kb.numpy())


def test_shared_keys_and_their_workspace():
    """dfss_attention_ragged_split: workspace given or allocated, poisoned, of exactly the size, guarded; shapes that share
    nothing and calls with a key bias are dfss_attention_ragged and take no workspace."""
    def case(BH, Lq, Lk, d):
        g = torch.Generator().manual_seed(8800 + Lk + d)
        s = Shape(BH, 1, Lq, Lk, d)
        return s, [torch.randn(BH, L, d, generator=g).to(DEV, torch.bfloat16) for L in (Lq, Lk, Lk)]

    for BH, Lq, Lk, d in ((12, 1, 3072, 64), (2, 16, 1540, 128), (104, 3, 3076, 64)):
        s, (Q, K, V) = case(BH, Lq, Lk, d)
        need = dfss.dfss_ragged_split_workspace_bytes(s)
        assert need > 0
        ref = dfss.dfss_attention_ragged(Q, K, V, None, s, 0.125)
        for fill in (0x00, 0xFF):
            ws = torch.full((need + 4096,), fill, dtype=torch.uint8, device=DEV)
            for call in (dfss.dfss_attention_ragged, dfss.dfss_attention_ragged_split):
                O = torch.full_like(Q, math.nan)
                assert call(Q, K, V, None, s, 0.125, O=O, ws=ws[:need]) is O
                torch.cuda.synchronize()
                assert torch.equal(O, ref) and bool((ws[need:] == fill).all())
        assert torch.equal(dfss.dfss_attention_ragged_split(Q, K, V, None, s, 0.125), ref)
        plain = _ragged_without_workspace(Q, K, V, None, s, 0.125)
        # the same weights, rounded to bfloat16 relative to another reference (2^-8), and one rounding of O
        assert (plain.float() - ref.float()).abs().max() <= 2.0 ** -7 * V.float().abs().max()
        with pytest.raises(dfss.DfssError, match="dfss_attention_ragged_split"):
            dfss.dfss_attention_ragged(Q, K, V, None, s, 0.125, ws=ws[:need - 256])
        bias = torch.zeros((BH, Lk), device=DEV)
        assert torch.equal(dfss.dfss_attention_ragged_split(Q, K, V, bias, s, 0.125),
                           dfss.dfss_attention_ragged(Q, K, V, bias, s, 0.125))
    for BH, Lq, Lk, d in ((12, 17, 4096, 64), (12, 1, 2048, 64), (3, 100, 332, 64)):
        s, (Q, K, V) = case(BH, Lq, Lk, d)
        assert dfss.dfss_ragged_split_workspace_bytes(s) == 0
        assert torch.equal(dfss.dfss_attention_ragged_split(Q, K, V, None, s, 0.125),
                           dfss.dfss_attention_ragged(Q, K, V, None, s, 0.125))


@pytest.mark.parametrize("variant", VARIANTS)
def test_weights_when_late_keys_raise_the_reference(variant):
    """Scores that grow along the key axis: the running reference of the softmax is raised in later blocks
    (the partial sums are rescaled, the block's scores re-centred) and the selection must not notice."""
    BH, L, d = 2, 384, 64
    Q, K, Qn, Kn = _int_qk(BH, L, L, d, seed=8242)
    ramp = (torch.arange(L) // 24).view(1, L, 1).float()                       # 0 .. 15 in steps
    K = (K.float() + ramp * torch.sign(Q.float().sum(1, keepdim=True))).to(torch.bfloat16)   # still integers
    Kn = synth.to_numpy_f32(K)
    s = Shape(1, BH, L, L, d, 2, 4)
    S = np.einsum("hqd,hkd->hqk", Qn, Kn) * 0.125
    assert (S.max(-1) - S[:, :, :64].max(-1)).max() > 16.0      # far above what the first block saw
    Qd, Kd = Q.to(DEV), K.to(DEV)
    W = _weights_through_identity_v(
        lambda V: binding.internal_attention_variant(Qd, Kd, V, None, s, 0.125, variant), BH, L, L, d, torch.bfloat16)
    _compare(W, Qn, Kn, 2, 4, 0.125)


@pytest.mark.parametrize("N,M", [(2, 4), (1, 2)])
def test_default_call_ragged_call_and_blocked_call(N, M):
    """The public one-kernel entry points: dfss_attention (whatever tiling it picks), dfss_attention_bias with
    a padding mask, dfss_attention_ragged on lengths that are no tile multiples, dfss_attention_blocked."""
    B, H, Lq, Lk, d = 2, 2, 192, 384, 64
    BH = B * H
    Q, K, Qn, Kn = _int_qk(BH, Lq, Lk, d, seed=8300 + N)
    s = Shape(B, H, Lq, Lk, d, N, M)
    Qd, Kd = Q.to(DEV), K.to(DEV)
    W = _weights_through_identity_v(lambda V: dfss.dfss_attention(Qd, Kd, V, s, 0.125), BH, Lq, Lk, d, torch.bfloat16)
    _compare(W, Qn, Kn, N, M, 0.125)
    # the two-kernel path (stage 1, then the product that applies the softmax on the way); 192 queries take the
    # 16-queries-per-wave stage 1, 128 of them the 32-queries-per-wave one
    W = _weights_through_identity_v(lambda V: dfss.dfss_attention_staged(Qd, Kd, V, s, 0.125), BH, Lq, Lk, d,
                                    torch.bfloat16)
    _compare(W, Qn, Kn, N, M, 0.125)
    s128 = Shape(B, H, 128, Lk, d, N, M)
    Q128 = Q[:, :128].contiguous().to(DEV)
    W = _weights_through_identity_v(lambda V: dfss.dfss_attention_staged(Q128, Kd, V, s128, 0.125), BH, 128, Lk, d,
                                    torch.bfloat16)
    _compare(W, Qn[:, :128], Kn, N, M, 0.125)
    # padding mask whose ends cut through runs of four
    lengths = torch.tensor([Lk, 203])
    bias = synth.key_padding_bias(lengths, Lk)
    bd = bias.to(DEV)
    W = _weights_through_identity_v(lambda V: dfss.dfss_attention_bias(Qd, Kd, V, bd, s, 0.125), BH, Lq, Lk, d,
                                    torch.bfloat16)
    _compare(W, Qn, Kn, N, M, 0.125, key_bias=bias.numpy(), H=H)
    W = _weights_through_identity_v(lambda V: dfss.dfss_attention_staged_bias(Qd, Kd, V, bd, s, 0.125), BH, Lq, Lk, d,
                                    torch.bfloat16)
    _compare(W, Qn, Kn, N, M, 0.125, key_bias=bias.numpy(), H=H)
    # unpadded lengths: 100 queries, 332 keys
    Lqr, Lkr = 100, 332
    sr = Shape(B, H, Lqr, Lkr, d, N, M)
    Qr, Kr = Q[:, :Lqr].contiguous().to(DEV), K[:, :Lkr].contiguous().to(DEV)
    W = _weights_through_identity_v(lambda V: dfss.dfss_attention_ragged(Qr, Kr, V, None, sr, 0.125), BH, Lqr, Lkr, d,
                                    torch.bfloat16)
    _compare(W, Qn[:, :Lqr], Kn[:, :Lkr], N, M, 0.125)
    # block pattern (window + global + random blocks)
    bm = synth.block_pattern(Lq // 64, Lk // 64, seed=77, window=1, n_global=1, n_random=1)
    bmd = bm.to(DEV)
    W = _weights_through_identity_v(lambda V: dfss.dfss_attention_blocked(Qd, Kd, V, None, bmd, s, 0.125), BH, Lq, Lk, d,
                                    torch.bfloat16)
    _compare(W, Qn, Kn, N, M, 0.125, block_mask=bm.numpy())


@pytest.mark.parametrize("BH,Lq,Lk,d,N,M,scale", [
    (2, 128, 384, 64, 2, 4, 0.125),                              # the mask is the initial value of the accumulators
    (2, 192, 256, 64, 1, 2, float(np.float32(1.0 / 3.0))),       # the mask is added after the scaling
    (1, 128, 256, 128, 2, 4, 0.125),
    (2, 100, 332, 64, 2, 4, 0.125),                              # unpadded lengths
    (1, 70, 140, 128, 1, 2, float(np.float32(1.0 / 3.0))),
    (96, 1024, 192, 64, 2, 4, 0.125),                            # many heads and row blocks: several launch tiles
    (96, 1000, 132, 64, 1, 2, float(np.float32(1.0 / 3.0))),     # the same on unpadded lengths
])
def test_general_mask_in_the_one_kernel_call(BH, Lq, Lk, d, N, M, scale):
    """dfss_attention_mask: quarter-integer terms and -inf entries (whole runs of four and whole 64-key blocks of a
    query hidden); with integer Q, K every biased score is exact on both sides, so the selection must agree with the
    oracle's, ties included."""
    Q, K, Qn, Kn = _int_qk(BH, Lq, Lk, d, seed=8500 + Lq + Lk)
    g = torch.Generator().manual_seed(8501 + Lq)
    mask = torch.zeros((Lq, Lk), dtype=torch.float32)
    r = torch.rand((Lq, Lk), generator=g)
    mask[r < 1 / 3] = (torch.randint(-8, 9, (Lq, Lk), generator=g).float() / 4)[r < 1 / 3]
    mask[r > 5 / 6] = float("-inf")
    mask[(torch.rand((Lq, Lk // 4), generator=g) < 0.1).repeat_interleave(4, dim=1)] = float("-inf")
    mask[Lq // 2:, :64] = float("-inf")            # the first block hidden from half of the queries
    mask[: Lq // 3, 64:128] = float("-inf")        # the second from a third
    mask[:, 130] = 0.0                             # every query sees a key
    s = Shape(1, BH, Lq, Lk, d, N, M)
    Qd, Kd, md = Q.to(DEV), K.to(DEV), mask.to(DEV)
    W = _weights_through_identity_v(lambda V: dfss.dfss_attention_mask(Qd, Kd, V, md, s, scale), BH, Lq, Lk, d,
                                    torch.bfloat16)
    ties = _compare(W, Qn, Kn, N, M, scale, mask=mask.numpy())
    assert ties > 100
    # the baseline: nothing is dropped
    W = _weights_through_identity_v(lambda V: dfss.dense_attention_fused_mask(Qd, Kd, V, md, s, scale), BH, Lq, Lk, d,
                                    torch.bfloat16)
    for h in range(BH):
        S = oracle.add_mask(oracle.scores(Qn[h], Kn[h], scale), mask.numpy()).astype(np.float64)
        P = np.exp(S - S.max(-1, keepdims=True))
        P /= P.sum(-1, keepdims=True)
        assert (np.abs(W[h] - P) <= REL * P + ABS).all()


@pytest.mark.parametrize("B,H,Lq,Lk,d,N,M,scale,lengths", [
    (3, 2, 128, 384, 64, 2, 4, 0.125, (384, 203, 1)),                       # 128-query workgroups; one key only
    (2, 2, 192, 256, 64, 1, 2, float(np.float32(1.0 / 3.0)), (64, 130)),    # 64-query workgroups; an end on a block edge
    (2, 1, 128, 256, 128, 2, 4, 0.125, (255, 66)),
])
def test_padded_batch_given_by_its_lengths(B, H, Lq, Lk, d, N, M, scale, lengths):
    """dfss_attention_varlen: the padding keys must carry weight exactly 0 and the selection among the real keys (runs
    of four that the end of a sequence cuts included) must be the oracle's with the equivalent -inf bias."""
    BH = B * H
    Q, K, Qn, Kn = _int_qk(BH, Lq, Lk, d, seed=8600 + Lk + d)
    s = Shape(B, H, Lq, Lk, d, N, M)
    lens = torch.tensor(lengths, dtype=torch.int32)
    bias = synth.key_padding_bias(lens, Lk)
    Qd, Kd, ld = Q.to(DEV), K.to(DEV), lens.to(DEV)
    W = _weights_through_identity_v(lambda V: dfss.dfss_attention_varlen(Qd, Kd, V, ld, s, scale), BH, Lq, Lk, d,
                                    torch.bfloat16)
    _compare(W, Qn, Kn, N, M, scale, key_bias=bias.numpy(), H=H)
    for b in range(B):
        assert (W[b * H:(b + 1) * H, :, lengths[b]:] == 0).all()


def test_ragged_call_on_a_grid_that_fills_the_chip():
    """dfss_attention_ragged on many heads runs the 32-queries-per-wave kernel: weight by weight, with a last
    query tile of 8 rows and a last key block of 4 keys."""
    BH, Lq, Lk, d, N, M = 64, 904, 260, 64, 2, 4
    Q, K, Qn, Kn = _int_qk(BH, Lq, Lk, d, seed=8700)
    s = Shape(1, BH, Lq, Lk, d, N, M)
    Qd, Kd = Q.to(DEV), K.to(DEV)
    W = _weights_through_identity_v(lambda V: dfss.dfss_attention_ragged(Qd, Kd, V, None, s, 0.125), BH, Lq, Lk, d,
                                    torch.bfloat16)
    ties = _compare(W[::8], Qn[::8], Kn[::8], N, M, 0.125)
    assert ties > 100


@pytest.mark.parametrize("BH,Lq,Lk,d,N,M,scale", [
    (200, 192, 256, 64, 2, 4, 0.125),
    (200, 192, 128, 128, 1, 2, 0.0625),
])
def test_default_call_with_half_a_workgroup_left_over_on_a_large_grid(BH, Lq, Lk, d, N, M, scale):
    """Lq an odd multiple of 64 on more than 384 workgroups: dfss_attention runs 128-query workgroups whose last
    one per head is half empty.  Weight by weight against the oracle, every eighth head."""
    Q, K, Qn, Kn = _int_qk(BH, Lq, Lk, d, seed=8800 + d)
    s = Shape(1, BH, Lq, Lk, d, N, M)
    Qd, Kd = Q.to(DEV), K.to(DEV)
    W = _weights_through_identity_v(lambda V: dfss.dfss_attention(Qd, Kd, V, s, scale), BH, Lq, Lk, d, torch.bfloat16)
    ties = _compare(W[::8], Qn[::8], Kn[::8], N, M, scale)
    assert ties > 100


@pytest.mark.parametrize("path,BH,Lq,Lk,d,N,M,scale", [
    ("attention", 288, 128, 128, 64, 2, 4, 0.125),     # two blocks: every mark but the first is missed
    ("attention", 136, 256, 384, 64, 1, 2, 0.125),     # six blocks
    ("attention", 160, 128, 1152, 64, 2, 4, 0.125),    # keys of a block split over two waves, 18 blocks
    ("attention", 264, 128, 256, 128, 2, 4, 0.0625),
    ("causal", 136, 256, 256, 128, 2, 4, 0.0625),      # (all at once: the causal form does not)
    ("causal", 136, 256, 256, 128, 1, 2, 0.0625),
    ("causal", 130, 512, 1024, 128, 2, 4, 0.0625),     # more than two rounds, workgroups of ten to sixteen blocks
    ("causal", 97, 256, 384, 64, 1, 2, 0.125),         # (1:2, the first grid that the 32-query kernel takes)
    ("causal", 96, 256, 384, 64, 1, 2, 0.125),         # (the last that it does not)
    ("lengths", 272, 128, 256, 64, 2, 4, 0.125),       # one block to four
])
def test_workgroups_that_keep_level_on_their_compute_unit(path, BH, Lq, Lk, d, N, M, scale):
    """More workgroups than compute units: the kernels give up wave priority at marks along the keys.  Weight by weight against the
    oracle, every sixteenth head."""
    Q, K, Qn, Kn = _int_qk(BH, Lq, Lk, d, seed=8900 + Lk + d)
    s = Shape(BH, 1, Lq, Lk, d, N, M)
    Qd, Kd = Q.to(DEV), K.to(DEV)
    lens = torch.arange(BH, dtype=torch.int32) * 37 % Lk + 1
    call, mask, bias = {
        "attention": (lambda V: dfss.dfss_attention(Qd, Kd, V, s, scale), None, None),
        "causal": (lambda V: dfss.dfss_attention_causal(Qd, Kd, V, None, s, scale),
                   np.triu(np.full((Lq, Lk), -np.inf, np.float32), 1 + Lk - Lq), None),
        "lengths": (lambda V: dfss.dfss_attention_varlen(Qd, Kd, V, lens.to(DEV), s, scale), None,
                    synth.key_padding_bias(lens, Lk).numpy()[::16]),
    }[path]
    W = _weights_through_identity_v(call, BH, Lq, Lk, d, torch.bfloat16)
    _compare(W[::16], Qn[::16], Kn[::16], N, M, scale, key_bias=bias, mask=mask)


@pytest.mark.parametrize("BH,Lq,Lk,d,N,M", [
    (272, 128, 256, 64, 2, 4), (272, 64, 128, 128, 1, 2),
    (272, 100, 132, 64, 1, 2), (272, 60, 100, 128, 2, 4),      # no tile multiples
])
def test_staged_call_on_workgroups_that_keep_level(BH, Lq, Lk, d, N, M):
    """The same in stage 1 and in the product on kept scores, some heads.  The scores are kept as bfloat16 numbers, at most 2^-8 |s|
    off: with |s| below 5 a weight is off by a factor of 1.02 at most, and O, a mean of V with |V| below 5, by less than 2e-2 on
    rows of 50 kept keys and more."""
    Q, K, V = synth.gaussian_qkv(BH, Lq, Lk, d, 1.0 if d == 64 else 0.5, seed=8930 + Lk + d)
    s = Shape(BH, 1, Lq, Lk, d, N, M)
    O = dfss.dfss_attention_staged(Q.to(DEV), K.to(DEV), V.to(DEV), s, 1.0 / math.sqrt(d))
    torch.cuda.synchronize()
    h = slice(None, None, 30)
    ref = oracle.attention(*(synth.to_numpy_f32(t[h]) for t in (Q, K, V)), N, M, 1.0 / math.sqrt(d))
    assert np.max(np.abs(O.float().cpu().numpy()[h] - ref)) <= 2e-2


@pytest.mark.parametrize("BH,Lq,Lk,d,N,M,scale", [
    (34, 128, 512, 64, 2, 4, 0.125),       # up to half a workgroup of 128 queries per compute unit: the 16-query kernel
    (17, 256, 1024, 64, 1, 2, 0.125),      # ... 1:2 at d = 64 up to 1024 keys
    (34, 128, 640, 128, 1, 2, 0.0625),     # ... and from more than 512 keys on two waves per tile of 32 queries
    (34, 128, 640, 64, 2, 4, 1.0 / 3.0),
    (128, 128, 384, 128, 2, 4, 0.0625),    # the last such grid, and the first that is none
    (129, 128, 384, 128, 2, 4, 0.0625),
    (140, 128, 2048, 128, 1, 2, 0.0625),   # d = 128, 2048 keys: two waves per tile up to 192
])
def test_default_call_on_grids_that_leave_compute_units_idle(BH, Lq, Lk, d, N, M, scale):
    """The tilings that dfss_attention takes for few workgroups, weight by weight against the oracle, some heads."""
    Q, K, Qn, Kn = _int_qk(BH, Lq, Lk, d, seed=8950 + Lk + d + N)
    s = Shape(1, BH, Lq, Lk, d, N, M)
    Qd, Kd = Q.to(DEV), K.to(DEV)
    W = _weights_through_identity_v(lambda V: dfss.dfss_attention(Qd, Kd, V, s, float(np.float32(scale))), BH, Lq, Lk, d, torch.bfloat16)
    h = slice(None, None, 24)
    assert _compare(W[h], Qn[h], Kn[h], N, M, float(np.float32(scale))) > 100


@pytest.mark.parametrize("path,BH,Lq,Lk,d,N,M", [
    ("ragged", 128, 100, 500, 64, 2, 4),     # two waves per tile: a partial last block that both tiles of keys reach
    ("ragged", 128, 70, 388, 64, 1, 2),      # ... four real keys in it, none in the second tile
    ("ragged", 128, 66, 484, 128, 1, 2),
    ("ragged", 130, 100, 1500, 128, 2, 4),   # ... more than 128 workgroups of 128 queries
    ("lengths", 5, 128, 384, 64, 2, 4),      # ... sequences that end in every block, some in its first tile
    ("lengths", 7, 192, 512, 128, 1, 2),     # ... an odd multiple of 64 queries
    ("lengths", 96, 192, 384, 64, 2, 4),     # ... on more workgroups than compute units, which keep level
    ("lengths", 135, 128, 1024, 64, 1, 2),
    ("lengths", 90, 192, 640, 128, 2, 4),
    ("lengths", 90, 192, 384, 128, 2, 4),    # (at d = 128 not on short rows: two-wave workgroups)
    ("ragged", 130, 100, 1100, 64, 2, 4),
])
def test_two_waves_per_tile_on_unpadded_and_padded_lengths(path, BH, Lq, Lk, d, N, M):
    """The keys of a block shared by two waves where the last block is partial, weight by weight against the oracle."""
    Q, K, Qn, Kn = _int_qk(BH, Lq, Lk, d, seed=9050 + Lk + d)
    s = Shape(BH, 1, Lq, Lk, d, N, M)
    Qd, Kd = Q.to(DEV), K.to(DEV)
    lens = torch.arange(BH, dtype=torch.int32) * 67 % Lk + 1
    h = slice(None, None, 1 if BH <= 40 else 40 if path == "ragged" else 8)
    if path == "ragged":
        W = _weights_through_identity_v(lambda V: dfss.dfss_attention_ragged(Qd, Kd, V, None, s, 0.125), BH, Lq, Lk, d, torch.bfloat16)
        assert _compare(W[h], Qn[h], Kn[h], N, M, 0.125) > 100
    else:
        W = _weights_through_identity_v(lambda V: dfss.dfss_attention_varlen(Qd, Kd, V, lens.to(DEV), s, 0.125), BH, Lq, Lk, d,
                                        torch.bfloat16)
        _compare(W[h], Qn[h], Kn[h], N, M, 0.125, key_bias=synth.key_padding_bias(lens, Lk).numpy()[h])


def test_float_one_kernel_path():
    """The 4-byte mode's one-kernel path (split products; integer inputs are exact in its bfloat16 pieces)."""
    BH, Lq, Lk, d = 2, 128, 256, 64
    Q, K, Qn, Kn = _int_qk(BH, Lq, Lk, d, seed=8400, tdtype=torch.float32)
    s = Shape(1, BH, Lq, Lk, d, 1, 2, DFSS_F32_BF16X3)
    Qd, Kd = Q.to(DEV), K.to(DEV)
    W = _weights_through_identity_v(lambda V: dfss.dfss_attention(Qd, Kd, V, s, 0.125), BH, Lq, Lk, d, torch.float32)
    # weights are split into two bfloat16 pieces (2^-17) and the output is fp32: far tighter than the 2-byte mode
    ties = _compare(W, Qn, Kn, 1, 2, 0.125, rel=2.0 ** -14)
    assert ties > 100
