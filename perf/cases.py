"""The work that a user of this library has it do, as cases to be timed.

A case names one public path (one call, or the calls of one training step), its sizes and its options.  ``listed``
holds one case for each kind of use, ``draw`` gives further ones from the same ranges.  Shapes are those of the
library's own workloads (``paper_2203_00091_amd.synth``) where it has one for the kind of use.

Paths
  attention   dfss_attention: the encoder's forward pass on tile-sized lengths
  ragged      dfss_attention_ragged without a mask: sequences taken as they are, any length; also one query per
              sequence against its cached keys
  padded      dfss_attention_bias with a padding mask of key biases (0 / -inf)
  lengths     dfss_attention_varlen: the same batch given by its lengths
  causal      dfss_attention_causal without a key bias
  training    the three stage calls, then dfss_attention_backward on what they leave: O, dQ, dK, dV
  float       dfss_attention with float32 arrays and products from bfloat16 pieces (DFSS_F32_BF16X3, 1:2)
"""
from __future__ import annotations

import math

import torch

import paper_2203_00091_amd as dfss
from paper_2203_00091_amd import Shape, synth


def _case(name, path, B, H, Lq, Lk, d, N, M, sigma=1.0):
    return {"name": name, "path": path, "B": B, "H": H, "Lq": Lq, "Lk": Lk, "d": d, "N": N, "M": M, "sigma": sigma}


def listed():
    return [
        # the smallest call: one head of a short sequence; launch and host time
        _case("one_head_L256", "attention", 1, 1, 256, 256, 64, 2, 4),
        # question answering with a BERT-base encoder, inference
        _case("bert_base_L384", "attention", 8, 12, 384, 384, 64, 2, 4),
        # the long-sequence encoder that the forward pass is quoted on
        _case("long_L4096", "attention", 2, 12, 4096, 4096, 64, 2, 4),
        # a model with large heads
        _case("large_head_L2048", "attention", 4, 16, 2048, 2048, 128, 2, 4, sigma=0.5),
        # document retrieval: sequences of 4000 tokens, taken without padding
        _case("retrieval_L4000", "ragged", 2, 12, 4000, 4000, 64, 2, 4),
        # generation: one new query per sequence against 4096 cached keys
        _case("one_query_L4096", "ragged", 8, 12, 1, 4096, 64, 2, 4),
        # a padded batch, its mask given as key biases; 1:2
        _case("padded_L512", "padded", 16, 12, 512, 512, 64, 1, 2),
        # a decoder with large heads reading its prompt
        _case("causal_L2048", "causal", 4, 16, 2048, 2048, 128, 2, 4, sigma=0.5),
        # finetuning steps: masked language modelling (1:2), a long sequence, a model with large heads
        _case("training_L512", "training", 16, 12, 512, 512, 64, 1, 2),
        _case("training_L4096", "training", 2, 12, 4096, 4096, 64, 2, 4),
        _case("training_large_head_L2048", "training", 4, 16, 2048, 2048, 128, 2, 4, sigma=0.5),
        # the 4-byte mode on the masked language modelling shape
        _case("float_L512", "float", 16, 12, 512, 512, 64, 1, 2),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: a path, a head size, lengths over the path's whole range, and as many heads as keep it between
    one head and the largest listed case of the path."""
    path = rng.choice(["attention", "attention", "ragged", "ragged", "padded", "lengths", "causal", "training",
                       "training", "float"])
    d = rng.choice([64, 64, 128])
    N, M = (1, 2) if path == "float" else rng.choice([(2, 4), (2, 4), (1, 2)])
    if path == "ragged":
        Lk = 4 * _log_uniform(rng, 256 // 4, 4096 // 4)
        Lq = rng.choice([1, rng.randint(2, 64), Lk, _log_uniform(rng, 64, 4096)])
    elif path == "training" and rng.random() < 0.4:      # lengths that are no multiples of the tiles
        Lk = 4 * _log_uniform(rng, 132 // 4, 4096 // 4)
        Lq = Lk
    else:
        Lk = 128 * _log_uniform(rng, 1, 32)
        Lq = Lk if path == "causal" or rng.random() < 0.7 else 64 * _log_uniform(rng, 1, Lk // 64)
    # heads: scores of the case between those of one head and the most that a listed case of the path computes
    most = {"padded": 16 * 12 * 512 * 512, "lengths": 16 * 12 * 512 * 512, "float": 16 * 12 * 512 * 512}
    scores = most.get(path, 2 * 12 * 4096 * 4096) * 64 // d
    BH = max(1, min(scores // (Lq * Lk), 1024, (1 << 25) // (Lk * d)))
    H = rng.choice([1, 4, 12, 16])
    B = max(1, _log_uniform(rng, 1, max(1, BH // H)))
    H = min(H, BH)
    return {"path": path, "B": B, "H": H, "Lq": Lq, "Lk": Lk, "d": d, "N": N, "M": M,
            "sigma": 1.0 if d == 64 else 0.5}


def _lengths(case, seed):
    """Real keys of every batch element of a padded batch: unaligned, between half of and all the padded length."""
    return synth.padding_lengths(case["B"], case["Lk"], seed + 7)


def prepare(case, seed):
    c = dict(case)
    f32 = c["path"] == "float"
    s = Shape(c["B"], c["H"], c["Lq"], c["Lk"], c["d"], c["N"], c["M"], dfss.DFSS_F32_BF16X3 if f32 else dfss.DFSS_BF16)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(L):
        return (torch.randn((s.BH, L, s.d), generator=g, device="cuda") * c["sigma"]).to(s.torch_dtype)

    state = {"path": c["path"], "s": s, "scale": 1.0 / math.sqrt(s.d),
             "Q": normal(s.Lq), "K": normal(s.Lk), "V": normal(s.Lk)}
    if c["path"] == "padded":
        state["bias"] = synth.key_padding_bias(_lengths(c, seed), s.Lk).cuda()
    elif c["path"] == "lengths":
        state["key_len"] = _lengths(c, seed).to(torch.int32).cuda()
    elif c["path"] == "training":
        state["dO"] = normal(s.Lq)
    return state


def run(state):
    path, s, scale = state["path"], state["s"], state["scale"]
    Q, K, V = state["Q"], state["K"], state["V"]
    if path in ("attention", "float"):
        return dfss.dfss_attention(Q, K, V, s, scale)
    if path == "ragged":
        return dfss.dfss_attention_ragged(Q, K, V, None, s, scale)
    if path == "padded":
        return dfss.dfss_attention_bias(Q, K, V, state["bias"], s, scale)
    if path == "lengths":
        return dfss.dfss_attention_varlen(Q, K, V, state["key_len"], s, scale)
    if path == "causal":
        return dfss.dfss_attention_causal(Q, K, V, None, s, scale)
    P, meta = dfss.dfss_sddmm_prune(Q, K, s, scale)
    dfss.dfss_sparse_softmax(P, s)
    O = dfss.dfss_spmm(P, meta, V, s)
    dQ, dK, dV = dfss.dfss_attention_backward(state["dO"], Q, K, V, O, P, meta, s, scale)
    return O, dQ, dK, dV


def work(case):
    """Bytes: every input read once and every output written once; a training step also hands the kept weights and the
    metadata from call to call (scores written, softmax in place, read by the product and by the backward pass).  Operations: Q K^T in full,
    the product with V over the kept half; in the backward pass dO V^T in full, dV, dQ and dK over the kept half."""
    c = case
    BH, Lq, Lk, d = c["B"] * c["H"], c["Lq"], c["Lk"], c["d"]
    elem = 4 if c["path"] == "float" else 2
    seen = BH * Lq * Lk
    if c["path"] == "causal":       # query i sees keys 0 .. i + Lk - Lq
        seen = BH * (Lq * (Lk - Lq) + Lq * (Lq + 1) // 2)
    elif c["path"] in ("padded", "lengths"):    # lengths are uniform in [Lk / 2, Lk]
        seen = seen * 3 // 4
    size = elem * BH * d * (2 * Lq + 2 * Lk)
    if c["path"] == "padded":
        size += 4 * c["B"] * Lk
    if c["path"] != "training":
        return {"bytes": size, "flops": 3 * seen * d}
    vals, meta = seen, seen // 8
    return {"bytes": elem * BH * d * (4 * Lq + 4 * Lk) + 5 * vals + 3 * meta, "flops": 8 * seen * d}


def tolerance(case):
    """Relative 2-norm errors, about four times what a comparison with the same function in 64 bits shows: 2.2e-3 to
    2.6e-3 for the bfloat16 forward pass (weights and O rounded to bfloat16; a few near-ties decided the other way),
    3e-3 to 4.9e-3 for O and the gradients of a training step (kept scores, weights, dS and the results rounded),
    1.1e-3 at most in the float mode (near-ties; 6e-6 in cases without one)."""
    return {"rel": {"training": 2e-2, "float": 5e-3}.get(case["path"], 1e-2)}
