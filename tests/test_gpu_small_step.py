"""GPU: decoding steps of models whose products are all small take three launches per layer with partial vectors between them.  Each
case is compared with the same stream through the kernels of the other models (option attn_split) and, for fp32, with the oracle in
64 bits: one to four query heads per kv head, rows that fill a wave's load and rows that do not, features that do not fill the last
workgroup, both caches of bf16, one layer, contexts up to and past the longest that these steps take."""
import numpy as np
import pytest
import torch

import asynclm_inputs as ai
from asynclm_inputs.configs import ModelConfig
from oracle import asynclm_oracle as orc

pytestmark = pytest.mark.gpu

# relative to the logits (2-norm), as for the rows of a pass: sums of fp32 in another order, stored values that round the other way
TOL = {"fp32": 1e-5, "pair": 5e-5, "bf16": 4e-3}


def _model(d, hq, hkv, dh, ffn, dtype, layers=2, vocab=520):
    return ModelConfig(n_layers=layers, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh, ffn=ffn, vocab=vocab, rms_eps=1e-5,
                       rope_theta=10000.0, dtype=dtype)


CASES = [
    ("fp32", _model(256, 4, 4, 64, 688, "fp32", vocab=1024)),       # the tiny preset's shape
    ("fp32", _model(264, 4, 2, 64, 712, "fp32", layers=3)),         # two loads per row, part empty; last workgroup half empty
    ("fp32", _model(512, 8, 8, 64, 1024, "fp32")),
    ("fp32", _model(136, 2, 1, 128, 8, "fp32", layers=1)),          # one workgroup for the features, one kv head
    ("fp32", _model(128, 12, 3, 64, 264, "fp32", vocab=17)),        # an odd number of kv heads, of columns of the head
    ("pair", _model(520, 8, 2, 64, 1000, "bf16")),
    ("pair", _model(1000, 6, 6, 64, 104, "bf16")),
    ("bf16", _model(256, 8, 2, 128, 512, "bf16")),
    ("bf16", _model(264, 8, 1, 64, 688, "bf16")),                   # eight query heads per kv head
    # Not all of the models above take the short step (at most 128 KB of the O projection per kv head).  These do, at the shorter contexts
    # at least: every variant of its kernels (heads per kv head, head_dim, cache), and two loads per row
    ("fp32", _model(264, 4, 4, 64, 712, "fp32", layers=3)),
    ("fp32", _model(128, 4, 2, 64, 264, "fp32")),
    ("fp32", _model(136, 2, 2, 128, 8, "fp32", layers=1)),
    ("fp32", _model(128, 4, 2, 128, 136, "fp32", layers=3)),
    ("pair", _model(256, 6, 6, 64, 104, "bf16")),
    ("pair", _model(264, 4, 2, 64, 200, "bf16")),
    ("pair", _model(128, 8, 2, 64, 344, "bf16")),
    ("pair", _model(120, 8, 1, 64, 264, "bf16", layers=1)),
    ("pair", _model(136, 3, 3, 128, 264, "bf16", layers=3)),
    ("pair", _model(136, 4, 2, 128, 264, "bf16")),
    ("pair", _model(120, 8, 2, 128, 264, "bf16")),
    ("bf16", _model(512, 4, 4, 64, 1000, "bf16")),
    ("bf16", _model(256, 8, 4, 64, 264, "bf16", layers=3)),
    ("bf16", _model(128, 8, 2, 64, 264, "bf16", vocab=33)),
    ("bf16", _model(128, 16, 2, 64, 264, "bf16")),
    ("bf16", _model(256, 2, 2, 128, 512, "bf16")),
    ("bf16", _model(128, 4, 2, 128, 264, "bf16")),
    ("bf16", _model(128, 8, 2, 128, 264, "bf16")),
]


def _rel(a, b):
    return float(np.linalg.norm(a.astype(np.float64) - b) / np.linalg.norm(b))


@pytest.mark.parametrize("kind,model", CASES, ids=["%s-d%d-h%d-f%d" % (k, m.d_model, m.n_q_heads, m.ffn) for k, m in CASES])
def test_small_steps_equal_the_other_kernels(kind, model):
    import paper_2412_07017_amd as pkg
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    fmt = pkg.KV_BF16 if kind == "bf16" else pkg.KV_AUTO
    toks = [int(t) for t in ai.uniform_tokens(ai.MASTER_SEED, 971, 600, model.vocab)]
    lms = [pkg.AsyncLM(model, w, max_positions=600, max_seqs=2, stream=torch.cuda.Stream(), kv_format=fmt) for _ in range(2)]
    lms[1].set_option("attn_split", 2)
    dec = orc.CachedDecoder(orc.Shape.of(model), ai.weights_to_numpy(w), dtype=np.float64) if kind == "fp32" else None
    for lm in lms:
        lm.prefill(1, toks[:7])
    at = 0
    for block in (1, 62, 65, 128, 119):                     # steps over 2, 66, 133, 263 and 384 keys, and the one after each
        for lm in lms:
            (lm.inject_interrupt if at else lm.prefill)(0, toks[at:at + block])
        if dec is not None:
            (dec.inject if at else dec.prefill)(toks[at:at + block])
        at += block
        for _ in range(2):
            assert all(lm.decode_step(0, forced_token=toks[at]) == toks[at] for lm in lms)
            a, b = lms[0].logits(0), lms[1].logits(0)
            assert np.isfinite(a).all() and _rel(a, b) <= TOL[kind], (at, _rel(a, b))
            assert lms[0].peek_choice(0) == int(np.argmax(a))
            if dec is not None:
                dec.decode_step(forced=toks[at])
                assert _rel(a, dec.logits) <= TOL[kind], (at, _rel(a, dec.logits))
            at += 1
    want = int(np.argmax(lms[0].logits(0)))                 # the greedy choice of a step, and the one after under a list
    assert lms[0].decode_step(0) == want
    order = np.argsort(lms[0].logits(0))
    lms[0].set_banned_tokens(0, [int(order[-1])])
    assert lms[0].decode_step(0) == int(order[-2])
    banned, logits = int(order[-1]), lms[0].logits(0).copy()
    logits[banned] = -np.inf
    assert lms[0].peek_choice(0) == int(np.argmax(logits))
    for lm in lms:                                          # the other sequence is untouched; graphs and plain launches agree
        lm.decode_step(1, forced_token=3)
    assert _rel(lms[0].logits(1), lms[1].logits(1)) <= TOL[kind]
    lms[0].set_option("graph", 0)
    for lm in lms:
        lm.decode_step(1, forced_token=5)
    assert _rel(lms[0].logits(1), lms[1].logits(1)) <= TOL[kind] and lms[0].seq_len(1) == lms[1].seq_len(1) == 9
    for lm in lms:
        lm.close()


# A step that the caller captures on its stream (plain launches, no token asked for): every replay appends one more token, because
# position and length are read from the device; small steps and, with forced key splits, those of the other kernels
@pytest.mark.parametrize("split", [0, 2])
@pytest.mark.parametrize("layers", [1, 2, 5])
def test_a_step_captured_by_the_caller_goes_on_with_every_replay(layers, split):
    import paper_2412_07017_amd as pkg
    model = _model(256, 4, 2, 64, 264, "fp32", layers=layers)
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    lms = [pkg.AsyncLM(model, w, max_positions=64, stream=s) for s in streams]
    lms[0].set_option("graph", 0)
    for lm in lms:
        lm.set_option("attn_split", split)
        lm.prefill(0, [1, 2, 3])
        lm.decode_step(0, forced_token=9)
        lm.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=streams[0], capture_error_mode="relaxed"):
        lms[0].decode_step(0, want_token=False)
    for _ in range(4):
        with torch.cuda.stream(streams[0]):
            graph.replay()
        torch.cuda.synchronize()
        lms[1].decode_step(0)
        assert np.array_equal(lms[0].logits(0), lms[1].logits(0))
    for lm in lms:                                          # and the context is as good as new
        lm.reset(0)
        lm.prefill(0, [4, 5])
        assert lm.decode_step(0, forced_token=6) == 6 and lm.seq_len(0) == 3
    assert np.array_equal(lms[0].logits(0), lms[1].logits(0))
    for lm in lms:
        lm.close()


# Models of four layers and more replay the short step as a graph behind its first kernel: the same bits as launch by launch, the oracle's
# logits, two sequences in turn, one of them over the end of the short step at `last` keys (an even and an odd number of layers: the
# residual stream alternates between two vectors)
GRAPHS = [("fp32", _model(256, 4, 2, 64, 264, "fp32", layers=4), 128), ("fp32", _model(256, 4, 4, 64, 264, "fp32", layers=5), 256),
          ("bf16", _model(256, 4, 2, 64, 264, "bf16", layers=5), 256), ("pair", _model(256, 4, 4, 64, 264, "bf16", layers=4), 256)]


@pytest.mark.parametrize("kind,model,last", GRAPHS, ids=["%s-%d" % (k, m.n_layers) for k, m, _ in GRAPHS])
def test_short_steps_as_a_graph(kind, model, last):
    import paper_2412_07017_amd as pkg
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    toks = [int(t) for t in ai.uniform_tokens(ai.MASTER_SEED, 973, 420, model.vocab)]
    lms = [pkg.AsyncLM(model, w, max_positions=420, max_seqs=2, stream=torch.cuda.Stream(), kv_format=pkg.KV_BF16 if kind == "bf16" else pkg.KV_AUTO) for _ in range(2)]
    lms[1].set_option("graph", 0)
    starts = [(0, 20), (1, last - 8)]
    for lm in lms:
        for seq, n in starts:
            lm.prefill(seq, toks[:n])
    for step in range(20):
        for seq, n in starts:
            for lm in lms:
                assert lm.decode_step(seq, forced_token=toks[n + step]) == toks[n + step]
            a = lms[0].logits(seq)
            assert np.isfinite(a).all() and np.array_equal(a, lms[1].logits(seq)), (seq, step)
    if kind == "fp32":
        for seq, n in starts:
            dec = orc.CachedDecoder(orc.Shape.of(model), ai.weights_to_numpy(w), dtype=np.float64)
            dec.prefill(toks[:n + 20])
            assert _rel(lms[0].logits(seq), dec.logits) <= TOL[kind]
    for lm in lms:
        lm.close()
