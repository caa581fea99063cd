"""GPU: bf16 models that keep their cache row by row (the single-plane format, head_dim 64) take prompts and interrupts through the
matrix cores with their fp32 activations as three bf16 planes.  Each case is compared with the same stream taken token by token
(option chunk = 1, the single-row kernels): pass lengths around row tiles of 32, workgroups of four of them and whole passes of
512, one to eight query heads per kv head, the smallest sizes (one block of 128 columns), several key splits."""
import numpy as np
import pytest
import torch

import asynclm_inputs as ai
import plane_model as pm
from asynclm_inputs.configs import ModelConfig
from oracle import asynclm_oracle as orc

pytestmark = pytest.mark.gpu

# Relative to the logits (2-norm).  A stored value may round the other way when sums are added in another order: a few 2^-17 with
# the paired cache, a few 2^-9 with the single plane (the same bounds as for the vector-unit rows).
TOL = {"pair": 5e-5, "bf16": 4e-3}


def _model(d, hq, hkv, dh, ffn, layers=2):
    return ModelConfig(n_layers=layers, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh, ffn=ffn, vocab=520, rms_eps=1e-5,
                       rope_theta=10000.0, dtype="bf16")


CASES = [
    ("bf16", _model(512, 8, 2, 128, 1152), [2, 31, 32, 33, 1, 128]),
    ("bf16", _model(512, 8, 2, 128, 1152), [257, 40]),               # key splits: 257 rows hold one, 40 rows two
    ("bf16", _model(1024, 4, 4, 128, 640), [96, 129, 64, 65]),
    ("bf16", _model(128, 2, 1, 64, 128), [3, 7]),                    # one block of columns in every product
    ("bf16", _model(128, 2, 1, 64, 128), [9, 40]),                   # ... in passes that do take the matrix cores
    ("bf16", _model(640, 8, 1, 128, 2432, layers=1), [200, 8]),      # one layer: the pass is its last row
    ("bf16", _model(384, 4, 2, 64, 256, layers=3), [513, 2]),        # a pass of 512 and a single row
    ("pair", _model(512, 8, 2, 64, 896), [24, 100, 300]),
    ("pair", _model(256, 8, 8, 64, 384), [514, 9]),
]


def _rel(a, b):
    return float(np.linalg.norm(a.astype(np.float64) - b) / np.linalg.norm(b))


@pytest.mark.parametrize("kind,model,blocks", CASES, ids=["%s-d%d-f%d-%d" % (k, m.d_model, m.ffn, b[0]) for k, m, b in CASES])
def test_wide_passes_equal_token_by_token(kind, model, blocks):
    import paper_2412_07017_amd as pkg
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    fmt = pkg.KV_BF16 if kind == "bf16" else pkg.KV_AUTO
    tk = lambda n, sub: [int(t) for t in ai.uniform_tokens(ai.MASTER_SEED, 961, n, model.vocab, sub=sub)]
    cap = sum(blocks) + 32
    lms = [pkg.AsyncLM(model, w, max_positions=cap, max_seqs=2, stream=torch.cuda.Stream(), kv_format=fmt) for _ in range(2)]
    lms[1].set_option("chunk", 1)
    for lm in lms:
        lm.prefill(1, tk(5, 99))                       # another sequence: rows of sequence 0 must not touch it
    for step, n in enumerate(blocks):
        toks = tk(n, step)
        for lm in lms:
            (lm.prefill if step == 0 else lm.inject_interrupt)(0, toks)
        a, b = lms[0].logits(0), lms[1].logits(0)
        assert np.isfinite(a).all()
        assert _rel(a, b) <= TOL[kind], (n, _rel(a, b))
        assert lms[0].seq_len(0) == lms[1].seq_len(0)
        assert lms[0].peek_choice(0) == int(np.argmax(a))
    for lm in lms:                                      # a token and its interrupt in one call, then a step, on both sequences
        assert list(lm.step_batch([0, 1], forced=[7, 9], interrupts=[tk(3, 50), tk(11, 51)])) == [7, 9]
        assert lm.decode_step(0, forced_token=3) == 3
    for seq in (0, 1):
        assert _rel(lms[0].logits(seq), lms[1].logits(seq)) <= TOL[kind]
    for lm in lms:
        lm.close()


# All three planes of every producer (first norm, norm of the residual, attention with and without a merge of key splits, SwiGLU, the last layer's
# K and V) in both kernels of the products: the logits are differences that only the third plane carries, against the oracle in 64 bits
@pytest.mark.parametrize("split", [0, 2])
@pytest.mark.parametrize("rows", [9, 32, 40, 140])
@pytest.mark.parametrize("kind,dh", [("pair", 64), ("bf16", 128), ("bf16", 64)])
def test_products_see_all_bits_of_their_inputs(kind, dh, rows, split):
    import paper_2412_07017_amd as pkg
    model, toks = pm.model(dh), pm.tokens(rows)
    w = pm.weights(dh, rows, torch.device("cuda:0"))
    torch.cuda.synchronize()
    dec = orc.CachedDecoder(orc.Shape.of(model), ai.weights_to_numpy(w), kv_round=kind == "bf16")
    dec.prefill(toks)
    lm = pkg.AsyncLM(model, w, max_positions=256, stream=torch.cuda.Stream(), kv_format=pkg.KV_BF16 if kind == "bf16" else pkg.KV_AUTO)
    lm.set_option("attn_split", split)
    lm.prefill(0, toks)
    errors = pm.errors(lm.logits(0), dec.logits)
    assert max(errors.values()) <= pm.BOUND, errors
    lm.close()
