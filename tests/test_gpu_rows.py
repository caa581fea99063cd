"""GPU: models outside the matrix-core append path take prompts and interrupts several rows per pass through the vector-unit
kernels.  Each case is compared with the same stream taken token by token (option chunk = 1) and, for fp32, with the oracle in
64 bits: a shape for every kernel variant, row counts around a full pass, contexts on both sides of one key split."""
import numpy as np
import pytest
import torch

import asynclm_inputs as ai
from asynclm_inputs.configs import ModelConfig
from oracle import asynclm_oracle as orc

pytestmark = pytest.mark.gpu

FP32, PAIR, BF16 = "fp32", "pair", "bf16"

# Differences of two correct orders of summation, relative to the logits (2-norm).  fp32: two layers of sums of up to 4104 terms,
# random signs: sqrt(4104) * 2^-24 = 4e-6 per product.  pair: values are stored with 2^-17, and a stored value may round the
# other way: a few 2^-17.  bf16: the same with 2^-9.
TOL = {FP32: 1e-5, PAIR: 5e-5, BF16: 4e-3}


def _model(d, hq, hkv, dh, ffn, dtype):
    return ModelConfig(n_layers=2, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=dh, ffn=ffn, vocab=520, rms_eps=1e-5,
                       rope_theta=10000.0, dtype=dtype)


# Every variant of the two kernels is taken by some product of these models (tests/test_host_rules.py checks it): k_rows_small
# (at most 1024 row pairs and 256 loads of 16 bytes per row), else k_rows_gemv with one row pair per wave at a time (up to 2048
# pairs) or two, the vectors in LDS as a whole (up to 4096 columns) or in segments.  On 256 compute units:
CASES = [
    (FP32, _model(256, 4, 4, 64, 688, "fp32")),        # all products small
    (FP32, _model(136, 4, 2, 128, 4104, "fp32")),      # QKV, O small; gate/up two pairs, odd counts; down one pair, segments
    (FP32, _model(2056, 2, 1, 64, 4104, "fp32")),      # QKV, O one pair; gate/up two pairs; down one pair, segments
    (FP32, _model(264, 32, 32, 64, 1032, "fp32")),     # QKV two pairs; O, gate/up, down one pair or small
    (FP32, _model(4104, 4, 4, 64, 264, "fp32")),       # QKV, gate/up one pair, segments; O, down two pairs
    (FP32, _model(4104, 32, 8, 128, 4104, "fp32")),    # QKV, gate/up (two rounds per wave), down two pairs, segments; O two pairs
    (PAIR, _model(520, 8, 2, 64, 1032, "bf16")),       # paired cache, head_dim 64: gate/up one pair, the others small
    (PAIR, _model(264, 32, 32, 64, 264, "bf16")),      # QKV two pairs; O small with four loads per row
    (PAIR, _model(4104, 4, 4, 64, 264, "bf16")),       # QKV, gate/up one pair, segments; O, down two pairs
    (BF16, _model(264, 8, 1, 128, 8200, "bf16")),      # single-plane cache, eight heads per kv head; down one pair, three segments
    (BF16, _model(2056, 2, 1, 64, 2056, "bf16")),      # QKV, O, down one pair; gate/up two pairs
    (BF16, _model(4104, 32, 8, 128, 4104, "bf16")),    # QKV, gate/up (two rounds per wave), down two pairs, segments; O two pairs
]


def _rel(a, b):
    return float(np.linalg.norm(a.astype(np.float64) - b) / np.linalg.norm(b))


@pytest.mark.parametrize("kind,model", CASES, ids=["%s-d%d-h%d-f%d" % (k, m.d_model, m.n_q_heads, m.ffn) for k, m in CASES])
def test_rows_of_a_pass_equal_token_by_token(kind, model):
    import paper_2412_07017_amd as pkg
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    fmt = pkg.KV_BF16 if kind == BF16 else pkg.KV_AUTO
    tk = lambda n, sub: [int(t) for t in ai.uniform_tokens(ai.MASTER_SEED, 931, n, model.vocab, sub=sub)]
    lms = [pkg.AsyncLM(model, w, max_positions=640, max_seqs=2, stream=torch.cuda.Stream(), kv_format=fmt) for _ in range(2)]
    lms[1].set_option("chunk", 1)
    dec = orc.CachedDecoder(orc.Shape.of(model), ai.weights_to_numpy(w), dtype=np.float64) if kind == FP32 else None
    for lm in lms:
        lm.prefill(1, tk(5, 99))                       # another sequence: rows of sequence 0 must not touch it
    for step, n in enumerate([2, 3, 8, 9, 231, 17, 25, 1, 7]):       # 253 tokens, then past one key split of 256
        toks = tk(n, step)
        for lm in lms:
            (lm.prefill if step == 0 else lm.inject_interrupt)(0, toks)
        a, b = lms[0].logits(0), lms[1].logits(0)
        assert np.isfinite(a).all()
        assert _rel(a, b) <= TOL[kind], (n, _rel(a, b))
        if dec is not None:
            (dec.prefill if step == 0 else dec.inject)(toks)
            assert _rel(a, dec.logits) <= TOL[kind], (n, _rel(a, dec.logits))
        assert lms[0].seq_len(0) == lms[1].seq_len(0)
    for lm in lms:
        lm.inject_interrupt(1, tk(11, 100))
    assert _rel(lms[0].logits(1), lms[1].logits(1)) <= TOL[kind]
    assert lms[0].decode_step(0, forced_token=3) == lms[1].decode_step(0, forced_token=3) == 3
    assert _rel(lms[0].logits(0), lms[1].logits(0)) <= TOL[kind]
    for lm in lms:
        lm.close()


# Models whose products are all small: passes of up to 128 rows, eight per workgroup; around that, around multiples of eight, and with
# key splits that 128 rows can hold no more than four of
@pytest.mark.parametrize("kind,model", [(FP32, _model(256, 4, 4, 64, 688, "fp32")), (PAIR, _model(264, 8, 2, 64, 1000, "bf16")), (BF16, _model(136, 4, 1, 128, 264, "bf16"))])
def test_long_passes_of_small_models(kind, model):
    import paper_2412_07017_amd as pkg
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    tk = lambda n, sub: [int(t) for t in ai.uniform_tokens(ai.MASTER_SEED, 932, n, model.vocab, sub=sub)]
    lms = [pkg.AsyncLM(model, w, max_positions=2000, stream=torch.cuda.Stream(), kv_format=pkg.KV_BF16 if kind == BF16 else pkg.KV_AUTO) for _ in range(2)]
    lms[1].set_option("chunk", 8)
    for step, n in enumerate([64, 127, 128, 129, 9, 1200, 121]):
        for lm in lms:
            (lm.prefill if step == 0 else lm.inject_interrupt)(0, tk(n, step))
        a, b = lms[0].logits(0), lms[1].logits(0)
        assert np.isfinite(a).all() and _rel(a, b) <= TOL[kind], (n, _rel(a, b))
    for lm in lms:
        lm.close()
