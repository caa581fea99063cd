"""Decoding steps whose output projection merges the attention's key splits: the 1, 2, 4 and 8 splits that the length of the context gives and every
other number up to eight by option, splits without keys, both head sizes, one head and as many as the early request of the partial results takes
(4096 columns), one head more, against the oracle."""
import numpy as np
import pytest
import torch

import asynclm_inputs as ai
from asynclm_inputs.configs import ModelConfig
from oracle import asynclm_oracle as orc

pytestmark = pytest.mark.gpu

# rows of the projection (d_model) above what the kernel for small products takes; tolerances as in test_gpu_weight_runs
MODELS = [
    ("bf16 64 x 64", ModelConfig(1, 2056, 64, 8, 64, 256, 264, 1e-5, 10000.0, "bf16"), 2e-4),
    ("bf16 one head of 64", ModelConfig(1, 2056, 1, 1, 64, 256, 264, 1e-5, 10000.0, "bf16"), 2e-4),
    ("bf16 65 x 64", ModelConfig(1, 2056, 65, 65, 64, 256, 264, 1e-5, 10000.0, "bf16"), 2e-4),
    ("fp32 32 x 128", ModelConfig(1, 2056, 32, 8, 128, 256, 264, 1e-5, 10000.0, "fp32"), 1e-5),
    ("fp32 3 x 128", ModelConfig(1, 2056, 3, 3, 128, 256, 264, 1e-5, 10000.0, "fp32"), 1e-5),
    ("fp32 18 x 64", ModelConfig(1, 2056, 18, 9, 64, 256, 264, 1e-5, 10000.0, "fp32"), 1e-5),
]


@pytest.mark.parametrize("name,model,rel", MODELS, ids=[m[0] for m in MODELS])
def test_merged_splits(name, model, rel):
    import paper_2412_07017_amd as pkg
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    conv = lambda t: t.detach().to("cpu").to(torch.float32).numpy()
    host = {k: ([conv(t) for t in v] if isinstance(v, list) else conv(v)) for k, v in w.items()}
    toks = [int(t) for t in ai.uniform_tokens(ai.MASTER_SEED, 975, 520, model.vocab)]
    lm = pkg.AsyncLM(model, w, max_positions=520, stream=torch.cuda.Stream())
    dec = orc.CachedDecoder(orc.Shape.of(model), host, dtype=np.float64)
    at = 0
    for n in (1, 63, 65, 128, 260, 300, 517):       # keys in the cache before a step: 1, 2, 4 and 8 splits
        (lm.inject_interrupt if at else lm.prefill)(0, toks[at:n])
        (dec.inject if at else dec.prefill)(toks[at:n])
        lm.decode_step(0, forced_token=toks[n])
        dec.inject(toks[n:n + 1])
        assert np.abs(lm.logits(0) - dec.logits).max() <= rel * np.abs(dec.logits).max(), (name, n)
        at = n + 1
    lm.close()


# Numbers of splits that only the option gives; of five keys some splits have none, and 200 keys do not divide evenly.
@pytest.mark.parametrize("nsplit", [3, 5, 6, 7])
@pytest.mark.parametrize("name,model,rel", [MODELS[i] for i in (0, 2, 3, 5)], ids=[MODELS[i][0] for i in (0, 2, 3, 5)])
def test_merged_splits_by_option(name, model, rel, nsplit):
    import paper_2412_07017_amd as pkg
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    conv = lambda t: t.detach().to("cpu").to(torch.float32).numpy()
    host = {k: ([conv(t) for t in v] if isinstance(v, list) else conv(v)) for k, v in w.items()}
    toks = [int(t) for t in ai.uniform_tokens(ai.MASTER_SEED, 976, 201, model.vocab)]
    lm = pkg.AsyncLM(model, w, max_positions=201, stream=torch.cuda.Stream())
    lm.set_option("attn_split", nsplit)
    dec = orc.CachedDecoder(orc.Shape.of(model), host, dtype=np.float64)
    at = 0
    for n in (1, 4, 199):                           # keys in the cache before a step
        (lm.inject_interrupt if at else lm.prefill)(0, toks[at:n])
        (dec.inject if at else dec.prefill)(toks[at:n])
        lm.decode_step(0, forced_token=toks[n])
        dec.inject(toks[n:n + 1])
        assert np.abs(lm.logits(0) - dec.logits).max() <= rel * np.abs(dec.logits).max(), (name, nsplit, n)
        at = n + 1
    lm.close()
