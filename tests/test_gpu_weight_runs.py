"""The streaming kernels request weights past the end of a wave's share; those requests are dropped by the loads' range check.  Rows that end
inside a tile of columns, waves without rows and with fewer tiles than the ring holds, against the oracle; and matrices that start at any
multiple of their element size give the same bits as aligned ones, because the same kernels run."""
import numpy as np
import pytest
import torch

import asynclm_inputs as ai
from asynclm_inputs.configs import ModelConfig
from oracle import asynclm_oracle as orc

pytestmark = pytest.mark.gpu

# name, model, largest error allowed relative to the largest logit: as in test_gpu_tiny (fp32 sums) and test_gpu_shapes (bf16 pairs in the cache)
MODELS = [
    ("bf16 rows of 257 pieces", ModelConfig(2, 2056, 4, 2, 64, 1000, 520, 1e-5, 10000.0, "bf16"), 2e-4),
    ("bf16 head_dim 128, three tiles a row", ModelConfig(1, 4616, 2, 2, 128, 264, 1030, 1e-5, 10000.0, "bf16"), 2e-4),
    ("fp32 rows of 258 pieces", ModelConfig(2, 1032, 4, 1, 64, 2504, 301, 1e-5, 10000.0, "fp32"), 1e-5),
]


def _stream(model, w, toks):
    import paper_2412_07017_amd as pkg
    lm = pkg.AsyncLM(model, w, max_positions=64, stream=torch.cuda.Stream())
    lm.prefill(0, toks[:1])
    out = [lm.logits(0)]
    for t in toks[1:]:
        lm.decode_step(0, forced_token=int(t))
        out.append(lm.logits(0))
    lm.close()
    return out


@pytest.mark.parametrize("name,model,rel", MODELS, ids=[m[0] for m in MODELS])
def test_rows_that_end_inside_a_tile(name, model, rel):
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    toks = [int(t) for t in ai.uniform_tokens(ai.MASTER_SEED, 971, 6, model.vocab)]
    conv = lambda t: t.detach().to("cpu").to(torch.float32).numpy()
    dec = orc.CachedDecoder(orc.Shape.of(model), {k: ([conv(t) for t in v] if isinstance(v, list) else conv(v)) for k, v in w.items()}, dtype=np.float64)
    got = _stream(model, w, toks)
    dec.prefill(toks[:1])
    for i, g in enumerate(got):
        if i:
            dec.inject(toks[i:i + 1])
        assert np.abs(g - dec.logits).max() <= rel * np.abs(dec.logits).max(), (name, i)


@pytest.mark.parametrize("elems", [1, 2, 4])
@pytest.mark.parametrize("name,model,rel", MODELS[::2], ids=[m[0] for m in MODELS[::2]])
def test_matrices_at_any_multiple_of_their_element_size(name, model, rel, elems):
    w = ai.make_weights(model, device=torch.device("cuda:0"))

    def moved(t):
        flat = torch.empty(t.numel() + elems, dtype=t.dtype, device=t.device)
        flat[elems:] = t.reshape(-1)
        return flat[elems:].view(t.shape)

    shifted = {k: ([moved(t) for t in v] if isinstance(v, (list, tuple)) else moved(v)) if "norm" not in k else v for k, v in w.items()}
    torch.cuda.synchronize()
    assert shifted["wdown"][0].data_ptr() % 16 == elems * w["wdown"][0].element_size() % 16
    toks = [int(t) for t in ai.uniform_tokens(ai.MASTER_SEED, 972, 4, model.vocab)]
    for a, b in zip(_stream(model, w, toks), _stream(model, shifted, toks)):
        assert np.array_equal(a, b)


# rows of a pass: one tile (weight stream), two (k-split), three and four (a wave per row tile); d and ffn leave runs of one block and of unequal length
@pytest.mark.parametrize("dh,kv", [(128, 0), (128, 1)], ids=["paired cache", "single plane"])
def test_products_of_several_rows_at_any_multiple_of_the_element_size(dh, kv):
    import paper_2412_07017_amd as pkg
    model = ModelConfig(2, 640, 4, 2, dh, 1408, 512, 1e-5, 10000.0, "bf16")
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    conv = lambda t: t.detach().to("cpu").to(torch.float32).numpy()
    host = {k: ([conv(t) for t in v] if isinstance(v, list) else conv(v)) for k, v in w.items()}

    def moved(t):
        flat = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        flat[1:] = t.reshape(-1)
        return flat[1:].view(t.shape)

    shifted = {k: ([moved(t) for t in v] if isinstance(v, (list, tuple)) else moved(v)) if "norm" not in k else v for k, v in w.items()}
    torch.cuda.synchronize()
    toks = [int(t) for t in ai.uniform_tokens(ai.MASTER_SEED, 973, 260, model.vocab)]
    cuts = [0, 23, 63, 147, 258, 260]
    got = []
    for ws in (w, shifted):
        lm = pkg.AsyncLM(model, ws, max_positions=300, stream=torch.cuda.Stream(), kv_format=kv)
        out = []
        for a, b in zip(cuts, cuts[1:]):
            (lm.prefill if a == 0 else lm.inject_interrupt)(0, toks[a:b])
            out.append(lm.logits(0))
        lm.close()
        got.append(out)
    dec = orc.CachedDecoder(orc.Shape.of(model), host, dtype=np.float32)
    for i, (a, b) in enumerate(zip(cuts, cuts[1:])):
        assert np.array_equal(got[0][i], got[1][i]), (a, b)
        if kv == 0:                             # (a single plane rounds keys and values, which the oracle here does not)
            (dec.prefill if a == 0 else dec.inject)(toks[a:b])
            assert np.abs(got[0][i] - dec.logits).max() <= 2e-4 * np.abs(dec.logits).max(), (a, b)


@pytest.mark.parametrize("rows", [[2, 31, 32], [33, 40, 48, 63, 64], [65, 96, 97, 127, 128], [129, 9]], ids=str)
@pytest.mark.parametrize("kv", [0, 1], ids=["paired cache", "single plane"])
def test_passes_that_end_inside_a_tile_of_rows(rows, kv):
    """Rows past a pass's last one are not fetched; runs of K of one and of three blocks, fewer than are in flight."""
    import paper_2412_07017_amd as pkg
    model = ModelConfig(2, 256, 2, 1, 128, 384, 128, 1e-5, 10000.0, "bf16")
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    conv = lambda t: t.detach().to("cpu").to(torch.float32).numpy()
    # the single plane rounds keys and values, in the oracle at the same place: a sum that falls on the other side of a rounding boundary moves an
    # element by 2^-8 of itself, hence the wider tolerance
    dec = orc.CachedDecoder(orc.Shape.of(model), {k: ([conv(t) for t in v] if isinstance(v, list) else conv(v)) for k, v in w.items()}, dtype=np.float32, kv_round=kv == 1)
    toks = [int(t) for t in ai.uniform_tokens(ai.MASTER_SEED, 974, sum(rows), model.vocab)]
    lm = pkg.AsyncLM(model, w, max_positions=sum(rows), stream=torch.cuda.Stream(), kv_format=kv)
    at = 0
    for n in rows:
        (lm.prefill if at == 0 else lm.inject_interrupt)(0, toks[at:at + n])
        (dec.prefill if at == 0 else dec.inject)(toks[at:at + n])
        at += n
        assert np.abs(lm.logits(0) - dec.logits).max() <= (2.5e-3 if kv else 2e-4) * np.abs(dec.logits).max(), (n, at)
    lm.close()


@pytest.mark.parametrize("ffn", [2176, 2432, 11008])
@pytest.mark.parametrize("kv", [0, 1], ids=["paired cache", "single plane"])
def test_gate_up_waves_without_rows(ffn, kv):
    """Gate rows that do not fill the last workgroup's waves (3, 3 and 11 rows a wave on 256 compute units): the idle waves request nothing."""
    import paper_2412_07017_amd as pkg
    model = ModelConfig(2, 256, 2, 1, 128, ffn, 128, 1e-5, 10000.0, "bf16")
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    conv = lambda t: t.detach().to("cpu").to(torch.float32).numpy()
    dec = orc.CachedDecoder(orc.Shape.of(model), {k: ([conv(t) for t in v] if isinstance(v, list) else conv(v)) for k, v in w.items()}, dtype=np.float32, kv_round=kv == 1)
    toks = [int(t) for t in ai.uniform_tokens(ai.MASTER_SEED, 976, 56, model.vocab)]
    lm = pkg.AsyncLM(model, w, max_positions=56, stream=torch.cuda.Stream(), kv_format=kv)
    for a, b in ((0, 32), (32, 56)):
        (lm.inject_interrupt if a else lm.prefill)(0, toks[a:b])
        (dec.inject if a else dec.prefill)(toks[a:b])
        assert np.abs(lm.logits(0) - dec.logits).max() <= (2.5e-3 if kv else 2e-4) * np.abs(dec.logits).max(), b    # as for passes that end inside a tile
    lm.close()
