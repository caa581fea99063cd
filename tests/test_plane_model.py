"""The model of plane_model.py does what it says, on the oracle: fp32 everywhere keeps every block, and a product's input rounded to two bf16
planes (planted in the oracle) spoils the block that is made for it."""
import numpy as np
import pytest
import torch

import asynclm_inputs as ai
import plane_model as pm
from oracle import asynclm_oracle as orc


def _two_planes(v):
    r = lambda u: torch.as_tensor(u).to(torch.bfloat16).float().numpy()
    v = np.asarray(v, np.float32)
    hi = r(v)
    return hi + r(v - hi)


@pytest.mark.parametrize("dh,n", [(64, 9), (64, 140), (128, 40), (128, 140)])
def test_blocks_show_a_lost_third_plane(dh, n, monkeypatch):
    w, shape = ai.weights_to_numpy(pm.weights(dh, n, "cpu")), orc.Shape.of(pm.model(dh))

    def run(dtype, diag=()):
        dec = orc.CachedDecoder(shape, w, dtype=dtype, diag_round=diag)
        dec.prefill(pm.tokens(n))
        return dec.logits
    want = run(np.float64)
    assert max(pm.errors(run(np.float32), want).values()) <= 0.02
    monkeypatch.setattr(orc, "round_to_bf16", _two_planes)
    for name, (cols, what) in pm.BLOCKS.items():
        assert np.abs(want[list(cols)]).mean() > 0.3, name
        assert pm.errors(run(np.float64, (what,)), want)[name] >= 2 * pm.BOUND, name
