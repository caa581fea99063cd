"""GPU: passes of more than 128 rows (large matrix-core product, up to 2048 rows per pass) against passes of 32 rows on the
same model.  What is compared is the whole cache image of every row, not only the last row's logits: the second layer's
keys and values depend on every product of the first."""

import numpy as np
import pytest
import torch

import asynclm_inputs as ai
from asynclm_inputs.configs import ModelConfig

pytestmark = pytest.mark.gpu

HEADER = 56                 # bytes of the image's description
# Both sides carry inputs of products as two bf16 (relative error 2^-17 each) and add in fp32; a second-layer key sees five
# products in a row: 5 * 2^-16 = 7.6e-5 of its norm.
TOL = 1e-4


def _planes(lm, model, n, seq=0):
    """Keys [layer, head, position, channel] and values [layer, head, tile, ...] of a sequence, hi + lo."""
    size = lm.kv_bytes(seq)
    buf = torch.empty(size, dtype=torch.uint8, pin_memory=True)
    lm.kv_swap_out(seq, buf.data_ptr(), size)
    L, H, dh = model.n_layers, model.n_kv_heads, model.head_dim
    k, v = H * n * dh, H * ((n + 31) // 32 * 32) * dh
    assert size == HEADER + L * 2 * (k + v) * 2 + model.vocab * 4
    raw = torch.frombuffer(buf.numpy(), dtype=torch.uint8, offset=HEADER, count=L * 2 * (k + v) * 2).view(torch.bfloat16)
    raw = raw.to(torch.float32).view(L, 2 * (k + v))
    keys = (raw[:, :k] + raw[:, k:2 * k]).view(L, H, n, dh)
    vals = (raw[:, 2 * k:2 * k + v] + raw[:, 2 * k + v:]).view(L, H, -1, 32 * dh)
    return keys.numpy(), vals.numpy()


def _worst(a, b):
    d = np.linalg.norm(a.astype(np.float64) - b, axis=-1)
    return float((d / np.linalg.norm(b, axis=-1)).max())


# F / 16 gate-up tiles against 32 per weight-row tile of a workgroup at eight row blocks: 2176 and 2432 take 5 (the last
# tile part empty), 2816 6, 3200 7 (both part empty), 3712 8; 1024 the smallest; rows: edges of row tiles, of
# 256-row blocks and of a pass
@pytest.mark.parametrize("n,ffn,heads,kv", [(129, 1024, 4, 4), (257, 1024, 4, 1), (1024, 1024, 8, 1), (1801, 2176, 4, 2), (2047, 2432, 4, 2),
                                            (2048, 2816, 4, 4), (1999, 3200, 4, 2), (2100, 3712, 4, 2)])
def test_large_passes_equal_passes_of_32_rows(n, ffn, heads, kv):
    import paper_2412_07017_amd as pkg
    model = ModelConfig(n_layers=2, d_model=512, n_q_heads=heads, n_kv_heads=kv, head_dim=128, ffn=ffn, vocab=1024, rms_eps=1e-5,
                        rope_theta=10000.0, dtype="bf16")
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    toks = ai.uniform_tokens(ai.MASTER_SEED, 941, n, model.vocab)
    got = []
    for chunk in (None, 32):
        lm = pkg.AsyncLM(model, w, max_positions=n + 8, stream=torch.cuda.Stream())
        if chunk:
            lm.set_option("chunk", chunk)
        lm.prefill(0, toks)
        got.append((*_planes(lm, model, n), lm.logits(0)))
        lm.close()
    (ka, va, la), (kb, vb, lb) = got
    assert np.isfinite(ka).all() and np.isfinite(va).all() and np.isfinite(la).all()
    assert not np.array_equal(ka[1], kb[1])              # the passes were not the same: sums in another order
    assert _worst(ka, kb) <= TOL, _worst(ka, kb)
    tail = n % 32                                        # a last tile of values that is part empty: compare as a whole
    assert _worst(va, vb) <= TOL, (_worst(va, vb), tail)
    assert np.linalg.norm(la - lb) / np.linalg.norm(lb) <= TOL


def test_pass_size_option_still_bounds_a_pass():
    import paper_2412_07017_amd as pkg
    model = ModelConfig(n_layers=2, d_model=256, n_q_heads=2, n_kv_heads=1, head_dim=128, ffn=256, vocab=512, rms_eps=1e-5,
                        rope_theta=10000.0, dtype="bf16")
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    toks = ai.uniform_tokens(ai.MASTER_SEED, 942, 1100, model.vocab)
    lm = pkg.AsyncLM(model, w, max_positions=1200, stream=torch.cuda.Stream())
    out = []
    for chunk in (0, 300, 512, 0):
        lm.set_option("chunk", chunk)
        with pytest.raises(pkg.AsyncLMError):
            lm.set_option("chunk", 513)
        lm.reset(0)
        lm.prefill(0, toks)
        out.append((*_planes(lm, model, 1100), lm.logits(0)))
    lm.close()
    for keys, vals, logits in out[1:]:
        assert _worst(keys, out[0][0]) <= TOL and _worst(vals, out[0][1]) <= TOL
        assert np.linalg.norm(logits - out[0][2]) / np.linalg.norm(out[0][2]) <= TOL
    # a pass of 300 rows sums in another order than one of 512 or 1100; the default again is the default
    assert not np.array_equal(out[0][0][1], out[1][0][1]) and not np.array_equal(out[1][0][1], out[2][0][1])
    assert all(np.array_equal(a, b) for a, b in zip(out[0], out[3]))


# The last layer of a pass over one sequence forms keys and values of all rows and goes on with the last row alone: with one layer
# that is the whole pass.  Prompt, interrupt, and an interrupt behind a chosen token, against the single-row kernels.
@pytest.mark.parametrize("n,kv,layers", [(2, 1, 1), (31, 4, 1), (33, 2, 1), (100, 4, 1), (129, 4, 1), (700, 1, 1), (65, 4, 2)])
def test_pass_that_ends_with_its_last_row(n, kv, layers):
    import paper_2412_07017_amd as pkg
    model = ModelConfig(n_layers=layers, d_model=512, n_q_heads=4, n_kv_heads=kv, head_dim=128, ffn=384, vocab=512, rms_eps=1e-5,
                        rope_theta=10000.0, dtype="bf16")
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    toks = ai.uniform_tokens(ai.MASTER_SEED, 946, 3 * n, model.vocab)
    lms = [pkg.AsyncLM(model, w, max_positions=3 * n + 8, stream=torch.cuda.Stream()) for _ in range(2)]
    lms[1].set_option("chunk", 1)
    for i, call in enumerate(("prefill", "inject", "batch")):
        blk = toks[i * n:(i + 1) * n]
        got = []
        for lm in lms:
            if call == "prefill":
                lm.prefill(0, blk)
            elif call == "inject":
                lm.inject_interrupt(0, blk)
            elif lm is lms[0]:
                assert list(lm.step_batch([0], forced=[9], interrupts=[blk])) == [9]
            else:
                lm.decode_step(0, forced_token=9)
                lm.inject_interrupt(0, blk)
            got.append((*_planes(lm, model, lm.seq_len(0)), lm.logits(0)))
        (ka, va, la), (kb, vb, lb) = got
        assert _worst(ka, kb) <= TOL and _worst(va, vb) <= TOL, (call, _worst(ka, kb), _worst(va, vb))
        assert np.linalg.norm(la - lb) / np.linalg.norm(lb) <= TOL, call
        assert lms[0].peek_choice(0) == int(np.argmax(la))
    for lm in lms:
        lm.close()


# Parts of K forced by option on a pass of more than 512 rows, where the partial planes hold fewer than asked for
@pytest.mark.parametrize("split", [1, 2, 3, 5, 8])
def test_forced_split_on_a_long_pass(split):
    import paper_2412_07017_amd as pkg
    model = ModelConfig(n_layers=2, d_model=1024, n_q_heads=8, n_kv_heads=2, head_dim=128, ffn=1152, vocab=512, rms_eps=1e-5,
                        rope_theta=10000.0, dtype="bf16")
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    toks = ai.uniform_tokens(ai.MASTER_SEED, 947, 1700, model.vocab)
    got = []
    for opt in (split, 0):
        lm = pkg.AsyncLM(model, w, max_positions=1800, stream=torch.cuda.Stream())
        lm.set_option("chunk_split", opt)
        lm.prefill(0, toks)
        got.append((*_planes(lm, model, 1700), lm.logits(0)))
        lm.close()
    (ka, va, la), (kb, vb, lb) = got
    assert _worst(ka, kb) <= TOL and _worst(va, vb) <= TOL
    assert np.linalg.norm(la - lb) / np.linalg.norm(lb) <= TOL


# k_chunk_attn_wide with every number of live waves in a block and of key splits: 1 to 9 query tiles over contexts below and
# above 3072 keys (where it also takes single tiles), against one split per wave (a batched step of one sequence at a time has
# the other kernel below 3072 keys)
@pytest.mark.parametrize("ctx", [70, 3040, 3300])
@pytest.mark.parametrize("rows", [2, 8, 9, 24, 31, 40, 72])
def test_shared_key_attention_on_short_interrupts(ctx, rows):
    import paper_2412_07017_amd as pkg
    model = ModelConfig(n_layers=2, d_model=512, n_q_heads=4, n_kv_heads=1, head_dim=128, ffn=256, vocab=512, rms_eps=1e-5,
                        rope_theta=10000.0, dtype="bf16")
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    toks = ai.uniform_tokens(ai.MASTER_SEED, 943, ctx + rows, model.vocab)
    got = []
    for chunk in (512, 1):                               # 1: the interrupt token by token through the single-row kernels
        lm = pkg.AsyncLM(model, w, max_positions=ctx + rows + 8, stream=torch.cuda.Stream())
        lm.prefill(0, toks[:ctx])
        lm.set_option("chunk", chunk)
        lm.inject_interrupt(0, toks[ctx:])
        got.append((*_planes(lm, model, ctx + rows), lm.logits(0)))
        lm.close()
    (ka, va, la), (kb, vb, lb) = got
    assert _worst(ka, kb) <= TOL, _worst(ka, kb)
    assert _worst(va, vb) <= TOL, _worst(va, vb)        # runs of values that start and end inside eight positions
    assert np.linalg.norm(la - lb) / np.linalg.norm(lb) <= TOL


# One sequence beyond 3072 keys among short ones: with fifteen others its key splits are few (a wave per task and split), with
# three the four waves of a workgroup share a tile; a batch of alike lengths beyond 3072 keys does so too.
@pytest.mark.parametrize("lens,intr", [([3400] + [40 + 3 * i for i in range(15)], {0: 5, 7: 24}), ([70, 3400, 33, 100], {1: 9}),
                                       ([3400, 3390, 3100, 3333, 3200, 3401], {2: 30})])
def test_batch_of_uneven_sequences_equals_one_at_a_time(lens, intr):
    import paper_2412_07017_amd as pkg
    model = ModelConfig(n_layers=2, d_model=1024, n_q_heads=8, n_kv_heads=8, head_dim=128, ffn=256, vocab=512, rms_eps=1e-5,
                        rope_theta=10000.0, dtype="bf16")
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    tk = lambda n, sub: ai.uniform_tokens(ai.MASTER_SEED, 944, n, model.vocab, sub=sub)
    blocks = [[int(t) for t in tk(intr.get(s, 0), 100 + s)] if s in intr else [] for s in range(len(lens))]
    forced = [(7 * s + 3) % model.vocab for s in range(len(lens))]
    lms = [pkg.AsyncLM(model, w, max_positions=3500, max_seqs=len(lens), stream=torch.cuda.Stream()) for _ in range(2)]
    for lm in lms:
        for s, n in enumerate(lens):
            lm.prefill(s, tk(n, s))
    for step in range(2):
        lms[0].step_batch(range(len(lens)), forced=forced, interrupts=blocks if step == 0 else None)
        for s in range(len(lens)):                                   # through the single-row kernels
            lms[1].decode_step(s, forced_token=forced[s])
            for t in blocks[s] if step == 0 else []:
                lms[1].decode_step(s, forced_token=t)
    for s, n in enumerate(lens):
        total = n + 2 + len(blocks[s])
        assert lms[0].seq_len(s) == lms[1].seq_len(s) == total
        (ka, va), (kb, vb) = _planes(lms[0], model, total, s), _planes(lms[1], model, total, s)
        assert _worst(ka, kb) <= TOL, (s, _worst(ka, kb))
        assert _worst(va, vb) <= TOL, (s, _worst(va, vb))
        la, lb = lms[0].logits(s), lms[1].logits(s)
        assert np.linalg.norm(la - lb) / np.linalg.norm(lb) <= TOL, s
    for lm in lms:
        lm.close()


# Interrupts of several tasks next to single rows, every sequence cut into another number of parts: blocks of one to four tasks
def test_blocks_of_several_tasks_cut_differently_in_one_batch():
    import paper_2412_07017_amd as pkg
    lens, intr = [3300, 1500, 700, 3000], {0: 40, 1: 24, 2: 70}
    model = ModelConfig(n_layers=2, d_model=1024, n_q_heads=8, n_kv_heads=2, head_dim=128, ffn=1024, vocab=512, rms_eps=1e-5,
                        rope_theta=10000.0, dtype="bf16")
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    tk = lambda n, sub: [int(t) for t in ai.uniform_tokens(ai.MASTER_SEED, 948, n, model.vocab, sub=sub)]
    blocks = [tk(intr[s], 100 + s) if s in intr else [] for s in range(len(lens))]
    lms = [pkg.AsyncLM(model, w, max_positions=3500, max_seqs=len(lens), stream=torch.cuda.Stream()) for _ in range(2)]
    for lm in lms:
        for s, n in enumerate(lens):
            lm.prefill(s, tk(n, s))
    lms[0].step_batch(range(len(lens)), forced=[3, 5, 7, 9], interrupts=blocks)
    for s, n in enumerate(lens):                            # through the single-row kernels
        lms[1].decode_step(s, forced_token=[3, 5, 7, 9][s])
        for t in blocks[s]:
            lms[1].decode_step(s, forced_token=t)
        total = n + 1 + len(blocks[s])
        (ka, va), (kb, vb) = _planes(lms[0], model, total, s), _planes(lms[1], model, total, s)
        assert _worst(ka, kb) <= TOL and _worst(va, vb) <= TOL, (s, _worst(ka, kb), _worst(va, vb))
        la, lb = lms[0].logits(s), lms[1].logits(s)
        assert np.linalg.norm(la - lb) / np.linalg.norm(lb) <= TOL, s
    for lm in lms:
        lm.close()


def test_weights_at_eight_bytes_past_an_alignment():
    """The same weights at addresses that are no multiple of 16: passes of at most 128 rows, through registers."""
    import paper_2412_07017_amd as pkg
    model = ModelConfig(n_layers=2, d_model=512, n_q_heads=4, n_kv_heads=2, head_dim=128, ffn=640, vocab=512, rms_eps=1e-5,
                        rope_theta=10000.0, dtype="bf16")
    w = ai.make_weights(model, device=torch.device("cuda:0"))

    def moved(t):
        flat = torch.empty(t.numel() + 4, dtype=t.dtype, device=t.device)
        flat[4:] = t.reshape(-1)
        return flat[4:].view(t.shape)

    shifted = {k: ([moved(t) for t in v] if isinstance(v, (list, tuple)) else moved(v)) if "norm" not in k else v for k, v in w.items()}
    assert shifted["wqkv"][0].data_ptr() % 16 == 8
    torch.cuda.synchronize()
    toks = ai.uniform_tokens(ai.MASTER_SEED, 945, 900, model.vocab)
    got = []
    for ws in (w, shifted):
        lm = pkg.AsyncLM(model, ws, max_positions=1000, max_seqs=2, stream=torch.cuda.Stream())
        lm.prefill(0, toks[:600])
        lm.prefill(1, toks[:7])
        lm.inject_interrupt(0, toks[600:650])
        lm.step_batch([0, 1], forced=[1, 2], interrupts=[toks[650:800], toks[800:830]])
        lm.decode_step(0, forced_token=5)
        got.append((*_planes(lm, model, 802), lm.logits(0), lm.logits(1)))
        lm.close()
    (ka, va, la, ma), (kb, vb, lb, mb) = got
    assert _worst(ka, kb) <= TOL and _worst(va, vb) <= TOL
    assert np.linalg.norm(la - lb) / np.linalg.norm(lb) <= TOL and np.linalg.norm(ma - mb) / np.linalg.norm(mb) <= TOL


# Keys that one workgroup streams: pieces of one tile and of two, with one tile left over, four tasks (32 rows are the streamed
# kernel's most; of 25 the last task has four columns).
@pytest.mark.parametrize("ctx", [0, 1, 32, 33, 64, 130, 290])
@pytest.mark.parametrize("rows", [25, 32])
def test_streamed_keys_in_pieces_of_one_and_two_tiles(ctx, rows):
    import paper_2412_07017_amd as pkg
    model = ModelConfig(n_layers=2, d_model=512, n_q_heads=4, n_kv_heads=1, head_dim=128, ffn=256, vocab=512, rms_eps=1e-5,
                        rope_theta=10000.0, dtype="bf16")
    w = ai.make_weights(model, device=torch.device("cuda:0"))
    torch.cuda.synchronize()
    toks = ai.uniform_tokens(ai.MASTER_SEED, 947, ctx + rows, model.vocab)
    got = []
    for chunk in (512, 1):                               # 1: token by token through the single-row kernels
        lm = pkg.AsyncLM(model, w, max_positions=ctx + rows, stream=torch.cuda.Stream())
        if ctx:
            lm.prefill(0, toks[:ctx])
        lm.set_option("chunk", chunk)
        (lm.inject_interrupt if ctx else lm.prefill)(0, toks[ctx:])
        got.append((*_planes(lm, model, ctx + rows), lm.logits(0)))
        lm.close()
    (ka, va, la), (kb, vb, lb) = got
    assert _worst(ka, kb) <= TOL, _worst(ka, kb)
    assert _worst(va, vb) <= TOL, _worst(va, vb)
    assert np.linalg.norm(la - lb) / np.linalg.norm(lb) <= TOL
