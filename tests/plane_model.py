"""A decoder whose logits lie in the low bits of what enters its products: every block of 32 (or 16) logits below is the difference of two
values that agree to 2^-17 or 2^-18, scaled up again by exact powers of two.  A product that sees its inputs with 16 bits of mantissa gets a block
wrong by its own size; one that sees all 24 gets it right to about a hundredth (an input rounded to 2^-24 is wrong by 2^-7 of the difference)."""
import numpy as np
import torch

from asynclm_inputs.configs import ModelConfig

D = 256
SPECIAL = 7                 # the token that the attention block weighs with about 2^-17
# Four roundings of 2^-24 against a difference of 2^-18 (fp32 on the CPU: 0.011 at most); two planes: 0.15 and more up to 140 rows
BOUND = 0.0625
# logits of a block -> the values whose low bits they are, and what rounds them in the oracle (see CachedDecoder.diag_round)
BLOCKS = {
    "QKV input, first layer (embedding and norm)": (range(96, 128), "h"),
    "gate/up input (residual and norm)": (range(128, 160), "h"),
    "attention output": (range(160, 176), "o"),
    "SwiGLU output": (range(192, 208), "a"),
    "K and V input, last layer": (range(224, 256), "h"),
}


def model(dh):
    return ModelConfig(n_layers=2, d_model=D, n_q_heads=4, n_kv_heads=2, head_dim=dh, ffn=256, vocab=D, rms_eps=1e-5, rope_theta=10000.0, dtype="bf16")


def tokens(n, seed=0):
    t = np.random.default_rng(seed).integers(0, D, size=n)
    t[t == SPECIAL] = 8
    t[3] = SPECIAL
    return [int(v) for v in t]


def weights(dh, n, device):
    """For a pass of n rows: the special token's score depends on it."""
    m, r = model(dh), np.random.default_rng(5)
    c0, c1 = 64, 65                                     # a constant column, and a flag of the special token
    embed = np.zeros((D, D))
    embed[:, :32] = r.uniform(0.5, 2.0, (D, 32))
    embed[:, 32:64] = embed[:, :32]
    embed[:, c0] = 1.0
    embed[SPECIAL, c1] = 1.0
    bf = lambda a: torch.as_tensor(a, dtype=torch.float32).to(torch.bfloat16)
    e = bf(embed).float().numpy()
    a0 = 1.0 / np.sqrt((e[:, :66] ** 2).sum(1).mean() / D)                      # about: the constant after a norm
    gain = np.ones(D)
    gain[32:64] = 1 + 2.0 ** -18                        # columns 32 + c: columns c, a little larger
    wqkv, wo = np.zeros((2, 8 * dh, D)), np.zeros((2, D, 4 * dh))
    wgu, wdown = np.zeros((2, 512, D)), np.zeros((2, D, 256))
    kv = lambda what, head, ch: (4 + 2 * what + head) * dh + ch                 # row of a key (0) or value (1)
    # query head 0 scores the special token so that e^score / n is about 2^-17, through the pair of channels that turns slowest
    score = np.log(n * 2.0 ** -17)
    wqkv[0, dh // 2 - 1, c0] = 8.0
    wqkv[0, kv(0, 0, dh // 2 - 1), c1] = score * np.sqrt(dh) / (8.0 * a0 * a0)
    for c in range(16):                                 # values 16 + c: values c, but for the special token
        wqkv[0, kv(1, 0, c), c] = wqkv[0, kv(1, 0, 16 + c), c] = wqkv[0, kv(1, 0, 16 + c), c1] = 1.0
        wo[0, 160 + c, c], wo[0, 160 + c, 16 + c] = 2.0 ** 17, -2.0 ** 17
    for c in range(32):                                 # values of the other kv head: differences of two columns; its query heads score all alike
        for l in range(2):
            wqkv[l, kv(1, 1, c), c], wqkv[l, kv(1, 1, c), 32 + c] = 2.0 ** 18, -2.0 ** 18
        wo[0, 96 + c, 2 * dh + c] = wo[1, 224 + c, 2 * dh + c] = 1.0
        wgu[0, c, c0], wgu[0, 256 + c, c], wgu[0, 256 + c, 32 + c] = 16.0, 2.0 ** 18, -2.0 ** 18
        wdown[0, 128 + c, c] = 0.125
    for c in range(16):                                 # features 96 + c: features 64 + c, a little larger
        for f in (64 + c, 96 + c):
            wgu[0, f, c0], wgu[0, 256 + f, c] = 16.0, 1.0
        wgu[0, 256 + 96 + c, c0] = 2.0 ** -17
        wdown[0, 192 + c, 64 + c], wdown[0, 192 + c, 96 + c] = 2.0 ** 14, -2.0 ** 14
    t = lambda a: bf(a).to(device).contiguous()
    f = lambda a: torch.as_tensor(a, dtype=torch.float32).to(device).contiguous()
    ones = np.ones(D)
    return {"embed": t(embed), "final_norm": f(ones), "lm_head": t(np.eye(D)), "attn_norm": [f(gain), f(gain)], "ffn_norm": [f(gain), f(ones)],
            "wqkv": [t(v) for v in wqkv], "wo": [t(v) for v in wo], "wgate_up": [t(v) for v in wgu], "wdown": [t(v) for v in wdown]}


def errors(got, want):
    """Relative error (2-norm) of every block."""
    out = {}
    for name, (cols, _) in BLOCKS.items():
        a, b = np.asarray(got, np.float64)[list(cols)], np.asarray(want, np.float64)[list(cols)]
        out[name] = float(np.linalg.norm(a - b) / np.linalg.norm(b))
    return out
