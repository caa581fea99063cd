"""Which kernels the host code launches, and with how many workgroups, on a HIP runtime without a device (host_hip.c is
preloaded into a child process; nothing is computed)."""
import json
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

CHILD = r'''
import ctypes as C, json, os, sys, types
sys.path.insert(0, os.environ["ASYNCLM_ROOT"])
import numpy as np
import paper_2412_07017_amd as pkg
hip = C.CDLL(os.environ["HOST_HIP_LIBRARY"])
hip.host_hip_peak.restype = hip.host_hip_used.restype = C.c_size_t

class Stream:
    cuda_stream = 4096

class Matrix:
    def __init__(self, a): self.a = a
    def data_ptr(self): return self.a

def context(max_positions, max_seqs=1, base=1 << 20, **model):
    m = dict(n_layers=2, d_model=512, n_q_heads=4, n_kv_heads=1, head_dim=128, ffn=512, vocab=512, rms_eps=1e-5, rope_theta=1e4, dtype="bf16")
    kv = model.pop("kv_format", 0)
    m.update(model)
    w = {k: Matrix(base) for k in ("embed", "final_norm", "lm_head")}
    w.update({k: [Matrix(base)] * m["n_layers"] for k in ("attn_norm", "wqkv", "wo", "ffn_norm", "wgate_up", "wdown")})
    return pkg.AsyncLM(types.SimpleNamespace(**m), w, max_positions=max_positions, max_seqs=max_seqs, stream=Stream(), kv_format=kv)

def tokens(n): return np.zeros(n, np.int32)

def launches(call):
    log = os.environ["HOST_HIP_LOG_FILE"]
    if os.path.exists(log): os.remove(log)
    os.environ["HOST_HIP_LOG"] = log
    call()
    del os.environ["HOST_HIP_LOG"]
    return [(l.split()[0], *map(int, l.split()[1:])) for l in open(log)] if os.path.exists(log) else []

def count(ls, name): return sum(name in l[0] for l in ls)
'''


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    if shutil.which("gcc") is None:
        pytest.skip("no C compiler")
    import paper_2412_07017_amd as pkg
    if not os.path.exists(pkg.library_path()):
        from paper_2412_07017_amd.build import build_library
        build_library()
    tmp = tmp_path_factory.mktemp("host_hip")
    so = str(tmp / "host_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", os.path.join(HERE, "host_hip.c"), "-o", so], check=True)

    def run(body, **env):
        preload = ":".join([so] + [p for p in (os.environ.get("LD_PRELOAD"),) if p])
        e = dict(os.environ, LD_PRELOAD=preload, HOST_HIP_LIBRARY=so, ASYNCLM_ROOT=ROOT, HOST_HIP_LOG_FILE=str(tmp / "log"), **{k: str(v) for k, v in env.items()})
        res = subprocess.run([sys.executable, "-c", CHILD + body], env=e, capture_output=True, text=True, timeout=120)
        assert res.returncode == 0, res.stderr
        return json.loads(res.stdout.splitlines()[-1])
    return run


# One sequence far longer than the others: the attention with a wave per task and split, which cuts it into four times as
# many parts.  Alike lengths, and few tasks: the attention whose four waves share a tile.
@pytest.mark.parametrize("lens,intr,wide", [([16000] + [512] * 15, {}, False), ([16000] + [512] * 31, {}, False), ([16000] + [500] * 5, {}, False),
                                            ([16000] + [512] * 15, {3: 24}, False), ([16000] + [512] * 15, {0: 48}, False),
                                            ([4000] + [300] * 15, {}, False), ([3500] * 16, {}, True), ([8000] * 4, {}, True),
                                            ([16000, 100], {}, True), ([16000] + [500] * 3, {}, True), ([2000] * 16, {}, False),
                                            ([600] * 4, {1: 200}, True)])
def test_attention_of_a_batch_follows_the_longest_chain(host, lens, intr, wide):
    got = host(f'''
lens, intr = {lens!r}, {intr!r}
lm = context(16400, len(lens), d_model=4096, n_q_heads=32, n_kv_heads=8, ffn=1024)
for s, n in enumerate(lens): lm.prefill(s, tokens(n))
ls = launches(lambda: lm.step_batch(range(len(lens)), forced=[1] * len(lens), interrupts=[tokens(intr.get(s, 0)) for s in range(len(lens))]))
print(json.dumps([count(ls, "k_chunk_attn_wide"), count(ls, "12k_chunk_attnE")]))
''')
    assert got == ([2, 0] if wide else [0, 2])


# A matrix that does not start at a multiple of 16 bytes: no pass reaches the product that loads weights straight to LDS
@pytest.mark.parametrize("off,big", [(0, True), (8, False), (2, False), (16, True)])
def test_unaligned_weights_stay_off_the_loads_to_lds(host, off, big):
    got = host(f'''
lm = context(2100, 4, base=(1 << 20) + {off})
a = launches(lambda: lm.prefill(0, tokens(1300)))
b = launches(lambda: [lm.prefill(s, tokens(3)) for s in (1, 2, 3)] + [lm.step_batch(range(4), interrupts=[tokens(n) for n in (200, 100, 50, 140)])])
print(json.dumps([count(a, "k_chunk_gemm_big"), count(b, "k_chunk_gemm_big"), count(a, "k_chunk_embed_norm"), lm.seq_len(0), lm.seq_len(3)]))
''')
    assert (got[0] > 0) == big and (got[1] > 0) == big
    assert got[2] == (1 if big else 11) and got[3:] == [1501, 144]


def test_pass_size_option_bounds_a_pass_and_can_be_taken_back(host):
    got = host('''
out = []
for lm, kernel, n in ((context(2100), "k_chunk_embed_norm", 1301), (context(2100, dtype="fp32", head_dim=64), "k_rows_embed", 34)):
    for value in (None, 512, 5, 1, 0):
        if value is not None: lm.set_option("chunk", value)
        lm.reset(0)
        out.append(count(launches(lambda: lm.prefill(0, tokens(n))), kernel))
    for bad in (-1, 513):
        try: lm.set_option("chunk", bad); out.append("taken")
        except pkg.AsyncLMError as e: out.append(e.code)
print(json.dumps(out))
''')
    # 1301 tokens: 2 passes of 512 and one of 277; 260 of five and the last token alone; 34: four of eight and one of two, or
    # six of five and one of four
    assert got[:7] == [1, 3, 260, 0, 1, -1, -1]
    assert got[7:] == [5, 5, 7, 0, 5, -1, -1]


# Memory too short for the buffers of 2048-row passes: the context is created with those of 512 rows, whether an allocation
# fails or the graphs of the decoding steps find no room; memory too short for these as well: an error, and nothing is left
def test_create_with_little_memory(host):
    full = host("context(4096); print(json.dumps(hip.host_hip_peak()))")
    body = '''
try:
    lm = context(4096)
    n = count(launches(lambda: lm.prefill(0, tokens(1300))), "k_chunk_embed_norm")
    lm.close()
except pkg.AsyncLMError as e: n = e.code
print(json.dumps([n, hip.host_hip_used()]))
'''
    assert host(body) == [1, 0]
    assert host(body, HOST_HIP_BUDGET=full) == [1, 0]
    assert host(body, HOST_HIP_BUDGET=full - 1) == [3, 0]
    assert host(body, HOST_HIP_GRAPHS=full - 1) == [3, 0]
    assert host(body, HOST_HIP_BUDGET=full // 4) == [-4, 0]
    assert host(body, HOST_HIP_GRAPHS=full // 4) == [-5, 0]


def test_every_variant_of_the_row_kernels_has_a_case(host):
    from test_gpu_rows import BF16, CASES
    models = [dict(m.__dict__, kv_format=1 if kind == BF16 else 0) for kind, m in CASES]
    names = set(host(f'''
names = set()
for m in {models!r}:
    lm = context(64, **m)
    names |= {{l[0] for l in launches(lambda: lm.prefill(0, tokens(8)))}}
    lm.close()
print(json.dumps(sorted(names)))
'''))
    for t in "ft":                                      # fp32, bf16 (unsigned short)
        for epi in (1, 2, 3):                           # residual, SwiGLU, QKV
            for pairs in (1, 2):
                for seg in (0, 1):
                    want = f"k_rows_gemvI{t}Li{epi}ELi{pairs}ELb{seg}E"
                    assert any(want in n for n in names), want
        for loads in (1, 2, 4):
            assert any(f"k_rows_smallI{t}" in n and f"ELi{loads}EEE" in n for n in names), (t, loads)


# Models of the wide rows path (bf16, the cache row by row): where their buffers find no room, or the graphs after them, the context is
# created without them and takes passes of eight rows; option chunk bounds a pass as everywhere
def test_wide_rows_and_little_memory(host):
    model = "context(1024, kv_format=1, d_model=1024, ffn=2048)"
    full = host(f"{model}; print(json.dumps(hip.host_hip_peak()))")
    body = f'''
try:
    lm = {model}
    out = []
    for value in (0, 100, 1):
        lm.set_option("chunk", value); lm.reset(0)
        ls = launches(lambda: lm.prefill(0, tokens(600)))
        out.append([count(ls, "k_chunk_embed_norm"), count(ls, "k_rows_embed")])
    lm.close()
except pkg.AsyncLMError as e: out = e.code
print(json.dumps([out, hip.host_hip_used()]))
'''
    wide, rows = [[2, 0], [6, 0], [0, 0]], [[0, 75], [0, 75], [0, 0]]
    assert host(body) == [wide, 0] and host(body, HOST_HIP_BUDGET=full) == [wide, 0]
    assert host(body, HOST_HIP_BUDGET=full - 1) == [rows, 0]
    assert host(body, HOST_HIP_GRAPHS=full - 1) == [rows, 0]
    assert host(body, HOST_HIP_BUDGET=full // 100) == [-4, 0]
    # sizes that are no multiples of 128, fp32: the rows path as before
    for other in ("ffn=2056", "d_model=1032", "dtype='fp32'"):
        kw = "kv_format=0, " if "fp32" in other else "kv_format=1, "
        assert host(f"lm = context(1024, {kw}{other}); print(json.dumps(count(launches(lambda: lm.prefill(0, tokens(16))), 'k_rows_embed')))") == 2


# Which of the two paths a pass of a row-major bf16 model takes: few rows of small models the vector units (five launches a layer and the
# head, eight tokens per launch of the embedding), all else the matrix cores
@pytest.mark.parametrize("model,rows,wide", [
    (dict(d_model=256, n_q_heads=4, n_kv_heads=4, head_dim=64, ffn=768), [2, 8], [9, 32, 200]),               # two layers
    (dict(d_model=256, n_q_heads=4, n_kv_heads=4, head_dim=64, ffn=768, n_layers=4), [2, 8, 9, 32], [33, 200]),
    (dict(d_model=1024, n_q_heads=16, n_kv_heads=4, head_dim=64, ffn=1024, n_layers=4), [8, 16], [17, 64]),
    (dict(d_model=1024, n_q_heads=16, n_kv_heads=4, head_dim=64, ffn=4096, n_layers=4), [2, 8], [9, 24]),      # not all products small
    (dict(d_model=2048, n_q_heads=16, n_kv_heads=8, ffn=6144, n_layers=3, kv_format=1), [2, 8], [9]),
    (dict(d_model=2048, n_q_heads=16, n_kv_heads=8, ffn=6144, n_layers=2, kv_format=1), [], [2, 8, 9]),
    (dict(d_model=4096, n_q_heads=32, n_kv_heads=8, ffn=14336, n_layers=4, kv_format=1), [], [2, 8, 24]),
])
def test_short_passes_of_small_models_take_the_vector_units(host, model, rows, wide):
    got = host(f'''
model = {model!r}
lm = context(1024, **model)
lm.prefill(0, tokens(40))
out = []
for n in {rows + wide!r}:
    ls = launches(lambda: lm.inject_interrupt(0, tokens(n)))
    out.append([count(ls, "k_rows_embed"), count(ls, "k_chunk_embed_norm"), len(ls)])
print(json.dumps(out))
''')
    nl = model.get("n_layers", 2)
    for n, g in zip(rows + wide, got):
        groups = (n + 7) // 8
        assert g == ([groups, 0, groups + 5 * nl + 1] if n in rows else [0, 1, g[2]]), n
        assert n in rows or g[2] == 8 * nl + 1, n


def test_every_pass_of_a_call_takes_its_own_path(host):
    assert host('''
lm = context(1024, d_model=256, n_q_heads=4, n_kv_heads=4, head_dim=64, ffn=768)
out = []
for chunk, n in ((0, 515), (8, 20), (1, 3)):
    lm.set_option("chunk", chunk); lm.reset(0)
    ls = launches(lambda: lm.prefill(0, tokens(n)))
    out.append([count(ls, "k_rows_embed"), count(ls, "k_chunk_embed_norm"), lm.seq_len(0)])
print(json.dumps(out))
''') == [[1, 1, 515], [3, 0, 20], [0, 0, 3]]


# The short step of small models: launch by launch up to three layers, from four on one kernel and a graph, past its last key the ordinary step
@pytest.mark.parametrize("layers,last", [(2, 384), (3, 384), (4, 256), (5, 256), (16, 256)])
def test_launches_of_the_short_step(host, layers, last):
    got = host(f'''
lm = context(500, dtype="fp32", d_model=256, n_kv_heads=4, head_dim=64, ffn=688, n_layers={layers})
out = []
for ctx, graph in ((20, 1), (20, 0), ({last} - 1, 1), ({last}, 1)):
    lm.set_option("graph", graph); lm.reset(0); lm.prefill(0, tokens(ctx))
    ls = launches(lambda: lm.decode_step(0, forced_token=1))
    out.append([sum(l[0] == "graph" for l in ls), len(ls), count(ls, "k_small_attn_o"), count(ls, "k_begin_step")])
print(json.dumps(out))
''')
    plain, graph = [0, 3 * layers + 1, layers, 0], [1, 2, 0, 0]
    short = graph if layers > 3 else plain
    assert got == [short, plain, short, [1, 2, 0, 1]]


def test_short_steps_of_the_device_tests_are_short_steps(host):
    from test_gpu_small_step import CASES, GRAPHS
    models = [dict(m.__dict__, kv_format=1 if kind == "bf16" else 0) for kind, m in CASES]
    graphs = [(dict(m.__dict__, kv_format=1 if kind == "bf16" else 0), last) for kind, m, last in GRAPHS]
    names, short = host(f'''
names, short = set(), []
for m in {models!r}:
    lm = context(64, **m)
    lm.prefill(0, tokens(1))
    names |= {{l[0] for l in launches(lambda: lm.decode_step(0, forced_token=1))}}
    lm.close()
for m, last in {graphs!r}:
    lm = context(420, **m)
    for ctx in (20, last - 1, last):
        lm.reset(0); lm.prefill(0, tokens(ctx))
        ls = launches(lambda: lm.decode_step(0, forced_token=1))
        short.append([sum(l[0] == "graph" for l in ls), count(ls, "k_begin_step")])
    lm.close()
print(json.dumps([sorted(names), short]))
''')
    assert short == [[1, 0], [1, 0], [1, 1]] * len(GRAPHS)
    want = ["k_small_attn_oIfLi%dELi%dELb0E" % v for v in ((64, 1), (64, 2), (64, 4), (128, 1), (128, 2))]
    want += ["k_small_attn_oItLi%dELi%dELb%dE" % (dh, G, pair) for dh in (64, 128) for G in (1, 2, 4, 8) if G * dh < 1024 for pair in (0, 1)]
    want += ["k_small_mlpIfLi1E", "k_small_mlpIfLi2E", "k_small_mlpItLi1E"]
    want += ["k_gemv_smallI%sLi%dELi%dELi%dEE" % (t, epi, ns, src) for t, ns in (("f", 1), ("f", 2), ("t", 1)) for epi, src in ((3, 1), (3, 2), (0, 1))]
    assert [w for w in want if not any(w in n for n in names)] == []


# Where the short step is the slower one: measured for each of these, the first two far beyond what it gains elsewhere
@pytest.mark.parametrize("model,ctx", [
    ("d_model=512, n_q_heads=8, n_kv_heads=4, head_dim=64, ffn=1024, n_layers=4", 340), ("d_model=128, n_q_heads=16, n_kv_heads=2, head_dim=64, ffn=384", 280),
    ("d_model=512, n_q_heads=8, n_kv_heads=8, head_dim=64, ffn=1024, n_layers=5", 20), ("d_model=1024, n_q_heads=8, n_kv_heads=8, head_dim=64, ffn=1024", 20),
    ("dtype='fp32', d_model=512, n_q_heads=8, n_kv_heads=8, head_dim=64, ffn=1024, n_layers=5", 20), ("dtype='fp32', d_model=128, n_q_heads=2, n_kv_heads=2, ffn=384", 360)])
def test_short_step_only_where_it_pays(host, model, ctx):
    assert host(f'''
lm = context(500, {model})
lm.prefill(0, tokens({ctx}))
print(json.dumps(count(launches(lambda: lm.decode_step(0, forced_token=1)), "k_begin_step")))
''') == 1


# A stream that has run dry without the word of the step's token having been written: the wait for it ends
@pytest.mark.parametrize("model", ["d_model=512", "dtype='fp32', d_model=256, head_dim=64, ffn=688", "dtype='fp32', d_model=256, n_kv_heads=4, head_dim=64, ffn=688"])
def test_wait_for_a_token_ends(host, model):
    assert host(f'''
lm = context(64, {model})
lm.prefill(0, tokens(5))
print(json.dumps([lm.decode_step(0, forced_token=3), lm.decode_step(0), lm.seq_len(0)]))
''') == [0, 0, 7]


# A step behind much other work: the host does not keep a core busy until its token is there
@pytest.mark.parametrize("model", ["n_layers=16, d_model=4096, n_q_heads=32, n_kv_heads=8, ffn=14336", "d_model=512", "dtype='fp32', d_model=256, n_kv_heads=4, head_dim=64, ffn=688"])
def test_wait_for_a_token_leaves_the_core(host, model):
    wall, cpu = host(f'''
import time
hip.host_hip_busy.argtypes = [C.c_double]
lm = context(64, {model})
lm.prefill(0, tokens(5))
hip.host_hip_busy(0.5)
t, p = time.monotonic(), time.thread_time()
assert lm.decode_step(0) == 0
print(json.dumps([time.monotonic() - t, time.thread_time() - p]))
''')
    assert wall >= 0.45 and cpu <= 0.1


# The shared-key attention of a batch: every sequence cut by its own length, at most two workgroups per compute unit, and no other cut
# with as many workgroups has a shorter longest part.  From the row table as it is uploaded (groups, tasks, blocks, pieces): every part of every
# block is there once, none is empty, and no two share the place of their partial results.  Single rows among interrupts (blocks of several
# tasks) too.  (The last case is that of a test on the device.)
@pytest.mark.parametrize("lens,intr,heads", [([3500] * 16, {}, (32, 8)), ([8000] * 4, {}, (32, 8)), ([16000, 100], {}, (32, 8)), ([16000] + [500] * 3, {}, (32, 8)),
                                             ([600] * 4, {1: 200}, (32, 8)), ([512 + 230 * i for i in range(16)], {0: 24}, (32, 8)),
                                             ([3300, 1500, 700, 3000], {0: 40, 1: 24, 2: 70}, (8, 2))])
def test_attention_of_a_batch_is_cut_evenly(host, lens, intr, heads):
    grids, tab = host(f'''
lens, intr = {lens!r}, {intr!r}
lm = context(16400, len(lens), d_model=1024, n_q_heads={heads[0]}, n_kv_heads={heads[1]}, ffn=1024)
for s, n in enumerate(lens): lm.prefill(s, tokens(n))
ls = launches(lambda: lm.step_batch(range(len(lens)), forced=[1] * len(lens), interrupts=[tokens(intr.get(s, 0)) for s in range(len(lens))]))
buf = (C.c_ubyte * (1 << 18))()
hip.host_hip_uploaded.restype = C.c_size_t
n = hip.host_hip_uploaded(buf, C.c_size_t(1 << 18))
print(json.dumps([[l[1] for l in ls if "k_chunk_attn_wide" in l[0]], list(buf)[:n]]))
''')
    rows = [1 + intr.get(s, 0) for s in range(len(lens))]
    G, Hkv = heads[0] // heads[1], heads[1]
    ntasks = [(G * r + 31) // 32 for r in rows]
    nblocks = sum((t + 3) // 4 for t in ntasks)
    npieces = grids[0] // Hkv
    assert grids == [npieces * Hkv] * 2 and npieces * Hkv <= 512
    tab, at = np.array(tab, np.uint8), 32 * len(lens)
    tasks = tab[at:at + 32 * sum(ntasks)].view(np.int32).reshape(-1, 8)         # seq, row0, n, pos0, tile, nsplit, unit0
    at += 32 * sum(ntasks)
    blocks = tab[at:at + 8 * nblocks].view(np.int32).reshape(-1, 2)             # task0, n
    at += (8 * nblocks + 31) // 32 * 32
    pieces = tab[at:at + 4 * npieces].view(np.int16).reshape(-1, 2)             # block, split
    assert list(tasks[:, 0]) == [s for s in range(len(lens)) for _ in range(ntasks[s])]
    assert [t for b, n in blocks for t in range(b, b + n)] == list(range(sum(ntasks)))
    tiles, splits = [], []                                  # key tiles and parts of every block
    for task0, n in blocks:
        seq, row0, r, pos0, tile = tasks[task0][:5]
        assert len({tuple(t[:4]) + (t[5],) for t in tasks[task0:task0 + n]}) == 1 and 1 <= n <= 4
        columns = range(32 * tile, min(32 * (tile + n), G * r))                 # (query head, row) pairs: a tile may run from one head into the next
        tiles.append(-(-(pos0 + max(c % r for c in columns) + 1) // 32))
        splits.append(int(tasks[task0][5]))
    assert sorted(map(tuple, pieces)) == [(b, s) for b in range(nblocks) for s in range(splits[b])]
    for t, k in zip(tiles, splits):
        per = -(-t // k)
        assert per * (k - 1) < t                            # the last part has tiles
    if any(k > 1 for k in splits):
        used = [u for t in tasks for u in range(t[6], t[6] + t[5])]
        assert len(set(used)) == len(used) and max(used) < 4096 // Hkv
    best = [1] * nblocks                                    # one more part for the longest, as long as there is room
    part = lambda i: -(-tiles[i] // best[i])
    while True:
        i = max(range(nblocks), key=part)
        k = next((k for k in range(best[i] + 1, tiles[i] + 1) if -(-tiles[i] // k) < part(i)), None)
        if k is None or part(i) <= 2 or (sum(best) - best[i] + k) * Hkv > 512:
            break
        best[i] = k
    assert max(-(-t // k) for t, k in zip(tiles, splits)) == max(map(part, range(nblocks)))


# ... and found in a few looks: the host's part of a batched step of 120 long sequences is a few times that of 16, not seven times
def test_cut_of_many_long_sequences_costs_the_host_little(host):
    few, many = host('''
import time
out = []
for n in (16, 120):
    lm = context(16600, n, d_model=1024, n_q_heads=32, n_kv_heads=8, ffn=1024)
    for s in range(n): lm.prefill(s, tokens(16000))
    ts = []
    for _ in range(30):
        t = time.perf_counter(); lm.step_batch(range(n), forced=[1] * n, want_tokens=False); ts.append(time.perf_counter() - t)
    out.append(min(ts))
    lm.close()
print(json.dumps(out))
''')
    assert many <= 4 * few


def test_attention_of_a_prompt_has_a_workgroup_per_block(host):
    assert host('''
lm = context(2100, d_model=4096, n_q_heads=32, n_kv_heads=8, ffn=1024)
out = []
for n in (1019, 2048):
    lm.reset(0)
    out.append([l[1] for l in launches(lambda: lm.prefill(0, tokens(n))) if "k_chunk_attn_wide" in l[0]])
print(json.dumps(out))
''') == [[256], [512]]


# Attention of the rows of a pass: its keys are cut only where the merge of the parts costs less than the shorter chain gives
@pytest.mark.parametrize("ctx,n,want", [(100, 8, 1), (300, 2, 2), (300, 24, 1), (300, 200, 1), (1000, 8, 4), (1000, 64, 1), (4000, 2, 16), (4000, 16, 4), (4000, 200, 1),
                                        (16000, 2, 32), (16000, 16, 8), (16000, 128, 4), (16000, 300, 1)])
def test_attention_of_rows_is_cut_where_the_merge_pays(host, ctx, n, want):
    got = host(f'''
lm = context(16400, 1, kv_format=1, d_model=4096, n_q_heads=32, n_kv_heads=8, ffn=1024)
lm.prefill(0, tokens({ctx}))
print(json.dumps([l[1:4] for l in launches(lambda: lm.inject_interrupt(0, tokens({n}))) if "k_attn_decode" in l[0]][0]))
''')
    assert got == [8, want, n]
