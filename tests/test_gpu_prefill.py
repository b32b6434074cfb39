"""The prefill pass (prompts of more tokens than a verify pass takes) against the same tokens given in pieces of at most 8
(float32: 16), which go through the verify pass: cache rows, greedy tokens of every position, kept logits and what a
following window sees, bit for bit.
The sizes put the edges of its row and column tiles, its workgroup shapes and the K ranges of the down projection in turn."""
import numpy as np
import pytest

from workload import GLOBAL_TENSORS, LAYER_TENSORS, SHAPES, WeightStore, prompt_tokens

pytestmark = pytest.mark.gpu

CASES = [
    # (shape, overrides, tokens cached before, prompt length)
    ("tiny_verify", {}, 0, 17), ("tiny_verify", {}, 5, 130), ("tiny_draft", {}, 0, 33),
    ("tiny_gqa_fp32", {}, 0, 300), ("tiny_wide_fp32", {}, 3, 65),
    ("tiny_gqa_bf16", {}, 0, 9), ("tiny_g8_bf16", {}, 130, 16), ("tiny_gqa_bf16", {}, 0, 17), ("tiny_gqa_bf16", {}, 7, 64), ("tiny_gqa_bf16", {}, 1, 300),
    ("tiny_gqa128_bf16", {}, 33, 129), ("tiny_g8_bf16", {}, 0, 200), ("tiny_wide_bf16", {}, 2, 97),
    ("tiny_gqa_bf16", {"d_model": 288, "d_ffn": 544, "vocab": 1008}, 0, 47),     # K blocks that do not split evenly over the waves
    ("tiny_wide_bf16", {"d_model": 320, "d_ffn": 4160}, 0, 80),
    ("tiny_gqa_bf16", {"d_model": 128, "n_q_heads": 2, "n_kv_heads": 1, "d_ffn": 96}, 0, 70),   # fewer K blocks than waves
    ("one_layer_8b_width_bf16", {"vocab": 16000}, 3, 24),
    ("one_layer_8b_width_bf16", {"vocab": 16000}, 0, 61), ("one_layer_8b_width_bf16", {}, 0, 128),
    ("one_layer_8b_width_bf16", {"d_ffn": 14336}, 0, 250), ("one_layer_8b_width_bf16", {"vocab": 16000}, 40, 400),
    ("one_layer_8b_width_bf16", {"vocab": 16000}, 0, 1100), ("one_layer_8b_width_bf16", {}, 9, 2190),
    # Attention runs of several key blocks: ceil(context / (256 / kv heads * runs * block)) blocks, 8 / G runs a chunk, so that
    # row tiles end after every number of blocks of the first and of the second run.  Odd runs end in a step of one block.
    ("tiny_gqa_bf16", {"d_model": 128, "n_q_heads": 128, "n_kv_heads": 32, "d_ffn": 128}, 33, 1030),     # G = 4: 3 blocks
    ("tiny_gqa_bf16", {"d_model": 128, "n_q_heads": 128, "n_kv_heads": 32, "d_ffn": 128}, 0, 2100),      # 5, in two passes
    ("tiny_gqa128_bf16", {"d_model": 128, "n_q_heads": 64, "n_kv_heads": 16, "d_ffn": 128}, 7, 2050),    # head_dim 128: 3
    ("tiny_g8_bf16", {"d_model": 128, "n_q_heads": 256, "n_kv_heads": 32, "d_ffn": 128}, 0, 400),        # G = 8, one run: 2
    ("tiny_g8_bf16", {"d_model": 128, "n_q_heads": 256, "n_kv_heads": 32, "d_ffn": 128}, 40, 660),       # 3
    ("tiny_g8_bf16", {"d_model": 128, "n_q_heads": 256, "n_kv_heads": 32, "d_ffn": 128}, 1, 1203),       # 5
    ("tiny_gqa_fp32", {"d_model": 128, "n_q_heads": 128, "n_kv_heads": 32, "d_ffn": 128}, 5, 700),       # G = 4: 3
    ("tiny_gqa_fp32", {"d_model": 128, "n_q_heads": 256, "n_kv_heads": 32, "d_ffn": 128}, 17, 300),      # G = 8: 3
    # walks that start at many places (42): a start's few tiles fill groups of 1, 2, 4, 8 and 16
    ("tiny_gqa_bf16", {"d_model": 1600, "n_q_heads": 25, "n_kv_heads": 25, "d_ffn": 672, "vocab": 2000}, 0, 11),
    ("tiny_gqa_bf16", {"d_model": 1600, "n_q_heads": 25, "n_kv_heads": 25, "d_ffn": 672, "vocab": 2000}, 3, 61),
    ("tiny_gqa_bf16", {"d_model": 1600, "n_q_heads": 25, "n_kv_heads": 25, "d_ffn": 4320, "vocab": 2000}, 0, 300),
    ("tiny_gqa_bf16", {"d_model": 1600, "n_q_heads": 25, "n_kv_heads": 25, "d_ffn": 4320, "vocab": 2000}, 0, 1400),
    # few column tiles and a long contraction: all K slices of a tile go to workgroups of their own, 16 (two K ranges) and 8
    ("tiny_wide_bf16", {"d_ffn": 16384}, 0, 140), ("tiny_wide_bf16", {"d_ffn": 16416}, 0, 140),
]


def _models(shape, max_ctx):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_17375_amd as A
    from paper_2410_17375_amd.harness import load_model
    store = WeightStore(shape)
    out = []
    for _ in range(2):
        m = load_model(shape, max_ctx, store=store)
        m.set_option(A.OPT_KEEP_LOGITS, 1)
        out.append(m)
    return out


def _bits(x):
    return np.ascontiguousarray(x, dtype=np.float32).view(np.uint32)


@pytest.mark.parametrize("name,over,before,n", CASES)
def test_prefill_pass_equals_short_passes(name, over, before, n):
    shape = SHAPES[name].with_(**over)
    total = before + n
    a, b = _models(shape, total + 40)
    toks = prompt_tokens(31, total + 16, shape.vocab)
    for m in (a, b):
        for s in range(0, before, 8):
            m.prefill(toks[s:min(s + 8, before)])
    group = 16 if shape.dtype == "fp32" else 8
    tail = (n - 1) % group + 1
    nxt = a.prefill(toks[before:total])                    # one prefill pass (or two)
    for s in range(before, total, group):
        ref = b.prefill(toks[s:min(s + group, total)])
    assert a.kv_len() == b.kv_len() == total and nxt == ref
    for layer in range(shape.n_layers):
        for which in (0, 1):
            assert np.array_equal(_bits(a.get_kv(layer, which, 0, total)), _bits(b.get_kv(layer, which, 0, total))), (layer, which)
    assert np.array_equal(a.get_greedy(tail), b.get_greedy(tail))
    assert np.array_equal(_bits(a.get_logits(tail)), _bits(b.get_logits(tail)))
    with pytest.raises(Exception):
        a.get_logits(tail + 1)
    window = toks[total:total + 9]
    res = []
    for m in (a, b):
        res.append((m.verify(total, window), _bits(m.get_logits(9))))
    assert res[0][0] == res[1][0] and np.array_equal(res[0][1], res[1][1])
    for pos in range(total, before, -1):                   # the model's own token is recorded for every position
        for m in (a, b):
            m.kv_rollback(pos)
        assert a.get_next() == b.get_next(), pos
    a.free()
    b.free()


def test_prefill_pass_into_second_sequence_and_stage_timing():
    import paper_2410_17375_amd as A
    from paper_2410_17375_amd.harness import load_model
    shape = SHAPES["tiny_gqa128_bf16"]
    store = WeightStore(shape)
    ms = [load_model(shape, 200, store=store, max_seqs=3) for _ in range(2)]
    toks = prompt_tokens(32, 120, shape.vocab)
    ms[1].set_option(A.OPT_TIME_STAGE, A.STAGES["qkv"])     # a timed stage is one of the verify pass
    for m in ms:
        m.seq_prefill(1, toks[:90])
        m.seq_prefill(2, toks[30:120])
    assert ms[1].stage_time()[1] == 2 * shape.n_layers * 12   # 90 tokens are 12 passes of at most 8
    for seq in (1, 2):
        assert ms[0].seq_len(seq) == 90 and ms[0].seq_get_next(seq) == ms[1].seq_get_next(seq)
        for which in (0, 1):
            assert np.array_equal(ms[0].seq_get_kv(seq, 1, which, 0, 90), ms[1].seq_get_kv(seq, 1, which, 0, 90))
    assert ms[0].seq_len(0) == 0 and ms[0].last_pass_ms() > 0
    for m in ms:
        m.free()


@pytest.mark.parametrize("max_k,n", [(7, 30721), (5, 32769), (3, 2050), (13, 61)])
def test_last_group_of_rows_is_kept_whole_for_any_max_k(max_k, n):
    """A long prompt goes through in stretches; its last group of rows, the last (n - 1) % group + 1 with groups of max_k,
    is in one of them."""
    import paper_2410_17375_amd as A
    from paper_2410_17375_amd.harness import load_model
    shape = SHAPES["tiny_draft"]
    store = WeightStore(shape)
    a, b = (load_model(shape, n + 20, max_k=max_k, store=store) for _ in range(2))
    toks = prompt_tokens(33, n, shape.vocab)
    rows = (n - 1) % max_k + 1
    for m in (a, b):
        m.set_option(A.OPT_KEEP_LOGITS, 1)
    nxt = a.prefill(toks)
    b.prefill(toks[:n - rows])
    assert b.prefill(toks[n - rows:]) == nxt               # at most max_k tokens: one verify pass
    assert np.array_equal(a.get_greedy(rows), b.get_greedy(rows))
    assert np.array_equal(_bits(a.get_logits(rows)), _bits(b.get_logits(rows)))
    a.free()
    b.free()


def test_rolled_back_rows_without_a_value_do_not_reach_rows_before_their_block():
    """A float32 cache may hold rolled-back rows that are not numbers.  A key block that no row of a pass sees is not
    multiplied, be the block before it visible or not; the cache's blocks are 16 keys and the unit's steps two of them."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_17375_amd as A
    shape = SHAPES["tiny_gqa_fp32"]
    store = WeightStore(shape)
    bad = 7
    embed = np.array(store.bits("embed", None), copy=True)
    embed[bad] = np.inf                                   # its keys and values are not numbers
    toks = prompt_tokens(34, 100, shape.vocab)
    toks[toks == bad] = bad + 1
    seen = []
    for poison in (False, True):
        m = A.Model(n_layers=shape.n_layers, d_model=shape.d_model, n_q_heads=shape.n_q_heads, n_kv_heads=shape.n_kv_heads,
                    head_dim=shape.head_dim, d_ffn=shape.d_ffn, vocab=shape.vocab, max_ctx=4200, dtype=A.DTYPE_FP32,
                    rope_theta=shape.rope_theta, rms_eps=shape.rms_eps)      # runs of two blocks, chunks of 64 keys
        for layer in [None] + list(range(shape.n_layers)):
            for name in GLOBAL_TENSORS if layer is None else LAYER_TENSORS:
                m.set_tensor(name, layer, embed if name == "embed" else store.bits(name, layer))
        m.finalize()
        m.set_option(A.OPT_KEEP_LOGITS, 1)
        m.prefill(toks[:80])
        if poison:
            m.prefill(np.full(10, bad, dtype=np.int32))   # positions 80 .. 89
            assert not np.isfinite(m.get_kv(1, 1, 80, 10)).any()
            with pytest.raises(A.AmusdError) as e:        # logits that are not numbers give no token to go on with
                m.draft_step()
            assert e.value.code == -5 and m.kv_len() == 90
        m.kv_rollback(60)
        m.prefill(toks[60:80])                            # a prefill pass: rows 60 .. 75 and 76 .. 79
        got = [_bits(m.get_logits(4))]
        m.kv_rollback(64)
        m.set_next(int(toks[64]))
        m.verify(64, toks[64:72])
        got.append(_bits(m.get_logits(8)))
        seen.append(got)
        m.free()
    assert np.isfinite(seen[0][0].view(np.float32)).all() and np.isfinite(seen[0][1].view(np.float32)).all()
    assert np.array_equal(seen[0][1], seen[1][1])         # the verify pass
    assert np.array_equal(seen[0][0], seen[1][0])         # the prefill pass


@pytest.mark.parametrize("name,over,before,n", [("tiny_gqa_bf16", {}, 7, 300), ("tiny_gqa_fp32", {}, 0, 70),
                                                ("one_layer_8b_width_bf16", {"vocab": 4096}, 0, 45)])
def test_prompts_without_the_workspace(name, over, before, n):
    """What a model does that has no memory for the workspace: the same through verify passes; and back again."""
    import paper_2410_17375_amd as A
    shape = SHAPES[name].with_(**over)
    m, other = _models(shape, before + n + 8)
    other.free()
    toks = prompt_tokens(35, before + n, shape.vocab)
    if before:
        m.prefill(toks[:before])
    held = m.prefill_workspace_bytes()
    assert held > 0
    tail = (n - 1) % (16 if shape.dtype == "fp32" else 8) + 1
    seen = []
    for on in (1, 0, 0, 1):
        m.set_option(A.OPT_PREFILL_WORKSPACE, on)
        assert m.prefill_workspace_bytes() == (held if on else 0)
        m.kv_rollback(before)
        nxt = m.prefill(toks[before:])
        seen.append([np.array([nxt]), m.get_greedy(tail), _bits(m.get_logits(tail))] +
                    [_bits(m.get_kv(layer, which, 0, before + n)) for layer in range(shape.n_layers) for which in (0, 1)])
    for other in seen[1:]:
        assert all(np.array_equal(x, y) for x, y in zip(seen[0], other))
    m.free()


@pytest.mark.parametrize("name", ["tiny_gqa_bf16", "tiny_gqa_fp32"])
def test_workspace_holds_no_more_than_its_buffers(name):
    s = SHAPES[name]
    m, other = _models(s, 360)
    other.free()
    cap, units = 384, 256 // s.n_kv_heads                  # rows in whole blocks of 128; chunks that a full context is cut into at most
    runs, keys = 8 // s.group, 16 if s.dtype == "fp32" else 32
    chunks = -(-360 // (runs * keys * -(-360 // (units * runs * keys))))
    rows = 4 * (2 * s.d_model + s.q_dim + s.d_ffn) + 4 * s.q_dim + s.d_model // 4 + 4      # activations, queries, sums of squares
    qkv, lm = -(-(s.q_dim + 2 * s.kv_dim) // 256) * 16, -(-s.vocab // 256) * 16              # column tiles, in groups of 16
    sums = 16 * cap * max(qkv, -(-s.d_model // 256) * 16) * 64
    expect = cap * rows + cap // 16 * s.n_kv_heads * chunks * s.group * 16 * (s.head_dim + 4) * 4 + min(sums, 64 << 20) + 4 * 4096 + 4 * cap * lm
    assert m.prefill_workspace_bytes() <= expect + 20 * 4096       # alignment, and the tile orders
    m.free()


def test_a_model_that_needs_the_memory_gets_an_idle_models_workspace():
    """Two models that fit the card fit it in any order of loading and prompting, whatever workspace the first one took."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_17375_amd as A
    from paper_2410_17375_amd.harness import load_model
    big, small = SHAPES["one_layer_8b_width_bf16"].with_(vocab=16000), SHAPES["tiny_gqa_bf16"]
    first = load_model(big, 2200)
    toks = prompt_tokens(36, 90, big.vocab)
    nxt = first.prefill(toks)
    held = first.prefill_workspace_bytes()
    assert held > 400 << 20
    fill = []                                              # the card is filled but for a gigabyte
    while torch.cuda.mem_get_info()[0] > (3 << 29) + (1 << 30):
        fill.append(torch.empty(min(torch.cuda.mem_get_info()[0] - (1 << 30), 16 << 30), dtype=torch.uint8, device="cuda"))
    left = torch.cuda.mem_get_info()[0]
    fill.append(torch.empty(left - (1 << 30), dtype=torch.uint8, device="cuda"))
    seqs = 5 * (1 << 28) // (4096 * 1024)                  # 1.25 GB of cache: a kilobyte a position
    try:
        second = load_model(small, 4096, max_seqs=seqs)
        assert first.prefill_workspace_bytes() == 0
        first.kv_rollback(0)
        assert first.prefill(toks) == nxt                  # through verify passes
        assert second.prefill(toks % small.vocab) >= 0
        second.free()
        first.set_option(A.OPT_PREFILL_WORKSPACE, 1)
        assert first.prefill_workspace_bytes() == held
        first.kv_rollback(0)
        assert first.prefill(toks) == nxt
        first.free()
    finally:
        fill.clear()
        torch.cuda.empty_cache()


def test_short_prompts_are_not_slower_than_verify_passes_where_walks_start_at_many_places():
    """Width 4672: slices of 18 and 19 K blocks, 256 starts of one or two tiles.  Filled up to groups of 16 they made twelve
    tokens take 1.34 times as long as in two verify passes; measured 0.70 since groups are filled to their own size."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import time
    import paper_2410_17375_amd as A
    d, heads, ffn, vocab = 4672, 73, 4672, 16000
    m = A.Model(n_layers=2, d_model=d, n_q_heads=heads, n_kv_heads=heads, head_dim=64, d_ffn=ffn, vocab=vocab, max_ctx=256,
                dtype=A.DTYPE_BF16, rope_theta=500000.0, rms_eps=1e-5)
    gen = torch.Generator(device="cuda").manual_seed(1)
    dims = {"embed": (vocab, d), "lm_head": (vocab, d), "wg": (ffn, d), "wu": (ffn, d), "wd": (d, ffn)}
    for layer in [None, 0, 1]:
        for name in GLOBAL_TENSORS if layer is None else LAYER_TENSORS:
            w = torch.randn(dims.get(name, (d,) if "norm" in name else (d, d)), generator=gen, device="cuda").mul_(0.02).to(torch.bfloat16)
            torch.cuda.synchronize()
            m.set_tensor(name, layer, w.data_ptr(), on_device=True)
    m.finalize()
    toks = prompt_tokens(37, 12, vocab)
    times = {}
    for on in (1, 0, 1, 0):
        m.set_option(A.OPT_PREFILL_WORKSPACE, on)
        for _ in range(20):
            m.kv_rollback(0)
            t0 = time.perf_counter()
            m.prefill(toks)
            times.setdefault(on, []).append(time.perf_counter() - t0)
    m.free()
    assert np.median(times[1]) < 1.1 * np.median(times[0]), {k: float(np.median(v)) for k, v in times.items()}
