"""Attention over tiles of (row, head) pairs, which verify passes of few rows and of several sequences take, against the same rows of
a prompt pass (another kernel), bit for bit: groups of 4 and 8 heads, one to eight tiles, runs of one to five key blocks that end in
a step of one, chunks whose second run has no visible key."""
import numpy as np
import pytest

from workload import SHAPES, WeightStore, prompt_tokens

pytestmark = pytest.mark.gpu


def _heads(kv_heads, group, head_dim):
    return {"d_model": 128, "d_ffn": 128, "n_q_heads": kv_heads * group, "n_kv_heads": kv_heads, "head_dim": head_dim}


# (shape, overrides, tokens of each sequence behind the pass, rows of each): 3 and 5 kv heads leave units of eight unfilled
@pytest.mark.parametrize("name,over,lens,rows", [
    ("tiny_gqa_bf16", _heads(8, 4, 64), (40,), (1,)), ("tiny_gqa_bf16", _heads(8, 4, 64), (1096, 72, 528), (1, 4, 3)),
    ("tiny_gqa_bf16", _heads(3, 4, 64), (72, 96, 40, 64), (5, 1, 8, 2)), ("tiny_gqa_bf16", _heads(32, 4, 64), (1944,), (4,)),
    ("tiny_gqa_bf16", _heads(8, 4, 64), (520,), (8,)), ("tiny_gqa_bf16", _heads(16, 4, 128), (1944, 32), (2, 3)),
    ("tiny_gqa_bf16", _heads(8, 4, 128), (1080,), (8,)), ("tiny_gqa_bf16", _heads(5, 4, 128), (488, 904, 1000, 968), (1, 2, 8, 5)),
    ("tiny_gqa_bf16", _heads(16, 8, 64), (1944,), (2,)), ("tiny_gqa_bf16", _heads(4, 8, 64), (200, 264), (8, 8)),
    ("tiny_gqa_bf16", _heads(8, 8, 128), (1880, 600, 72), (1, 7, 2)), ("tiny_gqa_fp32", _heads(8, 4, 64), (480, 496), (1, 9)),
    ("tiny_gqa_fp32", _heads(16, 4, 64), (1920,), (7,)), ("tiny_gqa_fp32", _heads(3, 8, 64), (208, 32, 112), (4, 11, 1)),
    ("tiny_gqa_fp32", _heads(32, 4, 128), (912,), (2,)), ("tiny_gqa_fp32", _heads(8, 8, 128), (960, 512), (3, 13)),
])
def test_pairs_equal_prompt_rows(name, over, lens, rows):
    _compare(name, over, lens, rows, max(lens) + 40)


# few keys, which a workgroup has all of: up to eight runs and 64 KB of them, one more; runs of several blocks (long contexts that are not
# used); groups of 1 and 2, one chunk and two
@pytest.mark.parametrize("name,over,lens,rows,max_ctx", [
    ("tiny_gqa_bf16", _heads(8, 4, 64), (256,), (1,), 300), ("tiny_gqa_bf16", _heads(8, 4, 64), (256, 16, 48, 136), (8, 1, 2, 5), 300),
    ("tiny_gqa_bf16", _heads(8, 4, 64), (264, 16), (8, 2), 300), ("tiny_gqa_bf16", _heads(3, 8, 64), (256, 72), (1, 8), 300),
    ("tiny_gqa_bf16", _heads(16, 4, 64), (200, 256), (8, 7), 4000), ("tiny_gqa_bf16", _heads(8, 4, 128), (128, 64), (8, 3), 200),
    ("tiny_gqa_bf16", _heads(8, 4, 128), (136,), (1,), 200), ("tiny_gqa_bf16", _heads(16, 8, 128), (128, 48), (3, 8), 3000),
    ("tiny_gqa_fp32", _heads(8, 4, 64), (128, 32), (13, 3), 200), ("tiny_gqa_fp32", _heads(8, 8, 64), (128, 64), (2, 14), 2000),
    ("tiny_gqa_fp32", _heads(5, 4, 128), (64, 32), (9, 1), 200), ("tiny_gqa_fp32", _heads(8, 8, 128), (64,), (16,), 700),
    ("tiny_gqa_fp32", _heads(4, 1, 64), (128, 112), (7, 9), 200), ("tiny_gqa_fp32", _heads(4, 1, 64), (144,), (16,), 200),
    ("tiny_gqa_fp32", _heads(4, 2, 128), (64, 48), (7, 9), 200), ("tiny_gqa_bf16", _heads(4, 1, 128), (256, 40), (8, 8), 300),
    ("tiny_gqa_bf16", _heads(4, 2, 64), (128, 40), (8, 1), 300),
])
def test_few_keys_equal_prompt_rows(name, over, lens, rows, max_ctx):
    _compare(name, over, lens, rows, max_ctx)


def _compare(name, over, lens, rows, max_ctx):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_17375_amd as A
    from paper_2410_17375_amd.harness import load_model
    shape = SHAPES[name].with_(**over)
    group = 16 if shape.dtype == "fp32" else 8               # rows whose logits a prompt leaves
    m = load_model(shape, max_ctx, store=WeightStore(shape), max_seqs=len(lens))
    m.set_option(A.OPT_KEEP_LOGITS, 1)
    want, new = [], []
    for i, (n, k) in enumerate(zip(lens, rows)):
        assert n % 8 == 0 and n > group and (n - 1) % group + 1 >= k
        toks = prompt_tokens(50 + i, n, shape.vocab)
        m.seq_prefill(i, toks)
        want.append(m.get_logits((n - 1) % group + 1)[-k:].copy())
        new.append(toks[n - k:])
        m.seq_rollback(i, n - k)
    m.verify_batch(list(range(len(lens))), [n - k for n, k in zip(lens, rows)], new)
    got = m.get_logits(sum(rows))
    assert np.isfinite(got).all()
    assert np.array_equal(got.view(np.uint32), np.concatenate(want).view(np.uint32))
    m.free()
