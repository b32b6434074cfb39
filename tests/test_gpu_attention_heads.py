"""Attention with a tile per head over runs of several blocks, which 16-bit verify passes of nine rows and more take, against the same
rows in passes of one (tiles of (row, head) pairs, another kernel), bit for bit.  tests/test_host_cpu.py checks that the passes take
the kernels that they are meant for."""
import numpy as np
import pytest

from workload import SHAPES, WeightStore, prompt_tokens

pytestmark = pytest.mark.gpu


def _heads(kv_heads, group, head_dim):
    return {"d_model": 128, "d_ffn": 128, "n_q_heads": kv_heads * group, "n_kv_heads": kv_heads, "head_dim": head_dim}


# (overrides, context of the model, blocks a run, tokens of each sequence before the window, rows of each): odd runs end in a step of one
# block, the last chunks in all of a run's blocks, in some and in none
CASES = [
    (_heads(32, 4, 64), 4000, 8, (3960,), (16,)), (_heads(32, 4, 64), 4200, 9, (4180,), (9,)), (_heads(32, 4, 64), 4200, 9, (1003,), (13,)),
    (_heads(32, 8, 64), 2040, 8, (2000,), (16,)), (_heads(32, 8, 64), 2200, 9, (2157,), (9,)), (_heads(32, 8, 64), 2500, 10, (700,), (11,)),
    (_heads(3, 4, 128), 2000, 1, (1900,), (16,)), (_heads(32, 4, 128), 1000, 2, (980,), (12,)), (_heads(32, 4, 128), 1500, 3, (1451,), (16,)),
    (_heads(32, 4, 128), 2500, 5, (2307,), (9,)),
    (_heads(16, 8, 128), 1000, 2, (984,), (16,)), (_heads(16, 8, 128), 1500, 3, (1433,), (9,)), (_heads(16, 8, 128), 2500, 5, (1801,), (13,)),
    (_heads(16, 4, 128), 1500, 3, (1440, 700), (12, 4)), (_heads(16, 8, 64), 2200, 9, (2100, 300), (14, 2)),
]


@pytest.mark.parametrize("over,max_ctx,blocks,lens,rows", CASES)
def test_heads_equal_single_rows(over, max_ctx, blocks, lens, rows):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_17375_amd as A
    from paper_2410_17375_amd.harness import load_model
    shape = SHAPES["tiny_gqa_bf16"].with_(**over)
    m = load_model(shape, max_ctx, store=WeightStore(shape), max_seqs=len(lens))
    m.set_option(A.OPT_KEEP_LOGITS, 1)
    toks = [prompt_tokens(70 + i, n + k, shape.vocab) for i, (n, k) in enumerate(zip(lens, rows))]
    want = []
    for i, n in enumerate(lens):
        m.seq_prefill(i, toks[i][:n])
        for at in range(n, len(toks[i])):
            m.seq_set_next(i, int(toks[i][at]))
            assert m.verify_batch([i], [at], [toks[i][at:at + 1]])[0][0] == 1
            want.append(m.get_logits(1)[0].copy())
        m.seq_rollback(i, n)
        m.seq_set_next(i, int(toks[i][n]))
    m.verify_batch(list(range(len(lens))), list(lens), [t[n:] for t, n in zip(toks, lens)])
    got = m.get_logits(sum(rows))
    assert np.isfinite(got).all()
    assert np.array_equal(got.view(np.uint32), np.stack(want).view(np.uint32))
    m.free()
