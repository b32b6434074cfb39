"""The ways of the logits to the caller's memory: with the pass (up to 256 KB), or when asked for, in chunks of 32 KB through a pinned
block of at most 4 MB.  Rows of a pass against the same rows of passes of one, bit for bit, at sizes around those limits."""
import ctypes as C

import numpy as np
import pytest

from workload import SHAPES, WeightStore, prompt_tokens

pytestmark = pytest.mark.gpu


# vocabulary: 16 rows in 256 KB, in one 16-column tile more, in 32 chunks and a half, in 4 MB, past it by a tile of 16 rows
@pytest.mark.parametrize("vocab", [16, 4096, 4112, 16640, 65536, 65552])
def test_rows_arrive_whole(vocab):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_17375_amd as A
    from paper_2410_17375_amd.harness import load_model
    shape = SHAPES["tiny_gqa_bf16"].with_(vocab=vocab, n_layers=1, d_ffn=64)
    g = load_model(shape, 96, store=WeightStore(shape))
    g.set_option(A.OPT_KEEP_LOGITS, 1)
    toks = prompt_tokens(5, 80, vocab)
    g.prefill(toks[:33])

    def window(at, n):
        g.kv_rollback(at)
        g.set_next(int(toks[at]))
        g.verify(at, toks[at:at + n])

    window(33, 16)
    buf = np.full(16 * vocab + 2, 7.5, dtype=np.float32)      # 4 bytes off, with a word before and behind
    for rows in (16, 5, 1, 16):
        buf[:] = 7.5
        assert A.lib.amusd_get_logits(g._h, C.cast(buf.ctypes.data + 4, C.POINTER(C.c_float)), rows) == 0
        got = buf[1:1 + rows * vocab].reshape(rows, vocab).copy()
        assert buf[0] == 7.5 and (buf[1 + rows * vocab:] == 7.5).all()
        assert np.array_equal(got.argmax(1), g.get_greedy(rows))
        if rows == 16:
            whole = got
        assert np.array_equal(got, whole[:rows])
    g.kv_rollback(33)
    g.prefill(toks[33:33 + 40])                              # the last group of 8 of a prompt pass: rows 65 .. 72
    prompt = g.get_logits(8).copy()
    for r in (0, 7, 15):
        g.kv_rollback(33)
        if r:
            g.prefill(toks[33:33 + r])
        window(33 + r, 1)
        assert np.array_equal(g.get_logits(1)[0], whole[r])
    g.kv_rollback(33)
    g.prefill(toks[33:65])
    window(65, 8)
    assert np.array_equal(g.get_logits(8), prompt)
    g.set_option(A.OPT_KEEP_LOGITS, 0)                       # a pass that keeps none leaves none of an earlier one either
    window(65, 1)
    with pytest.raises(A.AmusdError):
        g.get_logits(1)
    g.free()
