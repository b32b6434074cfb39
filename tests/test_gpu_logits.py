"""Logits on the host: arrays of the caller's own, ordinary memory, which hold what their pass computed for as long as they live."""
import ctypes as C
import re

import numpy as np
import pytest

from workload import SHAPES, WeightStore, prompt_tokens

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,rows,vocab", [("tiny_draft", 1, 4096), ("tiny_gqa_bf16", 16, 4096), ("tiny_gqa_bf16", 16, 4112)])
def test_logits_are_the_callers(name, rows, vocab):      # 16 KB and 256 KB
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_17375_amd as A
    from paper_2410_17375_amd.harness import load_model
    shape = SHAPES[name].with_(vocab=vocab)
    g = load_model(shape, 64, store=WeightStore(shape))
    g.set_option(A.OPT_KEEP_LOGITS, 1)
    toks = prompt_tokens(3, 64, vocab)
    g.prefill(toks[:20])

    def copied(n):
        out = np.empty((n, vocab), dtype=np.float32)
        assert A.lib.amusd_get_logits(g._h, out.ctypes.data_as(C.POINTER(C.c_float)), n) == 0
        return out

    kept = []
    for r in range(4):
        g.kv_rollback(20)
        g.set_next(int(toks[20 + r]))
        g.verify(20, toks[20 + r:20 + r + rows])
        want = copied(rows)
        kept.append((g.get_logits(rows), want, copied(rows)))
        for got, want, again in kept:
            assert np.array_equal(got, want) and np.array_equal(want, again)
        assert not np.array_equal(kept[0][0], kept[-1][0]) or r == 0
    kept[0][0][0, 0] = 5.0                                   # writable, and nobody else's
    assert kept[1][0][0, 0] != 5.0
    own = kept[1][0]
    del kept[1], got
    assert own.base is None and own.flags.owndata
    own.resize((rows + 1, vocab), refcheck=False)            # as any array that owns its data
    # .. and a child process has its copy of (memory that the GPU's driver maps, it has not)
    here, flags = False, None
    for line in open("/proc/self/smaps"):
        span = re.match(r"([0-9a-f]+)-([0-9a-f]+) ", line)
        if span:
            here = int(span.group(1), 16) <= kept[0][0].ctypes.data < int(span.group(2), 16)
        elif here and line.startswith("VmFlags"):
            flags = line.split()[1:]
    assert flags and "dc" not in flags
    with pytest.raises(A.AmusdError):
        g.get_logits(rows + 1)
    with pytest.raises(A.AmusdError):
        g.get_logits(0)
    last = kept[-1][0].copy(), kept[-1][0]
    g.free()
    assert kept[0][0][0, 0] == 5.0 and np.array_equal(*last)
