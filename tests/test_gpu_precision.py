"""What the sums of a pass keep: inputs on which a sum with fewer places, or in another unit, would give something else altogether."""
import numpy as np
import pytest

from workload import SHAPES, WeightStore, prompt_tokens
from workload.tensors import bf16_bits_to_f32, round_to_bf16_bits

pytestmark = pytest.mark.gpu


def _models_of(shape, max_ctx, store, n=1):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_17375_amd as A
    from paper_2410_17375_amd.harness import load_model
    ms = [load_model(shape, max_ctx, store=store) for _ in range(n)]
    for m in ms:
        m.set_option(A.OPT_KEEP_LOGITS, 1)
    return ms


class _Cancelling(WeightStore):
    """Layers that add nothing.  In every K block of the LM head one column's products are 4096, 4096, -4096, -4096 in turn, two more
    cancel in their high halves, and what is left is the low half of one activation, 2^-14: less than half a unit in the last place
    of a sum that holds 4096."""

    def bits(self, name, layer=None):
        b = super().bits(name, layer)
        if name in ("wo", "wd"):
            return np.zeros_like(b)
        x = np.ones(b.shape, dtype=np.float32)
        col = np.arange(self.shape.d_model)
        if name == "embed":
            x[:, col % 32 == 5] = 1 + 2.0 ** -7
            x[:, col % 32 == 11] = 1 + 2.0 ** -6
        elif name == "final_norm":
            x[col % 32 == 5] = 1 + 2.0 ** -7                 # times the embedding: 1 + 2^-6 and the low half 2^-14
        elif name == "lm_head":
            x[:] = 0
            big = np.where(col // 32 % 4 < 2, 4096.0, -4096.0)
            x[:, col % 32 == 5], x[:, col % 32 == 11] = 1, -1
            x[:, col % 32 == 20] = big[col % 32 == 20]
            x *= 2.0 ** (np.arange(len(x)) % 5)[:, None]
        else:
            return b
        return round_to_bf16_bits(x)


# rows: a window with both halves packed, one with a part each, prompts on the two larger workgroup shapes
@pytest.mark.parametrize("n", [3, 12, 40, 300])
def test_low_halves_are_summed_apart(n):
    shape = SHAPES["tiny_gqa_bf16"].with_(d_model=2048, vocab=16000 if n == 300 else 2048)
    m, = _models_of(shape, 320, _Cancelling(shape))
    toks = prompt_tokens(5, n + 1, shape.vocab)
    rows = n
    if n <= 16:
        m.prefill(toks[:1])
        m.set_next(int(toks[1]))
        m.verify(1, toks[1:])
    else:
        m.prefill(toks[:n])
        rows = (n - 1) % 8 + 1
    got = m.get_logits(rows)
    m.free()
    # 64 blocks of 2^-14, over the row's root mean square; float32 holds all sums exactly, the rest rounds a few times
    squares = (30 + (1 + 2.0 ** -7) ** 2 + (1 + 2.0 ** -6) ** 2) / 32
    want = 64 * 2.0 ** -14 / np.sqrt(squares + shape.rms_eps) * 2.0 ** (np.arange(shape.vocab) % 5)
    assert np.abs(got / want - 1).max() < 8 * 2.0 ** -24


class _Enormous(WeightStore):
    """Queries and keys of one direction, up to the largest that the cache's type holds: a row's score with itself is 2^31 (16-bit
    models) or 2^44 in units of log2, where a float's last place is worth 256 and more."""

    def bits(self, name, layer=None):
        if name not in ("wq", "wk"):
            return super().bits(name, layer)
        w = bf16_bits_to_f32(b) if (b := super().bits("wk", layer)).dtype == np.uint16 else b
        w = np.tile(w.reshape(self.shape.n_kv_heads, 1, self.shape.head_dim, -1), (1, self.shape.group if name == "wq" else 1, 1, 1))
        w = (w * np.float32(2.0 ** 15 if self.shape.dtype == "bf16" else 2.0 ** 20)).reshape(-1, self.shape.d_model)
        return round_to_bf16_bits(w) if self.shape.dtype == "bf16" else w


# groups of 2, 4, 8 and 1, both widths of a head; keys walked whole and, behind a context, in stretches
@pytest.mark.parametrize("name,ctx,n", [("tiny_gqa_bf16", 0, 60), ("tiny_gqa128_bf16", 0, 60), ("tiny_gqa128_bf16", 700, 20),
                                        ("tiny_g8_bf16", 0, 60), ("tiny_gqa_fp32", 0, 60), ("tiny_verify", 0, 60)])
def test_enormous_scores(name, ctx, n):
    from oracle import Decoder
    shape = SHAPES[name]
    store = _Enormous(shape)
    toks = prompt_tokens(6, ctx + n, shape.vocab)
    group = 16 if shape.dtype == "fp32" else 8
    rows = (n - 1) % group + 1
    out = []
    for m, piece in zip(_models_of(shape, ctx + n + 16, store, 2), (n, group)):     # one prefill pass; verify passes
        if ctx:
            m.prefill(toks[:ctx])
        for s in range(ctx, ctx + n, piece):
            m.prefill(toks[s:min(s + piece, ctx + n)])
        out.append(m.get_logits(rows))
        m.free()
    assert np.array_equal(out[0].view(np.uint32), out[1].view(np.uint32))
    # every weight is 0 or 1 and an output is one value row: what is left is the tolerance of any pass
    want = np.asarray(Decoder(shape, store, ctx + n).rows(toks, logits_from=ctx + n - rows))
    assert np.abs(want - out[0]).max() < (2e-5 if shape.dtype == "fp32" else 3e-2)


class _OneAmongMany(WeightStore):
    """Token 1 stands out of a context of token 2 by 29 in units of log2: 16 of the others, a chunk's, are less than half a unit in
    the last place of a float that holds the one, all of them 2^-17.  Its value is 1, theirs is 0; the output goes to the logits."""

    def bits(self, name, layer=None):
        s = self.shape
        x = np.zeros_like(super().bits(name, layer))
        if name.startswith("norm") or name == "final_norm":
            x[:] = 1
        elif name == "embed":
            x[1, 0] = x[2, 1] = 16                           # 16 again behind the norm, of 256 columns
        elif name == "wq":
            x[31::64, :2] = 8 / 16
        elif name == "wk":
            x[31::64, 0] = 29.0 / np.log2(np.e) / 16
        elif name == "wv":
            x[0::64, 0] = 1 / 16
        elif name == "wo":
            x[2, 0] = 1
        elif name == "lm_head":
            x[:, 2] = 2.0 ** (np.arange(len(x)) % 4)
        return x


# groups of 8 (chunks of one run), 4 and 1 (of more keys: fewer)
@pytest.mark.parametrize("heads,kv_heads,ctx", [(8, 1, 4080), (4, 1, 4080), (1, 1, 4080)])
def test_denominators_of_many_chunks(heads, kv_heads, ctx):
    from oracle import Decoder
    # one pair of columns that the rotation leaves alone
    shape = SHAPES["tiny_draft"].with_(d_model=256, n_q_heads=heads, n_kv_heads=kv_heads, d_ffn=16, vocab=64, rope_theta=1e30)
    store = _OneAmongMany(shape)
    toks = np.full(ctx + 16, 2, dtype=np.int32)
    toks[0] = 1
    out = []
    for m, pieces in zip(_models_of(shape, ctx + 16, store, 3), ([ctx + 16], [ctx - 16, ctx + 16], [ctx, ctx + 16])):
        start = 0
        for stop in pieces:                                  # keys walked whole; behind a context in stretches; a verify pass
            m.prefill(toks[start:stop])
            start = stop
        out.append(m.get_logits(16))
        m.free()
    for o in out[1:]:
        assert np.array_equal(out[0].view(np.uint32), o.view(np.uint32))
    want = np.asarray(Decoder(shape, store, ctx + 16).rows(toks, logits_from=ctx))
    # 1 over the denominator, and what follows it: some ten roundings
    assert np.abs(out[0] / want - 1).max() < 10 * 2.0 ** -24
