"""What a user of this package has it do, as cases that can be timed and checked.

A case is one call (or the few calls that belong together) through the package's
public entry points on one model: a verify window, a draft step, the same for
several sequences sharing a pass, or the prefill of a prompt.  Every case gives
the logits that the call computed besides its tokens.

Models have the shapes of `workload/shapes.py`.  "8b" with a handful of layers
and the smaller vocabulary stands for the decoder blocks of the 8B shape, which
are what a pass of that model repeats 32 times; "8b" with 32 layers and "1b" with
16 are whole models.  Weights, prompts and windows are drawn on the GPU from the
seed, in the distributions of `workload/tensors.py` and `workload/tokens.py`.
"""
import math

import numpy as np
import torch

import paper_2410_17375_amd as A
from workload import SHAPES

_MATRICES = ("wq", "wk", "wv", "wo", "wg", "wu", "wd")


def _case(name, kind, shape, layers, vocab, ctx, rows, seqs=1):
    """ctx: tokens in the cache before the call (of the longest sequence); rows: new tokens (of all sequences)."""
    c = {"kind": kind, "shape": shape, "layers": layers, "vocab": vocab, "ctx": ctx, "rows": rows, "seqs": seqs}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the tiny fp32 draft model of the parity workload: one step, nothing but launches
        _case("draft_tiny_fp32_ctx64", "draft", "tiny_draft", 1, 4096, 64, 1),
        # the draft model's step, the call that the draft process of Algorithm 1 makes most often
        _case("draft_1b_ctx512", "draft", "1b", 16, 32000, 512, 1),
        # its step for eight requests served together, at eight different lengths
        _case("draft_1b_8seqs_ctx1500", "draft", "1b", 16, 32000, 1500, 8, 8),
        # the 1B shape as a verify model: a window of five drafts
        _case("verify_1b_k5_ctx512", "verify", "1b", 16, 32000, 512, 5),
        # the headline workload: the whole 8B shape, eight drafts at context 2048
        _case("verify_8b_k8_ctx2048", "verify", "8b", 32, 128256, 2048, 8),
        # blocks of the 8B shape at long context with the largest window
        _case("verify_8b_blocks_k16_ctx16384", "verify", "8b", 4, 32000, 16384, 16),
        # four requests of different lengths with ragged windows sharing one pass
        _case("verify_8b_blocks_4seqs_13rows", "verify", "8b", 4, 32000, 3001, 13, 4),
        # a short chat turn
        _case("prefill_8b_blocks_61", "prefill", "8b", 4, 32000, 0, 61),
        # a prompt of the paper's usual size on the draft model, odd length
        _case("prefill_1b_509", "prefill", "1b", 16, 32000, 0, 509),
        # the headline context itself
        _case("prefill_8b_blocks_2048", "prefill", "8b", 4, 32000, 0, 2048),
        # a long document followed by a further turn of a conversation
        _case("prefill_8b_blocks_12288_more_4000", "prefill", "8b", 2, 32000, 12288, 4000),
        # exact-parity models are fp32
        _case("prefill_tiny_fp32_333", "prefill", "tiny_verify", 2, 4096, 0, 333),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    kind = rng.choice(("draft", "verify", "verify", "prefill", "prefill"))
    shape, layers, vocab = rng.choice((("tiny_draft", 1, 4096), ("tiny_verify", 2, 4096), ("1b", 16, 32000), ("1b", 16, 32000),
                                       ("8b", 2, 32000), ("8b", 4, 32000), ("8b", 4, 32000)))
    seqs = 1
    tiny = shape.startswith("tiny")
    if kind == "prefill":
        # from a handful of tokens to a long document; a later turn of a conversation starts behind what is cached
        rows = _log_int(rng, 17, 512 if tiny else 4000 if (shape, layers) == ("8b", 2) else 1800)
        ctx = rng.choice((0, 0, _log_int(rng, 33, 400 if tiny else 6000)))
    else:
        ctx = _log_int(rng, 33, 500 if tiny else 16384 if shape == "8b" else 4096)
        rows = 1 if kind == "draft" else rng.randint(2, 16)
        if rng.random() < 0.35 and not tiny:
            seqs = rng.randint(2, 6)
            ctx = min(ctx, 4096)
            rows = seqs if kind == "draft" else max(rows, seqs)
    return _case(None, kind, shape, layers, vocab, ctx, rows, seqs)


# ---------------------------------------------------------------- inputs
def _shape(case):
    return SHAPES[case["shape"]].with_(n_layers=case["layers"], vocab=case["vocab"])


def _dims(s, name):
    d, F = s.d_model, s.d_ffn
    return {"embed": (s.vocab, d), "lm_head": (s.vocab, d), "final_norm": (d,), "wq": (s.q_dim, d), "wk": (s.kv_dim, d),
            "wv": (s.kv_dim, d), "wo": (d, s.q_dim), "wg": (F, d), "wu": (F, d), "wd": (d, F), "norm_attn": (d,),
            "norm_mlp": (d,)}[name]


def _weights(s, seed):
    """(name, layer, tensor) in a fixed order, each in the model's storage type on the GPU."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.float32 if s.dtype == "fp32" else torch.bfloat16
    for layer in [None] + list(range(s.n_layers)):
        for name in ("embed", "lm_head", "final_norm") if layer is None else _MATRICES + ("norm_attn", "norm_mlp"):
            w = torch.randn(_dims(s, name), generator=gen, device="cuda", dtype=torch.float32).mul_(0.02)
            if "norm" in name:
                w.add_(1.0)
            yield name, layer, w.to(dt)


def _lengths(case, seed):
    """Cached tokens and new tokens of each sequence; the first is the longest."""
    rng, n = np.random.default_rng([seed, 1]), case["seqs"]
    ctx = [case["ctx"]] + [int(x) for x in rng.integers(max(1, case["ctx"] // 4), case["ctx"] + 1, size=n - 1)]
    if n == 1:
        return ctx, [case["rows"]]
    cuts = np.sort(rng.choice(np.arange(1, case["rows"]), size=n - 1, replace=False)) if case["rows"] > n else np.arange(1, n)
    return ctx, [int(x) for x in np.diff(np.concatenate([[0], cuts, [case["rows"]]]))]


def _tokens(case, seed):
    """For each sequence the tokens already cached and the new ones."""
    rng = np.random.default_rng([seed, 2])
    ctx, new = _lengths(case, seed)
    return [(rng.integers(0, case["vocab"], size=c).astype(np.int32), rng.integers(0, case["vocab"], size=k).astype(np.int32))
            for c, k in zip(ctx, new)]


def prepare(case, seed):
    s = _shape(case)
    toks = _tokens(case, seed)
    stream = torch.cuda.Stream()
    longest = max(len(c) + len(n) for c, n in toks)
    model = A.Model(n_layers=s.n_layers, d_model=s.d_model, n_q_heads=s.n_q_heads, n_kv_heads=s.n_kv_heads,
                    head_dim=s.head_dim, d_ffn=s.d_ffn, vocab=s.vocab, max_ctx=longest + 64,
                    dtype=A.DTYPE_FP32 if s.dtype == "fp32" else A.DTYPE_BF16, rope_theta=s.rope_theta, rms_eps=s.rms_eps,
                    max_seqs=case["seqs"], stream=stream.cuda_stream)
    for name, layer, w in _weights(s, seed):
        torch.cuda.synchronize()
        model.set_tensor(name, layer, w.data_ptr(), on_device=True)
    model.finalize()
    for i, (cached, _) in enumerate(toks):
        if len(cached):
            model.seq_prefill(i, cached)
    model.set_option(A.OPT_KEEP_LOGITS, 1)
    return {"kind": case["kind"], "model": model, "stream": stream, "ids": list(range(len(toks))),
            "ctx": [len(c) for c, _ in toks], "new": [n for _, n in toks]}


def _kept_rows(case):
    """Rows whose logits a call leaves: all of a pass; of a prefill, those of its last group of 8 (fp32: 16) tokens."""
    if case["kind"] != "prefill":
        return case["rows"]
    group = 16 if SHAPES[case["shape"]].dtype == "fp32" else 8
    return (case["rows"] - 1) % group + 1


# ---------------------------------------------------------------- one pass
def run(state):
    m, ctx, new, ids = state["model"], state["ctx"], state["new"], state["ids"]
    if state["kind"] == "prefill":
        m.kv_rollback(ctx[0])
        tokens = [m.prefill(new[0])]
        group = 16 if m.cfg.dtype == A.DTYPE_FP32 else 8
        rows = (len(new[0]) - 1) % group + 1
    else:
        # the token that each sequence is known to go on with is the first of its new ones, as in the decoding loops
        for i in ids:
            m.seq_rollback(i, ctx[i])
            m.seq_set_next(i, int(new[i][0]))
        rows = sum(len(n) for n in new)
        if state["kind"] == "draft":
            tokens = m.draft_step_batch(ids) if len(ids) > 1 else [m.draft_step()]
        elif len(ids) > 1:
            tokens = np.concatenate(m.verify_batch(ids, ctx, new))
        else:
            tokens = m.verify(ctx[0], new[0])
    return {"logits": m.get_logits(rows), "tokens": np.concatenate([np.asarray(tokens, dtype=np.int32), m.get_greedy(rows)])}


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    s = _shape(case)
    e = s.weight_elem_bytes
    n, kv = case["rows"], s.kv_dim
    ctx, new = _lengths(case, 0)
    ctx = ctx if case["seqs"] == 1 else [case["ctx"]] + [(case["ctx"] // 4 + case["ctx"]) // 2] * (case["seqs"] - 1)   # drawn: their mean
    new = new if case["seqs"] == 1 else [n / case["seqs"]] * case["seqs"]
    per_layer = s.d_model * (s.q_dim + 2 * kv) + s.q_dim * s.d_model + 3 * s.d_model * s.d_ffn
    nbytes = s.n_params_streamed() * e                                    # every weight read once
    nbytes += s.n_layers * 2 * kv * e * (sum(ctx) + n)                    # the cache read, the new rows written
    nbytes += n * s.d_model * e + _kept_rows(case) * s.vocab * 4          # embedding rows in, logits out
    flops = 2.0 * n * (s.n_layers * per_layer + s.vocab * s.d_model)
    # scores and values: a row sees what is cached and the rows up to itself
    flops += s.n_layers * 4.0 * s.q_dim * sum(k * c + k * (k + 1) / 2 for c, k in zip(ctx, new))
    return {"bytes": int(nbytes), "flops": int(flops)}


def tolerance(case):
    """bf16 models: the cache is held in half precision, activations enter the contractions with about 16 mantissa bits;
    fp32 models: sums in 32 bits.  About four times the distance from exact() that was measured (2.5e-3 for the 32-layer
    model, 6e-4 to 9.6e-4 for the others, 1e-7 to 4e-7 in fp32).  Tokens are arg-max values over random logits: a few of a
    pass's rows may be near ties."""
    if SHAPES[case["shape"]].dtype == "fp32":
        return {"rel": 2e-6, "differ": 0.1}
    return {"rel": 1e-2 if case["layers"] > 16 else 4e-3, "differ": 0.25}


# ---------------------------------------------------------------- the same in 64 bits
def _norm(x, gain, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * gain


def _rotate(v, cos, sin):
    """v: [n, heads, hd], pairs (i, i + hd/2)."""
    h = v.shape[-1] // 2
    a, b = v[..., :h], v[..., h:]
    return torch.cat([a * cos - b * sin, a * sin + b * cos], -1)


def _attention(q, k, v):
    """q, k, v: [n, hd] of one head; row j sees keys 0..j.  A few thousand rows at a time."""
    n = q.shape[0]
    out = torch.empty_like(q)
    for r0 in range(0, n, 2048):
        r1 = min(n, r0 + 2048)
        sc = (q[r0:r1] @ k[:r1].T) / math.sqrt(q.shape[1])
        sc.masked_fill_(torch.arange(r1, device="cuda")[None, :] > torch.arange(r0, r1, device="cuda")[:, None], float("-inf"))
        out[r0:r1] = torch.softmax(sc, -1) @ v[:r1]
    return out


def exact(case, seed):
    """The logits in float64, every sequence from its first token on."""
    s = _shape(case)
    toks = _tokens(case, seed)
    full = [torch.from_numpy(np.concatenate([c, n]).astype(np.int64)).cuda() for c, n in toks]
    keep = [len(n) for _, n in toks] if case["kind"] != "prefill" else [_kept_rows(case)]
    hd, group = s.head_dim, s.n_q_heads // s.n_kv_heads
    inv = torch.tensor(s.rope_theta, dtype=torch.float64) ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64) / hd)
    ang = [torch.arange(len(t), dtype=torch.float64)[:, None] * inv for t in full]
    rot = [(torch.cos(a).cuda()[:, None, :], torch.sin(a).cuda()[:, None, :]) for a in ang]
    w, xs, head = {}, None, None
    for name, layer, t in _weights(s, seed):
        if name == "embed":
            xs = [t[ids].double() for ids in full]
        elif name in ("lm_head", "final_norm"):
            head = (head or ()) + (t.double(),)
        else:
            w[name] = t.double()
        if name != "norm_mlp":
            continue
        for i, x in enumerate(xs):
            n = x.shape[0]
            a = _norm(x, w["norm_attn"], s.rms_eps)
            q = _rotate((a @ w["wq"].T).view(n, s.n_q_heads, hd), *rot[i])
            k = _rotate((a @ w["wk"].T).view(n, s.n_kv_heads, hd), *rot[i])
            v = (a @ w["wv"].T).view(n, s.n_kv_heads, hd)
            o = torch.stack([_attention(q[:, h].contiguous(), k[:, h // group].contiguous(), v[:, h // group].contiguous())
                             for h in range(s.n_q_heads)], 1)
            x = x + o.reshape(n, s.q_dim) @ w["wo"].T
            a = _norm(x, w["norm_mlp"], s.rms_eps)
            g = a @ w["wg"].T
            xs[i] = x + (g * torch.sigmoid(g) * (a @ w["wu"].T)) @ w["wd"].T
    z = torch.cat([_norm(x[-r:], head[1], s.rms_eps) @ head[0].T for x, r in zip(xs, keep)])
    return {"logits": z.cpu().numpy(), "tokens": None}
