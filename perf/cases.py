"""The work a user of the library has it do, as cases that can be timed and compared.

Such a user holds two models on the GPU, paired once, and a state per request; a request brings the token ids of a source
or a prompt.  The weights are therefore drawn once per process and pair; the ids, the uniform numbers of the sampling
variant, the drafts and the hidden rows come from the seed.

The pairs have the shapes of this repository's configurations: the fp32 pair of the first, the T5- and mT5-shaped pairs of
the second and third, and the 7B-shaped decoder-only pair of the fourth and fifth.  Weights are N(0, 0.02).  The small
model is cut out of the large one, except that a quarter of its embedding rows are weak: where the next token is one of
those, the small model is unsure, so that the fallback test fires (in a fixed window: the review rolls the draft back),
and the large model, whose rows are whole, decides.  Elsewhere both models are sure.  Fallbacks are then about as
frequent as in the paper's Table 4, and no decision hangs on the last bits of a sum.
"""
import math

import numpy as np
import torch

import paper_2302_07863_amd as bild

RELU, GEGLU, SWIGLU = 0, 1, 2       # bild.h: BILD_ACT_*
SINUS, ROPE, RELATIVE = 0, 1, 2     # BILD_POS_*
F32, BF16 = 0, 1                    # BILD_DT_*
REL_DIST = 128
WEAK_SHARE, WEAK_SCALE = 0.25, 0.3
ALPHA_FB, ALPHA_RB, N_MAX = 0.5, 2.0, 10   # the middle thresholds and the paper's cap on consecutive drafts
WEIGHT_SEED = 20230207


def _shape(enc, dec, d, heads, d_head, d_ff, act, pos, vocab, dtype, shift, embed_scale, logit_scale):
    return dict(enc=enc, dec=dec, d=d, heads=heads, d_head=d_head, d_ff=d_ff, act=act, pos=pos, vocab=vocab, dtype=dtype,
                shift=shift, embed_scale=embed_scale, logit_scale=logit_scale, tied=True, rel=REL_DIST if pos == RELATIVE else 0)


# (small, large).  With these embedding and logit scales both models give the next token about 0.99.
FAMILIES = {
    "tiny": (_shape(0, 2, 256, 4, 64, 1024, RELU, SINUS, 1024, F32, 331, 60.0, 2.8),
             _shape(4, 4, 256, 4, 64, 1024, RELU, SINUS, 1024, F32, 331, 60.0, 2.9)),
    "t5": (_shape(6, 6, 512, 8, 64, 2048, RELU, SINUS, 32128, BF16, 7919, 60.0, 2.1),
           _shape(24, 24, 1024, 16, 64, 4096, RELU, SINUS, 32128, BF16, 7919, 200.0, 0.95)),
    # the first six layers of the large model with its head are the small model (one cache for both)
    "t5-exit": (_shape(0, 6, 1024, 16, 64, 4096, RELU, SINUS, 32128, BF16, 7919, 200.0, 0.83),
                _shape(24, 24, 1024, 16, 64, 4096, RELU, SINUS, 32128, BF16, 7919, 200.0, 0.95)),
    # with the relative positions of that model family
    "mt5": (_shape(8, 8, 512, 6, 64, 1024, GEGLU, RELATIVE, 250112, BF16, 7919, 60.0, 1.8),
            _shape(24, 24, 1024, 16, 64, 2816, GEGLU, RELATIVE, 250112, BF16, 7919, 200.0, 0.93)),
    "llama": (_shape(0, 16, 2048, 16, 128, 5632, SWIGLU, ROPE, 32000, BF16, 7919, 60.0, 1.1),
              _shape(0, 32, 4096, 32, 128, 11008, SWIGLU, ROPE, 32000, BF16, 7919, 120.0, 1.1)),
}


# ------------------------------------------------------------------------------------------------ models
def _layer_shapes(m, cross):
    d, inner, f = m["d"], m["heads"] * m["d_head"], m["d_ff"]
    out = [("ln1", (d,)), ("wq", (d, inner)), ("wk", (d, inner)), ("wv", (d, inner)), ("wo", (inner, d))]
    if cross:
        out += [("lnc", (d,)), ("cwq", (d, inner)), ("cwk", (d, inner)), ("cwv", (d, inner)), ("cwo", (inner, d))]
    out += [("ln2", (d,)), ("w_in", (d, f))]
    if m["act"] != RELU:
        out.append(("w_up", (d, f)))
    return out + [("w_out", (f, d))]


def _tensor_shapes(m, cross):
    """Names and shapes in the order bild_model_create takes them."""
    out = [("emb", (m["vocab"], m["d"]))]
    if not m["tied"]:
        out.append(("head", (m["vocab"], m["d"])))
    if m["enc"]:
        out.append(("enc_norm", (m["d"],)))
    out.append(("dec_norm", (m["d"],)))
    if m["rel"]:
        rel = (m["heads"], 2 * m["rel"] + 1)
        out += ([("enc_rel", rel)] if m["enc"] else []) + [("dec_rel", rel)]
    for l in range(m["enc"]):
        out += [("enc%d.%s" % (l, n), s) for n, s in _layer_shapes(m, False)]
    for l in range(m["dec"]):
        out += [("dec%d.%s" % (l, n), s) for n, s in _layer_shapes(m, cross)]
    return out


def _weights(m, cross, gen):
    out = {}
    for name, shape in _tensor_shapes(m, cross):
        leaf = name.split(".")[-1]
        if leaf in ("enc_norm", "dec_norm", "ln1", "ln2", "lnc"):
            out[name] = torch.ones(shape, device="cuda")
        else:
            out[name] = torch.randn(shape, device="cuda", generator=gen)
            if leaf not in ("enc_rel", "dec_rel"):
                out[name] *= 0.02
    return out


def _weak_rows(vocab):
    gen = torch.Generator(device="cuda").manual_seed(WEIGHT_SEED + 1)
    return torch.rand(vocab, device="cuda", generator=gen) < WEAK_SHARE


def _cut(small, cross, large_weights):
    """The leading block of every tensor of the large model; a quarter of the embedding rows made weak."""
    out = {}
    for name, shape in _tensor_shapes(small, cross):
        out[name] = large_weights[name][tuple(slice(0, n) for n in shape)].contiguous()
    out["emb"] = torch.where(_weak_rows(small["vocab"])[:, None], WEAK_SCALE * out["emb"], out["emb"])
    return out


def _upload(m, cross, weights):
    cfg = bild.ModelConfig(n_enc_layers=m["enc"], n_dec_layers=m["dec"], d_model=m["d"], n_heads=m["heads"], d_head=m["d_head"],
                           d_ff=m["d_ff"], act=m["act"], pos=m["pos"], vocab=m["vocab"], tied_head=int(m["tied"]), dtype=m["dtype"],
                           cross_attn=int(cross), bos=0, tie_shift=m["shift"], logit_scale=m["logit_scale"],
                           embed_scale=m["embed_scale"], norm_eps=1e-6, rope_base=10000.0, rel_max_dist=m["rel"])
    return bild.Model(cfg, [weights[name].cpu().numpy() for name, _ in _tensor_shapes(m, cross)])


_kept = {}


def _keep(key, make):
    """What a process makes once and keeps (weights on the GPU); the oldest goes where there are many."""
    if key not in _kept:
        while len(_kept) >= 8:
            _kept.pop(next(iter(_kept)))
        _kept[key] = make()
    return _kept[key]


def _pair(family):
    def make():
        small, large = FAMILIES[family]
        cross = large["enc"] > 0
        gen = torch.Generator(device="cuda").manual_seed(WEIGHT_SEED)
        weights = _weights(large, cross, gen)
        if family == "t5-exit":
            return bild.Pair.early_exit(_upload(large, cross, weights), small["dec"], small["logit_scale"])
        cut = _cut(small, cross, weights)
        pair = bild.Pair(_upload(small, cross, cut), _upload(large, cross, weights))
        del weights, cut
        torch.cuda.empty_cache()
        return pair
    return _keep(family, make)


def _head_model(case):
    """One network of which only the LM head is used (a pruned or specialised vocabulary has any size)."""
    def make():
        d = case["d"]
        m = _shape(0, 1, d, d // 64, 64, d, RELU, ROPE, case["vocab"], case["dtype"], 0, 1.0, 1.0)
        gen = torch.Generator(device="cuda").manual_seed(WEIGHT_SEED)
        return _upload(m, False, _weights(m, False, gen))
    return _keep(("head", case["d"], case["vocab"], case["dtype"]), make)


# ------------------------------------------------------------------------------------------------ cases
def listed():
    return [
        # the vocabulary sweep alone: rescoring one hidden row of a T5-small-shaped model, the smallest call there is
        dict(name="head one row", kind="head", d=512, vocab=32128, dtype=BF16, rows=1, static=False),
        # the same for a batch of candidates at the largest vocabulary, through the call that allocates nothing
        dict(name="head 21 rows 250k", kind="head", d=1024, vocab=250112, dtype=BF16, rows=21, static=True),
        # a whole request of the fp32 pair
        dict(name="tiny fp32 request", kind="request", family="tiny", n_src=32, max_new=32, window=0, top_p=0.0),
        # summarisation: source of 512 tokens, 64 tokens streamed to the user step by step (Algorithm 1 over the calls)
        dict(name="t5 request", kind="request", family="t5", n_src=512, max_new=64, window=0, top_p=0.0),
        # the same by the one call that runs the loop itself, on a short odd source, drafting in a fixed window
        dict(name="t5 window generate", kind="generate", family="t5", n_src=77, max_new=48, window=5, top_p=0.0),
        # the sampling variant
        dict(name="t5 sampling", kind="request", family="t5", n_src=201, max_new=40, window=0, top_p=0.8),
        # early exit: the small model is the large one's trunk
        dict(name="t5 early exit", kind="generate", family="t5-exit", n_src=333, max_new=64, window=3, top_p=0.0),
        # translation: short source, 250 112 ids, relative positions
        dict(name="mt5 generate", kind="generate", family="mt5", n_src=64, max_new=64, window=0, top_p=0.0),
        # a long document up to its first reviewed token
        dict(name="t5 long first token", kind="first", family="t5", n_src=1531, window=0),
        # decoder-only: prompt up to the first reviewed token, and decoding behind a prompt
        dict(name="llama first token", kind="first", family="llama", n_src=1024, window=0),
        dict(name="llama decode", kind="decode", family="llama", n_src=1024, max_new=64, window=0, top_p=0.0),
        # one review of 31 drafts over a long cache
        dict(name="llama review 4096", kind="review", family="llama", n_src=4097, rows=32),
    ]


def _between(rng, lo, hi):
    """A whole number, its logarithm spread evenly."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["head", "request", "request", "generate", "first", "decode", "review"])
    if kind == "head":
        d, dtype = rng.choice([512, 1024, 2048, 4096]), rng.choice([BF16, BF16, F32])
        return dict(kind=kind, d=d, vocab=_between(rng, 1000, min(250112, 2 ** 28 // d)), dtype=dtype, rows=_between(rng, 1, 32),
                    static=rng.random() < 0.5)
    if kind in ("decode", "review"):
        if kind == "review":
            return dict(kind=kind, family="llama", n_src=_between(rng, 64, 4097), rows=_between(rng, 2, 32))
        return dict(kind=kind, family="llama", n_src=_between(rng, 16, 1024), max_new=_between(rng, 16, 64),
                    window=rng.choice([0, 0, rng.randint(2, 10)]), top_p=0.0)
    family = rng.choice(["tiny", "t5", "t5", "mt5", "llama"] if kind == "first" else ["tiny", "t5", "t5", "t5-exit", "mt5"])
    most = {"tiny": 128, "mt5": 512, "llama": 1024}.get(family, 1531)
    if kind == "first":
        return dict(kind=kind, family=family, n_src=_between(rng, 8, most), window=0)
    window = rng.randint(2, 10) if family == "t5-exit" else rng.choice([0, 0, rng.randint(2, 10)])
    return dict(kind=kind, family=family, n_src=_between(rng, 8, most), max_new=_between(rng, 12, 64), window=window,
                top_p=0.8 if kind == "request" and not window and rng.random() < 0.3 else 0.0)


def _ids(gen, vocab, n):
    """Ids with frequencies like those of text: Zipf, exponent 1.1."""
    cdf = np.cumsum(np.arange(1, vocab + 1, dtype=np.float64) ** -1.1)
    return np.minimum(np.searchsorted(cdf / cdf[-1], gen.random(n)), vocab - 1).astype(np.int32)


def prepare(case, seed):
    gen = np.random.default_rng([seed, 7863])
    if case["kind"] == "head":
        model = _head_model(case)
        tgen = torch.Generator(device="cuda").manual_seed(seed)
        x = torch.randn(case["rows"], case["d"], device="cuda", generator=tgen)
        targets = torch.randint(0, case["vocab"], (case["rows"],), device="cuda", generator=tgen).to(torch.int32)
        out = torch.zeros(case["rows"], 4, dtype=torch.int32, device="cuda")
        cols = {n: out[:, k].view(torch.float32) if n != "argmax" else out[:, k]
                for k, n in enumerate(("zmax", "lse", "argmax", "z_target"))}
        return dict(kind="head", model=model, x=x, targets=targets, out=out, cols=cols, rows=case["rows"],
                    entry="bild_head_stats_static" if case["static"] else "bild_head_stats")
    pair, (small, large) = _pair(case["family"]), FAMILIES[case["family"]]
    vocab, dec_only = large["vocab"], not large["enc"]
    src = _ids(gen, vocab, case["n_src"])
    kind, window = case["kind"], case.get("window", 0)
    state = dict(kind=kind, src=src, max_new=case.get("max_new", 1), n0=len(src) if dec_only else 1,
                 # a fixed window never falls back for lack of confidence
                 alpha_fb=0.0 if window else ALPHA_FB)
    # decoder-side prefix of an encoder-decoder request (a language or task token)
    state["prefix"] = gen.integers(0, vocab, 1).astype(np.int32)
    if kind == "review":
        state["draft"] = _ids(gen, vocab, case["rows"] - 1)
    max_len = state["n0"] + state["max_new"] + 40
    st = state["st"] = bild.State(pair, len(src), max_len, 31 if kind == "review" else (window or N_MAX))
    if case.get("top_p", 0.0) > 0:
        u = (gen.integers(0, 1 << 24, (2, max_len)) / float(1 << 24)).astype(np.float32)
        st.set_sampling(case["top_p"], u[0], u[1])
    if kind in ("decode", "review"):
        st.encode(src)
    return state


def _stream(st, max_new, alpha_fb):
    """Algorithm 1 over the calls, as a program runs it that hands out every token with the small model's confidence at
    its place and the large model's cost of the drafts it has kept."""
    tokens, n = np.zeros(max_new, dtype=np.int32), 0
    confidence, cost = np.zeros(max_new, dtype=np.float32), np.zeros(max_new, dtype=np.float32)
    start = 0  # drafts tokens[start:n] are unreviewed
    while n < max_new:
        token, fallback, confidence[n] = st.small_step(alpha_fb)
        if not fallback:
            tokens[n] = token
            n += 1
            continue
        got, kept, nll = st.large_verify(ALPHA_RB)
        tokens[start:start + len(got)] = got
        cost[start:start + kept] = nll[:kept]
        start = n = start + len(got)
    return {"tokens": tokens, "confidence": confidence, "cost": cost}


def run(state):
    kind = state["kind"]
    if kind == "head":
        bild.binding.head_stats(state["model"], state["x"].data_ptr(), state["rows"], state["targets"].data_ptr(),
                                state["out"].data_ptr(), entry=state["entry"])
        return state["cols"]
    st = state["st"]
    if kind == "review":
        st.seq_truncate(state["n0"])
        tokens, kept, nll = st.large_verify(math.inf, state["draft"])
        return {"tokens": np.array(tokens, dtype=np.int32), "cost": nll[:kept].copy()}
    if kind == "decode":
        st.seq_truncate(state["n0"])
        return _stream(st, state["max_new"], state["alpha_fb"])
    if kind == "generate":
        # the loop inside the library behind a decoder-side prefix; what is still unreviewed at the end is reviewed, so that
        # every token comes with the large model's word
        st.encode(state["src"])
        n0 = state["n0"]
        st.force_tokens(n0, state["prefix"], n0 + 1)
        tokens, stats = st.generate(None, state["alpha_fb"], ALPHA_RB, state["max_new"])
        last, kept, nll = st.large_verify(ALPHA_RB)
        tail, cost = np.full(N_MAX + 1, -1, dtype=np.int32), np.zeros(N_MAX + 1, dtype=np.float32)
        tail[:len(last)], cost[:kept] = last, nll[:kept]
        return {"tokens": np.array(tokens, dtype=np.int32), "counts": np.array(list(stats.values()), dtype=np.int32),
                "tail": tail, "cost": cost}
    st.encode(state["src"])
    if kind == "first":
        token, fallback, p = st.small_step(ALPHA_FB)
        tokens, kept, nll = st.large_verify(ALPHA_RB)
        return {"token": np.int32(tokens[0]), "confidence": np.float32(p), "cost": np.float32(nll[0] if kept else 0.0)}
    return _stream(st, state["max_new"], state["alpha_fb"])


# ------------------------------------------------------------------------------------------------ what a pass cannot do without
def _decoder(m, cross, cache, n_src, rows, head_rows):
    """(bytes, flops) of one pass of a decoder: every weight once, the cached keys and values once."""
    inner, b = m["heads"] * m["d_head"], 4 if m["dtype"] == F32 else 2
    layer = 4 * m["d"] * inner * (2 if cross else 1) + (2 if m["act"] == RELU else 3) * m["d"] * m["d_ff"]
    keys = cache + rows + (n_src if cross else 0)
    head = m["vocab"] * m["d"]
    return (b * (m["dec"] * (layer + 2 * inner * keys) + (head if head_rows else 0)),
            2 * rows * m["dec"] * (layer + 2 * inner * keys) + 2 * head_rows * head)


def _encode(small, large, n_src):
    bytes_, flops = 0, 0
    if not large["enc"]:
        for m in (small, large):
            w, f = _decoder(m, False, 0, 0, n_src, 0)
            bytes_, flops = bytes_ + w, flops + f
        return bytes_, flops
    for m in (small, large):
        inner, b = m["heads"] * m["d_head"], 4 if m["dtype"] == F32 else 2
        layer = 4 * m["d"] * inner + (2 if m["act"] == RELU else 3) * m["d"] * m["d_ff"]
        bytes_ += b * (m["enc"] * layer + m["dec"] * (2 * m["d"] * inner + 2 * inner * n_src))
        flops += 2 * n_src * (m["enc"] * (layer + 2 * inner * n_src) + m["dec"] * 2 * m["d"] * inner)
    return bytes_, flops


def work(case):
    if case["kind"] == "head":
        n = case["vocab"] * case["d"]
        return {"bytes": n * (2 if case["dtype"] == BF16 else 4) + case["rows"] * (4 * case["d"] + 20), "flops": 2 * n * case["rows"]}
    small, large = FAMILIES[case["family"]]
    cross, n_src = large["enc"] > 0, case["n_src"]
    n0 = 1 if cross else n_src
    if case["kind"] == "review":
        w, f = _decoder(large, cross, n0 - 1, n_src, case["rows"], case["rows"])
        return {"bytes": w, "flops": f}
    bytes_, flops = (0, 0) if case["kind"] == "decode" else _encode(small, large, n_src)
    if case["kind"] == "first":
        steps, reviews, rows = 1, 1, 1
    else:
        # a small step per token; a review per fallback (a quarter of the tokens) or per window
        steps = case["max_new"]
        reviews = max(1, round(steps * (WEAK_SHARE if not case["window"] else 1 / (case["window"] + 1))))
        rows = max(1, round(steps / reviews))
    middle = n0 + case.get("max_new", 1) // 2
    for m, passes, r in ((small, steps, 1), (large, reviews, rows)):
        w, f = _decoder(m, cross, middle, n_src, r, r)
        bytes_, flops = bytes_ + passes * w, flops + passes * f
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    if case["kind"] == "head":
        # fp32 sums; bf16 weights are exact and the hidden rows keep 16 bits or more
        return {"rel": 3e-5, "max": 1e-3}
    if case["family"] == "tiny":
        return {"rel": 3e-5, "max": 1e-3}
    # keys and values are cached in bf16: a value on a rounding boundary moves the logits by up to 1e-2
    return {"rel": 1e-2, "max": 0.1}
