"""Passes of a few rows on the thin GEMM and the attention whose workgroups join their keys themselves, at the edges of their row
tiles, key blocks, feature groups and slices, through the C ABI against the CPU oracle and the kernels they stand beside."""
import numpy as np
import pytest

import bild_inputs as bi
import oracle
import paper_2302_07863_amd as pkg
from tests import parity
from tests.test_gpu_parity import Rig
from tests.test_gpu_pass_wide import one_token_moves

pytestmark = pytest.mark.gpu

WIDE = dict(cross=False, act=bi.ACT_SWIGLU, pos=bi.POS_ROPE, d=2048, heads=16, d_head=128, d_ff=2112, n_large=1, vocab=300, logit_scale=4.0)  # (the large model is twice as wide)


@pytest.mark.parametrize("shape", [
    dict(),                                                                    # more waves than input tiles, cross-attention
    dict(act=bi.ACT_GATED_GELU, pos=bi.POS_RELATIVE, d_ff=224),                # the other attention kernel
    dict(cross=False, act=bi.ACT_SWIGLU, pos=bi.POS_ROPE, d_head=128, heads=2),
    dict(d=768, heads=12, d_ff=2080, vocab=9000),                              # several groups of the head, the last one short
    WIDE,                                                                      # slices
])
def test_rows_and_keys(shape, monkeypatch):
    """Reviews of 1 .. 32 rows over short and long caches: the two routes of a pass agree (each is within logit_tol of the oracle)."""
    cfg = bi.toy_pair(**{**dict(dtype=bi.DT_BF16, d=256, heads=4, d_head=64, d_ff=512, truncate=True, n_src=40, max_new=420), **shape})
    R = Rig(cfg)
    ref = oracle.bild_generate(R.req, 0.4, 1.0, 8, 6, keep_logits=True)
    monkeypatch.setenv("BILD_ONE_KERNEL", "0")
    got = {}
    for route in ("2", "99"):
        monkeypatch.setenv("BILD_THIN_MIN_ROWS", route)
        st = R.state(cfg.max_new, 31)
        st.encode(R.src)
        parity.teacher_forced(st, ref, R.n0, 0.4, 1.0, cfg)
        st.debug_enable_logits(True)
        rows_seen, nll = [], []
        for have in (R.n0, R.n0 + 31, R.n0 + 350):
            st.seq_truncate(R.n0)
            if have > R.n0:
                st.force_tokens(R.n0, bi.make_tokens(cfg.large.vocab, have - R.n0, seed=have), have)
            st.large_verify(float("inf"), draft=[])  # (brings the cache up)
            for rows in (1, 2, 8, 9, 16, 17, 32):
                st.seq_truncate(have)
                draft = [int(t) for t in bi.make_tokens(cfg.large.vocab, rows - 1, seed=40 + rows)]
                nll += list(st.large_verify(float("inf"), draft=draft)[2][:rows - 1])
                rows_seen += [st.debug_logits(pkg.LARGE, i) for i in range(rows)]
        got[route] = np.stack(rows_seen), np.array(nll)
    tol = 2 * parity.logit_tol(cfg)
    assert float(np.abs(got["2"][0] - got["99"][0]).max()) <= tol
    assert float(np.abs(got["2"][1] - got["99"][1]).max()) <= 2 * tol


def test_the_same_pass_twice_gives_the_same_bits(monkeypatch):
    """Whoever arrives last, slices and key ranges are joined in one order."""
    cfg = bi.toy_pair(**{**dict(dtype=bi.DT_BF16, truncate=True, n_src=300, max_new=8), **WIDE})
    R = Rig(cfg)
    st = R.state(40, 31)
    st.encode(R.src)
    st.debug_enable_logits(True)
    for rows in (1, 5, 12, 32):
        draft = [int(t) for t in bi.make_tokens(cfg.large.vocab, rows - 1, seed=rows)]
        seen = []
        for _ in range(6):
            st.seq_truncate(R.n0)
            st.large_verify(float("inf"), draft=draft)
            seen.append(np.stack([st.debug_logits(pkg.LARGE, i) for i in range(rows)]))
        assert all((s == seen[0]).all() for s in seen[1:]), rows


def test_single_rows_whose_producers_hand_over_planes(monkeypatch):
    """BILD_PRE_MIN_ROWS=1: the output projection of a single row reads the attention's planes, whichever kernel leaves them."""
    cfg = bi.toy_pair(**{**dict(dtype=bi.DT_BF16, truncate=True, n_src=40, max_new=8), **WIDE, "d": 1280, "heads": 10, "d_ff": 96})
    R = Rig(cfg)
    ref = oracle.bild_generate(R.req, 0.4, 1.0, 4, 8, keep_logits=True)
    monkeypatch.setenv("BILD_ONE_KERNEL", "0")
    monkeypatch.setenv("BILD_PRE_MIN_ROWS", "1")
    st = R.state(cfg.max_new, 4)
    st.encode(R.src)
    parity.teacher_forced(st, ref, R.n0, 0.4, 1.0, cfg)


@pytest.mark.parametrize("heads", [2, 16])
def test_long_caches(heads, monkeypatch):
    """Attention that joins its key ranges at more than 2048 keys: sixteen ranges a head, joined in two rounds (four heads), and more
    blocks of 32 keys than ranges x waves, so that a wave loads a second one (32 heads).  Against the kernels they stand beside, from
    which they differ by less than a quarter of what one other token among the earlier ones does."""
    cfg = bi.toy_pair(dtype=bi.DT_BF16, cross=False, act=bi.ACT_SWIGLU, pos=bi.POS_ROPE, d=256, heads=heads, d_head=128 if heads == 2 else 64, d_ff=256, n_small=1, n_large=2, vocab=300,
                      logit_scale=4.0, truncate=True, n_src=40, max_new=4240)
    R = Rig(cfg)
    monkeypatch.setenv("BILD_ONE_KERNEL", "0")
    got = {}
    for route in ("2", "99"):
        monkeypatch.setenv("BILD_THIN_MIN_ROWS", route)
        st = R.state(cfg.max_new, 31)
        st.encode(R.src)
        st.debug_enable_logits(True)
        rows_seen = []
        for have in (2040, 2049, 2100, 4170):
            st.seq_truncate(R.n0)
            st.force_tokens(R.n0, bi.make_tokens(cfg.large.vocab, have - R.n0, seed=have), have)
            st.large_verify(float("inf"), draft=[])
            for rows in (2, 8, 9, 17, 32):
                st.seq_truncate(have)
                st.large_verify(float("inf"), draft=[int(t) for t in bi.make_tokens(cfg.large.vocab, rows - 1, seed=40 + rows)])
                rows_seen += [st.debug_logits(pkg.LARGE, i) for i in range(rows)]
        got[route] = np.stack(rows_seen)
        moved = one_token_moves(st, R, 4170)
        st.close()
    worst = float(np.abs(got["2"] - got["99"]).max())
    print("worst", worst, "one token", moved, flush=True)
    assert worst <= min(moved / 4, 2 * parity.logit_tol(cfg))
