"""Passes of wide decoder-only models in one kernel (pass_wide.hip), at the edges of its key blocks, key ranges, row layouts and of the
cuts of its projections, through the C ABI against the separate kernels (which the other tests hold against the oracle)."""
import numpy as np
import pytest

import bild_inputs as bi
import oracle
import paper_2302_07863_amd as pkg
from tests import parity
from tests.test_gpu_early_exit import EERig
from tests.test_gpu_parity import Rig

pytestmark = pytest.mark.gpu

BASE = dict(dtype=bi.DT_BF16, cross=False, act=bi.ACT_SWIGLU, pos=bi.POS_ROPE, d=2048, heads=16, d_head=128, d_ff=2112, n_large=2, n_small=2, vocab=300,
            logit_scale=4.0, truncate=True, n_src=40, max_new=900)  # (the large model is twice as wide)


@pytest.mark.parametrize("shape", [dict(), dict(act=bi.ACT_RELU, pos=bi.POS_SINUSOIDAL, d=1280, heads=10, d_ff=96)])
def test_rows_and_keys(shape, monkeypatch):
    """Both models, reviews of 1 .. 8 rows, no earlier key up to four key ranges: the two routes of a pass agree (each is within
    logit_tol of the oracle), over layers enough for the hand-over memory to come round."""
    cfg = bi.toy_pair(**{**BASE, **shape})
    R = Rig(cfg)
    got = {}
    for one in ("1", "0"):
        monkeypatch.setenv("BILD_ONE_KERNEL", one)
        st = R.state(cfg.max_new, 31)
        st.encode(R.src)
        st.debug_enable_logits(True)
        rows_seen = []
        for have in (R.n0, R.n0 + 1, R.n0 + 24, R.n0 + 230, R.n0 + 520, R.n0 + 30):
            st.seq_truncate(R.n0)
            if have > R.n0:
                st.force_tokens(R.n0, bi.make_tokens(cfg.large.vocab, have - R.n0, seed=have), have)
            before = st.pass_routes()
            st.large_verify(float("inf"), draft=[])  # (brings the cache up)
            for rows in (1, 2, 3, 8):
                st.seq_truncate(have)
                st.large_verify(float("inf"), draft=[int(t) for t in bi.make_tokens(cfg.large.vocab, rows - 1, seed=40 + rows)])
                rows_seen += [st.debug_logits(pkg.LARGE, i) for i in range(rows)]
            st.seq_truncate(have)
            for _ in range(3):
                st.small_step(0.0)
                rows_seen.append(st.debug_logits(pkg.SMALL, 0))
            now = {k: v - before[k] for k, v in st.pass_routes().items() if v > before[k]}
            assert now == {"chip" if one == "1" else "kernels": 8}, (have, now)
        got[one] = np.stack(rows_seen)
        st.close()
    worst = float(np.abs(got["1"] - got["0"]).max())
    print("worst", worst, "tolerance", 2 * parity.logit_tol(cfg), flush=True)
    assert worst <= 2 * parity.logit_tol(cfg)


def test_early_exit_and_a_pass_that_gives_up(monkeypatch):
    """The upper layers start from the trunk's rows; then no poll is waited for: the pass commits nothing and runs as kernels."""
    cfg = bi.toy_pair(**{**BASE, "truncate": False, "n_large": 4, "d": 1280, "heads": 10, "max_new": 16})
    R = EERig(cfg)
    ref = oracle.bild_generate(R.req, 0.4, 1.0, 4, cfg.max_new, keep_logits=True)
    for spins, route in (("6000", "chip"), ("1", "gave_up")):
        monkeypatch.setenv("BILD_PASS_SPINS", spins)
        st = R.state(cfg.max_new, 4)
        st.encode(R.src)
        parity.teacher_forced(st, ref, R.n0, 0.4, 1.0, cfg)
        toks, stats = st.generate(R.src, 0.4, 1.0, cfg.max_new)
        print(parity.compare_generation(toks, stats, ref, 0.4, 1.0))
        assert st.pass_routes()[route] > 0, (spins, st.pass_routes())
