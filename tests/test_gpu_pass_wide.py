"""Passes of wide decoder-only models in one kernel (pass_wide.hip), at the edges of its key blocks, key ranges, row layouts and of the
cuts of its projections, through the C ABI against the separate kernels (which the other tests hold against the oracle)."""
import ctypes as C

import numpy as np
import pytest

import bild_inputs as bi
import oracle
import paper_2302_07863_amd as pkg
from tests import parity
from tests.test_gpu_early_exit import EERig
from tests.hipmem import hip
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


@pytest.mark.parametrize("shape", [dict(), dict(act=bi.ACT_RELU, pos=bi.POS_SINUSOIDAL, d=1280, heads=10, d_ff=96)])
def test_against_the_oracle(shape, monkeypatch):
    """Algorithm 1 of both cuts, logit by logit, every pass in one kernel."""
    cfg = bi.toy_pair(**{**BASE, **shape, "max_new": 12})
    R = Rig(cfg)
    ref = oracle.bild_generate(R.req, 0.4, 1.0, 4, cfg.max_new, keep_logits=True)
    st = R.state(cfg.max_new, 4)
    st.encode(R.src)
    before = st.pass_routes()
    print(parity.teacher_forced(st, ref, R.n0, 0.4, 1.0, cfg))
    now = st.pass_routes()
    assert now["chip"] - before["chip"] == len(ref.trace) and now["gave_up"] == 0, now


def one_token_moves(st, R, have):
    """Largest change of the last row's logits of the large model when one of `have` earlier tokens, in their middle, is another one."""
    seen = []
    for other in (0, 1):
        tokens = bi.make_tokens(R.cfg.large.vocab, have - R.n0, seed=have)
        if other:
            tokens[len(tokens) // 2] = (tokens[len(tokens) // 2] + 1) % R.cfg.large.vocab
        st.seq_truncate(R.n0)
        st.force_tokens(R.n0, tokens, have)
        st.large_verify(float("inf"), draft=[])
        seen.append(st.debug_logits(pkg.LARGE, 0))
    return float(np.abs(seen[0] - seen[1]).max())


@pytest.mark.parametrize("layers,have", [(7, (40, 41, 300)), (2, (990, 1017, 1018, 2041, 2049, 2110))])
def test_many_layers_and_long_caches(layers, have, monkeypatch):
    """More layers than places of the hand-over memory, so that places are filled and read again within a launch, pass behind pass; more
    than four key ranges a head (from 1025 keys on), a second block of 32 keys for the waves (from 2048 earlier keys on).  The small
    model is 1280 wide, the large one 2560: one of each cut.  Against the separate kernels, both within logit_tol of the oracle; the
    routes differ by less than a quarter of what one other token among the earlier ones does to the logits, so that a key left out,
    or taken twice, shows."""
    cfg = bi.toy_pair(**{**BASE, "d": 1280, "heads": 10, "d_ff": 96, "n_small": layers, "n_large": layers, "max_new": max(have) + 4})
    R = Rig(cfg)
    got = {}
    for one in ("1", "0"):
        monkeypatch.setenv("BILD_ONE_KERNEL", one)
        st = R.state(cfg.max_new, 31)
        st.encode(R.src)
        st.debug_enable_logits(True)
        rows_seen = []
        for n in have:
            st.seq_truncate(R.n0)
            if n > R.n0:
                st.force_tokens(R.n0, bi.make_tokens(cfg.large.vocab, n - R.n0, seed=n), n)
            st.large_verify(float("inf"), draft=[])
            before = st.pass_routes()
            for rows in (8, 1, 5, 8):
                st.seq_truncate(n)
                st.large_verify(float("inf"), draft=[int(t) for t in bi.make_tokens(cfg.large.vocab, rows - 1, seed=40 + rows)])
                rows_seen += [st.debug_logits(pkg.LARGE, i) for i in range(rows)]
            st.seq_truncate(n)
            for _ in range(4):
                st.small_step(0.0)
                rows_seen.append(st.debug_logits(pkg.SMALL, 0))
            now = {k: v - before[k] for k, v in st.pass_routes().items() if v > before[k]}
            assert now == {"chip" if one == "1" else "kernels": 8}, (n, now)
        got[one] = np.stack(rows_seen)
        moved = one_token_moves(st, R, have[-1])
        st.close()
    worst = [float(np.abs(a - b).max()) for a, b in zip(got["1"], got["0"])]
    print("worst", max(worst), "one token", moved, flush=True)
    assert max(worst) <= min(moved / 4, 2 * parity.logit_tol(cfg))


@pytest.mark.parametrize("shape", [dict(), dict(act=bi.ACT_RELU, pos=bi.POS_SINUSOIDAL, d=1280, heads=10, d_ff=96)])
def test_who_does_what_changes_with_the_length(shape, monkeypatch):
    """Models up to 2048 wide: workgroups have other parts from 1281 keys and from 2305 on, so that passes on both sides of the lines
    follow each other in the same hand-over memory; one, two and more rows, whose activations come in loads of their own kinds."""
    cfg = bi.toy_pair(**{**BASE, **shape, "truncate": False, "n_large": 4, "n_small": 4, "max_new": 2320})
    R = Rig(cfg)
    got = {}
    for one in ("1", "0"):
        monkeypatch.setenv("BILD_ONE_KERNEL", one)
        st = R.state(cfg.max_new, 31)
        st.encode(R.src)
        st.debug_enable_logits(True)
        rows_seen = []
        for n in (1278, 2302, 130):
            st.seq_truncate(R.n0)
            st.force_tokens(R.n0, bi.make_tokens(cfg.large.vocab, n - R.n0, seed=n), n)
            st.large_verify(float("inf"), draft=[])
            before = st.pass_routes()
            for rows in (1, 2, 3, 4, 5, 8, 2, 1):
                st.seq_truncate(n)
                st.large_verify(float("inf"), draft=[int(t) for t in bi.make_tokens(cfg.large.vocab, rows - 1, seed=40 + rows)])
                rows_seen += [st.debug_logits(pkg.LARGE, i) for i in range(rows)]
            st.seq_truncate(n)
            for _ in range(5):
                st.small_step(0.0)
                rows_seen.append(st.debug_logits(pkg.SMALL, 0))
            now = {k: v - before[k] for k, v in st.pass_routes().items() if v > before[k]}
            assert now == {"chip" if one == "1" else "kernels": 13}, (n, now)
        got[one] = np.stack(rows_seen)
        moved = one_token_moves(st, R, 130)
        st.close()
    worst = float(np.abs(got["1"] - got["0"]).max())
    print("worst", worst, "one token", moved, flush=True)
    assert worst <= min(moved / 4, 2 * parity.logit_tol(cfg))


@pytest.mark.parametrize("many", [(9, 16, 8, 11, 16, 1, 15), (17, 32, 16, 25, 32, 2, 31)])
@pytest.mark.parametrize("shape", [dict(), dict(act=bi.ACT_RELU, pos=bi.POS_SINUSOIDAL, d=1280, heads=10, d_ff=96, n_large=4), dict(act=bi.ACT_RELU, pos=bi.POS_SINUSOIDAL, d_ff=96)])
def test_nine_to_thirty_two_rows(shape, many, monkeypatch):
    """Models of the widest cut (the large ones): high and low parts in operands of their own, two row tiles, no earlier key up to eight key ranges, the new
    keys' block whole and short, passes of other rooms between; above sixteen rows the widest models, up to 4096 keys, from 25 rows on
    2048, beyond which the separate kernels stay.  Against the separate kernels, as above."""
    cfg = bi.toy_pair(**{**BASE, **shape, "max_new": 2100})
    R = Rig(cfg)
    got = {}
    for one in ("1", "0"):
        monkeypatch.setenv("BILD_ONE_KERNEL", one)
        st = R.state(cfg.max_new, 31)
        st.encode(R.src)
        st.debug_enable_logits(True)
        rows_seen = []
        for have in (R.n0, R.n0 + 24, 300, 1018, 2020):
            st.seq_truncate(R.n0)
            if have > R.n0:
                st.force_tokens(R.n0, bi.make_tokens(cfg.large.vocab, have - R.n0, seed=have), have)
            st.large_verify(float("inf"), draft=[])
            before = st.pass_routes()
            for rows in many:
                st.seq_truncate(have)
                st.large_verify(float("inf"), draft=[int(t) for t in bi.make_tokens(cfg.large.vocab, rows - 1, seed=40 + rows)])
                rows_seen += [st.debug_logits(pkg.LARGE, i) for i in range(rows)]
            now = {k: v - before[k] for k, v in st.pass_routes().items() if v > before[k]}
            chip = sum(r <= 16 or (cfg.large.d == 4096 and have + r <= (4096 if r <= 24 else 2048)) for r in many) if one == "1" else 0
            assert now == {k: n for k, n in (("chip", chip), ("kernels", 7 - chip)) if n}, (have, now)
        got[one] = np.stack(rows_seen)
        moved = one_token_moves(st, R, 300)
        st.close()
    worst = float(np.abs(got["1"] - got["0"]).max())
    print("worst", worst, "one token", moved, flush=True)
    assert worst <= min(moved / 4, 2 * parity.logit_tol(cfg))


def test_states_have_room_for_the_rows_of_their_own_drafts(monkeypatch):
    """Hand-over memory above eight rows: up to n_max + 1 of the large model, in rooms of 16 and 32.  A longer draft of the caller's own is
    reviewed by the separate kernels, with the same outcome."""
    monkeypatch.setenv("BILD_WIDE_ROWS", "32")
    cfg = bi.toy_pair(**{**BASE, "d_ff": 96, "max_new": 40})
    R = Rig(cfg)

    def free():
        now, total = C.c_size_t(), C.c_size_t()
        assert hip().hipMemGetInfo(C.byref(now), C.byref(total)) == 0
        return now.value

    taken, routes, kept = [], [], []
    for n_max in (7, 15, 31, 7):   # (the first one loads what the others find)
        before = free()
        st = R.state(cfg.max_new, n_max)
        taken.append(before - free())
        st.encode(R.src)
        st.large_verify(float("inf"), draft=[])
        for rows in (8, 9, 16, 17, 32):
            st.seq_truncate(R.n0)
            kept.append(st.large_verify(float("inf"), draft=[int(t) for t in bi.make_tokens(cfg.large.vocab, rows - 1, seed=rows)])[:2])
        r = st.pass_routes()
        routes.append((r["chip"], r["kernels"]))
        st.close()
    assert routes == [(2, 4), (4, 2), (6, 0), (2, 4)]
    assert kept[:5] == kept[5:10] == kept[10:15] == kept[15:]
    sixteen, thirty_two = taken[1] - taken[3], taken[2] - taken[1]
    print("MB", [t >> 20 for t in taken], flush=True)
    assert 6 << 20 <= sixteen <= 16 << 20 and 12 << 20 <= thirty_two <= 32 << 20
