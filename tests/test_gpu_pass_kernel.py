"""Decoder passes of narrow bf16 models as one kernel, at the edges of its shapes, rows and key blocks, through the C ABI against
the CPU oracle."""
import ctypes as C
import time

import numpy as np
import pytest

import bild_inputs as bi
import oracle
import paper_2302_07863_amd as pkg
from tests import parity
from tests.hipmem import hip
from tests.test_gpu_parity import Rig

pytestmark = pytest.mark.gpu


def _check(n_max=4, alpha_fb=0.4, max_new=8, **shape):
    cfg = bi.toy_pair(**{**dict(dtype=bi.DT_BF16, d=256, heads=4, d_head=64, d_ff=512, truncate=True, n_src=20, max_new=max_new), **shape})
    R = Rig(cfg)
    ref = oracle.bild_generate(R.req, alpha_fb, 1.0, n_max, cfg.max_new, keep_logits=True)
    st = R.state(cfg.max_new, n_max)
    st.encode(R.src)
    parity.teacher_forced(st, ref, R.n0, alpha_fb, 1.0, cfg)


@pytest.mark.parametrize("shape", [
    dict(d=256, heads=1, d_ff=32),                                           # fewer inputs and units than waves
    dict(d=512, heads=6, d_ff=1024, act=bi.ACT_GATED_GELU),                  # attention narrower than the model
    dict(d=768, heads=12, d_ff=2112),                                        # a wave's last inputs missing
    dict(d=1024, heads=16, d_ff=4096, vocab=300, n_large=2, logit_scale=4.0),  # the largest of each
    dict(d=512, heads=8, d_ff=1024, cross=False),
])
def test_shapes(shape):
    _check(**shape)


@pytest.mark.parametrize("n_max", [7, 8, 15])
def test_rows_of_a_review(n_max):
    """8, 9 and 16 rows: the packed operand, the plain one, and the most the kernel takes."""
    _check(n_max=n_max, alpha_fb=0.0, max_new=2 * n_max)


@pytest.mark.parametrize("d_ff", [2112, 4096])
def test_rows_of_a_review_of_a_wide_ffn(d_ff):
    """Sixteen rows: the hidden state's tiles in pieces, the last one short."""
    _check(n_max=15, alpha_fb=0.0, max_new=32, d=1024, heads=16, d_ff=d_ff, vocab=300, n_large=2, logit_scale=4.0)


@pytest.mark.parametrize("shape", [dict(), dict(pos=bi.POS_RELATIVE)])
def test_blocks_of_earlier_keys(shape, monkeypatch):
    """The new rows' keys are a block of their own, which the wave behind the last block of earlier keys takes; more than eight
    blocks of those.  Against the separate kernels: each is within logit_tol of the exact value."""
    cfg = bi.toy_pair(**{**dict(dtype=bi.DT_BF16, d=256, heads=4, d_head=64, d_ff=512, truncate=True, n_src=20, max_new=700), **shape})
    R = Rig(cfg)
    got = {}
    for form, env in FORMS.items():
        with monkeypatch.context() as m:
            for k, v in env.items():
                m.setenv(k, v)
            st = R.state(cfg.max_new, 15)
        st.encode(R.src)
        st.debug_enable_logits(True)
        logits = []
        for have in (1, 32, 33, 64, 225, 256, 257, 600):  # tokens before the review, the last of them not yet consumed
            st.seq_truncate(R.n0)
            st.force_tokens(R.n0, bi.make_tokens(cfg.large.vocab, have - R.n0, seed=have), have)
            st.large_verify(float("inf"), draft=[])  # (brings the cache up)
            for rows in (1, 4, 8, 13):
                st.seq_truncate(have)
                before = st.pass_routes()
                st.large_verify(float("inf"), draft=[int(t) for t in bi.make_tokens(cfg.large.vocab, rows - 1, seed=40 + rows)])
                assert {k for k, v in st.pass_routes().items() if v > before[k]} == {"chip" if form == "die" and rows > 4 else form}, (form, have, rows)
                logits += [st.debug_logits(pkg.LARGE, i) for i in range(rows)]
        got[form] = np.stack(logits)
    tol = 2 * parity.logit_tol(cfg)
    for form in ("die", "chip"):
        assert float(np.abs(got[form] - got["kernels"]).max()) <= tol, form


@pytest.mark.parametrize("dtype", [bi.DT_BF16, bi.DT_F32])
def test_the_longest_row_of_relative_biases(dtype, monkeypatch):
    """8193 biases of a head take its workgroup seventeen trips to bring to LDS, and the first layer's scores of one row, two and more
    read any of them: passes of states that have just been made, each against the separate kernels (both within logit_tol of the exact
    value)."""
    cfg = bi.toy_pair(dtype=dtype, pos=bi.POS_RELATIVE, rel_max_dist=4096, rel_buckets=64, d=256, heads=4, d_head=64, d_ff=512, truncate=dtype == bi.DT_BF16,
                      n_small=1, n_large=1, n_src=20, max_new=700)
    R = Rig(cfg)
    got = {}
    for form in ("die", "chip", "kernels") if dtype == bi.DT_BF16 else ("die", "kernels"):
        logits = []
        for rows in (1, 2, 4, 13):
            with monkeypatch.context() as m:
                for k, v in FORMS[form].items():
                    m.setenv(k, v)
                st = R.state(cfg.max_new, 15)
            st.encode(R.src)
            st.debug_enable_logits(True)
            st.force_tokens(R.n0, bi.make_tokens(cfg.large.vocab, 600 - R.n0, seed=7), 600)
            st.large_verify(float("inf"), draft=[])
            st.seq_truncate(600)
            st.large_verify(float("inf"), draft=[int(t) for t in bi.make_tokens(cfg.large.vocab, rows - 1, seed=40 + rows)])
            logits += [st.debug_logits(pkg.LARGE, i) for i in range(rows)]
            assert st.pass_routes()["gave_up"] == 0 and st.pass_routes()["chip" if form == "die" and dtype == bi.DT_BF16 and rows > 4 else form] > 0
            st.close()
        got[form] = np.stack(logits)
    for form in set(got) - {"kernels"}:
        assert float(np.abs(got[form] - got["kernels"]).max()) <= 2 * parity.logit_tol(cfg), form


def test_waves_without_keys_of_the_sequence(monkeypatch):
    """Every wave has keys of the source (530 tokens), one or two have keys of the sequence, over ten layers: a wave without any is through
    with the next layer's self-attention while others join this layer's cross-attention.  Against the separate kernels, as above."""
    cfg = bi.toy_pair(dtype=bi.DT_BF16, d=256, heads=4, d_head=64, d_ff=512, truncate=True, n_small=10, n_large=10, n_src=530, max_new=40)
    R = Rig(cfg)
    got = {}
    for form, env in FORMS.items():
        with monkeypatch.context() as m:
            for k, v in env.items():
                m.setenv(k, v)
            st = R.state(cfg.max_new, 15)
        st.encode(R.src)
        st.debug_enable_logits(True)
        logits = []
        for rows in (1, 2, 3, 8, 16):
            st.seq_truncate(R.n0)
            st.large_verify(float("inf"), draft=[int(t) for t in bi.make_tokens(cfg.large.vocab, rows - 1, seed=40 + rows)])
            logits += [st.debug_logits(pkg.LARGE, i) for i in range(rows)]
            st.small_step(0.0)
            logits.append(st.debug_logits(pkg.SMALL, 0))
        assert st.pass_routes()["gave_up"] == 0
        got[form] = np.stack(logits)
    for form in ("die", "chip"):
        assert float(np.abs(got[form] - got["kernels"]).max()) <= 2 * parity.logit_tol(cfg), form


@pytest.mark.parametrize("n_src", [1, 32, 33, 257, 530])
def test_source_lengths_around_the_key_blocks(n_src):
    _check(n_src=n_src)


def test_a_pass_that_gives_up_runs_again_as_kernels(monkeypatch):
    """No poll is waited for: the first pass is flagged, commits nothing, and the request goes on without the kernel."""
    monkeypatch.setenv("BILD_PASS_SPINS", "1")
    _check()


@pytest.mark.parametrize("how", ["passes", "measurement"])
def test_the_kernel_is_tried_again_after_a_pass_gave_up(how):
    """Both forms (one die up to four rows, the whole chip above): what made a pass give up may be gone, so the state comes back to
    the kernel, with the tokens it would have produced anyway."""
    cfg = bi.toy_pair(dtype=bi.DT_BF16, d=256, heads=4, d_head=64, d_ff=512, truncate=True, n_src=20, max_new=40)
    R = Rig(cfg)
    generate = lambda st: st.generate(R.src, cfg.alpha_fb, cfg.alpha_rb, cfg.max_new)
    sound = R.state(cfg.max_new, cfg.n_max)
    want = generate(sound)
    r = sound.pass_routes()
    assert r["chip"] > 0 and r["die"] > 0 and r["kernels"] == r["gave_up"] == 0
    st = R.state(cfg.max_new, cfg.n_max)
    st.debug_pass_spins(1)
    if how == "passes":
        assert generate(st) == want
    else:
        st.encode(R.src)
        st.bench_pass(pkg.SMALL, 1, 3)
    failed = st.pass_routes()["gave_up"]
    assert failed > 0
    st.debug_pass_spins(6000)
    for _ in range(8):                 # (a few attempts in vain: at most some hundred passes as kernels follow)
        before = st.pass_routes()
        assert generate(st) == want
        now = {k: v - before[k] for k, v in st.pass_routes().items()}
    assert now == r
    assert st.pass_routes()["gave_up"] == failed


FORMS = {"die": {}, "chip": {"BILD_ONE_DIE": "0"}, "kernels": {"BILD_ONE_KERNEL": "0"}}


@pytest.mark.parametrize("shape", [dict(), dict(act=bi.ACT_GATED_GELU, pos=bi.POS_RELATIVE, d_ff=256), dict(cross=False), dict(act=bi.ACT_SWIGLU, n_src=300)])
def test_the_forms_of_a_pass_agree(shape, monkeypatch):
    """Reviews of 1 .. 16 rows and a small step on one die (up to four rows), on the whole chip and as separate kernels.  Each form is
    within logit_tol of the oracle (teacher-forced), so two of them are within twice that of each other."""
    cfg = bi.toy_pair(**{**dict(dtype=bi.DT_BF16, d=256, heads=4, d_head=64, d_ff=512, truncate=True, n_src=20, max_new=24), **shape})
    R = Rig(cfg)
    ref = oracle.bild_generate(R.req, 0.4, 1.0, 15, 6, keep_logits=True)
    got = {}
    for form, env in FORMS.items():
        with monkeypatch.context() as m:
            for k, v in env.items():
                m.setenv(k, v)
            st = R.state(cfg.max_new, 15)
        st.encode(R.src)
        parity.teacher_forced(st, ref, R.n0, 0.4, 1.0, cfg)
        st.debug_enable_logits(True)
        logits = []
        for rows in (1, 2, 3, 4, 5, 8, 9, 16):
            st.seq_truncate(R.n0)
            before = st.pass_routes()
            st.large_verify(float("inf"), draft=[int(t) for t in bi.make_tokens(cfg.large.vocab, rows - 1, seed=40 + rows)])
            now = {k for k, v in st.pass_routes().items() if v > before[k]}
            assert now == {"chip" if form == "die" and rows > 4 else form}, (form, rows)
            logits += [st.debug_logits(pkg.LARGE, i) for i in range(rows)]
        before = st.pass_routes()[form]
        st.small_step(0.0)
        assert st.pass_routes()[form] == before + 1
        logits.append(st.debug_logits(pkg.SMALL, 0))
        got[form] = np.stack(logits)
    tol = 2 * parity.logit_tol(cfg)
    for a, b in (("die", "chip"), ("die", "kernels"), ("chip", "kernels")):
        worst = float(np.abs(got[a] - got[b]).max())
        print(a, b, worst)
        assert worst <= tol


@pytest.mark.parametrize("shape", [dict(d=512, heads=6, d_ff=1024, act=bi.ACT_GATED_GELU), dict(d=768, heads=12, d_ff=2112),
                                   dict(d=1024, heads=16, d_ff=4096, n_src=290), dict(d=1024, heads=16, d_ff=2816, act=bi.ACT_SWIGLU)])
def test_loads_of_several_tiles(shape, monkeypatch):
    """Loads that bring eight tiles' activations of one row, four of two rows, or one, whole and with the last tiles missing, and one
    row's attention, at the widths where a wave has more than one tile.  Against the separate kernels, as above."""
    cfg = bi.toy_pair(**{**dict(dtype=bi.DT_BF16, d_head=64, n_src=20, max_new=16, vocab=300, n_large=2, logit_scale=4.0), **shape})
    R = Rig(cfg)
    got = {}
    for form in ("chip", "kernels"):
        with monkeypatch.context() as m:
            for k, v in FORMS[form].items():
                m.setenv(k, v)
            st = R.state(cfg.max_new, 15)
        st.encode(R.src)
        st.debug_enable_logits(True)
        logits = []
        for rows in (1, 2, 3, 4, 5, 8, 2, 1):
            st.seq_truncate(R.n0)
            before = st.pass_routes()
            st.large_verify(float("inf"), draft=[int(t) for t in bi.make_tokens(cfg.large.vocab, rows - 1, seed=40 + rows)])
            assert {k for k, v in st.pass_routes().items() if v > before[k]} == {form}, (form, rows)
            logits += [st.debug_logits(pkg.LARGE, i) for i in range(rows)]
        got[form] = np.stack(logits)
    worst = float(np.abs(got["chip"] - got["kernels"]).max())
    print(worst)
    assert worst <= 2 * parity.logit_tol(cfg)


@pytest.mark.parametrize("shape", [dict(d=1024, heads=16, d_ff=4096), dict(d=1024, heads=16, d_ff=2816, act=bi.ACT_GATED_GELU), dict(d=768, heads=12, d_ff=2304, vocab=185000),
                                   dict(d=1024, heads=4, d_ff=3072)])
def test_who_does_what_with_weights_from_memory(shape, monkeypatch):
    """A head of more than 250 MiB: q, k, v and the FFN's input are the last workgroups' for one row, and for more where the FFN is three times as wide as the
    model; passes of both kinds follow each other in the same hand-over memory.  Against the separate kernels, as above."""
    cfg = bi.toy_pair(**{**dict(dtype=bi.DT_BF16, d_head=64, n_src=20, max_new=16, vocab=140000, n_small=1, n_large=3, logit_scale=4.0, tie_shift=0), **shape})
    R = Rig(cfg)
    got = {}
    for form in ("chip", "kernels"):
        with monkeypatch.context() as m:
            for k, v in FORMS[form].items():
                m.setenv(k, v)
            st = R.state(cfg.max_new, 15)
        st.encode(R.src)
        st.debug_enable_logits(True)
        logits = []
        for rows in (1, 2, 1, 5, 11, 1, 4, 16):
            st.seq_truncate(R.n0)
            before = st.pass_routes()
            st.large_verify(float("inf"), draft=[int(t) for t in bi.make_tokens(cfg.large.vocab, rows - 1, seed=40 + rows)])
            assert {k for k, v in st.pass_routes().items() if v > before[k]} == {form}, (form, rows)
            logits += [st.debug_logits(pkg.LARGE, i)[::37] for i in range(rows)]
        got[form] = np.stack(logits)
    worst = float(np.abs(got["chip"] - got["kernels"]).max())
    print(worst)
    assert worst <= 2 * parity.logit_tol(cfg)


F32 = dict(dtype=bi.DT_F32, truncate=False, d=256, heads=4, d_head=64, n_src=20)


@pytest.mark.parametrize("shape", [
    dict(d_ff=1024), dict(d_ff=32, heads=1), dict(d_ff=480, heads=3, act=bi.ACT_GATED_GELU),
    dict(d_ff=512, cross=False), dict(d_ff=256, act=bi.ACT_SWIGLU, pos=bi.POS_RELATIVE, n_src=300), dict(d_ff=512, n_src=33, tied=False)])
def test_fp32_models_on_one_die(shape):
    """Against the oracle, teacher-forced, and the route: rows of 1 .. 16 and keys past a block and past eight."""
    cfg = bi.toy_pair(**{**F32, "max_new": 700, **shape})
    R = Rig(cfg)
    ref = oracle.bild_generate(R.req, 0.4, 1.0, 15, 24, keep_logits=True)
    st = R.state(cfg.max_new, 15)
    st.encode(R.src)
    parity.teacher_forced(st, ref, R.n0, 0.4, 1.0, cfg)
    r = st.pass_routes()
    assert r["die"] > 0 and r["chip"] == r["kernels"] == r["gave_up"] == 0


@pytest.mark.parametrize("shape", [dict(d_ff=1024), dict(d_ff=256, act=bi.ACT_SWIGLU, pos=bi.POS_RELATIVE)])
def test_fp32_blocks_of_earlier_keys(shape, monkeypatch):
    """One die against the separate kernels (each is within logit_tol of the exact value)."""
    cfg = bi.toy_pair(**{**F32, "max_new": 700, **shape})
    R = Rig(cfg)
    got = {}
    for form in ("die", "kernels"):
        with monkeypatch.context() as m:
            for k, v in FORMS[form].items():
                m.setenv(k, v)
            st = R.state(cfg.max_new, 15)
        st.encode(R.src)
        st.debug_enable_logits(True)
        logits = []
        for have in (1, 32, 33, 225, 257, 600):
            st.seq_truncate(R.n0)
            st.force_tokens(R.n0, bi.make_tokens(cfg.large.vocab, have - R.n0, seed=have), have)
            st.large_verify(float("inf"), draft=[])
            for rows in (1, 3, 8, 16):
                st.seq_truncate(have)
                before = st.pass_routes()
                st.large_verify(float("inf"), draft=[int(t) for t in bi.make_tokens(cfg.large.vocab, rows - 1, seed=40 + rows)])
                assert {k for k, v in st.pass_routes().items() if v > before[k]} == {form}, (have, rows)
                logits += [st.debug_logits(pkg.LARGE, i) for i in range(rows)]
        got[form] = np.stack(logits)
    assert float(np.abs(got["die"] - got["kernels"]).max()) <= 2 * parity.logit_tol(cfg)


@pytest.mark.parametrize("one", ["1", "0"])
@pytest.mark.parametrize("shape", [dict(d=256, heads=4, d_head=64, d_ff=512, dtype=bi.DT_BF16, truncate=True), dict(d=256, heads=4, d_head=64, d_ff=512, n_small=2),
                                   dict(d=1280, heads=10, d_head=128, d_ff=96, dtype=bi.DT_BF16, truncate=True, cross=False, act=bi.ACT_SWIGLU, pos=bi.POS_ROPE, logit_scale=4.0)])
def test_embedding_rows_past_twice_the_vocabulary(shape, one, monkeypatch):
    """The row of token t is (t + tie_shift) mod vocab for every tie_shift: here five vocabularies and some more, bf16, fp32 and wide models,
    passes in one kernel and as kernels of their own."""
    monkeypatch.setenv("BILD_ONE_KERNEL", one)
    cfg = bi.toy_pair(**{**dict(n_large=2, vocab=200, tie_shift=5 * 200 + 137, max_new=8), **shape})
    R = Rig(cfg)
    ref = oracle.bild_generate(R.req, 0.4, 1.0, 4, cfg.max_new, keep_logits=True)
    st = R.state(cfg.max_new, 4)
    st.encode(R.src)
    parity.teacher_forced(st, ref, R.n0, 0.4, 1.0, cfg)
    routes = st.pass_routes()
    assert (routes["chip"] + routes["die"] > 0) == (one == "1"), routes


@pytest.mark.parametrize("dtype,vocab", [
    (bi.DT_BF16, 17), (bi.DT_BF16, 160), (bi.DT_BF16, 161), (bi.DT_BF16, 224 * 160), (bi.DT_BF16, 224 * 160 + 1), (bi.DT_BF16, 3 * 224 * 160 + 1000),
    (bi.DT_F32, 63), (bi.DT_F32, 65), (bi.DT_F32, 224 * 64 + 1), (bi.DT_F32, 40000)])
def test_head_and_policy_inside_the_pass(dtype, vocab):
    """Passes of one row whose head's workgroups are those of the other dies: less than a tile and than a unit of ten (fp32: four) tiles, a unit for each
    of the 224, one more, several rounds.  Against the oracle; then steps whose logits are kept, which run head and policy as kernels,
    between others in the same hand-over memory."""
    cfg = bi.toy_pair(dtype=dtype, d=256, heads=4, d_head=64, d_ff=512, truncate=dtype == bi.DT_BF16, n_src=20, max_new=8, vocab=vocab, tie_shift=min(37, vocab - 1))
    R = Rig(cfg)
    ref = oracle.bild_generate(R.req, 0.4, 1.0, 4, cfg.max_new, keep_logits=True)
    st = R.state(cfg.max_new, 4)
    st.encode(R.src)
    parity.teacher_forced(st, ref, R.n0, 0.4, 1.0, cfg, check_logits=False)
    steps = []
    for turn in range(6):
        st.debug_enable_logits(turn in (1, 2, 4))
        st.seq_truncate(R.n0)
        steps.append([st.small_step(0.0) for _ in range(3)])
    for other in steps[1:]:
        for (tok, flag, p), (tok0, flag0, p0) in zip(other, steps[0]):
            # (the same sums in another order: fp32 products of at most 512 inputs)
            assert (tok, flag) == (tok0, flag0) and abs(p - p0) <= 1e-4 * p0
    r = st.pass_routes()
    assert r["die"] > 0 and r["kernels"] == r["gave_up"] == 0


@pytest.mark.parametrize("dies", [0x1E, 0xFE, 0x01])
@pytest.mark.parametrize("dtype,vocab", [(bi.DT_BF16, 30000), (bi.DT_BF16, 224 * 160 + 1), (bi.DT_F32, 12000)])
def test_head_inside_the_pass_beside_other_work(dtype, vocab, dies):
    """Somebody else's kernel holds four dies, all dies but the one of the layers, and that one, for 40 ms: the head's workgroups that
    have started have the parts of those that have not, or all wait, and no pass gives up."""
    cfg = bi.toy_pair(dtype=dtype, d=256, heads=4, d_head=64, d_ff=512, truncate=dtype == bi.DT_BF16, n_src=20, max_new=16, vocab=vocab)
    R = Rig(cfg)
    st = R.state(cfg.max_new, 12)
    st.encode(R.src)
    streams = [C.c_void_p() for _ in range(8)]
    assert all(hip().hipStreamCreateWithFlags(C.byref(one), 1) == 0 for one in streams)

    def steps(n):
        st.seq_truncate(R.n0)
        t0 = time.perf_counter()
        return [(st.small_step(0.0), time.perf_counter() - t0) for _ in range(n)]

    want = [s for s, _ in steps(8)]
    # (streams share four hardware queues: one of another queue than the state's, whose kernel the first step does not wait for)
    for aside in streams:
        assert pkg.lib().bild_probe_occupy(aside, 0x1E, 40000) == 0
        time.sleep(0.005)
        first = steps(1)[0][1]
        assert hip().hipDeviceSynchronize() == 0
        if first < 0.025:
            break
    before = st.pass_routes()
    for _ in range(3):
        assert pkg.lib().bild_probe_occupy(aside, dies, 40000) == 0
        time.sleep(0.005)
        got = steps(8)
        print(dies, vocab, ["%.1f ms" % (1e3 * t) for _, t in got], flush=True)
        assert [s for s, _ in got] == want
        assert hip().hipDeviceSynchronize() == 0
        if dies == 0x1E:  # the first result is there before the other kernel's end; the next pass follows the first one's last workgroups
            assert got[0][1] < 0.025
        assert got[-1][1] > 0.02, "no work beside the passes"
    now = {k: v - before[k] for k, v in st.pass_routes().items()}
    assert now == {"chip": 0, "die": 24, "kernels": 0, "gave_up": 0}, now
    assert [s for s, _ in steps(8)] == want
    assert all(hip().hipStreamDestroy(one) == 0 for one in streams)
