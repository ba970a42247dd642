"""bild_head_stats: the fused final norm + LM head + softmax statistics as a call of its own, on hidden rows the
caller holds on the device, against the oracle's head and policy quantities (Sections 3.2-3.4)."""
import ctypes as C
import threading

import numpy as np
import pytest

import bild_inputs as bi
import oracle
import paper_2302_07863_amd as pkg
from paper_2302_07863_amd import binding as b
from tests import parity
from tests.hipmem import DeviceArray, hip

pytestmark = pytest.mark.gpu


def run_head_stats(model, x, targets, entry="bild_head_stats"):
    """x [rows][d] float32 numpy, targets [rows] int or None -> records of binding.ROW_STATS_DTYPE (numpy)."""
    xd = DeviceArray(np.ascontiguousarray(x, dtype=np.float32))
    td = DeviceArray(np.ascontiguousarray(targets, dtype=np.int32)) if targets is not None else None
    out = DeviceArray(nbytes=len(x) * b.ROW_STATS_DTYPE.itemsize)
    b.head_stats(model, xd.ptr.value, len(x), td.ptr.value if td is not None else None, out.ptr.value, None, entry)
    return out.to_host(b.ROW_STATS_DTYPE, len(x))


def check_against_oracle(shape, weights, x, targets, got, tol):
    m = oracle.Model(shape, weights)
    z = m.logits_from_hidden(np.asarray(x, dtype=np.float64))
    for t in range(len(x)):
        assert abs(float(got["zmax"][t]) - float(np.max(z[t]))) <= tol, t
        assert abs(float(got["lse"][t]) - oracle.policy.logsumexp(z[t])) <= tol, t
        assert int(got["argmax"][t]) == int(np.argmax(z[t])) or oracle.policy.top2_gap(z[t]) < parity.MARGIN, t
        if targets is None:
            assert np.isnan(got["z_target"][t])
        else:
            assert abs(float(got["z_target"][t]) - float(z[t][targets[t]])) <= tol, t
            # the two policy quantities built from the record
            assert abs(float(np.exp(got["zmax"][t] - got["lse"][t])) - oracle.policy.max_prob(z[t])) <= 2 * tol
            assert abs(float(got["lse"][t] - got["z_target"][t]) - oracle.policy.nll(z[t], int(targets[t]))) <= 2 * tol


@pytest.mark.parametrize("kw", [dict(), dict(dtype=bi.DT_BF16), dict(tied=False, vocab=1000, d=256, heads=3, d_head=32, d_ff=160),
                                dict(dtype=bi.DT_BF16, tied=False, vocab=40000)])
def test_head_stats_against_the_oracle(kw):
    cfg = bi.toy_pair(**kw)
    _, wl = bi.make_pair_weights(cfg)
    shape = cfg.large
    model = parity.make_gpu_model(shape, wl)
    rng = np.random.default_rng(11)
    tol = parity.logit_tol(cfg)
    for rows in (1, 3, 17, 32):
        x = rng.standard_normal((rows, shape.d)).astype(np.float32) * 3.0
        targets = rng.integers(0, shape.vocab, size=rows)
        check_against_oracle(shape, wl, x, targets, run_head_stats(model, x, targets), tol)
    x = rng.standard_normal((2, shape.d)).astype(np.float32)
    check_against_oracle(shape, wl, x, None, run_head_stats(model, x, None), tol)


def test_head_stats_t5_small_shape_and_errors():
    cfg = bi.t5_pair()
    ws, _ = bi.make_pair_weights(replace_large_with_small(cfg))
    shape = cfg.small
    model = parity.make_gpu_model(shape, ws)
    rng = np.random.default_rng(12)
    x = rng.standard_normal((11, shape.d)).astype(np.float32) * 2.0
    targets = rng.integers(0, shape.vocab, size=11)
    check_against_oracle(shape, ws, x, targets, run_head_stats(model, x, targets), parity.logit_tol(cfg))
    xd = DeviceArray(nbytes=40 * shape.d * 4)
    out = DeviceArray(nbytes=40 * 16)
    for rows, xp, op in ((0, xd.ptr.value, out.ptr.value), (33, xd.ptr.value, out.ptr.value), (4, 0, out.ptr.value),
                         (4, xd.ptr.value, 0), (4, xd.ptr.value + 4, out.ptr.value)):
        with pytest.raises(pkg.BildError) as e:
            b.head_stats(model, xp, rows, None, op)
        assert e.value.code == b.EINVAL


def replace_large_with_small(cfg):
    """A pair whose `large` is the small model's shape: weights of the small model alone, without drawing the large one."""
    from dataclasses import replace
    return replace(cfg, large=cfg.small)


def test_merge_of_many_partials_is_exact_to_the_sums_rounding():
    """One id at 0 and 250 111 ids at -x, x = 11.1 .. 12.2, where x log2(e) rounds by up to 9.5e-7: were the weight exp(-x) of each
    partial taken from the rounded product, all would be off the same way, by up to 6.6e-7 of the sum's larger part (5e-7 in the
    result, and the rest on top: 5.8e-7).  What 32 bits leave: about 20 additions on the way of a term, 3.4e-8 rms each, three
    times their root sum times the larger part's 0.7, and the last addition: 3 sqrt(20) 3.4e-8 0.7 + 1.2e-7 = 4.4e-7 (3.3e-7 seen)."""
    cfg = bi.toy_pair(vocab=250112, d=64)
    _, wl = bi.make_pair_weights(cfg)
    shape = cfg.large
    emb, norm = bi.tensor_names(shape)[0], next(n for n in bi.tensor_names(shape) if wl[n].shape == (64,) and "dec" in n and "norm" in n)
    wl = dict(wl)
    wl[emb] = np.full((shape.vocab, 64), -12.2 / 64 / shape.logit_scale, dtype=np.float32)
    wl[emb][0] = 0.0
    wl[norm] = np.ones(64, dtype=np.float32)
    model = parity.make_gpu_model(shape, wl)
    bend = np.linspace(0.0, 0.45, 32)[:, None] * np.where(np.arange(64) % 2, 1.0, -1.0)
    got = run_head_stats(model, 1.0 + bend, np.ones(32, dtype=np.int64))
    z = got["z_target"].astype(np.float64)
    assert np.all(got["zmax"] == 0) and np.all(got["argmax"] == 0) and z.max() < -11.0 and z.min() > -12.3
    err = got["lse"] - np.log1p((shape.vocab - 1) * np.exp(z))
    print("error of lse", np.abs(err).max(), np.sqrt(np.mean(err ** 2)))
    assert np.abs(err).max() < 4.4e-7


@pytest.mark.parametrize("d,vocab,dtype", [(64, 17, bi.DT_BF16), (512, 4100, bi.DT_BF16), (1056, 1030, bi.DT_BF16), (2048, 9000, bi.DT_BF16), (512, 66000, bi.DT_BF16),
                                           (4096, 600, bi.DT_BF16), (4096, 4100, bi.DT_BF16), (2112, 8300, bi.DT_BF16), (64, 17, bi.DT_F32), (256, 33000, bi.DT_F32), (512, 4100, bi.DT_F32), (1024, 9000, bi.DT_F32),
                                           (1056, 1030, bi.DT_F32), (2048, 9000, bi.DT_F32), (2112, 8300, bi.DT_F32), (4096, 8300, bi.DT_F32)])
def test_sweep_shapes(d, vocab, dtype):
    """Input tiles per wave (none for some waves, a short last one), feature tiles per group, several groups per workgroup, both
    entry points: the same results from a launch that joins and from one that does not."""
    cfg = bi.toy_pair(dtype=dtype, d=d, vocab=vocab, n_large=1)
    _, wl = bi.make_pair_weights(cfg)
    shape = cfg.large
    model = parity.make_gpu_model(shape, wl)
    rng = np.random.default_rng(13)
    x = rng.standard_normal((32, shape.d)).astype(np.float32)
    targets = rng.integers(0, shape.vocab, size=32)
    targets[:3] = (0, shape.vocab - 1, 16)
    for rows in (1, 2, 5, 8, 9, 16, 17, 32):
        for _ in range(2):  # (the second call finds the scratch of the first)
            got = run_head_stats(model, x[:rows], targets[:rows])
            check_against_oracle(shape, wl, x[:rows], targets[:rows], got, parity.logit_tol(cfg))
        other = run_head_stats(model, x[:rows], targets[:rows], "bild_head_stats_static")
        for k in ("zmax", "argmax", "z_target"):
            assert (got[k] == other[k]).all(), (rows, k)
        assert np.abs(got["lse"] - other["lse"]).max() <= 2e-6 * max(1.0, float(np.abs(got["lse"]).max()))


NON_BLOCKING = 1  # hipStreamNonBlocking


def _stream():
    s = C.c_void_p()
    assert hip().hipStreamCreateWithFlags(C.byref(s), NON_BLOCKING) == 0
    return s


@pytest.mark.parametrize("rows", [1, 9])  # joined by the sweep's last workgroup, and by a launch of its own
def test_first_calls_on_streams_that_do_not_wait_for_the_null_stream(rows):
    """A fresh scratch is made ready on the caller's stream: the call ends while the null stream still works, with the oracle's
    results; then two threads at once, each with a stream and a buffer of its own."""
    cfg = bi.toy_pair(dtype=bi.DT_BF16, tied=False, vocab=40000)
    _, wl = bi.make_pair_weights(cfg)
    shape = cfg.large
    rng = np.random.default_rng(5)
    x = rng.standard_normal((rows, shape.d)).astype(np.float32)
    targets = rng.integers(0, shape.vocab, size=rows).astype(np.int32)
    xd, td = DeviceArray(x), DeviceArray(targets)
    # (the kernels are loaded, and a model's first call is over, before the model that counts is made)
    run_head_stats(parity.make_gpu_model(shape, wl), x, targets)
    model, out, s = parity.make_gpu_model(shape, wl), DeviceArray(nbytes=rows * 16), _stream()
    a, c = DeviceArray(nbytes=1 << 30), DeviceArray(nbytes=1 << 30)
    for _ in range(200):  # 2 GiB of traffic each: some 80 ms on the null stream
        assert hip().hipMemcpyAsync(a.ptr, c.ptr, 1 << 30, 3, None) == 0
    b.head_stats(model, xd.ptr.value, rows, td.ptr.value, out.ptr.value, s.value)
    busy = hip().hipStreamQuery(None)
    got = out.to_host(b.ROW_STATS_DTYPE, rows)
    assert busy == 600  # hipErrorNotReady: nothing in the call has waited for the null stream
    check_against_oracle(shape, wl, x, targets, got, parity.logit_tol(cfg))
    model, outs, streams, start = parity.make_gpu_model(shape, wl), [DeviceArray(nbytes=rows * 16) for _ in range(2)], [_stream(), _stream()], threading.Barrier(2)

    def work(i):
        start.wait()
        for _ in range(20):
            b.head_stats(model, xd.ptr.value, rows, td.ptr.value, outs[i].ptr.value, streams[i].value)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for o in outs:
        assert (o.to_host(b.ROW_STATS_DTYPE, rows) == got).all()
    for q in [s] + streams:
        assert hip().hipStreamDestroy(q) == 0
