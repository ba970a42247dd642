"""What a process does once (loading the kernels, their attributes, streams) is done when the first state is made, not inside the
first encode or step."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

FIRST = """
import time
import bild_inputs as bi
import paper_2302_07863_amd as pkg
from tests import parity
cfg = bi.toy_pair(dtype=bi.DT_BF16, d=256, heads=4, d_head=64, d_ff=512, vocab=2000, truncate=True, n_src=200, max_new=8)
pair = parity.make_gpu_pair(cfg, *bi.make_pair_weights(cfg))
src = bi.make_source(cfg)
st = pkg.State(pair, len(src), cfg.max_new + 2, cfg.n_max)
def ms(f):
    t0 = time.perf_counter()
    f()
    return (time.perf_counter() - t0) * 1e3
print("encode", ms(lambda: st.encode(src)), min(ms(lambda: st.encode(src)) for _ in range(5)))
"""


def test_first_encode_of_a_process():
    """1 ms above a later one (6 where kernels were loaded and a stream was made inside it)."""
    r = subprocess.run([sys.executable, "-c", FIRST], cwd=ROOT, env=dict(os.environ), capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    print(r.stdout.strip())
    first, later = (float(v) for v in r.stdout.split()[1:3])
    assert first < later + 3.0


STEPS = """
import sys, time
import bild_inputs as bi
import paper_2302_07863_amd as pkg
from tests import parity
kw = dict(dtype=bi.DT_BF16, vocab=2000, truncate=True, n_src=200, max_new=8)
if sys.argv[1] == "wide":
    kw.update(cross=False, act=bi.ACT_SWIGLU, pos=bi.POS_ROPE, d=1280, heads=10, d_head=128, d_ff=96, n_small=1, n_large=1)
else:
    kw.update(d=256, heads=4, d_head=64, d_ff=512)
cfg = bi.toy_pair(**kw)
pair = parity.make_gpu_pair(cfg, *bi.make_pair_weights(cfg))
src = bi.make_source(cfg)
st = pkg.State(pair, len(src), len(src) + cfg.max_new + 2, cfg.n_max)
st.encode(src)
n = len(st.sequence())
def ms():
    st.seq_truncate(n)
    t0 = time.perf_counter()
    st.small_step(0.0)
    st.small_step(0.0)
    st.large_verify(2.0)
    return (time.perf_counter() - t0) * 1e3
print("steps", ms(), min(ms() for _ in range(5)))
"""


@pytest.mark.parametrize("shape", ["narrow", "wide"])
def test_first_steps_of_a_process(shape):
    """Two steps and a review of three rows: 0.3 ms above later ones, which is capturing the passes (narrow 1.6, wide 0.8 where the LM head's
    and the wide pass kernel were loaded inside them).  The best of three processes, whose host work is not disturbed."""
    over = []
    for _ in range(3):
        r = subprocess.run([sys.executable, "-c", STEPS, shape], cwd=ROOT, env=dict(os.environ), capture_output=True, text=True, timeout=30)
        assert r.returncode == 0, r.stderr[-2000:]
        print(r.stdout.strip())
        first, later = (float(v) for v in r.stdout.split()[1:3])
        over.append(first - later)
    assert min(over) < 0.6
