"""A state that serves one request after the other."""
import numpy as np
import pytest

import bild_inputs as bi
import paper_2302_07863_amd as pkg
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [bi.DT_F32, bi.DT_BF16])
def test_passes_over_another_source_take_its_launch_shapes(dtype, monkeypatch):
    """Separate kernels: passes captured over a short source are not replayed over a long one (whose keys are split over more
    workgroups), nor the other way round: the same launches and the same bits as a state made for that source."""
    monkeypatch.setenv("BILD_ONE_KERNEL", "0")
    cfg = bi.toy_pair(dtype=dtype, d=256, heads=4, d_head=64, d_ff=512, truncate=True, n_src=600, max_new=8)
    pair = parity.make_gpu_pair(cfg, *bi.make_pair_weights(cfg))
    src = bi.make_source(cfg)

    def passes(st, n):
        st.debug_enable_logits(True)
        st.encode(src[:n])
        out = []
        for which, call in ((pkg.SMALL, lambda: st.small_step(0.0)), (pkg.LARGE, lambda: st.large_verify(2.0))):
            call()
            out.append((st.pass_stages(), st.debug_logits(which, 0)))
        return out

    one = pkg.State(pair, len(src), 16, 4)
    for n in (20, 600, 20, 130):
        for (got_stages, got), (stages, want) in zip(passes(one, n), passes(pkg.State(pair, len(src), 16, 4), n)):
            assert np.array_equal(got, want) and got_stages == stages, n
